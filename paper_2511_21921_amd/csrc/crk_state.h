// Device state of one evaluation: the cell list and the cell-sorted
// structure-of-arrays intermediates, passed by value to every pass kernel.
#pragma once

#include "crk_device.h"
#include "crk_internal.h"

namespace crk {

constexpr int kLeaf = 16;        // tree path: particles per search leaf (a Morton run)
constexpr int kFan = 8;          // tree path: children per tree node
constexpr int kMaxLevels = 40;   // tree path: largest number of tree levels
// Particles up to which a pair pass gives each 16 lanes instead of 4: 16,384
// fill 4096 waves, four for each of the 1024 SIMDs. Force pass in FP32 (us, 16
// against 4 lanes): 11 and 23 at 4096, 20 and 24 at 16,384, 32 and 31 at 32,768,
// 56 and 51 at 65,536.
constexpr int64_t kRowsMaxN = 16384;
// The same for the passes over the candidates of the cell list, 16 lanes against
// a thread per particle. FP32 with ~64 neighbours, us (16 lanes / thread): h solve
// 34 / 71 at 16,384, 47 / 60 at 32,768, 97 / 72 at 65,536; lists 21 / 49 at 32,768, 38 /
// 52 at 65,536, 69 / 63 at 131,072. With ~268 neighbours (Wendland C4 at n_h = 4) the
// h solve 101 / 201, 178 / 152, 296 / 206; lists 59 / 174, 149 / 196, 278 / 275.
constexpr int64_t kRowsMaxSums = 16384;   // h solve, volume
constexpr int64_t kRowsMaxLists = 65536;

// Counters of one evaluation (unsigned long long, kCntSpread slots each).
enum Counter {
  CNT_HMAX_BITS = 0,   // max input h as double bits
  CNT_BAD_INPUT,       // h <= 0, m <= 0 or u <= 0
  CNT_PAIRS_GATHER,
  CNT_PAIRS_FORCE,
  CNT_H_ITER_MAX,
  CNT_H_UNCONV,
  CNT_H_CAPPED,
  CNT_SCR_OVERFLOW,    // largest candidate count beyond the candidate capacity
  CNT_LIST_OVERFLOW,   // largest gather count beyond the list capacity
  CNT_SLIST_OVERFLOW,  // largest scatter-only count beyond its capacity
  CNT_MMAX_BITS,       // max mass as double bits
  CNT_MINVMAX_BITS,    // max 1/mass as double bits
  CNT_RETRY,           // particles that need another candidate round (tree path)
  CNT_SINGULAR,
  CNT_RELAXED,
  CNT_NONFINITE,
  CNT_HMAX_OUT_BITS,   // max solved h as double bits
  CNT_CELL_MAX,        // largest cell occupancy of the cell list
  CNT_TOO_DENSE,       // a cell beyond the occupancy limit of a speculative cell list (slot 0 only)
  CNT_CANDIDATES,      // candidates kept by the neighbour search (all its passes)
  CNT_LONG_LISTS,      // tree path: scatter-only lists queued for the wave sort (slot 0 only)
  CNT_POOL,            // tree path: candidate pool entries taken by staged blocks (slot 0 only)
  CNT_MOVED,           // particles whose cell differs from the kept cell list's
  CNT_ACTIVE,          // hierarchy: particles active at the substep's end
  CNT_ACTLIST,         // hierarchy: length of the active list (slot 0 only)
  CNT_NEED4,           // tree path: room the unsolved particles ask for, in 4-entry units
  CNT_COUNT
};

// Every counter lives in kCntSpread slots; a block adds to the slot of its
// index modulo kCntSpread and the host folds the slots (sum, or max for the
// maxima). Atomics on one line serialise in the memory-side atomic unit: 1.7 ns
// each with the slots of a counter side by side in 512 bytes, which was all that
// bounded kernels with a counter per wave (4.2M waves at 16.8M particles). A
// slot therefore holds all counters, kCntStride words (256 bytes) apart from
// the next one.
constexpr int kCntSpread = 64;
constexpr int kCntStride = 32;
constexpr int kCntWords = kCntSpread * kCntStride;
static_assert(CNT_COUNT <= kCntStride, "the counters of a slot");
__device__ inline unsigned long long* cnt_at(unsigned long long* cnt, int c) {
  return cnt + c + (int)(blockIdx.x & (kCntSpread - 1)) * kCntStride;
}

// A wave's sum (or maximum) of v, added (or maxed) into *dst by its lane 0.
__device__ inline void wave_add_u64(unsigned long long* dst, unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(dst, v);
}
__device__ inline void wave_max_u64(unsigned long long* dst, unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    unsigned long long t = __shfl_xor(v, o, 64);
    v = t > v ? t : v;
  }
  if ((threadIdx.x & 63) == 0 && v) atomicMax(dst, v);
}

// Adds the number of the wave's (active) lanes with flag into *dst.
__device__ inline void wave_count(unsigned long long* dst, bool flag) {
  const uint64_t b = __ballot(flag);
  if (b != 0ull && (threadIdx.x & 63) == (unsigned)__builtin_ctzll(b))
    atomicAdd(dst, (unsigned long long)__popcll(b));
}

// Bits of a non-negative double, ordered as the value (counter maxima).
__device__ inline unsigned long long dbits(double d) {
  return (unsigned long long)__double_as_longlong(d);
}

template <class R>
struct State {
  int64_t n;
  int G;              // cells per side (lattice cells per side when lattice = 1)
  int lattice;        // 0: cell list with stencil codes; 1: tree over a fine lattice
  double box, ell_d;  // box side and cell side (FP64)
  R ell;              // cell side in Real
  // cell list
  const uint32_t* perm;        // sorted -> caller index
  const uint32_t* keys;        // sorted cell keys
  const uint32_t* cell_start;  // [G^3 + 1]
  uint32_t* cell3;             // packed cell coordinates x | y << 10 | z << 20
  // sorted particle data: position and velocity records side by side, so
  // that a neighbour's pair (one aligned 2 x Real4) is one fetch
  R4<R>* pv;    // [2 i]: (xi_x, xi_y, xi_z, 1/h); [2 i + 1]: (v_x, v_y, v_z, V)
  __device__ R4<R>& pos(int64_t i) const { return pv[2 * i]; }
  __device__ R4<R>& vel(int64_t i) const { return pv[2 * i + 1]; }
  R* mass;
  R* uu;
  R* hbuf;      // h (in: input or guess)
  R* Vbuf;
  R4<R>* gs4;   // 4 per particle: grad v rows in the first nine, then
                // (.., relaxed, lattice cell, 0) and (rho, P, c, den) with
                // den = sum V_j^2 W^R_ij
  R4<R>* kc4;   // 4 per particle: packed corrected-kernel coefficients
  R* mom;       // [40][n] moments kept for the adjoint (may be null)
  // large sets: A, B, grad A, grad B (4 Real4) and accel, du/dt per particle in
  // sorted order, over the candidates from the moment pass on (k_outputs writes the
  // caller's arrays; null: the passes write them), and the caller -> sorted index,
  // which every forward writes from the same size on (the adjoint of any of them
  // may read it)
  R4<R>* co4;
  double4* af4;
  uint32_t* inv;
  // neighbour lists (chunked SELL): gather entries (r < h_i) and
  // scatter-only entries (h_i <= r < h_j)
  uint32_t* nlist;
  uint32_t* slist;
  int* ng;
  int* ns;
  int list_cap;
  int slist_cap;
  // per-wave capacities (tree path): chunk-row offset of every wave's gather
  // and scatter-only lists, one entry per wave plus the total; null when
  // every wave has list_cap / slist_cap
  const uint32_t* grow;
  const uint32_t* srow;
  // candidates within rcap of each particle (16-entry groups, group_base):
  // packed entries, r, and m_j/m_i (the last only when the masses differ);
  // scr_cap is a multiple of 16
  uint32_t* cand;
  R* scr_r;
  R* scr_m;
  int* ccnt;
  int scr_cap;
  int equal_mass;
  R rcap;
  R* rad;             // per-particle candidate radius (tree path) or null; followed
                      // (at rad + n) by the largest radius known to lie below the root
  int* need;          // per-particle candidate capacity request (tree path) or null
  int* todo;          // per-particle "h not solved yet" flag (tree path) or null
  // tree path: rank of each particle among the unsolved ones; null on the
  // cell path
  const uint32_t* cslot;
  // tree path candidate pool (cand), every particle's candidates contiguous
  // from entry 4 cpos[s]: a round that stages them in LDS (the first, when
  // the capacity fits) appends each block's at a bump counter (the slot 0 of
  // CNT_POOL) below pool_cap entries; the other rounds give particle s the
  // room need[s] at 4 (pool_base4 + coff4[s]) (coff4: exclusive sums of the
  // requests of the round, in 4-entry units)
  const uint32_t* coff4;
  int64_t pool_base4;
  int64_t pool_cap;
  int shrink;         // tree path: adapt the radius of an overflowing particle
  // tree over leaves of kLeaf Morton-sorted particles (tree path): node boxes,
  // built as (x, y, z, h_max) low and (x, y, z, -) high corners, then kept as
  // (centre, h_max) in ncen and (half-widths, -) in nhw
  float4* ncen;
  float4* nhw;
  const int* lvl_off;  // [2 kMaxLevels]: node offset of each level (level 0 =
                       // leaves), then the node count of each level
  int nlevels;
  // tree path: where each particle's candidates start, in 4-entry units
  uint32_t* cpos;
  unsigned long long* cnt;
  // parameters
  double n_h3, gamma, alpha, beta, eps2, dt_relax, rtol;
  int max_iter;
  // timestep hierarchy (App. A.3, A.4; levels null: every particle active).
  // A particle of level L is passive at the end of substep jend unless
  // 2^(lev_max - L) divides jend. Passive particles collect no candidates or
  // lists, skip the volume, moment, density and force sums and take V, rho,
  // grad v and the corrections A, B, grad A, grad B from these caller-order
  // arrays (their state of the last evaluation, V and rho updated while
  // passive) when an active particle's force pair reads them.
  const int* levels;
  int lev_max;
  int jend;  // substep end, at most 2^30
  const R* pV;
  const R* prho;
  const R* pgv;
  const R* pA;
  const R* pB;
  const R* pgA;
  const R* pgB;
  // per sorted particle, set by the neighbour-list pass for the active
  // particles and their list partners: the passive particles whose stored
  // state a force pair reads (null: every particle's state is packed)
  uint8_t* needed;
  // a substep with few active particles: their sorted slots (as many as the
  // slot 0 of CNT_ACTLIST counts, in no particular order); the pair passes
  // then give each a 16-lane row, in grids of nact rows, a bound on that
  // number (act null: a thread per particle)
  const uint32_t* act;
  int64_t nact;
};

// The packed lattice coordinates (30 bits) carried in a Real of a record.
__device__ inline float cell_to_real(uint32_t c, float) { return __uint_as_float(c); }
__device__ inline double cell_to_real(uint32_t c, double) { return __hiloint2double(0, (int)c); }
__device__ inline uint32_t real_to_cell(float r) { return __float_as_uint(r); }
__device__ inline uint32_t real_to_cell(double r) { return (uint32_t)__double2loint(r); }

// The packed corrections and the grad v / state record of a particle from
// their Real4 (get(t): the t-th of the record, in memory or staged in LDS).
template <class R, class F>
__device__ inline void kc_from(F&& get, KC<R>& k) {
  const R4<R> q0 = get(0), q1 = get(1), q2 = get(2), q3 = get(3);
  k.a = q0.x;
  k.b[0] = q0.y;
  k.b[1] = q0.z;
  k.b[2] = q0.w;
  k.c[0] = q1.x;
  k.c[1] = q1.y;
  k.c[2] = q1.z;
  k.M[0] = q1.w;
  k.M[1] = q2.x;
  k.M[2] = q2.y;
  k.M[3] = q2.z;
  k.M[4] = q2.w;
  k.M[5] = q3.x;
  k.M[6] = q3.y;
  k.M[7] = q3.z;
  k.M[8] = q3.w;
}
template <class R, class F>
__device__ inline void gs_from(F&& get, R gv[9], R& relaxed, uint32_t& cell, R4<R>& st) {
  const R4<R> q0 = get(0), q1 = get(1), q2 = get(2);
  st = get(3);
  gv[0] = q0.x;
  gv[1] = q0.y;
  gv[2] = q0.z;
  gv[3] = q0.w;
  gv[4] = q1.x;
  gv[5] = q1.y;
  gv[6] = q1.z;
  gv[7] = q1.w;
  gv[8] = q2.x;
  relaxed = q2.y;
  cell = real_to_cell(q2.z);
}
template <class R>
__device__ inline void load_kc4(const State<R>& S, int64_t j, KC<R>& k) {
  kc_from<R>([&](int t) { return S.kc4[4 * j + t]; }, k);
}
template <class R>
__device__ inline void load_gs4(const State<R>& S, int64_t j, R gv[9], R& relaxed, R4<R>& st) {
  uint32_t cell;
  gs_from<R>([&](int t) { return S.gs4[4 * j + t]; }, gv, relaxed, cell, st);
}

// whether sorted particle s is passive (reads nothing without a hierarchy)
template <class R>
__device__ inline bool is_passive(const State<R>& S, int64_t s) {
  if (!S.levels) return false;
  const long long per = 1ll << (S.lev_max - S.levels[S.perm[s]]);
  return ((long long)S.jend & (per - 1)) != 0;
}

__device__ inline int wrap_cell(int c, int G) { return c < 0 ? c + G : (c >= G ? c - G : c); }

// Wave broadcast of lane k's value (k wave-uniform).
__device__ inline float bcast(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}
__device__ inline double bcast(double v, int k) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), k);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), k);
  return __hiloint2double(hi, lo);
}
__device__ inline int bcast(int v, int k) { return __builtin_amdgcn_readlane(v, k); }

// x_a - x_b of two positions on the 1024^3 lattice, in the nearest periodic
// image: the 10-bit coordinates are moved to the top of a word, where their
// difference wraps by itself into [-512, 511] and converts to a float that is
// 2^22 times the cell difference (a power of two: nothing is rounded). The
// roundings are written out: x_b - x_a is the exact negation in every kernel
// (for cells less than half a box apart, 512 of them).
template <class R>
__device__ inline void lattice_dx(const R4<R>& pa, uint32_t a, const R4<R>& pb, uint32_t b, R ell,
                                  R x[3]) {
  const R step = ell * R(1.0 / 4194304.0);
  const int dx = (int)((a << 22) - (b << 22));
  const int dy = (int)(((a << 12) & 0xFFC00000u) - ((b << 12) & 0xFFC00000u));
  const int dz = (int)(((a << 2) & 0xFFC00000u) - ((b << 2) & 0xFFC00000u));
  x[0] = Sc<R>::fma(R(dx), step, pa.x - pb.x);
  x[1] = Sc<R>::fma(R(dy), step, pa.y - pb.y);
  x[2] = Sc<R>::fma(R(dz), step, pa.z - pb.z);
}

// Periodic separation x_ij = x_i - x_j. Cell-list path: from the stencil
// code of the list entry. Lattice path: from both particles' lattice
// coordinates, the difference wrapped to the nearest periodic image.
template <class R>
__device__ inline void pair_x(const State<R>& S, int64_t s, const R4<R>& pi, const R4<R>& pj,
                              uint32_t e, R x[3]) {
  if (!S.lattice) {
    pair_sep<R>(pi, pj, e & kCodeMask, S.ell, x);
    return;
  }
  lattice_dx<R>(pi, S.cell3[s], pj, S.cell3[e >> kCodeBits], S.ell, x);
}

// The same with both lattice cells given (read on the lattice only).
template <class R>
__device__ inline void pair_x(const State<R>& S, const R4<R>& pi, uint32_t ci, const R4<R>& pj,
                              uint32_t cj, uint32_t e, R x[3]) {
  if (!S.lattice)
    pair_sep<R>(pi, pj, e & kCodeMask, S.ell, x);
  else
    lattice_dx<R>(pi, ci, pj, cj, S.ell, x);
}

// Index of this thread's particle, with the block index remapped so that
// each of the 8 XCDs (which receive blocks round-robin, block b on XCD
// b mod 8) takes runs of 2^kXcdRunLog consecutive blocks: particles that are close
// in the sorted order, and so share neighbours, then share that XCD's L2
// instead of being fetched by all eight, and crowded regions of the box, whose
// particles take many times the work, are shared out over the XCDs. (With an
// eighth of the blocks each, the tree's search of 16.8M clumped particles had
// the CUs busy 37% of the time: search 89 ms, gradient 255 ms; now 43 and 194.
// Runs of 2^3 to 2^9 blocks differ by 2%, and uniform sets do not care.)
constexpr int kXcdRunLog = 7;
template <int BLK = kBlock>
__device__ inline int64_t particle_id() {
  const uint32_t B = gridDim.x, b = blockIdx.x;
  constexpr uint32_t kRound = 8u << kXcdRunLog;
  const uint32_t full = B & ~(kRound - 1u);
  uint32_t blk;
  if (b < full) {
    blk = (b & ~(kRound - 1u)) + ((b & 7u) << kXcdRunLog) + ((b & (kRound - 1u)) >> 3);
  } else {  // the last, shorter round: an eighth each
    const uint32_t m = B - full, c = b - full;
    const uint32_t q = m >> 3, r = m & 7u, x = c & 7u;
    blk = full + (x < r ? x * (q + 1u) : r * (q + 1u) + (x - r) * q) + (c >> 3);
  }
  return (int64_t)blk * BLK + threadIdx.x;
}

// Tree path radius growth when the h root lies beyond the radius: by the
// factor that would bring the candidate count to the target (4 pi / 3) n_h^3
// at the density seen, x1.1, kept within [1.25, 4].
__device__ inline double grow_factor(double n_h3, int cnt) {
  const double g = 1.1 * cbrt(4.18879020478639098 * n_h3 / (double)(cnt > 1 ? cnt : 1));
  return g < 1.25 ? 1.25 : (g > 4.0 ? 4.0 : g);
}

// First h of the solve: the h at which cnt candidates within Rcap would be
// (4 pi / 3) n_h^3 at uniform density, Rcap (target / cnt)^(1/3), unless the
// caller's h lies within a factor 1.5 of it (a previous step's h); always
// inside (0, Rcap). The root does not depend on it, only the iterations do.
template <class R>
__device__ inline R first_h(R h_in, R Rcap, int cnt, double n_h3) {
  const double est = (double)Rcap * cbrt(4.18879020478639098 * n_h3 / (double)(cnt > 1 ? cnt : 1));
  double h = (double)h_in;
  if (!(h > est / 1.5 && h < est * 1.5)) h = est;
  if (!(h > 0.0 && h < (double)Rcap)) h = 0.5 * (double)Rcap;
  return (R)h;
}

// Capacity to request for the grown radius: the count scaled by the volume,
// with 30% room, in whole 4-entry chunks.
__device__ inline int need_after_growth(int cnt, double g) {
  const double v = 1.3 * (double)(cnt > 1 ? cnt : 1) * g * g * g;
  const int c = v < 1e8 ? (int)v : 100000000;
  return (c + 3) & ~3;
}

// Tree path: the room a round gives a particle that asks for need entries,
// in whole 4-entry chunks: in a retry round half as much again (an overflow
// of the estimate costs another round); in the first, where every particle
// asks for the uniform capacity, just that.
__device__ inline int room_for(int need, bool retry) {
  return (need + (retry ? need >> 1 : 0) + 3) & ~3;
}

// First word and capacity of particle s's candidate scratch on the cell
// path: slot s with the uniform capacity.
template <class R>
__device__ inline int64_t scratch_base(const State<R>& S, int64_t s, int& cap) {
  cap = S.scr_cap;
  return group_base((s >> 6) * (int64_t)(S.scr_cap >> 4), s);
}

// Where particle s's symmetric neighbour list lives: the gather part
// (r < h_s) and the scatter-only part (h_s <= r < h_j), with their lengths.
struct NbrRef {
  int64_t gb, sb;
  int ng, ns;
};

template <class R>
__device__ inline NbrRef nbr_ref(const State<R>& S, int64_t s) {
  const int64_t w = s >> 6;
  int64_t g0, s0;
  int gcap, scap;
  if (S.grow) {
    g0 = S.grow[w];
    s0 = S.srow[w];
    gcap = (int)(S.grow[w + 1] - S.grow[w]) * 4;
    scap = (int)(S.srow[w + 1] - S.srow[w]) * 4;
  } else {
    g0 = w * (S.list_cap >> 2);
    s0 = w * (S.slist_cap >> 2);
    gcap = S.list_cap;
    scap = S.slist_cap;
  }
  NbrRef r;
  r.gb = slot_base(g0, s);
  r.sb = slot_base(s0, s);
  r.ng = S.ng[s] < gcap ? S.ng[s] : gcap;
  r.ns = S.ns[s] < scap ? S.ns[s] : scap;
  return r;
}

}  // namespace crk
