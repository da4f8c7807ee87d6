// Neighbour search for strongly clustered particle sets.
//
// When smoothing lengths span orders of magnitude (gas clumps in a
// cosmological volume), a cell list sized to the largest h puts whole clumps
// into single cells. This path instead sorts the particles along a Morton
// curve over a 1024^3 lattice (positions are kept as lattice coordinates
// plus FP32/FP64 offsets from the lattice-cell centre), takes every run of
// kLeaf = 16 consecutive particles as a search leaf, and builds an implicit
// tree of leaf boxes with kFan = 8 children per node (a node is named by its
// level and index; its children are the kFan nodes that follow kFan times
// its index one level down). A wave walks the tree for four particles that
// follow each other on the curve, breadth first, and tests the particles of
// the reached leaves, four leaves at a time, against their spheres.
// Candidates within a particle's (padded) radius are kept as indices, each
// particle's contiguous in one pool: the h solve recomputes their distances,
// and the gather list is the candidates within the solved h.
#include "crk_pairs.h"
#include "crk_passes.h"

namespace crk {
namespace {


__device__ inline uint32_t spread10(uint32_t v) {
  v &= 1023u;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

__global__ void __launch_bounds__(kBlock) k_morton(const double* __restrict__ x, int64_t n,
                                                   double L, uint32_t* __restrict__ keys,
                                                   uint32_t* __restrict__ vals) {
  const int64_t i = particle_id();
  if (i >= n) return;
  const double inv = 1024.0 / L;
  uint32_t c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) c[a] = (uint32_t)cell_coord(wrap_pos(x[a * n + i], L), inv, 1024);
  keys[i] = spread10(c[0]) | (spread10(c[1]) << 1) | (spread10(c[2]) << 2);
  vals[i] = (uint32_t)i;
}

// Absolute position of a sorted particle (FP32, the rounding of the node
// boxes) from its lattice cell and its offset from the cell centre.
template <class R>
__device__ inline void abs_pos(const State<R>& S, uint32_t c3, const R4<R>& p, float a[3]) {
  const float ell = (float)S.ell;
  a[0] = ((float)(c3 & 1023u) + 0.5f) * ell + (float)p.x;
  a[1] = ((float)((c3 >> 10) & 1023u) + 0.5f) * ell + (float)p.y;
  a[2] = ((float)(c3 >> 20) + 0.5f) * ell + (float)p.z;
}

// Leaf boxes (absolute positions, FP32) and the largest h of each leaf; the
// absolute positions themselves go to absp (the search's leaf tests).
template <class R>
__global__ void __launch_bounds__(kBlock) k_leaf_boxes(State<R> S, const R* __restrict__ h,
                                                       float4* __restrict__ absp) {
  const int64_t leaf = particle_id();
  const int nleaf = S.lvl_off[kMaxLevels];  // level 0 count
  if (leaf >= nleaf) return;
  const int64_t b = leaf * kLeaf, e = (b + kLeaf < S.n) ? b + kLeaf : S.n;
  float lo[3] = {3e30f, 3e30f, 3e30f}, hi[3] = {-3e30f, -3e30f, -3e30f}, hm = 0.f;
  for (int64_t s = b; s < e; ++s) {
    float v[3];
    abs_pos(S, S.cell3[s], S.pos(s), v);
    absp[s] = make_float4(v[0], v[1], v[2], 0.f);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = fminf(lo[a], v[a]);
      hi[a] = fmaxf(hi[a], v[a]);
    }
    hm = fmaxf(hm, (float)h[s]);
  }
  S.ncen[leaf] = make_float4(lo[0], lo[1], lo[2], hm);  // corners until k_box_centres
  S.nhw[leaf] = make_float4(hi[0], hi[1], hi[2], 0.f);
}

// Node k of a level from its (up to kFan) children k kFan + c one level down.
__global__ void __launch_bounds__(kBlock) k_tree_up(float4* nlo, float4* nhi, int off_c,
                                                    int cnt_c, int off_p, int cnt_p) {
  const int k = blockIdx.x * kBlock + threadIdx.x;
  if (k >= cnt_p) return;
  float4 lo = nlo[off_c + kFan * k], hi = nhi[off_c + kFan * k];
  for (int c = 1; c < kFan && kFan * k + c < cnt_c; ++c) {
    const float4 l2 = nlo[off_c + kFan * k + c], h2 = nhi[off_c + kFan * k + c];
    lo = make_float4(fminf(lo.x, l2.x), fminf(lo.y, l2.y), fminf(lo.z, l2.z), fmaxf(lo.w, l2.w));
    hi = make_float4(fmaxf(hi.x, h2.x), fmaxf(hi.y, h2.y), fmaxf(hi.z, h2.z), 0.f);
  }
  nlo[off_p + k] = lo;
  nhi[off_p + k] = hi;
}

// Every node box from its corners to (centre, h_max) and (half-widths, 0).
__global__ void __launch_bounds__(kBlock) k_box_centres(float4* __restrict__ lo_c,
                                                        float4* __restrict__ hi_w, int nnode) {
  const int k = blockIdx.x * kBlock + threadIdx.x;
  if (k >= nnode) return;
  const float4 lo = lo_c[k], hi = hi_w[k];
  lo_c[k] = make_float4(0.5f * (lo.x + hi.x), 0.5f * (lo.y + hi.y), 0.5f * (lo.z + hi.z), lo.w);
  hi_w[k] = make_float4(0.5f * (hi.x - lo.x), 0.5f * (hi.y - lo.y), 0.5f * (hi.z - lo.z), 0.f);
}

// Radius widened against the FP32 rounding of positions and node boxes.
__device__ inline float pad_radius(float r, float L) { return r * 1.00001f + 4e-6f * L; }

// Distance of a pair from its two position records (their w holds the lattice
// cell until the lists are made). Every pass of the search takes it so: the
// offsets and differences negate exactly and the contraction of the sum is
// written out, so that r_ij = r_ji to the bit whatever the compiler unrolls.
template <class R>
__device__ inline R lattice_r(const State<R>& S, const R4<R>& pi, const R4<R>& pj) {
  R x[3];
  lattice_dx<R>(pi, real_to_cell(pi.w), pj, real_to_cell(pj.w), S.ell, x);
  return Sc<R>::sqrt(norm2(x));
}

// Sum over the lanes of a row.
__device__ inline int row_total(int v) {
  v += (int)dpp_mov<quad_perm(1, 0, 3, 2)>((uint32_t)v);
  v += (int)dpp_mov<quad_perm(2, 3, 0, 1)>((uint32_t)v);
  v += (int)dpp_mov<0x124>((uint32_t)v);
  v += (int)dpp_mov<0x128>((uint32_t)v);
  return v;
}

// First candidate radius of every particle, kept small so that the first
// walk stays cheap (particles whose h root lies beyond it grow it in later
// rounds): the least of the h that the target count would need at the
// density of the particle's 8 nearest wave-mates (the 64 particles of its
// wave), n_h r_8 (4 pi / 24)^(1/3), at the density of the wave's box, and
// 1.5x that of the mean density (the estimate lies a fifth above the root
// for the median particle and below it for a few percent). When the caller's
// h lies within [0.75, 1.33] of the estimate (a previous step's h), 1.05 h is
// taken where it is larger. With fixed h the radius is h.
template <class R>
__global__ void __launch_bounds__(kBlock) k_init_radius(State<R> S, int h_mode) {
  const int64_t s = particle_id();
  if ((s & ~(int64_t)63) >= S.n) return;
  const bool active = s < S.n;
  const int64_t sc = active ? s : 0;
  const int64_t wave = sc >> 6;
  R r = S.hbuf[sc];
  if (h_mode != 0) {
    const int lane = threadIdx.x & 63;
    const R4<R> pi = S.pos(sc);
    const uint32_t ci = S.cell3[sc];
    const int64_t b = wave * 64;
    const int cnt = (int)((b + 64 < S.n ? b + 64 : S.n) - b);
    // the wave's particles, broadcast to its lanes one at a time
    const int64_t jl = b + (lane < cnt ? lane : 0);
    const R4<R> pl = S.pos(jl);
    const int cl = (int)S.cell3[jl];
    float d[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) d[t] = 3e30f;
    for (int t = 0; t < cnt; ++t) {
      R4<R> pj;
      pj.x = bcast(pl.x, t);
      pj.y = bcast(pl.y, t);
      pj.z = bcast(pl.z, t);
      pj.w = R(0);
      const uint32_t cj = (uint32_t)bcast(cl, t);
      if (b + t == sc) continue;
      R x[3];
      lattice_dx<R>(pi, ci, pj, cj, S.ell, x);
      float v = (float)(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]);
#pragma unroll
      for (int q = 0; q < 8; ++q) {  // keep the 8 smallest, sorted
        const float lo = fminf(d[q], v);
        v = fmaxf(d[q], v);
        d[q] = lo;
      }
    }
    // the wave's box: the union of its (up to four) leaves
    const int nleaf = S.lvl_off[kMaxLevels];
    float lo[3] = {3e30f, 3e30f, 3e30f}, hi[3] = {-3e30f, -3e30f, -3e30f};
    for (int q = 0; q < 4 && wave * 4 + q < nleaf; ++q) {
      const float4 c = S.ncen[wave * 4 + q], w = S.nhw[wave * 4 + q];
      const float cc[3] = {c.x, c.y, c.z}, ww[3] = {w.x, w.y, w.z};
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lo[a] = fminf(lo[a], cc[a] - ww[a]);
        hi[a] = fmaxf(hi[a], cc[a] + ww[a]);
      }
    }
    const double pad = 0.5 * S.ell_d;  // coincident lattice cells have no volume
    const double vol = ((double)(hi[0] - lo[0]) + pad) * ((double)(hi[1] - lo[1]) + pad) *
                       ((double)(hi[2] - lo[2]) + pad);
    // (a wave of fewer than nine particles, the ragged last one, tells
    // nothing of the density: the mean density's h then)
    double est = cnt >= 9 ? cbrt(S.n_h3 * vol / (double)cnt) : cbrt(S.n_h3 / (double)S.n) * S.box;
    if (cnt >= 9)  // (4 pi / 24)^(1/3)
      est = fmin(est, cbrt(S.n_h3) * sqrt((double)d[7]) * 0.80599597700823482);
    est = fmin(est, 1.5 * cbrt(S.n_h3 / (double)S.n) * S.box);
    const double g = (double)r;
    const double h0 = (g > 0.75 * est && g < 1.33 * est) ? fmax(1.05 * g, est) : est;
    r = (R)fmin(h0, 0.45 * S.box);
  }
  if (active) {
    S.rad[s] = r;
    S.rad[S.n + s] = R(0);  // no radius known below the root yet
    S.need[s] = S.scr_cap;
    S.todo[s] = 1;
  }
}

// The h solve of k_hsolve (or the volume of k_volume for fixed h) with a
// 16-lane row per particle: lane sub takes the kept candidates 16 it + sub,
// recomputing their distances from the positions (the candidate pass keeps
// only the indices), holding those of the first kRegGroups groups in
// registers and recomputing any further ones at every evaluation. The sums over the row are butterfly
// reductions, which leave the same value in every lane, so the solve is
// uniform over the row and its lane 0 writes the results. The spread over
// the row keeps a particle with thousands of candidates (a sphere that
// takes in a dense clump core) from holding a wave for thousands of serial
// steps per evaluation. order null: row t takes particle t; else order[t].
constexpr int kRegGroups = 16;
template <class R, int K, bool EM>
__global__ void __launch_bounds__(kBlock) k_hsolve_rows(State<R> S,
                                                        const uint32_t* __restrict__ order,
                                                        int64_t nt) {
  const int64_t tid = particle_id();
  if (((tid & ~(int64_t)63) >> 4) >= nt) return;  // the wave's four rows past the end
  const int64_t t = tid >> 4;
  const int sub = threadIdx.x & 15;
  const int64_t s = t < nt ? (order ? (int64_t)order[t] : t) : S.n;
  // particles still to solve whose candidate pass fitted (uniform over the row)
  const bool work = s < S.n && S.todo[s] && S.ccnt[s] >= 0;
  unsigned long long iters = 0, unconv = 0, capped = 0, hbits = 0;
  if (__ballot(work) != 0ull) {
    int cnt = 0;
    int64_t base = 0;
    if (work) {
      base = 4 * (int64_t)S.cpos[s];
      cnt = S.ccnt[s];
    }
    const int ngroups = (cnt + 15) >> 4;
    // the distance and mass ratio of kept entry e, from the exact
    // separation (lattice offsets, as every later pass computes it)
    const int64_t sc = s < S.n ? s : 0;
    const R4<R> pi = S.pos(sc);
    const R mi_inv = EM ? R(1) : R(1) / S.mass[sc];
    // Lanes past the count load entry 0 of the row, or of the pool when the
    // row has no entry (the word at its position is then another row's or
    // was never written); the index is clamped below n, so that whatever
    // such a lane loaded addresses a particle (its terms are discarded).
    const int64_t at0 = cnt > 0 ? base : 0;
    const uint32_t jmax = (uint32_t)(S.n - 1);
    auto entry = [&](int e, R& r, R& mr) {
      const uint32_t w = S.cand[e < cnt ? base + e : at0] >> kCodeBits;
      const uint32_t j = w < jmax ? w : jmax;
      r = lattice_r(S, pi, S.pos(j));
      mr = EM ? R(1) : S.mass[j] * mi_inv;
    };
    R rk[kRegGroups], mk[kRegGroups];
    // four groups at once, without branches, so that their loads are in
    // flight together, as far as the wave's longest row goes
    const int most = max(max(__builtin_amdgcn_readlane(cnt, 0), __builtin_amdgcn_readlane(cnt, 16)),
                         max(__builtin_amdgcn_readlane(cnt, 32), __builtin_amdgcn_readlane(cnt, 48)));
#pragma unroll
    for (int q = 0; q < kRegGroups; q += 4)
      if (16 * q < most) {
#pragma unroll
        for (int it = q; it < q + 4; ++it) entry(16 * it + sub, rk[it], mk[it]);
      }
    auto sums = [&](R h, R& dsum) {
      const R hinv = R(1) / h;
      R sum = R(0), ds = R(0);
      auto add = [&](int e, R r, R mr) {
        // entries past the count are moved outside the support (w = w' = 0)
        const bool in = e < cnt;
        const R q = in ? r * hinv : R(2);
        R w, dw;
        Shape<K>::eval(q, w, dw);
        const R mt = EM ? R(1) : (in ? mr : R(0));
        sum += mt * w;
        ds += mt * dw * q;
      };
#pragma unroll
      for (int it = 0; it < kRegGroups; ++it)
        if (it < ngroups) add(16 * it + sub, rk[it], mk[it]);
      for (int it = kRegGroups; it < ngroups; ++it) {
        R r, mr;
        entry(16 * it + sub, r, mr);
        add(16 * it + sub, r, mr);
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        sum += __shfl_xor(sum, o, 16);
        ds += __shfl_xor(ds, o, 16);
      }
      dsum = ds;
      return sum + R(Shape<K>::w0);
    };
    const R C = R(Shape<K>::C);
    if (work && !S.shrink) {
      // fixed h: V_i = m_i / sum_j m_j W(r_ij, h_i), self term included
      const R h = S.hbuf[s];
      R dsum;
      const R sum = sums(h, dsum);
      if (sub == 0) {
        S.todo[s] = 0;
        if (!is_passive(S, s)) S.Vbuf[s] = h * h * h / (C * sum);
      }
    } else if (work) {
      // f(h) = C (w(0) + sum_j (m_j/m_i) w(r_ij / h)) - n_h^3, non-decreasing
      // in h: safeguarded Newton inside a bisection bracket, as k_hsolve
      const R Rcap = S.rad[s];
      const R n_h3 = R(S.n_h3);
      const R rtol = R(S.rtol);
      R h = first_h(S.hbuf[s], Rcap, cnt, S.n_h3);
      R dsum, sum = sums(h, dsum);
      R f = C * sum - n_h3;
      // the bracket [0, Rcap] holds the root only if f(Rcap) > 0
      bool cap_hit = false;
      if (!(f > R(0))) {
        R ds2;
        cap_hit = !(C * sums(Rcap, ds2) - n_h3 > R(0));
      }
      if (cap_hit) {
        // the root lies beyond the radius: grow it by what the candidate
        // count suggests; the particle is taken again in the next round
        if (sub == 0) {
          capped = 1;
          const double g = grow_factor(S.n_h3, cnt);
          S.rad[S.n + s] = Rcap;
          S.rad[s] = (R)((double)Rcap * g);
          S.need[s] = max(S.need[s], need_after_growth(cnt, g));
        }
      } else {
        R lo = R(0), hi = Rcap;
        bool conv = false;
        int it = 0;
        R hn = h;
        for (;;) {
          const R fp = -C * dsum / h;
          if (f > R(0)) hi = h; else lo = h;
          hn = R(0.5) * (lo + hi);
          if (fp > R(0)) {
            const R nt_ = h - f / fp;
            const R step = nt_ > h ? nt_ - h : h - nt_;
            if (step <= rtol * h) {
              hn = nt_ < lo ? lo : (nt_ > hi ? hi : nt_);
              conv = true;
              break;
            }
            if (nt_ > lo && nt_ < hi) hn = nt_;
          }
          if (hi - lo <= rtol * hn) {
            conv = true;
            break;
          }
          if (++it >= S.max_iter) break;
          h = hn;
          sum = sums(h, dsum);
          f = C * sum - n_h3;
        }
        // V at the final h from the last sums (first order in the step, which
        // is below the tolerance; an unconverged h gets its own pass)
        const R sum_f = conv ? sum - dsum / h * (hn - h) : sums(hn, dsum);
        if (sub == 0) {
          iters = (unsigned long long)(it + 1);
          unconv = conv ? 0 : 1;
          S.hbuf[s] = hn;
          S.Vbuf[s] = hn * hn * hn / (C * sum_f);
          hbits = dbits((double)hn);
          S.todo[s] = 0;
        }
      }
    }
  }
  wave_max_u64(cnt_at(S.cnt, CNT_H_ITER_MAX), iters);
  wave_add_u64(cnt_at(S.cnt, CNT_H_UNCONV), unconv);
  wave_add_u64(cnt_at(S.cnt, CNT_H_CAPPED), capped);
  wave_max_u64(cnt_at(S.cnt, CNT_HMAX_OUT_BITS), hbits);
}

// LDS staging capacity of a particle, in entries: 16 KB a block of 16
// particles, which leaves room in the LDS for seven blocks a CU.
constexpr int kStage = 256;
// Particles of a wave. The more share a walk and the leaves they load, the
// fewer instructions each takes (628 with eight, 770 with four), but the
// more staging they hold and the more scalar registers: at 16.8M clumped
// particles four take 29.7 ms, six 29.4, eight (half the waves in flight)
// 35.0; at 2.1M 5.0, 5.4 and 6.7.
constexpr int kSet = 4;
// Particles up to which a round gives each a wave of its own: the particles of
// a retry round lie apart, and with few waves of four the last ones leave the
// chip idle (the retry rounds at 2.1M: 4.4 ms in all the search with 65,536,
// 5.0 with 8192).
constexpr int64_t kAloneMax = 65536;

// Candidates of every unsolved particle: the j != s whose FP32 absolute
// position lies within its radius ri padded beyond the FP32 rounding (their
// indices, in ascending j), kept contiguous in the candidate pool from entry
// 4 cpos[s]. They hold every j with r_ij < ri and at most a thin shell
// beyond it, which adds nothing to the sums or lists of any h <= ri: the h
// solve and the list filter compute the exact separations themselves. A
// wave takes kSet consecutive particles (order null: rank t is particle t;
// else order[t], the unsolved particles of a retry round in rank order). Each
// works in its own room (room_for(need[s]) entries at pool_base4 + coff4[s]), or
// (STAGE) in an LDS stage of scr_cap entries, after which every block
// takes the room its particles' candidates need from the pool's bump counter and
// copies them there (a block that finds the pool full leaves its particles
// to the next round, with room of their own).
//    The particles of a wave, neighbours along the curve, reach much the same
//     leaves: the wave walks the levels once, breadth first on its 64 lanes,
//     for their common bounding box widened by the largest radius, keeps a
//     leaf when one of the spheres (padded beyond the FP32 rounding) reaches
//     it, and loads the particles of four leaves at a time, one per lane, to
//     test them against each sphere in turn. Positions, radii, counts and
//     masks of the spheres are wave-uniform and live in scalar registers, so
//     that a test is eight vector instructions for 64 particles. Particles far
//     apart, or so large a sphere that a level outgrows its buffer, walk
//     depth first or one after another.
// What bounds it is vector instructions: 2600 a wave of four particles, 87% of the
// issue slots (16.8M clumped particles; 3600 when each particle had 16 lanes that
// walked the lowest levels and tested by themselves, 19.8 ms a staged round
// against 11.3).
// A particle whose passed indices overflow its capacity is counted: the next
// round takes the radius that would hold 1.3 (4 pi / 3) n_h^3 of them at the
// density seen (at least half of ri), with capacity for 1.3 times what that
// density gives there; a radius that then falls short of the h root is grown
// by the h solve, and once that has happened radii only grow (an overflow
// keeps the radius and raises the capacity), so the rounds end. With fixed h
// the capacity is raised.
template <class R, bool STAGE>
__global__ void __launch_bounds__(kBlock) k_candidates_tree(State<R> S,
                                                            const float4* __restrict__ absp,
                                                            const uint32_t* __restrict__ order,
                                                            int64_t nt, int per) {
  constexpr int kWaves = kBlock / 64;
  constexpr int kQueue = 128;  // leaves queued (64 more fit whenever 64 or fewer wait)
  constexpr int kFront = 64;   // nodes of a level under expansion
  // largest half-diagonal of the particles' common box over their largest radius
  constexpr float kReach = 2.0f;
  static_assert(kFan == 8 && kLeaf == 16, "lanes: 8 nodes of 8 children, 4 leaves of 16");
  static_assert(kSet >= 1 && kSet <= 8, "a leaf's spheres are bits of a byte");
  __shared__ uint32_t leafq[kWaves][kQueue];
  __shared__ uint32_t front[kWaves][3][kFront];
  __shared__ uint4 stage4[STAGE ? kWaves * kSet : 1][STAGE ? kStage / 4 : 1];
  __shared__ uint32_t rcnt[kWaves * kSet];
  __shared__ unsigned long long rbase[kWaves * kSet];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63, sub = lane & 15;
  const int64_t t = (particle_id() >> 6) * per + lane;  // this lane's rank in the round
  // lanes 0 .. per - 1 hold the wave's particles
  const bool active = lane < per && t < nt;
  const int64_t s = active ? (order ? (int64_t)order[t] : t) : 0;
  const bool mine = active && S.todo[s];
  const uint64_t todo = __ballot(mine);
  if (!STAGE && todo == 0ull) return;
  unsigned long long kept = 0;
  bool retry = false;
  int np = 0;  // passed indices of the lane's particle
  int cap = 0;
  int64_t base = 0;
  if (todo != 0ull) {
    // level l's offset and node count, in lane l
    const int lv_off = lane < S.nlevels ? S.lvl_off[lane] : 0;
    const int lv_cnt = lane < S.nlevels ? S.lvl_off[kMaxLevels + lane] : 0;
    auto off_of = [&](int l) { return __builtin_amdgcn_readlane(lv_off, l); };
    auto cnt_of = [&](int l) { return __builtin_amdgcn_readlane(lv_cnt, l); };
    auto lane_f = [](float v, int l) {
      return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
    };
    auto wave_sync = [&]() {  // the wave's LDS writes before its reads, and the reverse
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    const R ri = mine ? S.rad[s] : R(0);
    if (mine) {
      if constexpr (STAGE) {
        cap = S.scr_cap;  // at most kStage
      } else {
        cap = room_for(S.need[s], order != nullptr);  // order: a retry round
        base = 4 * (S.pool_base4 + (int64_t)S.coff4[s]);
      }
    }
    float P[3];
    abs_pos(S, S.cell3[s], S.pos(s), P);
    const float L = (float)S.box;
    const float inv_L = 1.0f / L;
    const float rp = mine ? pad_radius((float)ri, L) : -1.f;
    const float rp2 = mine ? rp * rp : -1.f;
    // A sphere that stays a padded radius away from every face of the box
    // reaches no periodic image (box centres and positions lie in the box),
    // so its tests need no nearest-image shift; a wave with a sphere that
    // crosses a face takes it.
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) inside = inside && P[a] > rp + 1e-5f * L && P[a] < L - rp - 1e-5f * L;
    bool shifted = !inside;
    const uint32_t n32 = (uint32_t)S.n;
    const int top = S.nlevels - 1;
    // the particles' common box, from the first one's nearest images
    const int first = __builtin_ctzll(todo);
    float C0[3], W0[3], rm0 = rp;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float q0 = lane_f(P[a], first);
      float d = P[a] - q0;
      const float turn = rintf(d * inv_L);  // (particles of one wave on both sides of a face)
      shifted = shifted || turn != 0.f;
      d -= L * turn;
      float lo = mine ? d : 3e30f, hi = mine ? d : -3e30f;
#pragma unroll
      for (int o = kSet / 2; o > 0; o >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, o, 64));
        hi = fmaxf(hi, __shfl_xor(hi, o, 64));
      }
      C0[a] = q0 + 0.5f * lane_f(lo + hi, 0);
      W0[a] = 0.5f * lane_f(hi - lo, 0);
    }
#pragma unroll
    for (int o = kSet / 2; o > 0; o >>= 1) rm0 = fmaxf(rm0, __shfl_xor(rm0, o, 64));
    rm0 = lane_f(rm0, 0);
    const bool wrap = __ballot(mine && shifted) != 0ull;

    // The walk for the M particles of lanes g0 .. g0 + M - 1 (box centre C,
    // half widths W, largest radius rm), their passed indices in order.
    auto walk = [&](auto wrap_t, auto m_t, int g0, const float* C, const float* W, float rm) {
      constexpr bool WRAP = decltype(wrap_t)::value;
      constexpr int M = decltype(m_t)::value;
      float X[M][3], r2[M];
      uint32_t id[M];
      int cnt[M], room[M];
      int64_t at0[M];
#pragma unroll
      for (int k = 0; k < M; ++k) {
#pragma unroll
        for (int a = 0; a < 3; ++a) X[k][a] = lane_f(P[a], g0 + k);
        r2[k] = lane_f(rp2, g0 + k);  // -1 where there is no particle: nothing passes
        id[k] = (uint32_t)__builtin_amdgcn_readlane((int)s, g0 + k);
        room[k] = STAGE ? S.scr_cap : __builtin_amdgcn_readlane(cap, g0 + k);
        at0[k] = STAGE ? 0
                       : (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)base, g0 + k) |
                             ((int64_t)__builtin_amdgcn_readlane((int)(base >> 32), g0 + k) << 32);
        cnt[k] = 0;
      }
      // (the centre, the box's half widths and the radius widened beyond the
      // FP32 rounding, so that no box that a particle's own test reaches is lost)
      const float Rr = rm * 1.00001f + 4e-6f * L, Rr2 = Rr * Rr;
      auto near = [&](float4 c, float4 h) {  // the widened common box reaches this one
        const float cc[3] = {c.x, c.y, c.z}, hh[3] = {h.x, h.y, h.z};
        float g2 = 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          float d = cc[a] - C[a];
          if constexpr (WRAP) d = __builtin_fmaf(-L, rintf(d * inv_L), d);
          const float g = fmaxf(fabsf(d) - (hh[a] + W[a]), 0.f);
          g2 = __builtin_fmaf(g, g, g2);
        }
        return g2 < Rr2;
      };
      auto reached = [&](float4 c, float4 h) {  // the spheres that reach this box, a bit each
        const float cc[3] = {c.x, c.y, c.z}, hh[3] = {h.x, h.y, h.z};
        uint32_t which = 0u;
#pragma unroll
        for (int k = 0; k < M; ++k) {
          float g2 = 0.f;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            float d = cc[a] - X[k][a];
            if constexpr (WRAP) d = __builtin_fmaf(-L, rintf(d * inv_L), d);
            const float g = fmaxf(fabsf(d) - hh[a], 0.f);
            g2 = __builtin_fmaf(g, g, g2);
          }
          which |= g2 < r2[k] ? 1u << k : 0u;
        }
        return which;
      };
      // queued leaves, each with the spheres that reach it in the top byte
      uint32_t* queue = leafq[w];
      int qh = 0, qt = 0;  // the queue's head and tail (a ring)
      // up to four queued leaves: their particles, one per lane (on: there is
      // one), and the spheres that reach any of them
      struct Four {
        float a[3];
        uint32_t j;
        bool on;
        uint32_t which;
      };
      auto fetch = [&]() {
        Four f;
        const int q = qh + (lane >> 4);
        const uint32_t e = queue[(q < qt ? q : qh) & (kQueue - 1)];
        f.j = (e & 0xFFFFFFu) * (uint32_t)kLeaf + (uint32_t)sub;
        f.on = q < qt && f.j < n32;
        const float* a = reinterpret_cast<const float*>(absp + f.j);  // (padded to whole leaves)
#pragma unroll
        for (int b = 0; b < 3; ++b) f.a[b] = a[b];
        f.which = (uint32_t)(__builtin_amdgcn_readlane((int)e, 0) | __builtin_amdgcn_readlane((int)e, 16) |
                             __builtin_amdgcn_readlane((int)e, 32) | __builtin_amdgcn_readlane((int)e, 48)) >>
                  24;
        qh = qh + 4 < qt ? qh + 4 : qt;
        return f;
      };
      auto test = [&](const Four& f) {
        const float aa[3] = {f.on ? f.a[0] : __builtin_inff(), f.a[1], f.a[2]};
        const uint32_t j = f.j, v = j << kCodeBits;
#pragma unroll
        for (int k = 0; k < M; ++k) {
          if (M > 1 && !(f.which >> k & 1u)) continue;
          float d[3];
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            d[b] = aa[b] - X[k][b];
            if constexpr (WRAP) d[b] = __builtin_fmaf(-L, rintf(d[b] * inv_L), d[b]);
          }
          const float d2 = __builtin_fmaf(d[2], d[2], __builtin_fmaf(d[1], d[1], d[0] * d[0]));
          const bool near_k = d2 < r2[k], other = j != id[k];
          const uint64_t m =
              __builtin_amdgcn_ballot_w64(near_k) & __builtin_amdgcn_ballot_w64(other);
          if (m != 0ull) {
            const int c = __popcll(m);
            if (cnt[k] + c <= room[k]) {  // (an overflowed particle's indices are not read)
              const uint32_t at = __builtin_amdgcn_mbcnt_hi(
                  (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
              if (near_k & other) {
                if constexpr (STAGE)
                  (reinterpret_cast<uint32_t*>(stage4[w * kSet + g0 + k]) + cnt[k])[at] = v;
                else
                  (S.cand + (at0[k] + cnt[k]))[at] = v;
              }
            }
            cnt[k] += c;
          }
        }
      };
      // tests the queued leaves in fours until fewer than left + 1 wait
      auto drain = [&](int left) {
        if (qt - qh <= left) return;
        wave_sync();
        // four leaves in flight while four are tested (in turns: a copy would
        // wait for the load)
        Four f = fetch();
        for (;;) {
          if (qt - qh <= left) {
            test(f);
            break;
          }
          const Four g = fetch();
          test(f);
          if (qt - qh <= left) {
            test(g);
            break;
          }
          f = fetch();
          test(g);
        }
        wave_sync();
      };
      // queues the leaves (one per lane) that a sphere reaches, in order
      auto leaves = [&](uint32_t leaf, bool valid) {
        valid = valid && leaf < (uint32_t)cnt_of(0);
        const uint32_t node = (uint32_t)off_of(0) + (valid ? leaf : 0u);
        const uint32_t which = reached(S.ncen[node], S.nhw[node]);
        const bool hit = valid && which != 0u;
        const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
        const int at = qt + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (hit) queue[at & (kQueue - 1)] = leaf | which << 24;
        qt += __popcll(m);
        if (qt - qh > kQueue - 64) drain(3);
      };
      // the nodes ch of level l (one per lane) that the common box reaches,
      // appended to list[have ..]; returns how many there are then
      auto keep = [&](int l, uint32_t ch, bool valid, uint32_t* list, int have) {
        valid = valid && ch < (uint32_t)cnt_of(l);
        const uint32_t node = (uint32_t)off_of(l) + (valid ? ch : 0u);
        const bool hit = valid && near(S.ncen[node], S.nhw[node]);
        const uint64_t m = __builtin_amdgcn_ballot_w64(hit);
        const int at = have + (int)__builtin_amdgcn_mbcnt_hi(
                                  (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (hit && at < kFront) list[at] = ch;
        return have + __popcll(m);
      };
      // child of a listed node for this lane: lane 8 k + c takes child c of list[k0 + k]
      auto child = [&](const uint32_t* list, int k0, int have, bool& valid) {
        const int k = k0 + (lane >> 3);
        valid = k < have;
        return list[valid ? k : 0] * (uint32_t)kFan + (uint32_t)(lane & 7);
      };
      uint32_t *fa = front[w][0], *fb = front[w][1], *f1 = front[w][2];
      // the leaves under the n1 level-1 nodes of f1
      auto under = [&](int n1) {
        wave_sync();
        for (int k0 = 0; k0 < n1; k0 += 8) {
          bool valid;
          const uint32_t leaf = child(f1, k0, n1, valid);
          leaves(leaf, valid);
        }
        wave_sync();
      };
      // the walk starts at the lowest level of at most 64 nodes
      int l0 = 0;
      while (cnt_of(l0) > 64) ++l0;
      if (l0 == 0) {
        leaves((uint32_t)lane, true);
      } else if (l0 == 1) {
        under(keep(1, (uint32_t)lane, true, f1, 0));
      } else {
        int na = keep(l0, (uint32_t)lane, true, fa, 0);
        int l = l0;
        for (; l > 2 && na <= kFront; --l) {
          wave_sync();
          int nb = 0;
          for (int k0 = 0; k0 < na; k0 += 8) {
            bool valid;
            const uint32_t ch = child(fa, k0, na, valid);
            nb = keep(l - 1, ch, valid, fb, nb);
          }
          uint32_t* x = fa;
          fa = fb;
          fb = x;
          na = nb;
        }
        if (na <= kFront) {  // fa: the reached level-2 nodes
          wave_sync();
          for (int k0 = 0; k0 < na; k0 += 8) {
            bool valid;
            const uint32_t ch = child(fa, k0, na, valid);
            under(keep(1, ch, valid, f1, 0));
          }
        } else {
          // A level outgrew its buffer (nothing is queued yet): depth first,
          // the children of one node a step, those still to visit as bits of
          // one word, 8 per level, so that the walk needs no stack.
          int cur = 0, level = top;
          uint64_t pend = 0;
          for (;;) {
            const int cl = level - 1;
            const uint32_t ch = (uint32_t)cur * (uint32_t)kFan + (uint32_t)(lane & 7);
            if (cl == 0) {
              leaves(ch, lane < 8);
            } else {
              const bool valid = lane < 8 && ch < (uint32_t)cnt_of(cl);
              const uint32_t node = (uint32_t)off_of(cl) + (valid ? ch : 0u);
              const uint64_t m = __ballot(valid && near(S.ncen[node], S.nhw[node]));
              pend |= m << (8 * cl);
            }
            if (pend == 0ull) break;
            const int b = __builtin_ctzll(pend);  // the deepest; its parent is an ancestor of cur
            pend &= pend - 1;
            const int nl = b >> 3;
            cur = ((cur >> (3 * (nl + 1 - level))) << 3) + (b & 7);
            level = nl;
          }
        }
      }
      drain(0);
#pragma unroll
      for (int k = 0; k < M; ++k) np = lane == g0 + k ? cnt[k] : np;
    };
    auto walks = [&](auto wrap_t) {
      const float w2 = W0[0] * W0[0] + W0[1] * W0[1] + W0[2] * W0[2];
      if ((todo & (todo - 1)) != 0ull && w2 <= kReach * kReach * rm0 * rm0) {
        walk(wrap_t, std::integral_constant<int, kSet>(), 0, C0, W0, rm0);
      } else {
        for (uint64_t left = todo; left != 0ull; left &= left - 1) {
          const int g = __builtin_ctzll(left);
          const float C[3] = {lane_f(P[0], g), lane_f(P[1], g), lane_f(P[2], g)};
          const float W[3] = {0.f, 0.f, 0.f};
          walk(wrap_t, std::integral_constant<int, 1>(), g, C, W, lane_f(rp, g));
        }
      }
    };
    if (wrap)
      walks(std::true_type());
    else
      walks(std::false_type());
    // every passed index fitted the particle's room: they are its candidates
    if (mine) {
      if (np > cap && S.shrink && S.rad[S.n + s] == R(0)) {
        const double want = 1.3 * 4.18879020478639098 * S.n_h3;
        const double f = fmax(cbrt(want / (double)np), 0.5);
        S.rad[s] = (R)((double)ri * f);
        const int ns = (int)(1.3 * (double)np * f * f * f) + 1;
        S.need[s] = ((ns > 4 ? ns : 4) + 3) & ~3;
        S.ccnt[s] = -1;
        retry = true;
      } else if (np > cap) {
        S.need[s] = (np + 3) & ~3;
        S.ccnt[s] = -1;
        retry = true;
      } else if (!STAGE) {
        S.ccnt[s] = np;
        S.cpos[s] = (uint32_t)(base >> 2);
        kept = (unsigned long long)np;
      }
    }
  }
  if constexpr (STAGE) {
    // the block's kept candidates go to the pool in one piece: each
    // particle's count rounded up to 4 entries, their sum taken from the
    // bump counter
    const bool fits = mine && np <= cap;
    const int c4 = fits ? (np + 3) & ~3 : 0;
    if (lane < kSet) rcnt[w * kSet + lane] = (uint32_t)c4;
    __syncthreads();
    constexpr int kAll = kWaves * kSet;
    static_assert(kAll == 16, "a row of lanes sums the block's counts");
    if (threadIdx.x < kAll) {
      const uint32_t own = rcnt[lane];
      uint32_t upto = own;
#pragma unroll
      for (int o = 1; o < kAll; o <<= 1) {
        const uint32_t v = __shfl_up(upto, o, kAll);
        if (lane >= o) upto += v;
      }
      unsigned long long b = 0;
      if (lane == kAll - 1 && upto)
        b = atomicAdd(S.cnt + CNT_POOL, (unsigned long long)upto);
      b = __shfl(b, kAll - 1, kAll);
      rbase[lane] = b + (upto - own);
    }
    __syncthreads();
    bool in = false;
    if (fits) {
      const unsigned long long b = rbase[w * kSet + lane];
      in = b + (unsigned long long)c4 <= (unsigned long long)S.pool_cap;
      if (in) {
        S.ccnt[s] = np;
        S.cpos[s] = (uint32_t)(b >> 2);
        kept = (unsigned long long)np;
      } else {
        // the pool is full: the next round gives the particle room of its own
        S.need[s] = (np + 3) & ~3;
        S.ccnt[s] = -1;
        retry = true;
      }
    }
    for (uint64_t left = __ballot(in); left != 0ull; left &= left - 1) {
      const int k = __builtin_ctzll(left);
      const int m4 = __builtin_amdgcn_readlane(c4, k);
      if (4 * lane < m4)
        *reinterpret_cast<uint4*>(S.cand + rbase[w * kSet + k] + 4 * lane) =
            stage4[w * kSet + k][lane];
    }
  }
  // (the lanes past the set's hold zero)
  static_assert(kSet == 4, "a quad of lanes");
  kept += __shfl_xor(kept, 1, 64);
  kept += __shfl_xor(kept, 2, 64);
  if (lane == 0 && kept) atomicAdd(cnt_at(S.cnt, CNT_CANDIDATES), kept);
  wave_count(cnt_at(S.cnt, CNT_RETRY), retry);
}

// The room every unsolved particle gets in a retry round, in 4-entry units
// (zero for the solved ones; need4[n] = 0 closes the exclusive sums). Their sum
// goes to CNT_NEED4 in 64 bits: the 32-bit prefix sums wrap where it needs more,
// and the host refuses such a pool by it.
template <class R>
__global__ void __launch_bounds__(kBlock) k_need4(State<R> S, uint32_t* __restrict__ need4,
                                                  bool retry) {
  const int64_t s = particle_id();
  uint32_t v = 0u;
  if (s < S.n) {
    v = S.todo[s] ? (uint32_t)(room_for(S.need[s], retry) >> 2) : 0u;
    need4[s] = v;
  }
  if (s == 0) need4[S.n] = 0u;
  wave_add_u64(cnt_at(S.cnt, CNT_NEED4), (unsigned long long)v);
}

// The unsolved particles in rank order.
template <class R>
__global__ void __launch_bounds__(kBlock) k_rank_order(State<R> S, uint32_t* __restrict__ order) {
  const int64_t s = particle_id();
  if (s < S.n && S.todo[s]) order[S.cslot[s]] = (uint32_t)s;
}

// Neighbour lists from the stored candidates of every particle (the
// candidates hold every j with r_ij below the particle's radius, which is at
// least its solved h): the gather list (r_ij < h_i, in candidate order, which
// is ascending j) and the scatter-only list, the j that gather i but are not
// gathered by it (h_i <= r_ij < h_j). Where r_ij lies below i's radius, j is
// among i's candidates and i finds it there; where it does not, j puts itself
// on i's list with an atomic. The separation is recomputed as the candidate
// walk computed it; from the other side it is the exact negation (lattice
// offsets and differences negate exactly), so that both sides decide alike.
//    k_filter_tree decides, counts (the gather lengths, the entries found by
// i itself in own[i], those of others in ns[i]) and leaves the decisions in the
// free low bits of the candidate's entry; with per-wave capacities from those
// counts k_fill_tree writes the entries from the bits alone, the others' from
// own[i] on (unordered; sorted afterwards). At 16.8M particles with 1.9G
// candidates and 172M scatter-only entries, when all of these were appended
// by the other side and both passes read three words of each candidate, the
// two took 9.2 and 15.9 ms; now 8.3, bound by gathered addresses (x with the
// lattice cell in its w, and h_j: about one a cycle and CU), and 5.1.
//    A 16-lane row per particle: the row takes 16 candidates at a time, one per
// lane, several such groups a step (the filter eight, four in FP64; the fill six),
// so that most rows take one step or two and nothing waits for its stores. The fill collects the gather entries in LDS and writes whole
// 16-byte chunks of the list.
constexpr uint32_t kGathered = 1u, kTold = 2u, kFound = 4u;  // bits of a candidate's entry

template <class R>
__global__ void __launch_bounds__(kBlock) k_filter_tree(State<R> S, int* __restrict__ own) {
  constexpr int kStep = sizeof(R) == 4 ? 8 : 4;  // groups a step
  const int64_t s = particle_id() >> 4;
  const int sub = threadIdx.x & 15;
  if (s >= S.n) return;  // the whole row
  const int cnt = S.ccnt[s];  // uniform over the row
  const int64_t base = 4 * (int64_t)S.cpos[s];
  const R h = S.hbuf[s], rad = S.rad[s];
  const R4<R> pi = S.pos(s);
  int ng = 0, nf = 0;  // of this lane
  // (lanes past the count take entry 0 of the row, whose record they load and
  // discard: the row has an entry whenever the loop runs)
  for (int k = 0; k < cnt; k += 16 * kStep) {
    uint32_t ent[kStep];
    R4<R> pj[kStep];
    R hj[kStep];
#pragma unroll
    for (int t = 0; t < kStep; ++t) {
      const int e = k + 16 * t + sub;
      ent[t] = S.cand[base + (e < cnt ? e : 0)];
    }
#pragma unroll
    for (int t = 0; t < kStep; ++t) {
      pj[t] = S.pos(ent[t] >> kCodeBits);
      hj[t] = S.hbuf[ent[t] >> kCodeBits];
    }
    // the decisions, and the radius of those that may not find this particle
#pragma unroll
    for (int t = 0; t < kStep; ++t) {
      const bool in = k + 16 * t + sub < cnt;
      const R r = lattice_r(S, pi, pj[t]);
      const bool g = in && r < h, back = r < hj[t];
      const bool found = in && !g && back && r < rad;
      ent[t] |= g ? kGathered : (found ? kFound : 0u);
      ng += g ? 1 : 0;
      nf += found ? 1 : 0;
      hj[t] = R(3e38);
      if (g && !back) hj[t] = S.rad[ent[t] >> kCodeBits];
      pj[t].x = r;
    }
#pragma unroll
    for (int t = 0; t < kStep; ++t) {
      const int e = k + 16 * t + sub;
      if (!(pj[t].x < hj[t])) {  // told to j
        ent[t] |= kTold;
        atomicAdd(&S.ns[ent[t] >> kCodeBits], 1);
      }
      if (e < cnt) S.cand[base + e] = ent[t];
    }
  }
  ng = row_total(ng);
  nf = row_total(nf);
  if (sub == 0) {
    S.ng[s] = ng;
    own[s] = nf;
  }
}

template <class R>
__global__ void __launch_bounds__(kBlock) k_fill_tree(State<R> S, int* __restrict__ fillc) {
  constexpr int kStep = 6;
  __shared__ uint4 buf4[kBlock / 16][4 * kStep + 1];  // 3 entries left over and the new ones
  const int64_t s = particle_id() >> 4;
  const int lane = threadIdx.x & 63, sub = lane & 15;
  uint4* const chunk = buf4[threadIdx.x >> 4];
  uint32_t* const buf = reinterpret_cast<uint32_t*>(chunk);
  const uint32_t below = (1u << sub) - 1u;
  const bool on = s < S.n;  // uniform over the row
  const int64_t sc = on ? s : 0;
  const int cnt = on ? S.ccnt[sc] : 0;
  const int64_t base = 4 * (int64_t)S.cpos[sc];
  const int64_t gb = slot_base(S.grow[sc >> 6], sc), sb = slot_base(S.srow[sc >> 6], sc);
  int ng = 0, wait = 0, nf = 0;  // entries written, waiting in buf, found
  auto place = [&](bool f, int& n) {  // this lane's entry among the row's
    const uint32_t b = (uint32_t)(__ballot(f) >> (lane & 48)) & 0xFFFFu;
    const int at = n + __popc(b & below);
    n += __popc(b);
    return at;
  };
  auto wave_sync = [&]() {  // the wave's LDS writes before its reads, and the reverse
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  for (int k = 0; k < cnt; k += 16 * kStep) {
    uint32_t ent[kStep];
    int u[kStep];
    uint32_t s0[kStep], s1[kStep];
#pragma unroll
    for (int t = 0; t < kStep; ++t) {
      const int e = k + 16 * t + sub;
      ent[t] = e < cnt ? S.cand[base + e] : 0u;
    }
    // the entries told to others: their places all asked for at once
#pragma unroll
    for (int t = 0; t < kStep; ++t)
      if (ent[t] & kTold) {
        const uint32_t j = ent[t] >> kCodeBits;
        u[t] = atomicAdd(&fillc[j], 1);
        s0[t] = S.srow[j >> 6];
        s1[t] = S.srow[(j >> 6) + 1];
      }
#pragma unroll
    for (int t = 0; t < kStep; ++t) {
      const uint32_t e = ent[t] & ~(uint32_t)kCodeMask;
      const bool g = (ent[t] & kGathered) != 0u, f = (ent[t] & kFound) != 0u;
      const int ag = place(g, wait), af = place(f, nf);
      if (g) buf[ag] = e;
      if (f) S.slist[slot_at(sb, af)] = e;
    }
    wave_sync();
    const int full = wait >> 2;  // at most 4 kStep chunks
    for (int c = sub; c < full; c += 16)
      *reinterpret_cast<uint4*>(S.nlist + slot_at(gb, ng + 4 * c)) = chunk[c];
    const uint32_t rest = buf[4 * full + (sub & 3)];
    wave_sync();
    ng += 4 * full;
    wait -= 4 * full;
    if (sub < wait) buf[sub] = rest;
#pragma unroll
    for (int t = 0; t < kStep; ++t)
      if ((ent[t] & kTold) && u[t] < (int)(s1[t] - s0[t]) * 4)
        S.slist[slot_at(slot_base(s0[t], ent[t] >> kCodeBits), u[t])] = (uint32_t)s << kCodeBits;
  }
  wave_sync();
  if (sub == 0 && wait > 0) *reinterpret_cast<uint4*>(S.nlist + slot_at(gb, ng)) = chunk[0];
}

// Per-wave capacity in chunk rows from per-particle counts: the largest of
// its lanes' counts, rounded up to 4 entries. own (or null): the particles' own
// share, added to cnt.
__global__ void __launch_bounds__(kBlock) k_wave_rows(int* __restrict__ cnt,
                                                      const int* __restrict__ own, int64_t n,
                                                      uint32_t* __restrict__ rows) {
  const int64_t s = particle_id();
  if ((s & ~(int64_t)63) >= n) return;
  int c = s < n ? cnt[s] : 0;
  if (own && s < n) {
    c += own[s];
    cnt[s] = c;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c = max(c, __shfl_xor(c, o, 64));
  if ((threadIdx.x & 63) == 0) rows[s >> 6] = (uint32_t)((c + 3) >> 2);
}

// Ascending bitonic sorting network over N values held in registers (every
// index is a compile-time constant once the loops unroll).
template <int N>
__device__ inline void bitonic_sort(uint32_t (&a)[N]) {
#pragma unroll
  for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int l = i ^ j;
        if (l > i) {
          const uint32_t lo = min(a[i], a[l]), hi = max(a[i], a[l]);
          a[i] = (i & k) == 0 ? lo : hi;
          a[l] = (i & k) == 0 ? hi : lo;
        }
      }
    }
  }
}

// One lane's list of ns <= N entries, read as 16-byte chunks, padded with
// 0xffffffff, sorted in registers and written back chunk by chunk.
template <int N>
__device__ inline void sort_list_regs(uint32_t* __restrict__ list, int64_t sb, int ns) {
  uint32_t a[N];
#pragma unroll
  for (int c = 0; c < N / 4; ++c) {
    uint4 q = make_uint4(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu);
    if (4 * c < ns) q = *reinterpret_cast<const uint4*>(list + slot_at(sb, 4 * c));
    a[4 * c] = 4 * c < ns ? q.x : 0xffffffffu;
    a[4 * c + 1] = 4 * c + 1 < ns ? q.y : 0xffffffffu;
    a[4 * c + 2] = 4 * c + 2 < ns ? q.z : 0xffffffffu;
    a[4 * c + 3] = 4 * c + 3 < ns ? q.w : 0xffffffffu;
  }
  bitonic_sort<N>(a);
#pragma unroll
  for (int c = 0; c < N / 4; ++c)
    if (4 * c < ns)
      *reinterpret_cast<uint4*>(list + slot_at(sb, 4 * c)) =
          make_uint4(a[4 * c], a[4 * c + 1], a[4 * c + 2], a[4 * c + 3]);
}

// Sorts every scatter-only list by j, giving the order a walk would produce
// and making runs reproducible; counts the force pairs. Lists of at most 32
// entries are sorted in their lane's registers (a network of the wave's size
// class); longer ones are queued (queue[], their number in the slot 0 of
// CNT_LONG_LISTS) for k_sort_long.
constexpr int kShortList = 32;
template <class R>
__global__ void __launch_bounds__(kBlock) k_scatter_sort(State<R> S, uint32_t* __restrict__ queue) {
  const int64_t s = particle_id();
  if ((s & ~(int64_t)63) >= S.n) return;
  unsigned long long f = 0, g = 0;
  int ns = 0;
  int64_t sb = 0;
  if (s < S.n) {
    const int64_t w = s >> 6;
    const int scap = (int)(S.srow[w + 1] - S.srow[w]) * 4;
    ns = S.ns[s] < scap ? S.ns[s] : scap;
    sb = slot_base(S.srow[w], s);
    g = (unsigned long long)S.ng[s];
    f = g + (unsigned long long)S.ns[s];
  }
  if (ns > kShortList) {
    queue[atomicAdd(S.cnt + CNT_LONG_LISTS, 1ull)] = (uint32_t)s;
    ns = 0;
  }
  int big = ns;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) big = max(big, __shfl_xor(big, o, 64));
  if (big > 16) {
    sort_list_regs<32>(S.slist, sb, ns);
  } else if (big > 8) {
    sort_list_regs<16>(S.slist, sb, ns);
  } else if (big > 1) {
    sort_list_regs<8>(S.slist, sb, ns);
  }
  wave_add_u64(cnt_at(S.cnt, CNT_PAIRS_GATHER), g);
  wave_add_u64(cnt_at(S.cnt, CNT_PAIRS_FORCE), f);
}

// The queued long scatter-only lists, one per single-wave block in turn: up
// to kLongSort entries are padded to a power of two with 0xffffffff and
// sorted by a bitonic network in LDS (each compare-exchange owned by the lane
// of its lower index, a barrier between steps); a longer list takes an
// insertion sort in memory by one lane.
constexpr int kLongSort = 4096;
template <class R>
__global__ void __launch_bounds__(64) k_sort_long(State<R> S, const uint32_t* __restrict__ queue) {
  __shared__ uint32_t buf[kLongSort];
  const unsigned long long nq = S.cnt[CNT_LONG_LISTS];
  const int lane = threadIdx.x;
  for (unsigned long long q = blockIdx.x; q < nq; q += gridDim.x) {
    const int64_t s = queue[q];
    const int64_t w = s >> 6;
    const int scap = (int)(S.srow[w + 1] - S.srow[w]) * 4;
    const int ns = S.ns[s] < scap ? S.ns[s] : scap;
    const int64_t sb = slot_base(S.srow[w], s);
    if (ns > kLongSort) {
      if (lane == 0) {
        for (int a = 1; a < ns; ++a) {
          const uint32_t v = S.slist[slot_at(sb, a)];
          int b = a - 1;
          while (b >= 0 && S.slist[slot_at(sb, b)] > v) {
            S.slist[slot_at(sb, b + 1)] = S.slist[slot_at(sb, b)];
            --b;
          }
          S.slist[slot_at(sb, b + 1)] = v;
        }
      }
      continue;
    }
    int P = 64;
    while (P < ns) P <<= 1;
    for (int k = lane; k < P; k += 64) buf[k] = k < ns ? S.slist[slot_at(sb, k)] : 0xffffffffu;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = lane; i < P; i += 64) {
          const int l = i ^ j;
          if (l > i) {
            const uint32_t a = buf[i], b = buf[l];
            if ((a > b) == ((i & k) == 0)) {
              buf[i] = b;
              buf[l] = a;
            }
          }
        }
        __syncthreads();
      }
    }
    for (int k = lane; k < ns; k += 64) S.slist[slot_at(sb, k)] = buf[k];
    __syncthreads();  // the reads above before the next list's writes
  }
}

}  // namespace

void launch_morton(const double* x, int64_t n, double box, uint32_t* keys, uint32_t* vals,
                   hipStream_t s) {
  hipLaunchKernelGGL(k_morton, dim3(grid_for(n)), dim3(kBlock), 0, s, x, n, box, keys, vals);
}

template <class R>
void launch_tree_build(const State<R>& S, const R* h, float4* absp, const int* host_off,
                       const int* host_cnt, hipStream_t s) {
  hipLaunchKernelGGL(k_leaf_boxes<R>, dim3(grid_for(host_cnt[0])), dim3(kBlock), 0, s, S, h,
                     absp);
  for (int l = 0; l + 1 < S.nlevels; ++l)
    hipLaunchKernelGGL(k_tree_up, dim3(grid_for(host_cnt[l + 1])), dim3(kBlock), 0, s, S.ncen,
                       S.nhw, host_off[l], host_cnt[l], host_off[l + 1], host_cnt[l + 1]);
  const int nnode = host_off[S.nlevels - 1] + host_cnt[S.nlevels - 1];
  hipLaunchKernelGGL(k_box_centres, dim3(grid_for(nnode)), dim3(kBlock), 0, s, S.ncen, S.nhw,
                     nnode);
}

template <class R>
void launch_init_radius(const State<R>& S, int h_mode, hipStream_t s) {
  hipLaunchKernelGGL(k_init_radius<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, h_mode);
}

template <class R>
void launch_rank_order(const State<R>& S, uint32_t* order, hipStream_t s) {
  hipLaunchKernelGGL(k_rank_order<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, order);
}

template <class R>
void launch_candidates_tree(const State<R>& S, const float4* absp, bool stage,
                            const uint32_t* order, int64_t nt, hipStream_t s) {
  if (nt <= 0) return;
  // particles per wave; a block has four waves
  const int per = nt <= kAloneMax ? 1 : kSet;
  const dim3 g(grid_for(nt, 4 * per)), b(kBlock);
  if (stage)
    hipLaunchKernelGGL((k_candidates_tree<R, true>), g, b, 0, s, S, absp, order, nt, per);
  else
    hipLaunchKernelGGL((k_candidates_tree<R, false>), g, b, 0, s, S, absp, order, nt, per);
}

bool stage_fits(int scr_cap) { return scr_cap <= kStage; }

template <class R>
void launch_hsolve_tree(const State<R>& S, int kernel, const uint32_t* order, int64_t nt,
                        hipStream_t s) {
  if (nt <= 0) return;
  const dim3 g(grid_for(16 * nt)), b(kBlock);  // a 16-lane row per particle
  if (S.equal_mass) {
    if (kernel == 0)
      hipLaunchKernelGGL((k_hsolve_rows<R, 0, true>), g, b, 0, s, S, order, nt);
    else
      hipLaunchKernelGGL((k_hsolve_rows<R, 1, true>), g, b, 0, s, S, order, nt);
  } else {
    if (kernel == 0)
      hipLaunchKernelGGL((k_hsolve_rows<R, 0, false>), g, b, 0, s, S, order, nt);
    else
      hipLaunchKernelGGL((k_hsolve_rows<R, 1, false>), g, b, 0, s, S, order, nt);
  }
}

template <class R>
void launch_need4(const State<R>& S, uint32_t* need4, bool retry, hipStream_t s) {
  hipLaunchKernelGGL(k_need4<R>, dim3(grid_for(S.n + 1)), dim3(kBlock), 0, s, S, need4, retry);
}

template <class R>
void launch_filter_tree(const State<R>& S, int* own, hipStream_t s) {
  hipLaunchKernelGGL(k_filter_tree<R>, dim3(grid_for(16 * S.n)), dim3(kBlock), 0, s, S, own);
}

template <class R>
void launch_fill_tree(const State<R>& S, int* fillc, uint32_t* queue, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_tree<R>, dim3(grid_for(16 * S.n)), dim3(kBlock), 0, s, S, fillc);
  hipLaunchKernelGGL(k_scatter_sort<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, queue);
  // ten blocks a CU, as many as the LDS holds (1024 in all: 1.35 ms at 16.8M clumped
  // particles, now 1.08)
  hipLaunchKernelGGL(k_sort_long<R>, dim3(2560), dim3(64), 0, s, S, (const uint32_t*)queue);
}

void launch_wave_rows(int* cnt, const int* own, int64_t n, uint32_t* rows, hipStream_t s) {
  hipLaunchKernelGGL(k_wave_rows, dim3(grid_for(n)), dim3(kBlock), 0, s, cnt, own, n, rows);
}

#define CRK_INSTANTIATE_TREE(R)                                                               \
  template void launch_tree_build<R>(const State<R>&, const R*, float4*, const int*, const int*,      \
                                     hipStream_t);                                           \
  template void launch_init_radius<R>(const State<R>&, int, hipStream_t);                    \
  template void launch_rank_order<R>(const State<R>&, uint32_t*, hipStream_t);              \
  template void launch_candidates_tree<R>(const State<R>&, const float4*, bool,              \
                                          const uint32_t*, int64_t, hipStream_t);            \
  template void launch_hsolve_tree<R>(const State<R>&, int, const uint32_t*, int64_t,       \
                                      hipStream_t);                                          \
  template void launch_need4<R>(const State<R>&, uint32_t*, bool, hipStream_t);               \
  template void launch_filter_tree<R>(const State<R>&, int*, hipStream_t);                   \
  template void launch_fill_tree<R>(const State<R>&, int*, uint32_t*, hipStream_t);

CRK_INSTANTIATE_TREE(float)
CRK_INSTANTIATE_TREE(double)

}  // namespace crk
