// Forward CRKSPH pair passes on gfx950.
//
// Particles are taken in cell order, so that the lanes of a wave share almost
// all of their neighbours and the neighbour records stay in the L2. A cell-sorted
// particle has 16 lanes in the candidate walk; 4 lanes in the moment, density and
// force passes (the force pass 16 for small sets); one lane, or 16 for small sets,
// in the h solve, volume and list passes; 16 everywhere in a hierarchy substep
// with few active particles. Pair arithmetic is in Real (FP32 or FP64); the 3x3
// second-moment solve and the force / energy accumulators are FP64.
//
// Passes (paper: arXiv:2511.21921):
//   k_hsolve   smoothing length from the Thacker fixed point Delta_N = 1
//              (App. A.3, eq. thacker) and the volume of App. A.2, eq. Vg;
//   k_volume   the volume alone for fixed h;
//   k_nlist    symmetric neighbour list r_ij < max(h_i, h_j);
//   k_moments  geometric moments and the corrections A, B, grad A, grad B of
//              W^R_ij = A_i (1 + B_i . x_ij) W_ij(h_i) (App. A.1, eq. RK);
//   k_density  density (Sec. 2.5.1, eq. rhow), velocity gradient
//              (App. A.1, eq. gradv), ideal-gas EOS and the relaxation flag
//              exp(|div v| dt) > 8 (App. A.1);
//   k_force    pairwise momentum and compatible energy with the limited
//              artificial viscosity (Sec. 2.1).
#include "crk_pairs.h"
#include "crk_passes.h"

namespace crk {
namespace {

template <class R>
__device__ inline R dot3(const R a[3], const R b[3]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// ------------------------------------------------------------- inputs ----

// Grid-stride over the inputs; each block reduces in LDS and issues one
// atomic per counter (per-wave atomics on four shared addresses serialise).
template <class R>
__global__ void __launch_bounds__(kBlock) k_check_inputs(const double* __restrict__ x,
                                                         const R* __restrict__ h,
                                                         const R* __restrict__ m,
                                                         const R* __restrict__ u, int64_t n,
                                                         unsigned long long* cnt) {
  unsigned long long hb = 0, bad = 0, mb = 0, ib = 0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock) {
    const double hv = (double)h[i], mv = (double)m[i], uv = (double)u[i];
    const double x0 = fabs(x[i]), x1 = fabs(x[n + i]), x2 = fabs(x[2 * n + i]);
    const bool ok = hv > 0.0 && mv > 0.0 && uv > 0.0 && hv < 1e300 && uv < 1e300 && mv < 1e300 &&
                    x0 < 1e300 && x1 < 1e300 && x2 < 1e300;
    bad += ok ? 0 : 1;
    if (ok) {
      const unsigned long long a = dbits(hv), b = dbits(mv), c = dbits(1.0 / mv);
      hb = a > hb ? a : hb;  // positive doubles order as their bit patterns
      mb = b > mb ? b : mb;
      ib = c > ib ? c : ib;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    bad += __shfl_xor(bad, o, 64);
    unsigned long long t = __shfl_xor(hb, o, 64);
    hb = t > hb ? t : hb;
    t = __shfl_xor(mb, o, 64);
    mb = t > mb ? t : mb;
    t = __shfl_xor(ib, o, 64);
    ib = t > ib ? t : ib;
  }
  __shared__ unsigned long long part[kBlock / 64][4];
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    part[w][0] = hb;
    part[w][1] = bad;
    part[w][2] = mb;
    part[w][3] = ib;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kBlock / 64; ++k) {
      hb = part[k][0] > hb ? part[k][0] : hb;
      bad += part[k][1];
      mb = part[k][2] > mb ? part[k][2] : mb;
      ib = part[k][3] > ib ? part[k][3] : ib;
    }
    if (hb) atomicMax(cnt_at(cnt, CNT_HMAX_BITS), hb);
    if (bad) atomicAdd(cnt_at(cnt, CNT_BAD_INPUT), bad);
    if (mb) atomicMax(cnt_at(cnt, CNT_MMAX_BITS), mb);
    if (ib) atomicMax(cnt_at(cnt, CNT_MINVMAX_BITS), ib);
  }
}

__global__ void __launch_bounds__(kBlock) k_keys(const double* __restrict__ x, int64_t n,
                                                 double L, int G, uint32_t* __restrict__ keys,
                                                 uint32_t* __restrict__ vals) {
  const int64_t i = particle_id();
  if (i >= n) return;
  const double inv = (double)G / L;
  int c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    c[a] = cell_coord(wrap_pos(x[a * n + i], L), inv, G);
  }
  keys[i] = ((uint32_t)c[2] * G + (uint32_t)c[1]) * G + (uint32_t)c[0];
  vals[i] = (uint32_t)i;
}

// The kept cell list against new positions: every sorted slot s recomputes
// the cell of its particle perm[s] and counts it in CNT_MOVED when that
// differs from keys[s] (the list then no longer sorts these positions).
__global__ void __launch_bounds__(kBlock) k_keys_check(const double* __restrict__ x, int64_t n,
                                                       double L, int G,
                                                       const uint32_t* __restrict__ keys,
                                                       const uint32_t* __restrict__ perm,
                                                       unsigned long long* __restrict__ cnt) {
  const int64_t s = particle_id();
  if ((s & ~(int64_t)63) >= n) return;
  unsigned long long moved = 0;
  if (s < n) {
    const double inv = (double)G / L;
    const uint32_t p = perm[s];
    if (p < (uint32_t)n) {
      int c[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) c[a] = cell_coord(wrap_pos(x[a * n + p], L), inv, G);
      moved = ((uint32_t)c[2] * G + (uint32_t)c[1]) * G + (uint32_t)c[0] != keys[s] ? 1ull : 0ull;
    } else {
      moved = 1;  // not a permutation of these particles
    }
  }
  wave_add_u64(cnt_at(cnt, CNT_MOVED), moved);
}

// Hierarchy: the particles (caller order) active at the end of substep jend,
// counted in CNT_ACTIVE.
__global__ void __launch_bounds__(kBlock) k_count_active(const int* __restrict__ levels,
                                                         int64_t n, int lmax, int64_t jend,
                                                         unsigned long long* __restrict__ cnt) {
  const int64_t p = particle_id();
  if ((p & ~(int64_t)63) >= n) return;
  unsigned long long a = 0;
  if (p < n) a = (jend & ((1ll << (lmax - levels[p])) - 1)) == 0 ? 1ull : 0ull;
  wave_add_u64(cnt_at(cnt, CNT_ACTIVE), a);
}

// The sorted slots of the active particles, appended to list (a wave's at
// once; the order is not kept).
template <class R>
__global__ void __launch_bounds__(kBlock) k_active_list(State<R> S, uint32_t* __restrict__ list) {
  const int64_t s = particle_id();
  if ((s & ~(int64_t)63) >= S.n) return;
  const bool a = s < S.n && !is_passive(S, s);
  const uint64_t b = __ballot(a);
  if (b == 0ull) return;
  const int lane = threadIdx.x & 63;
  unsigned long long base = 0;
  if (lane == __ffsll((unsigned long long)b) - 1)
    base = atomicAdd(S.cnt + CNT_ACTLIST, (unsigned long long)__popcll(b));
  base = __shfl(base, __ffsll((unsigned long long)b) - 1, 64);
  if (a) list[base + __popcll(b & ((1ull << lane) - 1ull))] = (uint32_t)s;
}

// cell_start[c] = first sorted position whose key is >= c, for c = 0..ncell
// (searches of the sorted keys; no atomics). The largest
// occupancy start[c + 1] - start[c] is reduced per block into one atomic;
// a block whose largest occupancy exceeds occ_limit raises CNT_TOO_DENSE.
// What bounds it is the chain of dependent loads: two waves of a block search
// for its first and last cell with 64 probes a step, and each thread for its
// own between the two (a search per cell over all keys: 10.8 us at 64^3).
__global__ void __launch_bounds__(kBlock) k_cell_bounds(const uint32_t* __restrict__ keys,
                                                        int64_t n, int64_t ncell,
                                                        uint32_t* __restrict__ start,
                                                        unsigned long long occ_limit,
                                                        unsigned long long* __restrict__ cnt) {
  __shared__ int64_t ends[2];
  __shared__ uint32_t first[kBlock + 1];
  const int64_t c0 = (int64_t)blockIdx.x * kBlock, c = c0 + threadIdx.x;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (w < 2) {
    const int64_t v = w == 0 ? c0 : c0 + kBlock;
    int64_t lo = 0, hi = n;  // keys[lo - 1] < v <= keys[hi]
    while (lo < hi) {
      const int64_t step = (hi - lo + 63) >> 6;
      const int64_t at = lo + lane * step;
      const int below = __popcll(__ballot(at < hi && (int64_t)keys[at < hi ? at : lo] < v));
      const int64_t end = lo + below * step;
      hi = end < hi ? end : hi;
      lo = below > 0 ? lo + (below - 1) * step + 1 : hi;
    }
    if (lane == 0) ends[w] = lo;
  }
  __syncthreads();
  int64_t lo = ends[0], hi = ends[1];
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)keys[mid] < c) lo = mid + 1; else hi = mid;
  }
  first[threadIdx.x] = (uint32_t)lo;
  if (threadIdx.x == 0) first[kBlock] = (uint32_t)ends[1];
  if (c <= ncell) start[c] = (uint32_t)lo;
  __syncthreads();
  unsigned long long occ = 0;
  if (c < ncell) occ = (unsigned long long)(first[threadIdx.x + 1] - (uint32_t)lo);
  __shared__ unsigned long long red[kBlock / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long t = __shfl_xor(occ, o, 64);
    occ = t > occ ? t : occ;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = occ;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long m = 0;
    for (int w = 0; w < kBlock / 64; ++w) m = red[w] > m ? red[w] : m;
    if (m) atomicMax(cnt_at(cnt, CNT_CELL_MAX), m);
    if (m > occ_limit) cnt[CNT_TOO_DENSE] = 1ull;
  }
}

template <class R>
__global__ void __launch_bounds__(kBlock) k_gather(State<R> S, const double* __restrict__ x,
                                                   const R* __restrict__ v,
                                                   const R* __restrict__ m,
                                                   const R* __restrict__ u,
                                                   const R* __restrict__ h) {
  const int64_t s = particle_id();
  if (s >= S.n) return;
  const int64_t n = S.n;
  const uint32_t p = S.perm[s];
  if (p >= (uint32_t)n) return;
  int c[3];
  R xi[3];
  const double inv = (double)S.G / S.box;
  // the cell list's own cell of the slot (on a kept list the particle may
  // have left it: its offset from that cell's centre is then beyond half a
  // side, but the walk stays consistent with the list)
  const uint32_t key = S.lattice ? 0u : S.keys[s];
  const uint32_t G = (uint32_t)S.G;
  const uint32_t kz = key / (G * G);
  const int kc[3] = {(int)(key % G), (int)((key / G) % G), (int)(kz < G ? kz : G - 1)};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double t = wrap_pos(x[a * n + p], S.box);
    c[a] = S.lattice ? cell_coord(t, inv, S.G) : kc[a];
    xi[a] = (R)(t - ((double)c[a] + 0.5) * S.ell_d);
  }
  R4<R> q;
  q.x = xi[0];
  q.y = xi[1];
  q.z = xi[2];
  // the cell's x index (tree path: the lattice cell) until 1/h takes its place
  const uint32_t c3 = (uint32_t)c[0] | ((uint32_t)c[1] << 10) | ((uint32_t)c[2] << 20);
  q.w = S.lattice ? cell_to_real(c3, R()) : R(c[0]);
  S.pos(s) = q;
  R4<R> w;
  w.x = v[p];
  w.y = v[n + p];
  w.z = v[2 * n + p];
  w.w = R(0);
  S.vel(s) = w;
  if (S.inv) S.inv[p] = (uint32_t)s;
  S.mass[s] = m[p];
  S.uu[s] = u[p];
  S.hbuf[s] = h[p];
  S.cell3[s] = c3;
}

// The row of a pair pass: sorted slot s of the lanes' particle, and whether
// there is one to sum. HIER: a substep of the timestep hierarchy, where only
// the active particles are (all of them in place, or a list of few).
template <class R, int L, bool HIER>
__device__ inline bool pair_row(const State<R>& S, int64_t row, int64_t& s) {
  if (HIER && S.act) {
    const bool on = row < (int64_t)S.cnt[CNT_ACTLIST];
    s = on ? (int64_t)S.act[row] : 0;
    return on;
  }
  const bool on = row < S.n;
  s = on ? row : 0;
  return on && !(HIER && is_passive(S, s));
}

// ---------------------------------------------------------- candidates ----
// One traversal of the stencil cells per particle collects every j != i
// with r_ij < rcap (rcap >= every h, at most two cell sides), storing the
// packed entry and (r, m_j / m_i). The h solve, the fixed-h volume and the
// neighbour list all read this list instead of walking the cells again.
// EM: all masses equal (m_j / m_i = 1 is not stored).
//    A row of 16 lanes per particle. Of its 5x5x5 cells those within reach form,
// in each of the 25 cell rows, one run of dx (the distance to a cell is convex
// in dx), and consecutive cells of a row hold consecutive particles: a
// contiguous range of particles, split where the row wraps. The lanes first
// find these runs (a lane a cell row) and number the particles of all of them
// through; then they test the numbers 32 at a time, whatever runs these fall
// in, and append the accepted ones in order. A number's run is the count of
// run starts up to it, from a bit per number (a search of the starts where there
// are more than 2048). A particle's cell within the run comes from the x index
// kept in its position record's w.
//    What bounds it is instructions and the latency of the particles' loads. A
// thread that walked the runs of its own particle, four particles at a time,
// took 25,000 instructions a wave, as its lanes' runs never ended together:
// FP32, ~64 neighbours, 322 us at 262,144 particles against 163 now, 1203 against
// 680 at 1,048,576 (FP64 491 against 254 and 1809 against 1087); 16 lanes that
// walked the runs in turn, 41 us at 4096 against 16, 185 against 90 at 131,072;
// with ~268 neighbours (Wendland C4 at n_h = 4) 756 against 612 at 262,144.
template <class R, bool EM>
__global__ void __launch_bounds__(kBlock) k_candidates(State<R> S) {
  constexpr int kRuns = 75, kWords = 64;
  struct Runs {
    // a run's first number; its first particle less that; bytes: stencil code of
    // dx = 0, dy + 2, dz + 2; x offset (a float)
    uint4 run[kRuns + 1];
    uint32_t start[kWords];  // bit f: a run starts at number f
  };
  __shared__ Runs runs[kBlock / 16];
  const int lane = threadIdx.x & 63, sub = lane & 15;
  const uint64_t rowbits = 0xFFFFull << (lane & 48);
  const uint64_t below = rowbits & ((1ull << lane) - 1ull);
  const int64_t r = particle_id() >> 4;
  int64_t s;
  const bool on = pair_row<R, 16, true>(S, r, s);  // uniform over the row
  // A speculative cell list found too dense (strong clustering): the host discards
  // this evaluation, so the quadratic walk is left out. The count is set all the
  // same: the later passes run, and the entries that an older count stands for
  // may hold the workspace of an adjoint by now.
  if (!on || S.cnt[CNT_TOO_DENSE] != 0ull) {
    if (sub == 0 && (on || (!S.act && r < S.n))) S.ccnt[s] = 0;
    return;
  }
  Runs& T = runs[threadIdx.x >> 4];
  const R4<R> pi = S.pos(s);
  const R mi_inv = EM ? R(1) : R(1) / S.mass[s];
  const R rc2 = S.rcap * S.rcap;
  int cap;
  const int64_t base = scratch_base(S, s, cap);
  const uint32_t c3 = S.cell3[s];
  const int G = S.G;
  const int cx = (int)(c3 & 1023u), cy = (int)((c3 >> 10) & 1023u), cz = (int)(c3 >> 20);
  const R ell = S.ell;
  const uint32_t n = (uint32_t)S.n;
  auto wave_sync = [&]() {  // the wave's LDS writes before its reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto upto = [](uint32_t v) {  // sum over the row's lanes up to this one
    v += dpp_mov<0x111>(v);
    v += dpp_mov<0x112>(v);
    v += dpp_mov<0x114>(v);
    v += dpp_mov<0x118>(v);
    return v;
  };
  auto gap2 = [&](R xi, int d) {
    const R lo = (R(d) - R(0.5)) * ell - xi, hi = xi - (R(d) + R(0.5)) * ell;
    const R g = lo > hi ? lo : hi;
    return g > R(0) ? g * g : R(0);
  };
#pragma unroll
  for (int w = sub; w < kWords; w += 16) T.start[w] = 0u;
  wave_sync();
  uint32_t total = 0, nrun = 0;  // uniform over the row
  for (int q0 = 0; q0 < 25; q0 += 16) {
    const int q = q0 + sub, dz = q / 5 - 2, dy = q % 5 - 2;
    uint32_t b[3] = {0u, 0u, 0u}, len[3] = {0u, 0u, 0u};
    int xoff[3] = {0, 0, 0};
    const R gz = gap2(pi.z, dz), gyz = gz + gap2(pi.y, dy);
    if (q < 25 && gz < rc2 && gyz < rc2) {
      const int z = wrap_cell(cz + dz, G), y = wrap_cell(cy + dy, G);
      const uint32_t rowbase = ((uint32_t)z * G + (uint32_t)y) * G;
      int dlo = 3, dhi = -3;
#pragma unroll
      for (int dx = -2; dx <= 2; ++dx)
        if (gyz + gap2(pi.x, dx) < rc2) {
          dlo = dx < dlo ? dx : dlo;
          dhi = dx;
        }
      // cells dx = d0 .. d1 of the row, stored from x index x0 on
      auto piece = [&](int k, int x0, int d0, int d1) {
        if (d0 > d1) return;
        b[k] = S.cell_start[rowbase + (uint32_t)x0];
        uint32_t e = S.cell_start[rowbase + (uint32_t)(x0 + d1 - d0 + 1)];
        if (e > n) e = n;
        len[k] = e > b[k] ? e - b[k] : 0u;
        xoff[k] = d0 - x0;
      };
      // the run split where the row wraps (G >= 2): x < 0, 0 <= x < G, x >= G
      const int b0 = max(dlo, -cx), c0 = max(dlo, G - cx);
      piece(0, cx + dlo + G, dlo, min(dhi, -cx - 1));
      piece(1, cx + b0, b0, min(dhi, G - 1 - cx));
      piece(2, cx + c0 - G, c0, dhi);
    }
    const uint32_t all = len[0] + len[1] + len[2];
    const uint32_t has = (len[0] ? 1u : 0u) + (len[1] ? 1u : 0u) + (len[2] ? 1u : 0u);
    const uint32_t al = upto(all), hs = upto(has);
    uint32_t o = total + al - all, at = nrun + hs - has;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (len[k]) {
        T.run[at] = make_uint4(o, b[k] - o,
                               (uint32_t)(dz + 2) << 16 | (uint32_t)(dy + 2) << 8 |
                                   stencil_code(0, dy, dz),
                               __float_as_uint((float)xoff[k]));
        if (o < 32u * kWords) atomicOr(&T.start[o >> 5], 1u << (o & 31u));
        o += len[k];
        ++at;
      }
    total += dpp_mov<0x15F>(al);  // lane 15's
    nrun += dpp_mov<0x15F>(hs);
  }
  wave_sync();
  int cnt = 0;         // uniform over the row
  uint32_t before = 0;  // runs that start before the word
  for (uint32_t f0 = 0; f0 < total; f0 += 32) {
    const uint32_t word = f0 < 32u * kWords ? T.start[f0 >> 5] : 0u;
    uint32_t j[2];
    uint4 run[2];
    R4<R> pj[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t f = min(f0 + 16u * u + (uint32_t)sub, total - 1u);
      uint32_t id;
      if (total <= 32u * kWords) {
        id = before + (uint32_t)__popc(word & ((2u << (f & 31u)) - 1u)) - 1u;
      } else {
        uint32_t lo = 0, hi = nrun;  // off[lo] <= f < off[hi]
        while (hi - lo > 1u) {
          const uint32_t mid = (lo + hi) >> 1;
          if (T.run[mid].x <= f) lo = mid; else hi = mid;
        }
        id = lo;
      }
      run[u] = T.run[id];
      j[u] = run[u].y + f;
      pj[u] = S.pos(j[u]);
    }
    before += (uint32_t)__popc(word);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t f = f0 + 16u * u + (uint32_t)sub;
      // (small whole numbers of cells: their products with ell are exact)
      const R dx = pj[u].w + R(__uint_as_float(run[u].w));
      R x[3];
      x[0] = (pi.x - pj[u].x) - dx * ell;
      x[1] = (pi.y - pj[u].y) - Sc<R>::fma(R(run[u].z >> 8 & 255u), ell, R(-2) * ell);
      x[2] = (pi.z - pj[u].z) - Sc<R>::fma(R(run[u].z >> 16), ell, R(-2) * ell);
      const R r2 = test_norm2(x, f - run[u].x);
      const int code = (int)(run[u].z & 255u) + (int)dx;
      const bool ok = f < total && r2 < rc2 && !(j[u] == (uint32_t)s && code == kSelfCode);
      const uint64_t bm = __ballot(ok) & rowbits;
      const int at = cnt + __popcll(bm & below);
      if (ok && at < cap) {
        const int64_t q = group_at(base, at);
        S.cand[q] = (j[u] << kCodeBits) | (uint32_t)code;
        S.scr_r[q] = Sc<R>::sqrt(r2);
        if (!EM) S.scr_m[q] = S.mass[j[u]] * mi_inv;
      }
      cnt += __popcll(bm);
    }
  }
  if (sub == 0) {
    S.ccnt[s] = cnt < cap ? cnt : cap;
    if (cnt > cap) atomicMax(cnt_at(S.cnt, CNT_SCR_OVERFLOW), (unsigned long long)cnt);
  }
}

// A listed substep's passive particles have no candidates.
template <class R>
__global__ void __launch_bounds__(kBlock) k_no_candidates(State<R> S) {
  const int64_t s = particle_id();
  if (s < S.n && is_passive(S, s)) S.ccnt[s] = 0;
}

// sum_k (m_k/m_i) w(r_k / h) over the candidates plus the self term w(0), and
// dsum = sum_k (m_k/m_i) w'(q_k) q_k. The list is read a 16-entry group at a
// time, its loads issued together.
template <class R, int K>
__device__ inline R candidate_sum(const State<R>& S, int64_t base, int cnt, R h, R& dsum) {
  const R hinv = R(1) / h;
  R sum = R(Shape<K>::w0), ds = R(0);
  for (int k = 0; k < cnt; k += 16) {
    const int64_t e = group_at(base, k);
    R rr[16], mm[16];
    load_group(S.scr_r + e, rr);
    if (!S.equal_mass) load_group(S.scr_m + e, mm);
    const int left = cnt - k;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      // entries past the count are moved outside the support (w = w' = 0)
      const bool in = t < left;
      const R q = in ? rr[t] * hinv : R(2);
      R w, dw;
      Shape<K>::eval(q, w, dw);
      const R mt = S.equal_mass ? R(1) : (in ? mm[t] : R(0));
      sum += mt * w;
      ds += mt * dw * q;
    }
  }
  dsum = ds;
  return sum;
}

// ------------------------------------------------------------- h solve ----
// f(h) = C (w(0) + sum_{j != i} (m_j/m_i) w(r_ij / h)) - n_h^3, which is
// h^3 sum_j (m_j/m_i) W(r_ij, h) - n_h^3: zero exactly when Delta_N = 1.
// f is non-decreasing in h; safeguarded Newton inside a bisection bracket,
// stopping when a Newton step falls below the tolerance.

// The solve of particle s from sums(h, dsum), the candidate sums; write: this
// lane stores the results and counts.
template <class R, int K, class F>
__device__ inline void hsolve_steps(const State<R>& S, int64_t s, int cnt, F&& sums, bool write,
                                    unsigned long long& iters, unsigned long long& unconv,
                                    unsigned long long& capped, unsigned long long& hbits) {
  const R C = R(Shape<K>::C);
  const R n_h3 = R(S.n_h3);
  const R Rcap = S.rcap;
  const R rtol = R(S.rtol);
  R h = first_h(S.hbuf[s], Rcap, cnt, S.n_h3);
  R dsum, sum = sums(h, dsum);
  R f = C * sum - n_h3;
  // the bracket [0, Rcap] holds the root only if f(Rcap) > 0; that needs
  // its own pass, taken only when the starting h is below the root
  bool cap_hit = false;
  if (!(f > R(0))) {
    R ds2;
    cap_hit = !(C * sums(Rcap, ds2) - n_h3 > R(0));
  }
  if (cap_hit) {
    if (write) capped = 1;  // the root lies beyond the candidate radius
    return;
  }
  R lo = R(0), hi = Rcap;
  bool conv = false;
  int it = 0;
  R hn = h;
  for (;;) {
    const R fp = -C * dsum / h;
    if (f > R(0)) hi = h; else lo = h;
    hn = R(0.5) * (lo + hi);
    if (fp > R(0)) {
      const R nt = h - f / fp;
      const R step = nt > h ? nt - h : h - nt;
      if (step <= rtol * h) {
        hn = nt < lo ? lo : (nt > hi ? hi : nt);
        conv = true;
        break;
      }
      if (nt > lo && nt < hi) hn = nt;
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
  // V at the final h from the last sums: the step is below the
  // tolerance, so the first-order term leaves an error of order rtol^2
  // (an unconverged h gets its own pass)
  const R sum_f = conv ? sum - dsum / h * (hn - h) : sums(hn, dsum);
  if (write) {
    iters = (unsigned long long)(it + 1);
    unconv = conv ? 0 : 1;
    S.hbuf[s] = hn;
    S.Vbuf[s] = hn * hn * hn / (C * sum_f);
    hbits = dbits((double)hn);
  }
}

// Cell path: a thread per particle (the tree path solves with k_hsolve_rows,
// small sets with k_hsolve_small).
template <class R, int K>
__global__ void __launch_bounds__(kBlock) k_hsolve(State<R> S) {
  const int64_t s = particle_id();
  unsigned long long iters = 0, unconv = 0, capped = 0, hbits = 0;
  if (s < S.n) {
    int scap;
    const int64_t q = scratch_base(S, s, scap);
    const int cnt = S.ccnt[s] < scap ? S.ccnt[s] : scap;
    hsolve_steps<R, K>(
        S, s, cnt, [&](R h, R& dsum) { return candidate_sum<R, K>(S, q, cnt, h, dsum); }, true,
        iters, unconv, capped, hbits);
  }
  wave_max_u64(cnt_at(S.cnt, CNT_H_ITER_MAX), iters);
  wave_add_u64(cnt_at(S.cnt, CNT_H_UNCONV), unconv);
  wave_add_u64(cnt_at(S.cnt, CNT_H_CAPPED), capped);
  wave_max_u64(cnt_at(S.cnt, CNT_HMAX_OUT_BITS), hbits);
}

// Fixed h: V_i = m_i / sum_j m_j W(r_ij, h_i), self term included.
template <class R, int K>
__global__ void __launch_bounds__(kBlock) k_volume(State<R> S) {
  const int64_t s = particle_id();
  if (s >= S.n) return;
  if (is_passive(S, s)) return;  // V comes from the stored state (k_pack)
  const R h = S.hbuf[s];
  int scap;
  const int64_t base = scratch_base(S, s, scap);
  R dsum;
  const R sum = candidate_sum<R, K>(S, base, S.ccnt[s] < scap ? S.ccnt[s] : scap, h, dsum);
  S.Vbuf[s] = h * h * h / (R(Shape<K>::C) * sum);
}

template <class R>
__global__ void __launch_bounds__(kBlock) k_pack(State<R> S, R* __restrict__ h_out,
                                                 R* __restrict__ V_out) {
  const int64_t s = particle_id();
  if (s >= S.n) return;
  const uint32_t p = S.perm[s];
  const bool pas = is_passive(S, s);
  const R h = S.hbuf[s], V = pas ? S.pV[p] : S.Vbuf[s];
  S.pos(s).w = R(1) / h;
  S.vel(s).w = V;
  if (!h_out || pas) return;  // an input still (a speculative forward), or stored
  h_out[p] = h;
  V_out[p] = V;
}

// --------------------------------------------------------- neighbour list --
// A pair is classified by its distance r: j is on i's gather list where
// r < h_i, on its scatter-only list where h_i <= r < h_j, that is where i is on j's
// gather list. Both sides have to decide alike, and the candidates' r may differ
// between them by a few roundings (test_norm2): where it lies that close to the
// h it is compared with, r is taken anew with one contraction from both sides
// (the separation negates exactly). Three roundings of x.x and one of the root
// on either side are below 8 units in the last place. In FP32 with 64 neighbours
// one particle in 500 has such a pair. (The look costs 3 us of 114 at 262,144
// particles, 13 of 494 at ~268 neighbours. Appending a group with such a pair one
// entry at a time instead took 20 and 13 us more: 98 registers for 85.)
template <class R> struct EdgeTol { static constexpr R v = R(8.0 * 2.220446049250313e-16); };
template <> struct EdgeTol<float> { static constexpr float v = 8.0f * 1.1920929e-7f; };
template <class R>
__device__ inline bool at_edge(R r, R h) {
  return fabs(r - h) <= EdgeTol<R>::v * h;
}
template <class R>
__device__ inline R edge_r(const State<R>& S, int64_t s, uint32_t e) {
  R x[3];
  pair_sep<R>(S.pos(s), S.pos(e >> kCodeBits), e & kCodeMask, S.ell, x);
  return Sc<R>::sqrt(norm2(x));
}

template <class R>
__global__ void __launch_bounds__(kBlock) k_nlist(State<R> S) {
  const int64_t s = particle_id();
  unsigned long long g = 0, f = 0, ovf = 0, sovf = 0, cands = 0;
  // (a listed active particle: k_nlist_rows)
  if (s < S.n && !(S.act && !is_passive(S, s))) {
    const R hi = S.hbuf[s];
    int ng = 0, ns = 0;
    const int cap = S.list_cap, scap = S.slist_cap;
    Stage4<uint32_t> sg, ss;
    int ccap;
    const int64_t base = scratch_base(S, s, ccap);
    // passive particles keep no lists (their force is not summed)
    const int cc = is_passive(S, s) ? 0 : (S.ccnt[s] < ccap ? S.ccnt[s] : ccap);
    cands = (unsigned long long)cc;
    auto append = [&](uint32_t e, bool gather, bool scatter) {
      if (gather) {
        if (ng < cap) {
          sg.put(ng & 3, e);
          if ((ng & 3) == 3) sg.flush(S.nlist, s, cap, ng);
        }
        ++ng;
        if (S.needed) S.needed[e >> kCodeBits] = 1;
      } else if (scatter) {
        if (ns < scap) {
          ss.put(ns & 3, e);
          if ((ns & 3) == 3) ss.flush(S.slist, s, scap, ns);
        }
        ++ns;
        if (S.needed) S.needed[e >> kCodeBits] = 1;
      }
    };
    for (int k = 0; k < cc; k += 16) {
      const int64_t c = group_at(base, k);
      uint32_t ee[16];
      R rr[16], hj[16];
      load_group(S.cand + c, ee);
      load_group(S.scr_r + c, rr);
      // h_j only where the pair is not a gather pair of i, all loads at once
#pragma unroll
      for (int t = 0; t < 16; ++t)
        hj[t] = (k + t < cc && !(rr[t] < hi)) ? S.hbuf[ee[t] >> kCodeBits] : R(0);
      uint32_t edge = 0u;
#pragma unroll
      for (int t = 0; t < 16; ++t)
        edge |= at_edge(rr[t], hi) | at_edge(rr[t], hj[t]) ? 1u << t : 0u;
      uint32_t mg = 0u, ms = 0u;  // gather, scatter-only
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const bool in = k + t < cc;
        mg |= in && rr[t] < hi ? 1u << t : 0u;
        ms |= in && rr[t] < hj[t] ? 1u << t : 0u;
      }
      while (edge) {  // (rare)
        const int t = __builtin_ctz(edge);
        edge &= edge - 1u;
        if (k + t >= cc) break;
        const uint32_t e = S.cand[c + t];
        const R r = edge_r(S, s, e);
        mg = (mg & ~(1u << t)) | (r < hi ? 1u << t : 0u);
        ms = (ms & ~(1u << t)) | (r < S.hbuf[e >> kCodeBits] ? 1u << t : 0u);
      }
#pragma unroll
      for (int t = 0; t < 16; ++t) append(ee[t], mg >> t & 1u, ms >> t & 1u);
    }
    const int gst = ng < cap ? ng : cap, sst = ns < scap ? ns : scap;
    if (gst & 3) sg.flush(S.nlist, s, cap, gst - 1);
    if (sst & 3) ss.flush(S.slist, s, scap, sst - 1);
    S.ng[s] = ng;
    S.ns[s] = ns;
    g = (unsigned long long)ng;
    f = (unsigned long long)(ng + ns);
    if (ng > cap) ovf = (unsigned long long)ng;
    if (ns > scap) sovf = (unsigned long long)ns;
  }
  wave_add_u64(cnt_at(S.cnt, CNT_PAIRS_GATHER), g);
  wave_add_u64(cnt_at(S.cnt, CNT_PAIRS_FORCE), f);
  wave_add_u64(cnt_at(S.cnt, CNT_CANDIDATES), cands);
  wave_max_u64(cnt_at(S.cnt, CNT_LIST_OVERFLOW), ovf);
  wave_max_u64(cnt_at(S.cnt, CNT_SLIST_OVERFLOW), sovf);
}

// ------------------------------------------------ moments + corrections ----
// Moments over j with r_ij < h_i, self included (V_j, h_i fixed; d_g is
// the derivative with respect to the evaluation point x_i):
//   m0 = sum V W, m1_a = sum V x_a W, m2_ab = sum V x_a x_b W,
//   d_g m0 = sum V d_g W, d_g m1_a = delta_ag m0 + sum V x_a d_g W,
//   d_g m2_ab = delta_ag m1_b + delta_bg m1_a + sum V x_a x_b d_g W.
// Corrections from sum V W^R = 1 and sum V x W^R = 0:
//   B = -m2^-1 m1, A = 1 / (m0 + B.m1),
//   d_g B = -m2^-1 (d_g m1 + d_g m2 B), d_g A = -A^2 (d_g m0 + d_g B.m1 + B.d_g m1).

// Symmetric-pair index of (a, b) in (xx, xy, xz, yy, yz, zz).
__device__ inline constexpr int sym6(int a, int b) {
  return a <= b ? (a == 0 ? b : (a == 1 ? 2 + b : 5)) : (b == 0 ? a : (b == 1 ? 2 + a : 5));
}

// Full moment set (40 values, FP64) from the accumulated sums.
struct Mom64 {
  double m0, m1[3], m2[9], dm0[3], dm1[9], dm2[27];
};

template <class R>
__device__ inline void expand_moments(const Moments<R>& M, Mom64& D) {
  D.m0 = (double)M.m0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    D.m1[a] = (double)M.m1[a];
    D.dm0[a] = (double)M.dm0[a];
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) D.m2[a * 3 + b] = (double)M.m2[sym6(a, b)];
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      D.dm1[g * 3 + a] = (double)M.X1[g * 3 + a] + (a == g ? D.m0 : 0.0);
#pragma unroll
      for (int b = 0; b < 3; ++b)
        D.dm2[(g * 3 + a) * 3 + b] = (double)M.X2[g * 6 + sym6(a, b)] +
                                     (a == g ? D.m1[b] : 0.0) + (b == g ? D.m1[a] : 0.0);
    }
}

struct Corr64 {
  double A, B[3], dA[3], dB[9], inv[9];
  bool singular;
};

template <class R>
__device__ inline void solve_corrections(const Mom64& D, Corr64& o) {
  const double* m2 = D.m2;
  double cof[9];
  cof[0] = m2[4] * m2[8] - m2[5] * m2[7];
  cof[1] = m2[2] * m2[7] - m2[1] * m2[8];
  cof[2] = m2[1] * m2[5] - m2[2] * m2[4];
  cof[3] = m2[5] * m2[6] - m2[3] * m2[8];
  cof[4] = m2[0] * m2[8] - m2[2] * m2[6];
  cof[5] = m2[2] * m2[3] - m2[0] * m2[5];
  cof[6] = m2[3] * m2[7] - m2[4] * m2[6];
  cof[7] = m2[1] * m2[6] - m2[0] * m2[7];
  cof[8] = m2[0] * m2[4] - m2[1] * m2[3];
  const double det = m2[0] * cof[0] + m2[1] * cof[3] + m2[2] * cof[6];
  const double tr = fabs(m2[0]) + fabs(m2[4]) + fabs(m2[8]);
  o.singular = !(fabs(det) > SingularTol<R>::v * tr * tr * tr);
  if (o.singular) {
    o.A = 1.0;
#pragma unroll
    for (int t = 0; t < 3; ++t) o.B[t] = o.dA[t] = 0.0;
#pragma unroll
    for (int t = 0; t < 9; ++t) o.dB[t] = o.inv[t] = 0.0;
    return;
  }
  const double id = 1.0 / det;
#pragma unroll
  for (int t = 0; t < 9; ++t) o.inv[t] = cof[t] * id;
#pragma unroll
  for (int a = 0; a < 3; ++a)
    o.B[a] = -(o.inv[a * 3 + 0] * D.m1[0] + o.inv[a * 3 + 1] * D.m1[1] + o.inv[a * 3 + 2] * D.m1[2]);
  o.A = 1.0 / (D.m0 + o.B[0] * D.m1[0] + o.B[1] * D.m1[1] + o.B[2] * D.m1[2]);
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    double rhs[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      rhs[b] = D.dm1[g * 3 + b];
#pragma unroll
      for (int e = 0; e < 3; ++e) rhs[b] += D.dm2[(g * 3 + b) * 3 + e] * o.B[e];
    }
    double t = D.dm0[g];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      o.dB[g * 3 + a] = -(o.inv[a * 3 + 0] * rhs[0] + o.inv[a * 3 + 1] * rhs[1] +
                          o.inv[a * 3 + 2] * rhs[2]);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) t += o.dB[g * 3 + a] * D.m1[a] + o.B[a] * D.dm1[g * 3 + a];
    o.dA[g] = -(o.A * o.A) * t;
  }
}

template <class R>
__device__ inline void store_kc(const State<R>& S, int64_t s, const Corr64& c) {
  // packed form: a = A, b = A B, c_g = dA_g + A B_g, M_ga = dA_g B_a + A dB_ga
  R v[16];
  v[0] = (R)c.A;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    v[1 + t] = (R)(c.A * c.B[t]);
    v[4 + t] = (R)(c.dA[t] + c.A * c.B[t]);
  }
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int a = 0; a < 3; ++a) v[7 + g * 3 + a] = (R)(c.dA[g] * c.B[a] + c.A * c.dB[g * 3 + a]);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    R4<R> q;
    q.x = v[4 * t];
    q.y = v[4 * t + 1];
    q.z = v[4 * t + 2];
    q.w = v[4 * t + 3];
    S.kc4[4 * s + t] = q;
  }
}

// Corrections from the sums of particle s: stored (moments when kept,
// packed corrections) and written in caller order; whether the second moment
// was singular.
template <class R>
__device__ inline bool moments_finish(const State<R>& S, int64_t s,
                                                    const Moments<R>& M, CorrOut o) {
  Mom64 D;
  expand_moments(M, D);
  if (S.mom) {
    const int64_t n = S.n;
    S.mom[s] = (R)D.m0;
#pragma unroll
    for (int t = 0; t < 3; ++t) S.mom[(1 + t) * n + s] = M.m1[t];
#pragma unroll
    for (int t = 0; t < 6; ++t) S.mom[(4 + t) * n + s] = M.m2[t];
#pragma unroll
    for (int t = 0; t < 3; ++t) S.mom[(10 + t) * n + s] = M.dm0[t];
#pragma unroll
    for (int t = 0; t < 9; ++t) S.mom[(13 + t) * n + s] = M.X1[t];
#pragma unroll
    for (int t = 0; t < 18; ++t) S.mom[(22 + t) * n + s] = M.X2[t];
  }
  Corr64 c;
  solve_corrections<R>(D, c);
  store_kc(S, s, c);
  if (S.co4) {  // kept in sorted order: k_outputs writes the caller's arrays
    R v[16];
    v[0] = (R)c.A;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      v[1 + t] = (R)c.B[t];
      v[4 + t] = (R)c.dA[t];
    }
#pragma unroll
    for (int t = 0; t < 9; ++t) v[7 + t] = (R)c.dB[t];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      R4<R> q;
      q.x = v[4 * t];
      q.y = v[4 * t + 1];
      q.z = v[4 * t + 2];
      q.w = v[4 * t + 3];
      S.co4[4 * s + t] = q;
    }
  } else {
    const int64_t n = S.n;
    const uint32_t p = S.perm[s];
    R* A = (R*)o.A;
    R* B = (R*)o.B;
    R* gA = (R*)o.gradA;
    R* gB = (R*)o.gradB;
    A[p] = (R)c.A;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      B[t * n + p] = (R)c.B[t];
      gA[t * n + p] = (R)c.dA[t];
    }
#pragma unroll
    for (int t = 0; t < 9; ++t) gB[t * n + p] = (R)c.dB[t];
  }
  return c.singular;
}

// Moment sums with L lanes per particle (262,144 particles FP32 123 -> 106 us, 16.8M
// clustered 12.3 -> 6.6 ms, 4096 particles 46 -> 17 us against a thread each, the
// outputs kept in sorted order included); the block then gathers its particles'
// sums in LDS and solves them with one thread each (the FP64 solve takes about
// as many instructions as four pairs: on one lane of four it would cost the
// wave as much as sixteen).
template <class R, int K, int L, bool HIER>
__global__ void __launch_bounds__(kBlock) k_moments(State<R> S, CorrOut o) {
  __shared__ MomentStage<R, L> sh;
  const int64_t row = particle_id() / L;
  int64_t s;
  const bool on = pair_row<R, L, HIER>(S, row, s);
  moment_sums<R, K, L>(S, s, on, sh);
  // (particle_id() - threadIdx.x is the block's first thread)
  if (threadIdx.x < kBlock / L &&
      pair_row<R, L, HIER>(S, (particle_id() - threadIdx.x) / L + threadIdx.x, s)) {
    Moments<R> M;
    sh.get(threadIdx.x, M);
    wave_count(cnt_at(S.cnt, CNT_SINGULAR), moments_finish<R>(S, s, M, o));
  }
}

// ------------------------------------------------ density, grad v, EOS ----

// The record of grad v, the relaxation flag, the lattice cell and the state.
template <class R>
__device__ inline void store_gs(const State<R>& S, int64_t s, const R gv[9], R relaxed, R rho, R P,
                                R c, R den) {
  R4<R> g0, g1, g2, st;
  g0.x = gv[0]; g0.y = gv[1]; g0.z = gv[2]; g0.w = gv[3];
  g1.x = gv[4]; g1.y = gv[5]; g1.z = gv[6]; g1.w = gv[7];
  g2.x = gv[8]; g2.y = relaxed; g2.z = cell_to_real(S.cell3[s], R()); g2.w = R(0);
  st.x = rho; st.y = P; st.z = c; st.w = den;
  S.gs4[4 * s] = g0;
  S.gs4[4 * s + 1] = g1;
  S.gs4[4 * s + 2] = g2;
  S.gs4[4 * s + 3] = st;
}

// rho, P, c and the relaxation flag from the sums of particle s, stored and
// written in caller order; whether it is relaxed.
template <class R>
__device__ inline bool density_finish(const State<R>& S, int64_t s,
                                                    const R sums[11], R* rho_out,
                                                    R* gradv_out) {
  bool nrel = false;
  {
    const R num = sums[0], den = sums[1];
    R gv[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) gv[t] = sums[2 + t];
    const R rho = num / den;
    const R u = S.uu[s];
    const R gam = R(S.gamma);
    const R P = (gam - R(1)) * rho * u;
    const R c = Sc<R>::sqrt(gam * (gam - R(1)) * u);
    R relaxed = R(0);
    if (S.dt_relax > 0.0) {
      const double div = (double)gv[0] + (double)gv[4] + (double)gv[8];
      // exp(|div v| dt) > 8  <=>  |div v| dt > ln 8
      if (fabs(div) * S.dt_relax > 2.0794415416798357) {
        relaxed = R(1);
        nrel = true;
      }
    }
    store_gs(S, s, gv, relaxed, rho, P, c, den);
    if (!S.co4) {  // (else k_outputs writes the caller's arrays from the record)
      const int64_t n = S.n;
      const uint32_t p = S.perm[s];
      rho_out[p] = rho;
#pragma unroll
      for (int t = 0; t < 9; ++t) gradv_out[t * n + p] = gv[t];
    }
  }
  return nrel;
}

// Num, Den and the nine grad v sums with L lanes per particle; a neighbour's
// position, velocity and volume staged in LDS (262,144 particles FP32 116 -> 95 us,
// 16.8M clustered 12.2 -> 5.6 ms, 4096 particles 38 -> 16 us against a thread each).
template <class R, int K, int L, bool HIER>
__global__ void __launch_bounds__(kBlock) k_density(State<R> S, R* __restrict__ rho_out,
                                                    R* __restrict__ gradv_out) {
  using Pv = Rec<R, 2>;
  __shared__ uint4 stage[kBlock / 64][Pv::kWords];
  const int sub = threadIdx.x & (L - 1);
  int64_t s;
  const bool on = pair_row<R, L, HIER>(S, particle_id() / L, s);
  if (__ballot(on) == 0ull) return;  // the whole wave
  uint4* const wpv = stage[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
  const R4<R> pi = S.pos(s);
  const R4<R> vi = S.vel(s);
  const R mi = S.mass[s];
  const R hinv = pi.w;
  const R C3 = R(Shape<K>::C) * hinv * hinv * hinv;
  const R C4 = C3 * hinv;
  KC<R> ki;
  load_kc4(S, s, ki);
  const uint32_t ci = S.cell3[s];
  // equal FP32 masses are the same number (FP64 ones may differ in the last bit)
  const bool same_mass = sizeof(R) == 4 && S.equal_mass;
  constexpr int N = L == 4 ? 3 : 12;
  R v[N];  // the sums of group g < 3: grad v_g; of group 3: Num, Den
#pragma unroll
  for (int t = 0; t < N; ++t) v[t] = R(0);
  if (sub == (L == 4 ? 3 : 0)) {  // self term: x = 0, W^R_ii = A_i W(0)
    const R W0 = C3 * R(Shape<K>::w0);
    v[N - 3] = mi * vi.w * ki.a * W0;
    v[N - 2] = vi.w * vi.w * ki.a * W0;
  }
  NbrRef nb = nbr_ref(S, s);
  if (!on) nb.ng = 0;
  nb.ns = 0;
  const int total = nb.ng;
  const int most = wave_max_int(total);
  R mn = mi;
  uint32_t cn = 0;
  auto fetch = [&](uint32_t e) {
    const uint32_t j = e >> kCodeBits;
    Pv::load(S.pv, j, wpv);
    if (!same_mass) mn = S.mass[j];
    if (S.lattice) cn = S.cell3[j];
  };
  uint32_t e = entry_or_self(S, nb, s, sub), en = 0;
  if (most > 0) {
    fetch(e);
    en = entry_or_self(S, nb, s, sub + L);
  }
  for (int k = 0; k < most; k += L) {
    wait_loads();
    const R4<R> pj = rec4<2>(wpv, 0, R()), vj = rec4<2>(wpv, 1, R());
    const R mj = mn;
    const uint32_t cj = cn;
    wait_lds();
    const uint32_t ec = e;
    e = en;
    if (k + L < most) {
      fetch(e);
      en = entry_or_self(S, nb, s, k + 2 * L + sub);
    }
    R WR = R(0), gWR[3] = {R(0), R(0), R(0)}, dvV[3] = {R(0), R(0), R(0)}, mV = R(0), VV = R(0);
    if (k + sub < total) {
      R x[3];
      pair_x<R>(S, pi, ci, pj, cj, ec, x);
      const R r2 = norm2(x);
      const R rinv = Sc<R>::rsqrt(r2);
      R w, dw;
      Shape<K>::eval(r2 * rinv * hinv, w, dw);
      const R W = C3 * w;
      const R fg = C4 * dw * rinv;
      const R gW[3] = {fg * x[0], fg * x[1], fg * x[2]};
      kc_apply(ki, x, W, gW, WR, gWR);
      mV = mj * vj.w;
      VV = vj.w * vj.w;
      dvV[0] = vj.w * (vi.x - vj.x);
      dvV[1] = vj.w * (vi.y - vj.y);
      dvV[2] = vj.w * (vi.z - vj.z);
    }
    if constexpr (L == 4) {  // in list order, each lane its group (see moment_sums)
      auto turn = [&](auto lane) {
        constexpr int T = decltype(lane)::value;
        constexpr int B = quad_perm(T, T, T, T);
        const R d0 = dpp_mov<B>(dvV[0]), d1 = dpp_mov<B>(dvV[1]), d2 = dpp_mov<B>(dvV[2]);
        const R wr = dpp_mov<B>(WR);
        const R d = -(sub == 0 ? d0 : (sub == 1 ? d1 : d2));
        const R g0 = dpp_mov<B>(gWR[0]), g1 = dpp_mov<B>(gWR[1]), g2 = dpp_mov<B>(gWR[2]);
        const R m = dpp_mov<B>(mV), q = dpp_mov<B>(VV);
        v[0] = Sc<R>::fma(sub == 3 ? m : d, sub == 3 ? wr : g0, v[0]);
        v[1] = Sc<R>::fma(sub == 3 ? q : d, sub == 3 ? wr : g1, v[1]);
        v[2] = Sc<R>::fma(d, g2, v[2]);  // (of lane 3: not used)
      };
      turn(std::integral_constant<int, 0>());
      turn(std::integral_constant<int, 1>());
      turn(std::integral_constant<int, 2>());
      turn(std::integral_constant<int, 3>());
    } else {
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int g = 0; g < 3; ++g) v[a * 3 + g] = Sc<R>::fma(-dvV[a], gWR[g], v[a * 3 + g]);
      v[9] = Sc<R>::fma(mV, WR, v[9]);
      v[10] = Sc<R>::fma(VV, WR, v[10]);
    }
  }
  R sums[11];  // Num, Den, grad v
  if constexpr (L == 4) {
    auto from = [&](auto lane, int t) {
      constexpr int T = decltype(lane)::value;
      return dpp_mov<quad_perm(T, T, T, T)>(v[t]);
    };
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      sums[2 + t] = from(std::integral_constant<int, 0>(), t);
      sums[5 + t] = from(std::integral_constant<int, 1>(), t);
      sums[8 + t] = from(std::integral_constant<int, 2>(), t);
    }
    sums[0] = from(std::integral_constant<int, 3>(), 0);
    sums[1] = from(std::integral_constant<int, 3>(), 1);
  } else {
#pragma unroll
    for (int t = 0; t < 9; ++t) sums[2 + t] = lane_sum<L>(v[t]);
    sums[0] = lane_sum<L>(v[9]);
    sums[1] = lane_sum<L>(v[10]);
  }
  if (on && sub == 0)
    wave_count(cnt_at(S.cnt, CNT_RELAXED), density_finish<R>(S, s, sums, rho_out, gradv_out));
}

// Hierarchy: the stored state of the passive particles that an active one's
// force pair reads: the corrections of their last evaluation, the carried
// density, grad v of the last evaluation, P and c from that density and u.
template <class R>
__global__ void __launch_bounds__(kBlock) k_passive(State<R> S) {
  const int64_t s = particle_id();
  if (s >= S.n || !is_passive(S, s) || (S.needed && !S.needed[s])) return;
  const int64_t n = S.n;
  const uint32_t p = S.perm[s];
  Corr64 c;
  c.A = (double)S.pA[p];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    c.B[t] = (double)S.pB[t * n + p];
    c.dA[t] = (double)S.pgA[t * n + p];
  }
#pragma unroll
  for (int t = 0; t < 9; ++t) c.dB[t] = (double)S.pgB[t * n + p];
  store_kc(S, s, c);
  const R rho = S.prho[p];
  R gv[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) gv[t] = S.pgv[t * n + p];
  const R u = S.uu[s];
  const R gam = R(S.gamma);
  R relaxed = R(0);
  if (S.dt_relax > 0.0) {
    const double div = (double)gv[0] + (double)gv[4] + (double)gv[8];
    if (fabs(div) * S.dt_relax > 2.0794415416798357) relaxed = R(1);
  }
  store_gs(S, s, gv, relaxed, rho, (gam - R(1)) * rho * u, Sc<R>::sqrt(gam * (gam - R(1)) * u),
           R(0));
}

// ------------------------------------------------------ force and du/dt ----
// For j != i with r_ij < max(h_i, h_j):
//   G_ij = grad_i W^R_ij - grad_j W^R_ji (uncorrected on both sides when
//   either particle is relaxed),
//   limiter phi = clamp(4 n d / (n + d)^2, 0, 1) with n = x.(grad v_i x),
//   d = x.(grad v_j x); midpoint velocity jump
//   v' = (v_i - phi/2 grad v_i x) - (v_j + phi/2 grad v_j x);
//   mu_k = min(0, v'.x h_k / (r^2 + eps2 h_k^2)), Q_k = rho_k (-alpha c_k mu_k + beta mu_k^2);
//   F_ij = -1/2 V_i V_j (P_i + P_j + Q_i + Q_j) G_ij;
//   a_i = sum F_ij / m_i, du_i/dt = -1/(2 m_i) sum (v_i - v_j).F_ij.

template <class R, int K>
__device__ inline void side_grad(const KC<R>& k, const R x[3], R r2, R rinv, R hinv,
                                 R out[3]) {
  const R C3 = R(Shape<K>::C) * hinv * hinv * hinv;
  R w, dw;
  Shape<K>::eval(r2 * rinv * hinv, w, dw);
  const R W = C3 * w;
  const R fg = C3 * hinv * dw * rinv;
  const R gW[3] = {fg * x[0], fg * x[1], fg * x[2]};
  R WR;
  kc_apply(k, x, W, gW, WR, out);
}

// One side of a force pair: position and 1/h, velocity and V, the packed
// corrections, grad v, the relaxation flag, the lattice cell and the state.
template <class R>
struct ForceSide {
  R4<R> p, v, st;
  KC<R> kc;
  R gv[9], relaxed;
  uint32_t cell;
};

// Adds the force pair of particle i with its neighbour j (the record kj of
// which is spent) at separation x to acc and du.
template <class R, int K>
__device__ __forceinline__ void force_term(const ForceSide<R>& I, ForceSide<R>& J, const R x[3],
                                           R hi, bool relax_on, R alpha, R beta, R eps2,
                                           double acc[3], double& du) {
  const R r2 = dot3(x, x);
  const R rinv = Sc<R>::rsqrt(r2);
  KC<R> kiu = I.kc;
  if (relax_on && (I.relaxed != R(0) || J.relaxed != R(0))) {
    kc_plain(kiu);
    kc_plain(J.kc);
  }
  const R4<R>&vi = I.v, &vj = J.v;
  R Gi[3], Gj[3];
  side_grad<R, K>(kiu, x, r2, rinv, I.p.w, Gi);
  const R xm[3] = {-x[0], -x[1], -x[2]};
  side_grad<R, K>(J.kc, xm, r2, rinv, J.p.w, Gj);
  R G[3] = {Gi[0] - Gj[0], Gi[1] - Gj[1], Gi[2] - Gj[2]};
  // limited artificial viscosity
  R gix[3], gjx[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    gix[a] = I.gv[a * 3] * x[0] + I.gv[a * 3 + 1] * x[1] + I.gv[a * 3 + 2] * x[2];
    gjx[a] = J.gv[a * 3] * x[0] + J.gv[a * 3 + 1] * x[1] + J.gv[a * 3 + 2] * x[2];
  }
  const R nn = dot3(x, gix), dd = dot3(x, gjx);
  const R sum = nn + dd;
  const R s2 = sum * sum;
  R phi = R(0);
  if (s2 > R(0)) {
    phi = Sc<R>::div(R(4) * nn * dd, s2);
    phi = phi < R(0) ? R(0) : (phi > R(1) ? R(1) : phi);
  }
  const R hp = R(0.5) * phi;
  const R vp[3] = {(vi.x - vj.x) - hp * (gix[0] + gjx[0]), (vi.y - vj.y) - hp * (gix[1] + gjx[1]),
                   (vi.z - vj.z) - hp * (gix[2] + gjx[2])};
  const R vpx = dot3(vp, x);
  const R hj = Sc<R>::rcp(J.p.w);
  R mui = Sc<R>::div(vpx * hi, r2 + eps2 * hi * hi);
  R muj = Sc<R>::div(vpx * hj, r2 + eps2 * hj * hj);
  mui = mui < R(0) ? mui : R(0);
  muj = muj < R(0) ? muj : R(0);
  const R Qi = I.st.x * (-alpha * I.st.z * mui + beta * mui * mui);
  const R Qj = J.st.x * (-alpha * J.st.z * muj + beta * muj * muj);
  const R sfac = R(-0.5) * vi.w * vj.w * (I.st.y + J.st.y + Qi + Qj);
  const R F[3] = {sfac * G[0], sfac * G[1], sfac * G[2]};
  const R work = (vi.x - vj.x) * F[0] + (vi.y - vj.y) * F[1] + (vi.z - vj.z) * F[2];
  acc[0] += (double)F[0];
  acc[1] += (double)F[1];
  acc[2] += (double)F[2];
  du += (double)work;
}

// The force pass, L lanes per particle with the neighbours' records (160 B in
// FP32) staged in LDS (crk_pairs.h): what bounds it then is instruction issue
// (~275 VALU instructions a pair). Against a thread per particle, FP32: 262,144
// particles 320 -> 173 us (FP64 660 -> 306), the same at ~268 neighbours 1225 ->
// 634, 16.8M clustered 24.0 -> 14.3 ms, 4096 particles 37 -> 8 us. HIER: a substep of the timestep hierarchy (the passive
// particles keep their acceleration: nothing to sum or write, and a list of
// few active particles may stand in for all of them); a separate instance, so
// that the ordinary forward's code is not shaped by the extra branch.
template <class R, int K, int L, bool HIER>
__global__ void __launch_bounds__(kBlock) k_force(State<R> S, double* __restrict__ accel,
                                                  double* __restrict__ dudt) {
  using Pv = Rec<R, 2>;
  using Kc = Rec<R, 4>;
  using Gs = Rec<R, 4>;
  constexpr int kStageWords = Pv::kWords + Kc::kWords + Gs::kWords;
  __shared__ uint4 stage[kBlock / 64][kStageWords];
  const int sub = threadIdx.x & (L - 1);
  int64_t s;
  const bool on = pair_row<R, L, HIER>(S, particle_id() / L, s);
  if (__ballot(on) == 0ull) return;  // the whole wave
  uint4* const wpv = stage[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
  uint4* const wkc = wpv + Pv::kWords;
  uint4* const wgs = wkc + Kc::kWords;
  ForceSide<R> I;
  I.p = S.pos(s);
  I.v = S.vel(s);
  load_kc4(S, s, I.kc);
  load_gs4(S, s, I.gv, I.relaxed, I.st);
  I.cell = S.cell3[s];
  const bool relax_on = S.dt_relax > 0.0;
  const R alpha = R(S.alpha), beta = R(S.beta), eps2 = R(S.eps2);
  const R hi = R(1) / I.p.w;
  double acc[3] = {0.0, 0.0, 0.0}, du = 0.0;
  NbrRef nb = nbr_ref(S, s);
  if (!on) nb.ng = nb.ns = 0;
  const int total = nb.ng + nb.ns;
  const int most = wave_max_int(total);
  auto fetch = [&](uint32_t e) {
    const uint32_t j = e >> kCodeBits;
    Pv::load(S.pv, j, wpv);
    Kc::load(S.kc4, j, wkc);
    Gs::load(S.gs4, j, wgs);
  };
  uint32_t e = entry_or_self(S, nb, s, sub), en = 0;
  if (most > 0) {
    fetch(e);
    en = entry_or_self(S, nb, s, sub + L);
  }
  for (int k = 0; k < most; k += L) {
    wait_loads();
    ForceSide<R> J;
    J.p = rec4<2>(wpv, 0, R());
    J.v = rec4<2>(wpv, 1, R());
    kc_from<R>([&](int t) { return rec4<4>(wkc, t, R()); }, J.kc);
    gs_from<R>([&](int t) { return rec4<4>(wgs, t, R()); }, J.gv, J.relaxed, J.cell, J.st);
    wait_lds();
    const uint32_t ec = e;
    e = en;
    if (k + L < most) {
      fetch(e);
      en = entry_or_self(S, nb, s, k + 2 * L + sub);
    }
    if (k + sub < total) {
      R x[3];
      pair_x<R>(S, I.p, I.cell, J.p, J.cell, ec, x);
      force_term<R, K>(I, J, x, hi, relax_on, alpha, beta, eps2, acc, du);
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) acc[a] = lane_sum<L>(acc[a]);
  du = lane_sum<L>(du);
  if (on && sub == 0) {
    const int64_t n = S.n;
    const double minv = 1.0 / (double)S.mass[s];
    const double out[4] = {acc[0] * minv, acc[1] * minv, acc[2] * minv, -0.5 * du * minv};
    if (S.co4) {
      S.af4[s] = make_double4(out[0], out[1], out[2], out[3]);
    } else {
      const uint32_t p = S.perm[s];
      accel[p] = out[0];
      accel[n + p] = out[1];
      accel[2 * n + p] = out[2];
      dudt[p] = out[3];
    }
  }
}

// ------------------------------------------------------------- outputs ---
// The caller's arrays from the sorted records, a thread per particle of the
// caller: a few whole records fetched from the particle's slot, 38 arrays
// written in order. Written from the passes in sorted order instead, each of
// a particle's 38 words lands in a sector of its own, and at 16.8M particles
// in random order the moment and density passes spent as long on that as on
// their pairs (10.5 and 6.8 GB written for 1.1 and 0.7).
template <class R>
__global__ void __launch_bounds__(kBlock) k_outputs(State<R> S, R* __restrict__ rho, CorrOut o,
                                                    R* __restrict__ gradv,
                                                    double* __restrict__ accel,
                                                    double* __restrict__ dudt) {
  const int64_t p = particle_id(), n = S.n;
  if (p >= n) return;
  const int64_t s = S.inv[p];
  R4<R> c[4], g[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) c[t] = S.co4[4 * s + t];
#pragma unroll
  for (int t = 0; t < 4; ++t) g[t] = S.gs4[4 * s + t];
  const double4 f = S.af4[s];
  R *A = (R*)o.A, *B = (R*)o.B, *gA = (R*)o.gradA, *gB = (R*)o.gradB;
  A[p] = c[0].x;
  B[p] = c[0].y;
  B[n + p] = c[0].z;
  B[2 * n + p] = c[0].w;
  gA[p] = c[1].x;
  gA[n + p] = c[1].y;
  gA[2 * n + p] = c[1].z;
  gB[p] = c[1].w;
#pragma unroll
  for (int t = 2; t < 4; ++t) {
    gB[(4 * t - 7) * n + p] = c[t].x;
    gB[(4 * t - 6) * n + p] = c[t].y;
    gB[(4 * t - 5) * n + p] = c[t].z;
    gB[(4 * t - 4) * n + p] = c[t].w;
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    gradv[4 * t * n + p] = g[t].x;
    gradv[(4 * t + 1) * n + p] = g[t].y;
    gradv[(4 * t + 2) * n + p] = g[t].z;
    gradv[(4 * t + 3) * n + p] = g[t].w;
  }
  gradv[8 * n + p] = g[2].x;
  rho[p] = g[3].x;
  accel[p] = f.x;
  accel[n + p] = f.y;
  accel[2 * n + p] = f.z;
  dudt[p] = f.w;
}

// ------------------------------------------------------------ checks -----

__global__ void __launch_bounds__(kCntSpread) k_clear_counters(unsigned long long* cnt, int c,
                                                                int count) {
  for (int k = c; k < c + count; ++k) cnt[threadIdx.x * kCntStride + k] = 0ull;
}

template <class R>
__global__ void __launch_bounds__(kBlock) k_nonfinite(const R* __restrict__ a, int64_t na,
                                                      unsigned long long* cnt) {
  const int64_t i = particle_id();
  unsigned long long bad = 0;
  if (i < na) {
    const double v = (double)a[i];
    bad = (v - v == 0.0) ? 0 : 1;
  }
  wave_add_u64(cnt_at(cnt, CNT_NONFINITE), bad);
}


// ------------------------------------------------- rows for small sets ----
// With few particles (all of a small set, or the listed active ones of a
// hierarchy substep) a thread each leaves most of the chip idle and every pass
// lasts one lane's serial walk: the h, volume and neighbour-list
// passes give each a 16-lane row instead, with the entry order, the values and
// the order of the sums of the thread kernels, so that either gives the same
// bits.

// The candidate sums of a particle by its row, lane sub taking entry 16 g + sub
// of group g (kept in registers for the first kRowGroups groups) and the row
// adding the 16 terms one after another, lane by lane: the order, and so the
// bits, of candidate_sum.
template <class R, int K, bool EM>
struct RowSums {
  static constexpr int kRowGroups = 12;
  const State<R>& S;
  int64_t base;
  int cnt, sub;
  R r[kRowGroups], m[EM ? 1 : kRowGroups];
  __device__ inline RowSums(const State<R>& S_, int64_t s, int sub_) : S(S_), sub(sub_) {
    int cap;
    base = scratch_base(S, s, cap);
    cnt = S.ccnt[s] < cap ? S.ccnt[s] : cap;
#pragma unroll
    for (int g = 0; g < kRowGroups; ++g) {
      const bool in = 16 * g + sub < cnt;
      const int64_t e = group_at(base, in ? 16 * g + sub : 0);
      r[g] = S.scr_r[e];
      if (!EM) m[g] = S.scr_m[e];
    }
  }
  template <int T>
  __device__ inline void add_from(R w, R t, R q, R mt, R& sum, R& ds) {
    if constexpr (T < 16) {
      constexpr int B = 0x150 + T;  // lane T of the row to all of it
      if constexpr (EM)
        sum += dpp_mov<B>(w);
      else
        sum = Sc<R>::fma(dpp_mov<B>(mt), dpp_mov<B>(w), sum);
      ds = Sc<R>::fma(dpp_mov<B>(q), dpp_mov<B>(t), ds);
      add_from<T + 1>(w, t, q, mt, sum, ds);
    }
  }
  __device__ inline void group(int g, R rr, R mm, R hinv, R& sum, R& ds) {
    const bool in = 16 * g + sub < cnt;
    const R q = in ? rr * hinv : R(2);
    R w, dw;
    Shape<K>::eval(q, w, dw);
    const R mt = EM ? R(1) : (in ? mm : R(0));
    add_from<0>(w, mt * dw, q, mt, sum, ds);
  }
  __device__ inline R operator()(R h, R& dsum) {
    const R hinv = R(1) / h;
    R sum = R(Shape<K>::w0), ds = R(0);
#pragma unroll
    for (int g = 0; g < kRowGroups; ++g)
      if (16 * g < cnt) group(g, r[g], EM ? R(1) : m[EM ? 0 : g], hinv, sum, ds);
    for (int g = kRowGroups; 16 * g < cnt; ++g) {
      const int64_t e = group_at(base, 16 * g + sub < cnt ? 16 * g + sub : 0);
      const R rr = S.scr_r[e];
      const R mm = EM ? R(1) : S.scr_m[e];
      group(g, rr, mm, hinv, sum, ds);
    }
    dsum = ds;
    return sum;
  }
};

// The fixed-h volume of k_volume by a row.
template <class R, int K, bool EM>
__global__ void __launch_bounds__(kBlock) k_volume_rows(State<R> S) {
  int64_t s;
  if (!pair_row<R, 16, true>(S, particle_id() >> 4, s)) return;  // the whole row
  const int sub = threadIdx.x & 15;
  const R h = S.hbuf[s];
  RowSums<R, K, EM> sums(S, s, sub);
  R dsum;
  const R sum = sums(h, dsum);
  if (sub == 0) S.Vbuf[s] = h * h * h / (R(Shape<K>::C) * sum);
}

// The h solve of k_hsolve by a row (every lane of it takes the same steps).
template <class R, int K, bool EM>
__global__ void __launch_bounds__(kBlock) k_hsolve_small(State<R> S) {
  const int64_t s = particle_id() >> 4;
  const int sub = threadIdx.x & 15;
  unsigned long long iters = 0, unconv = 0, capped = 0, hbits = 0;
  if (s < S.n) {
    RowSums<R, K, EM> sums(S, s, sub);
    hsolve_steps<R, K>(S, s, sums.cnt, sums, sub == 0, iters, unconv, capped, hbits);
  }
  wave_max_u64(cnt_at(S.cnt, CNT_H_ITER_MAX), iters);
  wave_add_u64(cnt_at(S.cnt, CNT_H_UNCONV), unconv);
  wave_add_u64(cnt_at(S.cnt, CNT_H_CAPPED), capped);
  wave_max_u64(cnt_at(S.cnt, CNT_HMAX_OUT_BITS), hbits);
}

// The neighbour lists of k_nlist by a row: 16 candidates at a time, the
// gather and scatter-only entries appended in candidate order.
template <class R>
__global__ void __launch_bounds__(kBlock) k_nlist_rows(State<R> S) {
  const int lane = threadIdx.x & 63, sub = lane & 15;
  const uint64_t rowbits = 0xFFFFull << (lane & 48);
  const uint64_t below = rowbits & ((1ull << lane) - 1ull);
  const int64_t r = particle_id() >> 4;
  int64_t s;
  const bool on = pair_row<R, 16, true>(S, r, s);  // uniform over the row
  const R hi = S.hbuf[s];
  int ccap;
  const int64_t base = scratch_base(S, s, ccap);
  const int cc = !on ? 0 : (S.ccnt[s] < ccap ? S.ccnt[s] : ccap);
  const int cap = S.list_cap, scap = S.slist_cap;
  int ng = 0, ns = 0;  // uniform over the row
  for (int k = 0; k < cc; k += 16) {
    const int t = k + sub;
    const bool in = t < cc;
    const int64_t c = group_at(base, in ? t : 0);
    const uint32_t e = S.cand[c];
    R rr = S.scr_r[c];
    if (in && at_edge(rr, hi)) rr = edge_r(S, s, e);
    const bool g = in && rr < hi;
    const R hj = in && !g ? S.hbuf[e >> kCodeBits] : R(0);
    if (in && at_edge(rr, hj)) rr = edge_r(S, s, e);
    const bool sc = in && !g && rr < hj;
    const uint64_t gm = __ballot(g) & rowbits, sm = __ballot(sc) & rowbits;
    if (g) {
      const int at = ng + __popcll(gm & below);
      if (at < cap) S.nlist[list_index(s, cap, at)] = e;
    }
    if (sc) {
      const int at = ns + __popcll(sm & below);
      if (at < scap) S.slist[list_index(s, scap, at)] = e;
    }
    if (S.needed && (g || sc)) S.needed[e >> kCodeBits] = 1;
    ng += __popcll(gm);
    ns += __popcll(sm);
  }
  // (passive particles keep no lists)
  if (sub == 0 && (on || (!S.act && r < S.n))) {
    S.ng[s] = ng;
    S.ns[s] = ns;
  }
  const bool one = sub == 0;
  wave_add_u64(cnt_at(S.cnt, CNT_PAIRS_GATHER), one ? (unsigned long long)ng : 0ull);
  wave_add_u64(cnt_at(S.cnt, CNT_PAIRS_FORCE), one ? (unsigned long long)(ng + ns) : 0ull);
  wave_add_u64(cnt_at(S.cnt, CNT_CANDIDATES), one ? (unsigned long long)cc : 0ull);
  wave_max_u64(cnt_at(S.cnt, CNT_LIST_OVERFLOW), one && ng > cap ? (unsigned long long)ng : 0ull);
  wave_max_u64(cnt_at(S.cnt, CNT_SLIST_OVERFLOW), one && ns > scap ? (unsigned long long)ns : 0ull);
}
}  // namespace

// ----------------------------------------------------------- launchers ----

template <class R>
void launch_check_inputs(const double* x, const R* h, const R* m, const R* u, int64_t n,
                         unsigned long long* cnt, hipStream_t s) {
  const unsigned blocks = grid_for(n) < 1024u ? grid_for(n) : 1024u;
  hipLaunchKernelGGL(k_check_inputs<R>, dim3(blocks > 0 ? blocks : 1), dim3(kBlock), 0, s, x, h,
                     m, u, n, cnt);
}

void launch_keys(const double* x, int64_t n, double box, int G, uint32_t* keys, uint32_t* vals,
                 hipStream_t s) {
  hipLaunchKernelGGL(k_keys, dim3(grid_for(n)), dim3(kBlock), 0, s, x, n, box, G, keys, vals);
}

void launch_keys_check(const double* x, int64_t n, double box, int G, const uint32_t* keys,
                       const uint32_t* perm, unsigned long long* cnt, hipStream_t s) {
  hipLaunchKernelGGL(k_keys_check, dim3(grid_for(n)), dim3(kBlock), 0, s, x, n, box, G, keys,
                     perm, cnt);
}

void launch_clear_counters(unsigned long long* cnt, int c, int count, hipStream_t s) {
  hipLaunchKernelGGL(k_clear_counters, dim3(1), dim3(kCntSpread), 0, s, cnt, c, count);
}

void launch_count_active(const int* levels, int64_t n, int lmax, int64_t jend,
                         unsigned long long* cnt, hipStream_t s) {
  hipLaunchKernelGGL(k_count_active, dim3(grid_for(n)), dim3(kBlock), 0, s, levels, n, lmax, jend,
                     cnt);
}
template <class R>
void launch_active_list(const State<R>& S, uint32_t* list, hipStream_t s) {
  hipLaunchKernelGGL(k_active_list<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, list);
}

void launch_cell_bounds(const uint32_t* keys, int64_t n, int64_t ncell, uint32_t* start,
                        unsigned long long occ_limit, unsigned long long* cnt, hipStream_t s) {
  hipLaunchKernelGGL(k_cell_bounds, dim3((unsigned)((ncell + kBlock) / kBlock)), dim3(kBlock), 0,
                     s, keys, n, ncell, start, occ_limit, cnt);
}

template <class R>
void launch_gather(const State<R>& S, const double* x, const R* v, const R* m, const R* u,
                   const R* h, hipStream_t s) {
  hipLaunchKernelGGL(k_gather<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, x, v, m, u, h);
}

// How many 16-lane rows a search pass takes (0: a thread per particle): the
// listed active particles', or every particle's of a set of at most most.
template <class R>
int64_t search_rows(const State<R>& S, int64_t most) {
  return S.act ? S.nact : (S.n <= most ? S.n : 0);
}
template <class R>
void launch_candidates(const State<R>& S, hipStream_t s) {
  if (S.act) hipLaunchKernelGGL(k_no_candidates<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S);
  const int64_t rows = S.act ? S.nact : S.n;
  if (rows <= 0) return;
  const dim3 rg(grid_for(16 * rows));
  if (S.equal_mass)
    hipLaunchKernelGGL((k_candidates<R, true>), rg, dim3(kBlock), 0, s, S);
  else
    hipLaunchKernelGGL((k_candidates<R, false>), rg, dim3(kBlock), 0, s, S);
}
// KFN<R, kernel, equal masses>
#define CRK_ROWS_KEM(KFN, grid, ...)                                                    \
  do {                                                                                  \
    if (kernel == 0 && S.equal_mass)                                                    \
      hipLaunchKernelGGL((KFN<R, 0, true>), grid, dim3(kBlock), 0, s, __VA_ARGS__);     \
    else if (kernel == 0)                                                               \
      hipLaunchKernelGGL((KFN<R, 0, false>), grid, dim3(kBlock), 0, s, __VA_ARGS__);    \
    else if (S.equal_mass)                                                              \
      hipLaunchKernelGGL((KFN<R, 1, true>), grid, dim3(kBlock), 0, s, __VA_ARGS__);     \
    else                                                                                \
      hipLaunchKernelGGL((KFN<R, 1, false>), grid, dim3(kBlock), 0, s, __VA_ARGS__);    \
  } while (0)
template <class R>
void launch_hsolve(const State<R>& S, int kernel, hipStream_t s) {
  if (S.n == 0) return;
  const dim3 g(grid_for(S.n)), b(kBlock);
  if (S.n <= kRowsMaxSums)
    CRK_ROWS_KEM(k_hsolve_small, dim3(grid_for(16 * S.n)), S);
  else if (kernel == 0)
    hipLaunchKernelGGL((k_hsolve<R, 0>), g, b, 0, s, S);
  else
    hipLaunchKernelGGL((k_hsolve<R, 1>), g, b, 0, s, S);
}
template <class R>
void launch_volume(const State<R>& S, int kernel, hipStream_t s) {
  if (S.n == 0) return;
  const dim3 g(grid_for(S.n)), b(kBlock);
  const int64_t rows = search_rows(S, kRowsMaxSums);
  if (rows > 0)
    CRK_ROWS_KEM(k_volume_rows, dim3(grid_for(16 * rows)), S);
  else if (S.act)
    return;  // no active particle
  else if (kernel == 0)
    hipLaunchKernelGGL((k_volume<R, 0>), g, b, 0, s, S);
  else
    hipLaunchKernelGGL((k_volume<R, 1>), g, b, 0, s, S);
}
template <class R>
void launch_pack(const State<R>& S, R* h_out, R* V_out, hipStream_t s) {
  hipLaunchKernelGGL(k_pack<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, h_out, V_out);
}
template <class R>
void launch_nlist(const State<R>& S, hipStream_t s) {
  const int64_t rows = search_rows(S, kRowsMaxLists);
  const bool small = rows > 0;
  if (!small || S.act)  // (beside a list it clears the passive particles' lists)
    hipLaunchKernelGGL(k_nlist<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S);
  if (small)
    hipLaunchKernelGGL(k_nlist_rows<R>, dim3(grid_for(16 * rows)), dim3(kBlock), 0, s, S);
}
// Instances of a forward pair pass: 4 or 16 lanes per particle (16 always for
// the listed active particles of a hierarchy substep; the moment and density
// sums, taken in list order, have 4 otherwise), with or without levels.
#define CRK_PAIRS_HL(KFN, K, L, H, rows, ...)                                                  \
  hipLaunchKernelGGL((KFN<R, K, L, H>), dim3(grid_for(L * (rows))), dim3(kBlock), 0, s,        \
                     __VA_ARGS__)
#define CRK_PAIRS_K(KFN, K, lanes, ...)                                                        \
  do {                                                                                         \
    if (S.act) {                                                                               \
      if (S.nact > 0) CRK_PAIRS_HL(KFN, K, 16, true, S.nact, __VA_ARGS__);                     \
    } else if (S.levels) {                                                                     \
      if ((lanes) == 16)                                                                       \
        CRK_PAIRS_HL(KFN, K, 16, true, S.n, __VA_ARGS__);                                      \
      else                                                                                     \
        CRK_PAIRS_HL(KFN, K, 4, true, S.n, __VA_ARGS__);                                       \
    } else if ((lanes) == 16) {                                                                \
      CRK_PAIRS_HL(KFN, K, 16, false, S.n, __VA_ARGS__);                                       \
    } else {                                                                                   \
      CRK_PAIRS_HL(KFN, K, 4, false, S.n, __VA_ARGS__);                                        \
    }                                                                                          \
  } while (0)
#define CRK_PAIRS(kernel, KFN, lanes, ...)                                                     \
  do {                                                                                         \
    if ((kernel) == 0)                                                                         \
      CRK_PAIRS_K(KFN, 0, lanes, __VA_ARGS__);                                                 \
    else                                                                                       \
      CRK_PAIRS_K(KFN, 1, lanes, __VA_ARGS__);                                                 \
  } while (0)

template <class R>
void launch_moments(const State<R>& S, int kernel, CorrOut o, hipStream_t s) {
  CRK_PAIRS(kernel, k_moments, 4, S, o);
}
template <class R>
void launch_density(const State<R>& S, int kernel, R* rho_out, R* gradv_out, hipStream_t s) {
  CRK_PAIRS(kernel, k_density, 4, S, rho_out, gradv_out);
}
template <class R>
void launch_force(const State<R>& S, int kernel, double* accel, double* dudt, hipStream_t s) {
  if (S.levels) hipLaunchKernelGGL(k_passive<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S);
  CRK_PAIRS(kernel, k_force, pair_lanes(S.n), S, accel, dudt);
}
template <class R>
void launch_outputs(const State<R>& S, R* rho, CorrOut o, R* gradv, double* accel, double* dudt,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_outputs<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, rho, o, gradv,
                     accel, dudt);
}
template <class R>
void launch_count_nonfinite(const R* a, int64_t na, unsigned long long* cnt, hipStream_t s) {
  hipLaunchKernelGGL(k_nonfinite<R>, dim3(grid_for(na)), dim3(kBlock), 0, s, a, na, cnt);
}
void launch_count_nonfinite_f64(const double* a, int64_t na, unsigned long long* cnt,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_nonfinite<double>, dim3(grid_for(na)), dim3(kBlock), 0, s, a, na, cnt);
}

#define CRK_INSTANTIATE(R)                                                                   \
  template void launch_check_inputs<R>(const double*, const R*, const R*, const R*, int64_t, \
                                       unsigned long long*, hipStream_t);                    \
  template void launch_gather<R>(const State<R>&, const double*, const R*, const R*,         \
                                 const R*, const R*, hipStream_t);                           \
  template void launch_candidates<R>(const State<R>&, hipStream_t);                          \
  template void launch_hsolve<R>(const State<R>&, int, hipStream_t); \
  template void launch_volume<R>(const State<R>&, int, hipStream_t); \
  template void launch_pack<R>(const State<R>&, R*, R*, hipStream_t);                        \
  template void launch_nlist<R>(const State<R>&, hipStream_t);                               \
  template void launch_moments<R>(const State<R>&, int, CorrOut, hipStream_t);               \
  template void launch_density<R>(const State<R>&, int, R*, R*, hipStream_t);                \
  template void launch_force<R>(const State<R>&, int, double*, double*, hipStream_t);        \
  template void launch_outputs<R>(const State<R>&, R*, CorrOut, R*, double*, double*,        \
                                  hipStream_t);                                              \
  template void launch_active_list<R>(const State<R>&, uint32_t*, hipStream_t);              \
  template void launch_count_nonfinite<R>(const R*, int64_t, unsigned long long*, hipStream_t);

CRK_INSTANTIATE(float)
CRK_INSTANTIATE(double)

}  // namespace crk
