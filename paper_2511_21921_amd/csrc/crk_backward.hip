// Adjoint (reverse-mode) CRKSPH passes on gfx950, in gather form.
//
// For the loss L = sum_i gA_i . a_i + sum_i gU_i du_i/dt, each pass gives
// every particle the derivatives of L with respect to its own quantities:
//   k_bwd_force    pairwise momentum/energy with viscosity -> x, v, h, V,
//                  packed corrections, rho, P, c, grad v, alpha, beta;
//                  the EOS adjoint (P, c -> rho, u) closes the kernel;
//   k_bwd_density  density and velocity gradient (own sums and the
//                  particle's share in its neighbours' sums) -> x, v, h, V,
//                  packed corrections;
//   k_bwd_corr     corrections -> the 40 moment sums through the FP64 solve
//                  (moments recomputed, or read when the forward kept them);
//   k_bwd_moments  moments -> x, h, V (own and neighbours' sums), then the
//                  volume / smoothing-length coefficient kappa;
//   k_bwd_volume   V_i = m_i / sum_j m_j W(r_ij, h_i) and, for solved h, the
//                  implicit-function term of the Thacker fixed point
//                  (App. A.3) -> x;
//   k_bwd_finish   caller order and the alpha, beta totals.
// Pair arithmetic in Real; accumulators in FP64, but for the sums of the packed
// corrections' and grad v's adjoints, in Real (one term per pair); no float atomics.
#include "crk_adjoint.h"
#include "crk_pairs.h"
#include "crk_passes.h"

namespace crk {
namespace {

template <class R>
__device__ inline R dot3b(const R a[3], const R b[3]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// One side of a force pair from its records: get_pw, get_kc and get_gs give
// the Real4 of the position / velocity / weight, correction and state records.
template <class R, class FP, class FK, class FG>
__device__ inline void side_from(FP&& get_pw, FK&& get_kc, FG&& get_gs, PairSide<R>& o, R4<R>& p,
                                 R& relaxed, uint32_t& cell) {
  p = get_pw(0);
  const R4<R> v = get_pw(1), w = get_pw(2);
  R4<R> st;
  kc_from<R>(get_kc, o.kc);
  gs_from<R>(get_gs, o.gv, relaxed, cell, st);
  o.hinv = p.w;
  o.h = Sc<R>::rcp(p.w);
  o.V = v.w;
  o.rho = st.x;
  o.P = st.y;
  o.c = st.z;
  o.v[0] = v.x;
  o.v[1] = v.y;
  o.v[2] = v.z;
  o.wam[0] = w.x;
  o.wam[1] = w.y;
  o.wam[2] = w.z;
  o.wum = w.w;
}

// The density adjoint's record of a particle.
template <class R>
struct GvcRec {
  R gvb[9], Numb, Denb, m;
  uint32_t cell;
};
template <class R, class F>
__device__ inline void gvc_from(F&& get, GvcRec<R>& o) {
  const R4<R> q0 = get(0), q1 = get(1), q2 = get(2), q3 = get(3);
  o.gvb[0] = q0.x;
  o.gvb[1] = q0.y;
  o.gvb[2] = q0.z;
  o.gvb[3] = q0.w;
  o.gvb[4] = q1.x;
  o.gvb[5] = q1.y;
  o.gvb[6] = q1.z;
  o.gvb[7] = q1.w;
  o.gvb[8] = q2.x;
  o.Numb = q2.y;
  o.Denb = q2.z;
  o.m = q2.w;
  o.cell = real_to_cell(q3.x);
}

// Loss weights gathered into sorted order, beside the position and velocity.
template <class R>
__global__ void __launch_bounds__(kBlock) k_bwd_prep(State<R> S, AdjState<R> G) {
  const int64_t s = particle_id();
  if (s >= S.n) return;
  const int64_t n = S.n;
  const uint32_t q = S.perm[s];
  // the force adjoint uses the weights only as w_a / m and w_u / (2 m)
  const R m = S.mass[s];
  R4<R> w;
  w.x = (R)G.w_a[q] / m;
  w.y = (R)G.w_a[n + q] / m;
  w.z = (R)G.w_a[2 * n + q] / m;
  w.w = (R)G.w_u[q] / (R(2) * m);
  G.pw4[4 * s] = S.pos(s);
  G.pw4[4 * s + 1] = S.vel(s);
  G.pw4[4 * s + 2] = w;
}

// ------------------------------------------------------------------ B1+B2 --
// L lanes per particle, the neighbours' records (192 B in FP32) staged in LDS
// (crk_pairs.h). Bound by instruction issue (~610 VALU instructions a pair; 256
// VGPRs, two waves per SIMD). Against a thread per particle that gathered its
// records: FP32 262,144 particles 412 -> 334 us (FP64 908 -> 793), 16.8M clustered
// 33.0 -> 22.5 ms, 4096 particles 141 -> 17 us.
template <class R, int K, int L>
__global__ void __launch_bounds__(kAdjBlock<R>) k_bwd_force(State<R> S, AdjState<R> G) {
  constexpr int BLK = kAdjBlock<R>;
  using Pw = Rec<R, 4>;
  using Kc = Rec<R, 4>;
  using Gs = Rec<R, 4>;
  __shared__ uint4 stage[BLK / 64][Pw::kWords + Kc::kWords + Gs::kWords];
  __shared__ double part[BLK / 64][2];
  const int64_t row = particle_id<BLK>() / L;
  const int sub = threadIdx.x & (L - 1);
  const bool on = row < S.n;
  const int64_t s = on ? row : S.n - 1, n = S.n;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint4* const wpw = stage[wave];
  uint4* const wkc = wpw + Pw::kWords;
  uint4* const wgs = wkc + Kc::kWords;
  PairSide<R> I;
  R4<R> pi;
  R reli;
  uint32_t ci;
  side_from<R>([&](int t) { return G.pw4[4 * s + t]; }, [&](int t) { return S.kc4[4 * s + t]; },
               [&](int t) { return S.gs4[4 * s + t]; }, I, pi, reli, ci);
  const bool relax_on = S.dt_relax > 0.0;
  const R alpha = R(S.alpha), beta = R(S.beta), eps2 = R(S.eps2);
  // x, v, h, V and the EOS adjoints accumulate in FP64; the 16 correction
  // and 9 velocity-gradient adjoint sums (one term per pair) in the
  // working precision, like the density adjoint's own correction sums
  ForceBar<double, R> ob;
  ob.zero();
  NbrRef nb = nbr_ref(S, s);
  if (!on) nb.ng = nb.ns = 0;
  const int total = nb.ng + nb.ns;
  const int most = wave_max_int(total);
  auto fetch = [&](uint32_t e) {
    const uint32_t j = e >> kCodeBits;
    Pw::load(G.pw4, j, wpw);
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
    PairSide<R> J;
    R4<R> pj;
    R relj;
    uint32_t cj;
    side_from<R>([&](int t) { return rec4<4>(wpw, t, R()); },
                 [&](int t) { return rec4<4>(wkc, t, R()); },
                 [&](int t) { return rec4<4>(wgs, t, R()); }, J, pj, relj, cj);
    wait_lds();
    const uint32_t ec = e;
    e = en;
    if (k + L < most) {
      fetch(e);
      en = entry_or_self(S, nb, s, k + 2 * L + sub);
    }
    if (k + sub < total) {
      R x[3];
      pair_x<R>(S, pi, ci, pj, cj, ec, x);
      KC<R> ki = I.kc;
      const bool plain = relax_on && (reli != R(0) || relj != R(0));
      if (plain) {
        kc_plain(ki);
        kc_plain(J.kc);
      }
      force_pair_adj<R, double, R, K>(I, ki, J, x, alpha, beta, eps2, !plain, ob);
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    ob.x[a] = lane_sum<L>(ob.x[a]);
    ob.v[a] = lane_sum<L>(ob.v[a]);
    ob.kc.b[a] = lane_sum<L>(ob.kc.b[a]);
    ob.kc.c[a] = lane_sum<L>(ob.kc.c[a]);
  }
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    ob.gv[t] = lane_sum<L>(ob.gv[t]);
    ob.kc.M[t] = lane_sum<L>(ob.kc.M[t]);
  }
  ob.kc.a = lane_sum<L>(ob.kc.a);
  ob.h = lane_sum<L>(ob.h);
  ob.V = lane_sum<L>(ob.V);
  ob.rho = lane_sum<L>(ob.rho);
  ob.P = lane_sum<L>(ob.P);
  ob.c = lane_sum<L>(ob.c);
  if (on && sub == 0) {
    // equation of state: P = (gamma - 1) rho u, c = sqrt(gamma (gamma - 1) u)
    const double gam = S.gamma;
    const double u = (double)S.uu[s];
    const double rhob = ob.rho + ob.P * (gam - 1.0) * u;
    const double ub = ob.P * (gam - 1.0) * (double)I.rho +
                      ob.c * gam * (gam - 1.0) / (2.0 * (double)I.c);
    for (int a = 0; a < 3; ++a) {
      G.gx[a * n + s] = ob.x[a];
      G.gv[a * n + s] = ob.v[a];
    }
    G.gh[s] = ob.h;
    G.gV[s] = ob.V;
    G.gu[s] = ub;
    G.gkc[s] = ob.kc.a;
    for (int t = 0; t < 3; ++t) {
      G.gkc[(1 + t) * n + s] = ob.kc.b[t];
      G.gkc[(4 + t) * n + s] = ob.kc.c[t];
    }
    for (int t = 0; t < 9; ++t) G.gkc[(7 + t) * n + s] = ob.kc.M[t];
    // density adjoint coefficients: rho = Num / Den
    const double den = (double)S.gs4[4 * s + 3].w;
    R4<R> q0, q1, q2, q3;
    q0.x = (R)ob.gv[0]; q0.y = (R)ob.gv[1]; q0.z = (R)ob.gv[2]; q0.w = (R)ob.gv[3];
    q1.x = (R)ob.gv[4]; q1.y = (R)ob.gv[5]; q1.z = (R)ob.gv[6]; q1.w = (R)ob.gv[7];
    q2.x = (R)ob.gv[8];
    q2.y = (R)(rhob / den);                       // Num bar
    q2.z = (R)(-rhob * (double)I.rho / den);      // Den bar
    q2.w = S.mass[s];
    q3.x = cell_to_real(S.cell3[s], R());
    q3.y = q3.z = q3.w = R(0);
    G.gvc4[4 * s] = q0;
    G.gvc4[4 * s + 1] = q1;
    G.gvc4[4 * s + 2] = q2;
    G.gvc4[4 * s + 3] = q3;
  }
  // per-block alpha, beta partial sums (a fixed order: deterministic; lanes
  // without a pair hold zeros)
  const double pa = wave_sum64(ob.alpha), pb = wave_sum64(ob.beta);
  if ((threadIdx.x & 63) == 0) {
    part[wave][0] = pa;
    part[wave][1] = pb;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double t = part[0][threadIdx.x];
    for (int w = 1; w < BLK / 64; ++w) t += part[w][threadIdx.x];
    G.gab[2 * blockIdx.x + threadIdx.x] = t;
  }
}

// --------------------------------------------------------------------- B3 --
// The particle's own sums (gather entries) and its share in the sums of every
// neighbour j with r < h_j, from one fetch of the neighbour's records (two
// passes over the list, to keep registers free, fetched them twice: 387 -> 225 us
// at 262,144 particles in FP32, 744 -> 614 in FP64, 28.5 -> 15.7 ms at 16.8M
// clustered). Three waves per SIMD, bound by instruction issue.
template <class R, int K, int L>
__global__ void __launch_bounds__(kBlock) k_bwd_density(State<R> S, AdjState<R> G) {
  using Pv = Rec<R, 2>;
  using Kc = Rec<R, 4>;
  using Gv = Rec<R, 4>;
  __shared__ uint4 stage[kBlock / 64][Pv::kWords + Kc::kWords + Gv::kWords];
  const int64_t row = particle_id() / L;
  const int sub = threadIdx.x & (L - 1);
  const bool on = row < S.n;
  if (__ballot(on) == 0ull) return;  // the whole wave
  const int64_t s = on ? row : S.n - 1, n = S.n;
  uint4* const wpv = stage[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
  uint4* const wkc = wpv + Pv::kWords;
  uint4* const wgv = wkc + Kc::kWords;
  const R4<R> pi = S.pos(s);
  const R4<R> vi = S.vel(s);
  KC<R> ki;
  load_kc4(S, s, ki);
  GvcRec<R> gi;
  gvc_from<R>([&](int t) { return G.gvc4[4 * s + t]; }, gi);
  // the 16 correction adjoints of the own sums accumulate in the working
  // precision (64 gather pairs; they feed the FP64 correction adjoint)
  KCBar<R> kb;
  kb.zero();
  double xb[3] = {0, 0, 0}, vb[3] = {0, 0, 0}, hb = 0, Vb = 0;
  if (sub == 0) {
    R W0, dW0;
    kernel_self<R, K>(pi.w, W0, dW0);
    density_self_adj<R, double, R>(ki.a, gi.m, vi.w, W0, dW0, gi.Numb, gi.Denb, &kb, Vb, hb);
  }
  NbrRef nb = nbr_ref(S, s);
  if (!on) nb.ng = nb.ns = 0;
  const int total = nb.ng + nb.ns;
  const int most = wave_max_int(total);
  auto fetch = [&](uint32_t e) {
    const uint32_t j = e >> kCodeBits;
    Pv::load(S.pv, j, wpv);
    Kc::load(S.kc4, j, wkc);
    Gv::load(G.gvc4, j, wgv);
  };
  uint32_t e = entry_or_self(S, nb, s, sub), en = 0;
  if (most > 0) {
    fetch(e);
    en = entry_or_self(S, nb, s, sub + L);
  }
  for (int k = 0; k < most; k += L) {
    wait_loads();
    const R4<R> pj = rec4<2>(wpv, 0, R()), vj = rec4<2>(wpv, 1, R());
    KC<R> kj;
    kc_from<R>([&](int t) { return rec4<4>(wkc, t, R()); }, kj);
    GvcRec<R> gj;
    gvc_from<R>([&](int t) { return rec4<4>(wgv, t, R()); }, gj);
    wait_lds();
    const uint32_t ec = e;
    e = en;
    if (k + L < most) {
      fetch(e);
      en = entry_or_self(S, nb, s, k + 2 * L + sub);
    }
    if (k + sub < total) {
      R x[3];
      pair_x<R>(S, pi, gi.cell, pj, gj.cell, ec, x);
      const R r2 = dot3b(x, x);
      const R rinv = Sc<R>::rsqrt(r2);
      const R r = r2 * rinv;
      const R vij[3] = {vi.x - vj.x, vi.y - vj.y, vi.z - vj.z};
      if (k + sub < nb.ng) {
        KEval<R> ev;
        kernel_eval<R, K>(r, rinv, pi.w, ev);
        density_own_adj<R, double, R>(ki, x, r, rinv, ev, gj.m, vj.w, vij, gi.Numb, gi.Denb,
                                      gi.gvb, &kb, xb, hb, vb);
      }
      if (r2 * (pj.w * pj.w) < R(1)) {
        KEval<R> ej;
        kernel_eval<R, K>(r, rinv, pj.w, ej);
        density_rev_adj<R, double>(kj, x, r, rinv, ej, gi.m, vi.w, vij, gj.Numb, gj.Denb, gj.gvb,
                                   xb, Vb, vb);
      }
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    xb[a] = lane_sum<L>(xb[a]);
    vb[a] = lane_sum<L>(vb[a]);
    kb.b[a] = lane_sum<L>(kb.b[a]);
    kb.c[a] = lane_sum<L>(kb.c[a]);
  }
#pragma unroll
  for (int t = 0; t < 9; ++t) kb.M[t] = lane_sum<L>(kb.M[t]);
  kb.a = lane_sum<L>(kb.a);
  hb = lane_sum<L>(hb);
  Vb = lane_sum<L>(Vb);
  if (!on || sub != 0) return;
  G.gh[s] += hb;
  G.gkc[s] += (double)kb.a;
  for (int q = 0; q < 3; ++q) {
    G.gkc[(1 + q) * n + s] += (double)kb.b[q];
    G.gkc[(4 + q) * n + s] += (double)kb.c[q];
  }
  for (int q = 0; q < 9; ++q) G.gkc[(7 + q) * n + s] += (double)kb.M[q];
  for (int a = 0; a < 3; ++a) {
    G.gx[a * n + s] += xb[a];
    G.gv[a * n + s] += vb[a];
  }
  G.gV[s] += Vb;
}

// --------------------------------------------------------------------- B4 --
// The moment sums as in the forward (4 lanes per particle, then a thread each
// for the FP64 adjoint of the solve), or read when the forward kept them.
// At least three waves per SIMD (168 VGPRs, a few spilled): measured at 16.8M
// clustered particles 10.5 -> 8.7 ms against the two the register count gives
// otherwise.
template <class R, int K, int L>
__global__ void __launch_bounds__(kBlock, 3) k_bwd_corr(State<R> S, AdjState<R> G) {
  __shared__ MomentStage<R, L> sh;
  const int64_t n = S.n;
  if (!S.mom) {
    const int64_t row = particle_id() / L;
    moment_sums<R, K, L>(S, row < n ? row : 0, row < n, sh);
  }
  const int64_t s = (particle_id() - threadIdx.x) / L + threadIdx.x;
  if (threadIdx.x >= kBlock / L || s >= n) return;
  double raw[40];
  if (S.mom) {
    for (int t = 0; t < 40; ++t) raw[t] = (double)S.mom[t * n + s];
  } else {
    for (int t = 0; t < 40; ++t) raw[t] = (double)sh.sum[threadIdx.x][t];
  }
  double kcb[16];
  for (int t = 0; t < 16; ++t) kcb[t] = G.gkc[t * n + s];
  double out[40];
  corr_solve_adj(raw, kcb, out, SingularTol<R>::v);
#pragma unroll
  for (int t = 0; t < 10; ++t) {
    R4<R> q;
    q.x = (R)out[4 * t];
    q.y = (R)out[4 * t + 1];
    q.z = (R)out[4 * t + 2];
    q.w = (R)out[4 * t + 3];
    G.mom4[4 * ((t >> 2) * G.npad + s) + (t & 3)] = q;
  }
  R4<R> a;
  a.x = S.vel(s).w;
  a.y = S.mass[s];
  a.z = cell_to_real(S.cell3[s], R());
  a.w = R(0);
  G.mom4[4 * (2 * G.npad + s) + 2] = S.pos(s);
  G.mom4[4 * (2 * G.npad + s) + 3] = a;
}

// ------------------------------------------------------------------ B5+B6 --
// The moment adjoint's record: the 40 adjoints, then position and 1/h, and V,
// mass and lattice cell (get(t): its Real4 t of 12).
template <class R>
struct MomRec {
  R mb[40];
  R4<R> p;
  R V, m;
  uint32_t cell;
};
template <class R, class F>
__device__ inline void mom_from(F&& get, MomRec<R>& o) {
#pragma unroll
  for (int t = 0; t < 10; ++t) {
    const R4<R> q = get(t);
    o.mb[4 * t] = q.x;
    o.mb[4 * t + 1] = q.y;
    o.mb[4 * t + 2] = q.z;
    o.mb[4 * t + 3] = q.w;
  }
  o.p = get(10);
  const R4<R> q = get(11);
  o.V = q.x;
  o.m = q.y;
  o.cell = real_to_cell(q.z);
}

// Own moment sums (gather entries) and the particle's share in the sums of
// every neighbour j with r < h_j, from one fetch of the neighbour's record:
// 440 -> 217 us at 262,144 particles in FP32 (FP64 807 -> 552), 29.1 -> 15.5 ms at
// 16.8M clustered, against a thread per particle. Bound by instruction issue.
template <class R, int K, int L>
__global__ void __launch_bounds__(kAdjBlock<R>) k_bwd_moments(State<R> S, AdjState<R> G,
                                                              int h_mode) {
  constexpr int BLK = kAdjBlock<R>;
  using Mo = Rec<R, 4>;  // each third of the record
  __shared__ uint4 stage[BLK / 64][3 * Mo::kWords];
  const int64_t row = particle_id<BLK>() / L;
  const int sub = threadIdx.x & (L - 1);
  const bool on = row < S.n;
  if (__ballot(on) == 0ull) return;  // the whole wave
  const int64_t s = on ? row : S.n - 1, n = S.n;
  uint4* const w = stage[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
  const R4<R>* const mo[3] = {G.mom4, G.mom4 + 4 * G.npad, G.mom4 + 8 * G.npad};
  MomRec<R> I;
  mom_from<R>([&](int t) { return mo[t >> 2][4 * s + (t & 3)]; }, I);
  const R hinv = I.p.w;
  double Vb = 0.0, hb = 0.0, sh = 0.0, xb[3] = {0, 0, 0};
  if (sub == 0) {
    R W0, dW0;
    kernel_self<R, K>(hinv, W0, dW0);
    Vb = (double)(I.mb[0] * W0);
    hb = (double)(I.mb[0] * I.V * dW0);
    sh = (double)(I.m * dW0);
  }
  NbrRef nb = nbr_ref(S, s);
  if (!on) nb.ng = nb.ns = 0;
  const int total = nb.ng + nb.ns;
  const int most = wave_max_int(total);
  auto fetch = [&](uint32_t e) {
    const uint32_t j = e >> kCodeBits;
#pragma unroll
    for (int t = 0; t < 3; ++t) Mo::load(mo[t], j, w + t * Mo::kWords);
  };
  uint32_t e = entry_or_self(S, nb, s, sub), en = 0;
  if (most > 0) {
    fetch(e);
    en = entry_or_self(S, nb, s, sub + L);
  }
  for (int k = 0; k < most; k += L) {
    wait_loads();
    MomRec<R> J;
    mom_from<R>([&](int t) { return rec4<4>(w + (t >> 2) * Mo::kWords, t & 3, R()); }, J);
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
      const R r2 = dot3b(x, x);
      const R rinv = Sc<R>::rsqrt(r2);
      const R r = r2 * rinv;
      if (k + sub < nb.ng) {
        KEval<R> ev;
        kernel_eval<R, K>(r, rinv, hinv, ev);
        R gx[3], gh;
        mom_pair_adj<R>(I.mb, x, rinv, ev, gx, gh);
        for (int a = 0; a < 3; ++a) xb[a] += (double)(J.V * gx[a]);
        hb += (double)(J.V * gh);
        sh += (double)(J.m * ev.dWdh);
      }
      if (r2 * (J.p.w * J.p.w) < R(1)) {
        KEval<R> ej;
        kernel_eval<R, K>(r, rinv, J.p.w, ej);
        const R xm[3] = {-x[0], -x[1], -x[2]};
        R gx[3], gh;
        const R l = mom_pair_adj<R>(J.mb, xm, rinv, ej, gx, gh);
        Vb += (double)l;
        for (int a = 0; a < 3; ++a) xb[a] -= (double)(I.V * gx[a]);
      }
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) xb[a] = lane_sum<L>(xb[a]);
  Vb = lane_sum<L>(Vb);
  hb = lane_sum<L>(hb);
  sh = lane_sum<L>(sh);
  if (!on || sub != 0) return;
  for (int a = 0; a < 3; ++a) G.gx[a * n + s] += xb[a];
  const double hbt = G.gh[s] + hb;
  const double Vbt = G.gV[s] + Vb;
  // volume and smoothing-length coefficient (V = m / S, S = sum m_j W(r, h_j))
  const double V = (double)I.V, m = (double)I.m;
  const double Ssum = m / V;
  double kappa = -Vbt * V / Ssum;
  if (h_mode == 1) {
    const double h = (double)S.hbuf[s];
    const double dVdh = -V * sh / Ssum;
    const double htot = hbt + Vbt * dVdh;
    const double dFdh = 3.0 * h * h * Ssum / m + h * h * h * sh / m;
    kappa += -htot * (h * h * h / m) / dFdh;
  }
  R4<R> q;
  q.x = I.m;
  q.y = (R)kappa;
  q.z = cell_to_real(I.cell, R());
  q.w = R(0);
  G.vol4[2 * s] = I.p;
  G.vol4[2 * s + 1] = q;
}

// --------------------------------------------------------------------- B7 --
// (101 -> 49 us at 262,144 particles in FP32, 9.3 -> 4.3 ms at 16.8M clustered)
template <class R, int K, int L>
__global__ void __launch_bounds__(kBlock) k_bwd_volume(State<R> S, AdjState<R> G) {
  using Vo = Rec<R, 2>;
  __shared__ uint4 stage[kBlock / 64][Vo::kWords];
  const int64_t row = particle_id() / L;
  const int sub = threadIdx.x & (L - 1);
  const bool on = row < S.n;
  if (__ballot(on) == 0ull) return;  // the whole wave
  const int64_t s = on ? row : S.n - 1, n = S.n;
  uint4* const w = stage[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
  const R4<R> pi = G.vol4[2 * s], qi = G.vol4[2 * s + 1];
  const uint32_t ci = real_to_cell(qi.z);
  double xb[3] = {0, 0, 0};
  NbrRef nb = nbr_ref(S, s);
  if (!on) nb.ng = nb.ns = 0;
  const int total = nb.ng + nb.ns;
  const int most = wave_max_int(total);
  uint32_t e = entry_or_self(S, nb, s, sub), en = 0;
  if (most > 0) {
    Vo::load(G.vol4, e >> kCodeBits, w);
    en = entry_or_self(S, nb, s, sub + L);
  }
  for (int k = 0; k < most; k += L) {
    wait_loads();
    const R4<R> pj = rec4<2>(w, 0, R()), qj = rec4<2>(w, 1, R());
    wait_lds();
    const uint32_t ec = e;
    e = en;
    if (k + L < most) {
      Vo::load(G.vol4, e >> kCodeBits, w);
      en = entry_or_self(S, nb, s, k + 2 * L + sub);
    }
    if (k + sub < total) {
      R x[3];
      pair_x<R>(S, pi, ci, pj, real_to_cell(qj.z), ec, x);
      const R r2 = dot3b(x, x);
      const R rinv = Sc<R>::rsqrt(r2);
      const R r = r2 * rinv;
      R c = R(0);
      if (k + sub < nb.ng) {
        KEval<R> ev;
        kernel_eval<R, K>(r, rinv, pi.w, ev);
        c += qi.y * qj.x * ev.f;
      }
      if (r2 * (pj.w * pj.w) < R(1)) {
        KEval<R> ej;
        kernel_eval<R, K>(r, rinv, pj.w, ej);
        c += qj.y * qi.x * ej.f;
      }
      for (int a = 0; a < 3; ++a) xb[a] += (double)(c * x[a]);
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) xb[a] = lane_sum<L>(xb[a]);
  if (!G.out8) {
    if (on && sub == 0)
      for (int a = 0; a < 3; ++a) G.gx[a * n + s] += xb[a];
  } else if (on && sub < 4) {  // four lanes write the particle's record
    auto part = [&](int c) {
      if (c < 3) return G.gx[c * n + s] + (c == 0 ? xb[0] : (c == 1 ? xb[1] : xb[2]));
      return c < 6 ? G.gv[(c - 3) * n + s] : (c == 6 ? G.gu[s] : 0.0);
    };
    reinterpret_cast<double2*>(G.out8)[4 * s + sub] = make_double2(part(2 * sub), part(2 * sub + 1));
  }
}

// ----------------------------------------------------------------- finish --
template <class R>
__global__ void __launch_bounds__(kBlock) k_bwd_unpermute(State<R> S, AdjState<R> G,
                                                          double* __restrict__ g_x,
                                                          double* __restrict__ g_v,
                                                          double* __restrict__ g_u) {
  const int64_t i = particle_id();
  if (i >= S.n) return;
  const int64_t n = S.n;
  if (G.out8) {
    // particle i of the caller: its record is one line, the writes are
    // coalesced (scattered 8-byte writes of seven arrays took 26 us at 262,144
    // particles and 2.7 ms at 16.8M, this 8 and 0.5)
    const double2* r = reinterpret_cast<const double2*>(G.out8) + 4 * (int64_t)S.inv[i];
    const double2 a = r[0], b = r[1], c = r[2], d = r[3];
    g_x[i] = a.x;
    g_x[n + i] = a.y;
    g_x[2 * n + i] = b.x;
    g_v[i] = b.y;
    g_v[n + i] = c.x;
    g_v[2 * n + i] = c.y;
    g_u[i] = d.x;
    return;
  }
  const uint32_t p = S.perm[i];
  for (int a = 0; a < 3; ++a) {
    g_x[a * n + p] = G.gx[a * n + i];
    g_v[a * n + p] = G.gv[a * n + i];
  }
  g_u[p] = G.gu[i];
}

// Deterministic sum of the per-block alpha, beta partials: block b of the grid
// sums its share (fixed strided order, fixed tree) into out[2 b .. 2 b + 1].
__global__ void __launch_bounds__(kBlock) k_bwd_reduce_ab(const double* __restrict__ part,
                                                          int64_t nb, double* __restrict__ out) {
  __shared__ double sa[kBlock], sb[kBlock];
  double a = 0.0, b = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < nb;
       i += (int64_t)gridDim.x * kBlock) {
    a += part[2 * i];
    b += part[2 * i + 1];
  }
  sa[threadIdx.x] = a;
  sb[threadIdx.x] = b;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      sa[threadIdx.x] += sa[threadIdx.x + w];
      sb[threadIdx.x] += sb[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[2 * blockIdx.x] = sa[0];
    out[2 * blockIdx.x + 1] = sb[0];
  }
}

__global__ void __launch_bounds__(kBlock) k_zero_f64(double* __restrict__ a, int64_t na) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < na) a[i] = 0.0;
}

}  // namespace

void launch_zero_f64(double* a, int64_t na, hipStream_t s) {
  if (na > 0) hipLaunchKernelGGL(k_zero_f64, dim3(grid_for(na)), dim3(kBlock), 0, s, a, na);
}

template <class R>
void launch_bwd_prep(const State<R>& S, const AdjState<R>& G, hipStream_t s) {
  hipLaunchKernelGGL(k_bwd_prep<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, G);
}
// a pair pass: pair_lanes(n) lanes per particle
#define CRK_DISPATCH_PAIRS(kernel, KFN, BLK, ...)                                               \
  do {                                                                                          \
    const dim3 pg(grid_for(pair_lanes(S.n) * S.n, BLK)), pb(BLK);                               \
    if (pair_lanes(S.n) == 16) {                                                                \
      if ((kernel) == 0)                                                                        \
        hipLaunchKernelGGL((KFN<R, 0, 16>), pg, pb, 0, s, __VA_ARGS__);                         \
      else                                                                                      \
        hipLaunchKernelGGL((KFN<R, 1, 16>), pg, pb, 0, s, __VA_ARGS__);                         \
    } else {                                                                                    \
      if ((kernel) == 0)                                                                        \
        hipLaunchKernelGGL((KFN<R, 0, 4>), pg, pb, 0, s, __VA_ARGS__);                          \
      else                                                                                      \
        hipLaunchKernelGGL((KFN<R, 1, 4>), pg, pb, 0, s, __VA_ARGS__);                          \
    }                                                                                           \
  } while (0)

template <class R>
void launch_bwd_force(const State<R>& S, const AdjState<R>& G, int kernel, hipStream_t s) {
  CRK_DISPATCH_PAIRS(kernel, k_bwd_force, kAdjBlock<R>, S, G);
}
template <class R>
void launch_bwd_density(const State<R>& S, const AdjState<R>& G, int kernel, hipStream_t s) {
  CRK_DISPATCH_PAIRS(kernel, k_bwd_density, kBlock, S, G);
}
template <class R>
void launch_bwd_corr(const State<R>& S, const AdjState<R>& G, int kernel, hipStream_t s) {
  const dim3 g(grid_for(4 * S.n)), b(kBlock);  // (list-ordered sums: 4 lanes)
  if (kernel == 0)
    hipLaunchKernelGGL((k_bwd_corr<R, 0, 4>), g, b, 0, s, S, G);
  else
    hipLaunchKernelGGL((k_bwd_corr<R, 1, 4>), g, b, 0, s, S, G);
}
template <class R>
void launch_bwd_moments(const State<R>& S, const AdjState<R>& G, int kernel, int h_mode,
                        hipStream_t s) {
  CRK_DISPATCH_PAIRS(kernel, k_bwd_moments, kAdjBlock<R>, S, G, h_mode);
}
template <class R>
void launch_bwd_volume(const State<R>& S, const AdjState<R>& G, int kernel, hipStream_t s) {
  CRK_DISPATCH_PAIRS(kernel, k_bwd_volume, kBlock, S, G);
}
template <class R>
void launch_bwd_finish(const State<R>& S, const AdjState<R>& G, double* g_x, double* g_v,
                       double* g_u, double* g_ab, hipStream_t s) {
  hipLaunchKernelGGL(k_bwd_unpermute<R>, dim3(grid_for(S.n)), dim3(kBlock), 0, s, S, G, g_x, g_v,
                     g_u);
  // up to 256 blocks sum the partials (into the room after them), one the rest
  const int64_t blocks = bwd_force_blocks(S.n, sizeof(R) == 8);
  const int64_t first = blocks < 256 * (int64_t)kBlock ? grid_for(blocks) : 256;
  double* mid = first > 1 ? G.gab + 2 * blocks : g_ab;
  hipLaunchKernelGGL(k_bwd_reduce_ab, dim3((unsigned)first), dim3(kBlock), 0, s,
                     (const double*)G.gab, blocks, mid);
  if (first > 1)
    hipLaunchKernelGGL(k_bwd_reduce_ab, dim3(1), dim3(kBlock), 0, s, (const double*)mid, first,
                       g_ab);
}

#define CRK_INSTANTIATE_BWD(R)                                                                 \
  template void launch_bwd_prep<R>(const State<R>&, const AdjState<R>&, hipStream_t);          \
  template void launch_bwd_force<R>(const State<R>&, const AdjState<R>&, int, hipStream_t);    \
  template void launch_bwd_density<R>(const State<R>&, const AdjState<R>&, int, hipStream_t);  \
  template void launch_bwd_corr<R>(const State<R>&, const AdjState<R>&, int, hipStream_t);     \
  template void launch_bwd_moments<R>(const State<R>&, const AdjState<R>&, int, int,           \
                                      hipStream_t);                                            \
  template void launch_bwd_volume<R>(const State<R>&, const AdjState<R>&, int, hipStream_t);   \
  template void launch_bwd_finish<R>(const State<R>&, const AdjState<R>&, double*, double*,    \
                                     double*, double*, hipStream_t);

CRK_INSTANTIATE_BWD(float)
CRK_INSTANTIATE_BWD(double)

}  // namespace crk
