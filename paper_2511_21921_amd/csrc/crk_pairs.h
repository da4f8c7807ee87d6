// Pair loops by groups of lanes with the neighbour records staged in LDS.
//
// A pair pass reads ~160 B of records per neighbour. With a thread per
// particle every 16-byte load of a wave touches 64 different lines, and the
// vector memory path takes about one line a cycle: at 64^3 that alone is
// ~14 ps a pair (a loop that only loads the records: 254 us for 18.7M pairs,
// where the whole force pass took 320 us). Here L = 4 (or 16) lanes share a
// particle, lane sub taking the entries k = sub mod L, and a wave fetches the
// records of its 64 current pairs together: the four lanes of a quad load the
// four 16-byte pieces of one 64-byte record, record by record, straight into
// LDS (global_load_lds, no registers held), and every lane then reads the
// record of its own pair from there. The same loads take 7.2-7.6 ps a pair,
// and the next pairs' records are in flight while the current ones are
// computed.
#pragma once

#include "crk_state.h"

namespace crk {

typedef __attribute__((address_space(3))) void LdsVoid;
typedef const __attribute__((address_space(1))) void GlobalVoid;

// ---- exchanges inside a quad or a row of 16 lanes (DPP, no LDS) ----------
constexpr int quad_perm(int a, int b, int c, int d) { return a | b << 2 | c << 4 | d << 6; }

template <int CTRL>
__device__ inline uint32_t dpp_mov(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ inline float dpp_mov(float v) {
  return __uint_as_float(dpp_mov<CTRL>(__float_as_uint(v)));
}
template <int CTRL>
__device__ inline double dpp_mov(double v) {
  const uint32_t lo = dpp_mov<CTRL>((uint32_t)__double2loint(v));
  const uint32_t hi = dpp_mov<CTRL>((uint32_t)__double2hiint(v));
  return __hiloint2double((int)hi, (int)lo);
}

// Sum over the L lanes (an aligned quad or row of 16) that share a particle.
// Every lane gets a sum in an order of its own, fixed from run to run.
template <int L, class T>
__device__ inline T lane_sum(T v) {
  static_assert(L == 4 || L == 16, "a quad or a row");
  v += dpp_mov<quad_perm(1, 0, 3, 2)>(v);
  v += dpp_mov<quad_perm(2, 3, 0, 1)>(v);
  if (L == 16) {
    v += dpp_mov<0x124>(v);  // row rotated by 4
    v += dpp_mov<0x128>(v);  // and by 8
  }
  return v;
}

// Sum over the wave's 64 lanes, in a fixed order, the same in every lane.
__device__ inline double wave_sum64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The wave's largest v, as a scalar.
__device__ inline int wave_max_int(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return __builtin_amdgcn_readfirstlane(v);
}

// ------------------------------------------------- staged records ----------
// Records of P 16-byte pieces (P a multiple of 4, or 2), one per lane of the
// wave, in 64 P uint4 of LDS. Load t of a group of four pieces has each quad
// fetch the record of its lane t: lane q of the quad takes piece q ^ t, and
// the load writes its 64 lanes' pieces side by side. Lane t then finds piece
// p of its record at position p ^ t, so that the lanes of a quad read
// different banks. Records of two pieces go the same way, two to a load of a
// quad. Offsets are 32-bit: a record array holds less than 2^32 bytes (2^25
// particles of at most 128 bytes).
template <int P>
struct Staged {
  static_assert(P == 2 || P % 4 == 0, "pieces of a staged record");
  static constexpr int kWords = 64 * P;  // uint4 of LDS a wave

  // j: this lane's record; w: the wave's LDS (the same in every lane)
  static __device__ inline void load(const void* base, uint32_t j, uint4* w) {
    const uint32_t q = threadIdx.x & 3u;
    if constexpr (P == 2) {
      load_pair<0>(base, j, q, w);
      load_pair<1>(base, j, q, w);
    } else {
      load_quad<0>(base, j, q, w);
      load_quad<1>(base, j, q, w);
      load_quad<2>(base, j, q, w);
      load_quad<3>(base, j, q, w);
    }
  }

  // piece p of this lane's record
  static __device__ inline uint4 piece(const uint4* w, int p) {
    const int lane = threadIdx.x & 63, q = lane & 3, quad = lane & ~3;
    if constexpr (P == 2) return w[(q & 1) * 64 + quad + (q & 2) + (p ^ (q & 1))];
    return w[(p >> 2) * 256 + q * 64 + quad + ((p & 3) ^ q)];
  }

 private:
  static __device__ inline void to_lds(const void* base, uint32_t off, uint4* w) {
    __builtin_amdgcn_global_load_lds((GlobalVoid*)((const char*)base + off), (LdsVoid*)w, 16, 0,
                                     0);
  }
  template <int T>
  static __device__ inline void load_quad(const void* base, uint32_t j, uint32_t q, uint4* w) {
    const uint32_t off = dpp_mov<quad_perm(T, T, T, T)>(j) * (16u * P) + ((q ^ T) << 4);
#pragma unroll
    for (int g = 0; g < P / 4; ++g) to_lds(base, off + 64u * g, w + g * 256 + T * 64);
  }
  template <int T>
  static __device__ inline void load_pair(const void* base, uint32_t j, uint32_t q, uint4* w) {
    const uint32_t off = dpp_mov<quad_perm(T, T, T + 2, T + 2)>(j) * 32u + (((q & 1u) ^ T) << 4);
    to_lds(base, off, w + T * 64);
  }
};

// A Real4 is one piece in FP32 and two in FP64.
template <class R> constexpr int kPieces = (int)sizeof(R4<R>) / 16;

// Staged records of N Real4, and Real4 t of the lane's record.
template <class R, int N> using Rec = Staged<N * kPieces<R>>;
template <int N>
__device__ inline float4 rec4(const uint4* w, int t, float) {
  const uint4 a = Rec<float, N>::piece(w, t);
  return make_float4(__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z),
                     __uint_as_float(a.w));
}
template <int N>
__device__ inline double4 rec4(const uint4* w, int t, double) {
  const uint4 a = Rec<double, N>::piece(w, 2 * t), b = Rec<double, N>::piece(w, 2 * t + 1);
  return make_double4(__hiloint2double((int)a.y, (int)a.x), __hiloint2double((int)a.w, (int)a.z),
                      __hiloint2double((int)b.y, (int)b.x), __hiloint2double((int)b.w, (int)b.z));
}

// The wave's outstanding loads (into LDS among them) have arrived.
__device__ inline void wait_loads() {
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  asm volatile("" ::: "memory");
}
// The wave's LDS reads have returned: the stage may be written again.
__device__ inline void wait_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_sched_barrier(0);
}

// Entry t of the symmetric list of particle s (gather part first), or s
// itself past its end (a record that may be loaded and is not used).
template <class R>
__device__ inline uint32_t entry_or_self(const State<R>& S, const NbrRef& nb, int64_t s, int t) {
  if (t < nb.ng) return S.nlist[slot_at(nb.gb, t)];
  if (t < nb.ng + nb.ns) return S.slist[slot_at(nb.sb, t - nb.ng)];
  return ((uint32_t)s << kCodeBits) | (uint32_t)kSelfCode;
}

// ------------------------------------------------------- moment sums ------
// The 40 geometric moment sums of a particle over its gather entries (the
// corrections' solve and its adjoint take them): m0, m1, m2 (xx, xy, xz, yy,
// yz, zz), dm0, X1 and X2 (sum V x_a d_g W and sum V x_a x_b d_g W).
template <class R>
struct Moments {
  R m0, m1[3], m2[6], dm0[3], X1[9], X2[18];
};

// A neighbour's factors in the sums, at separation x with volume Vj (1/h hinv,
// C h^-3 and C h^-4): VW = vc w and Vg_g = fg x_g.
template <class R>
struct MomentPair {
  R x[3], vc, w, fg;
};
template <class R, int K>
__device__ __forceinline__ void moment_pair(R Vj, R hinv, R C3, R C4, MomentPair<R>& o) {
  const R r2 = norm2(o.x);
  const R rinv = Sc<R>::rsqrt(r2);
  R dw;
  Shape<K>::eval(r2 * rinv * hinv, o.w, dw);
  o.vc = Vj * C3;
  o.fg = Vj * C4 * dw * rinv;
}

// LDS of a block's moment sums: the staged records while they are summed, then
// the sums of each of its particles (an odd stride: no bank conflicts).
template <class R, int L>
struct MomentStage {
  union {
    uint4 rec[kBlock / 64][Rec<R, 2>::kWords];
    R sum[kBlock / L][41];
  };
  __device__ inline void get(int row, Moments<R>& M) const {
    R* v = reinterpret_cast<R*>(&M);
#pragma unroll
    for (int t = 0; t < 40; ++t) v[t] = sum[row][t];
  }
};

// The moment sums of particle s, left in sh (row threadIdx.x / L of the block)
// behind a barrier; every thread of the block calls.
//
// The limiter of the force adjoint jumps where its argument changes sign, so a
// last bit of grad v in FP32 may decide a term of the gradient: each sum is
// therefore taken in list order, whatever the number of lanes. With L = 4 each
// lane computes the pair of every fourth entry and owns ten of the forty sums:
// lane g < 3 those with d_g W (dm0_g, X1_g, X2_g), lane 3 those with W (m0, m1,
// m2). The four pairs then go round the quad in order, and every lane adds
// q (1, x_a, x_a x_b) with its own q = x_g fg or vc w. (Sums of every lane's own
// entries instead took 87 us where this takes 106, at 262,144 particles, but
// moved 16.8M clustered particles' gradient by 1.6e-4 in norm. L = 16, the short lists
// of active particles of a hierarchy substep, takes every sixteenth entry and
// adds the lanes' sums.)
template <class R, int K, int L>
__device__ inline void moment_sums(const State<R>& S, int64_t s, bool on,
                                   MomentStage<R, L>& sh) {
  using Pv = Rec<R, 2>;
  const int sub = threadIdx.x & (L - 1);
  uint4* const wpv = sh.rec[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
  const R4<R> pi = S.pos(s);
  const R hinv = pi.w;
  const R C3 = R(Shape<K>::C) * hinv * hinv * hinv;
  const R C4 = C3 * hinv;
  const R self = S.vel(s).w * C3 * R(Shape<K>::w0);
  constexpr int N = L == 4 ? 10 : 40;
  R v[N];
#pragma unroll
  for (int t = 0; t < N; ++t) v[t] = R(0);
  if (sub == (L == 4 ? 3 : 0)) v[0] = self;
  const uint32_t ci = S.cell3[s];
  NbrRef nb = nbr_ref(S, s);
  if (!on) nb.ng = 0;
  nb.ns = 0;
  const int total = nb.ng;
  const int most = wave_max_int(total);
  uint32_t cn = 0;
  auto fetch = [&](uint32_t e) {
    const uint32_t j = e >> kCodeBits;
    Pv::load(S.pv, j, wpv);
    if (S.lattice) cn = S.cell3[j];
  };
  uint32_t e = entry_or_self(S, nb, s, sub), en = 0;
  if (most > 0) {
    fetch(e);
    en = entry_or_self(S, nb, s, sub + L);
  }
  for (int k = 0; k < most; k += L) {
    wait_loads();
    const R4<R> pj = rec4<2>(wpv, 0, R());
    const R Vj = rec4<2>(wpv, 1, R()).w;
    const uint32_t cj = cn;
    wait_lds();
    const uint32_t ec = e;
    e = en;
    if (k + L < most) {
      fetch(e);
      en = entry_or_self(S, nb, s, k + 2 * L + sub);
    }
    MomentPair<R> p;
    p.x[0] = p.x[1] = p.x[2] = p.vc = p.w = p.fg = R(0);
    if (k + sub < total) {
      pair_x<R>(S, pi, ci, pj, cj, ec, p.x);
      moment_pair<R, K>(Vj, hinv, C3, C4, p);
    }
    auto add = [&](R* acc, const R x[3], R a, R b) {  // the ten sums of one q = a b
      const R q = a * b;
      acc[0] = Sc<R>::fma(a, b, acc[0]);
#pragma unroll
      for (int t = 0; t < 3; ++t) acc[1 + t] = Sc<R>::fma(x[t], q, acc[1 + t]);
      acc[4] = Sc<R>::fma(x[0] * x[0], q, acc[4]);
      acc[5] = Sc<R>::fma(x[0] * x[1], q, acc[5]);
      acc[6] = Sc<R>::fma(x[0] * x[2], q, acc[6]);
      acc[7] = Sc<R>::fma(x[1] * x[1], q, acc[7]);
      acc[8] = Sc<R>::fma(x[1] * x[2], q, acc[8]);
      acc[9] = Sc<R>::fma(x[2] * x[2], q, acc[9]);
    };
    if constexpr (L == 4) {
      auto turn = [&](auto lane) {
        constexpr int T = decltype(lane)::value;
        constexpr int B = quad_perm(T, T, T, T);
        const R x[3] = {dpp_mov<B>(p.x[0]), dpp_mov<B>(p.x[1]), dpp_mov<B>(p.x[2])};
        const R vc = dpp_mov<B>(p.vc), w = dpp_mov<B>(p.w), fg = dpp_mov<B>(p.fg);
        const R xg = sub == 0 ? x[0] : (sub == 1 ? x[1] : x[2]);
        add(v, x, sub == 3 ? vc : xg, sub == 3 ? w : fg);
      };
      turn(std::integral_constant<int, 0>());
      turn(std::integral_constant<int, 1>());
      turn(std::integral_constant<int, 2>());
      turn(std::integral_constant<int, 3>());
    } else {
      add(v, p.x, p.vc, p.w);
#pragma unroll
      for (int g = 0; g < 3; ++g) add(v + 10 + 10 * g, p.x, p.x[g], p.fg);
    }
  }
  if constexpr (L != 4) {
#pragma unroll
    for (int t = 0; t < N; ++t) v[t] = lane_sum<L>(v[t]);
  }
  __syncthreads();  // every wave is done with its records
  R* to = sh.sum[threadIdx.x / L];
  // ten sums of group g (0..2: d_g W, 3: W) into the order of Moments
  auto put = [&](const R* acc, int g) {
    to[g < 3 ? 10 + g : 0] = acc[0];
#pragma unroll
    for (int t = 0; t < 3; ++t) to[g < 3 ? 13 + 3 * g + t : 1 + t] = acc[1 + t];
#pragma unroll
    for (int t = 0; t < 6; ++t) to[g < 3 ? 22 + 6 * g + t : 4 + t] = acc[4 + t];
  };
  if constexpr (L == 4) {
    put(v, sub);
  } else if (sub == 0) {
    put(v, 3);
#pragma unroll
    for (int g = 0; g < 3; ++g) put(v + 10 + 10 * g, g);
  }
  __syncthreads();
}

}  // namespace crk
