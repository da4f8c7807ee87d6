// Deterministic device-wide primitives for building the cell list:
// an exclusive prefix sum and a stable LSD radix sort of (key, value) pairs.
// Both are written for 64-wide wavefronts: the sort ranks equal digits
// inside a wave with a ballot per bit (wave multisplit), so the output order
// never depends on atomic ordering and repeated runs are bitwise equal.
#include "crk_internal.h"

#include <algorithm>
#include <type_traits>

namespace crk {
namespace {

constexpr int kItems = 8;                  // items per thread
constexpr int kTile = kBlock * kItems;     // 2048 items per block
constexpr int kWaves = kBlock / 64;

__device__ inline uint32_t wave_incl_scan(uint32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

// Block-wide exclusive scan of one value per thread; returns the block total.
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t& total) {
  __shared__ uint32_t wsum[kWaves];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = wave_incl_scan(v);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    uint32_t s = wsum[k];
    off += (k < w) ? s : 0u;
    tot += s;
  }
  __syncthreads();
  total = tot;
  return off + inc - v;
}

__global__ void __launch_bounds__(kBlock) k_chunk_sums(const uint32_t* __restrict__ in, int64_t n,
                                                       uint32_t* __restrict__ part) {
  const int64_t base = (int64_t)blockIdx.x * kTile + threadIdx.x * kItems;
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k)
    if (base + k < n) s += in[base + k];
  uint32_t tot;
  block_excl_scan(s, tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// One block scans the chunk sums in place (exclusive), 2048 at a time.
__global__ void __launch_bounds__(kBlock) k_scan_parts(uint32_t* part, int64_t m) {
  uint32_t carry = 0;
  for (int64_t base = 0; base < m; base += kTile) {
    uint32_t v[kItems], s = 0;
    const int64_t my = base + threadIdx.x * kItems;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      v[k] = (my + k < m) ? part[my + k] : 0u;
      s += v[k];
    }
    uint32_t tot;
    uint32_t off = block_excl_scan(s, tot) + carry;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      if (my + k < m) part[my + k] = off;
      off += v[k];
    }
    carry += tot;
    __syncthreads();
  }
}

// SELF: part holds the chunk sums themselves, and every block adds up those
// before its own (up to kSelfParts of them cost less than a launch between:
// 128 blocks of 2048 take 4.5 us against 9.5).
constexpr int64_t kSelfParts = 1024;
template <bool SELF>
__global__ void __launch_bounds__(kBlock) k_scan_apply(const uint32_t* in, uint32_t* out,
                                                       int64_t n,
                                                       const uint32_t* __restrict__ part) {
  uint32_t before = 0;
  if constexpr (SELF) {
    uint32_t p = 0;
    for (uint32_t k = threadIdx.x; k < blockIdx.x; k += kBlock) p += part[k];
    block_excl_scan(p, before);
  } else {
    before = part[blockIdx.x];
  }
  const int64_t base = (int64_t)blockIdx.x * kTile + threadIdx.x * kItems;
  uint32_t v[kItems], s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    v[k] = (base + k < n) ? in[base + k] : 0u;
    s += v[k];
  }
  uint32_t tot;
  uint32_t off = block_excl_scan(s, tot) + before;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    if (base + k < n) out[base + k] = off;
    off += v[k];
  }
}

// ------------------------------------------------------------ radix sort --
// NB bits a pass. A pass over few keys costs its launches and the latency of
// its scattered accesses, so up to kWideMax of them take digits of up to ten
// bits (18-bit cell keys: two passes and no copy back instead of three);
// larger sets take eight, whose runs of equal digits in a block stay longer
// (2048 keys in 256 digits) and fill their lines (at 16.8M keys four passes of
// eight bits scatter for 0.55 ms, three of ten for 1.05; at 2M the two are equal).

template <int NB>
__global__ void __launch_bounds__(kBlock) k_radix_hist(const uint32_t* __restrict__ keys,
                                                       int64_t n, int shift, int64_t nblk,
                                                       uint32_t* __restrict__ hist) {
  constexpr int D = 1 << NB;
  __shared__ uint32_t cnt[D];
#pragma unroll
  for (int d = threadIdx.x; d < D; d += kBlock) cnt[d] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    int64_t i = (int64_t)blockIdx.x * kTile + r * kBlock + threadIdx.x;
    if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & (uint32_t)(D - 1)], 1u);
  }
  __syncthreads();
#pragma unroll
  for (int d = threadIdx.x; d < D; d += kBlock) hist[(int64_t)d * nblk + blockIdx.x] = cnt[d];
}

// Each wave of a block ranks the equal digits of its own 512 keys, in order,
// with counters of its own in LDS; the block then adds up the waves' counters
// once and scatters: two barriers a block.
template <int NB>
__global__ void __launch_bounds__(kBlock) k_radix_scatter(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
    uint32_t* __restrict__ vout, int64_t n, int shift, int64_t nblk,
    const uint32_t* __restrict__ offs) {
  constexpr int D = 1 << NB;
  __shared__ uint32_t wcnt[kWaves][D];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  auto wave_sync = [&]() {  // the wave's LDS accesses in program order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
#pragma unroll
  for (int d = lane; d < D; d += 64) wcnt[w][d] = 0;
  wave_sync();
  const int64_t first = (int64_t)blockIdx.x * kTile + w * (kTile / kWaves) + lane;
  uint32_t key[kItems], val[kItems], rank[kItems];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int64_t i = first + r * 64;
    key[r] = i < n ? kin[i] : 0u;
    val[r] = i < n ? vin[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const bool valid = first + r * 64 < n;
    const uint32_t d = (key[r] >> shift) & (uint32_t)(D - 1);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const uint32_t before = wcnt[w][d], lower = __popcll(peers & lt);
    rank[r] = before + lower;
    wave_sync();
    if (valid && lower == 0) wcnt[w][d] = before + __popcll(peers);
    wave_sync();
  }
  __syncthreads();
#pragma unroll
  for (int d = t; d < D; d += kBlock) {
    uint32_t run = offs[(int64_t)d * nblk + blockIdx.x];
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
      const uint32_t c = wcnt[k][d];
      wcnt[k][d] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const uint32_t pos = wcnt[w][(key[r] >> shift) & (uint32_t)(D - 1)] + rank[r];
    // (pos < n always for a consistent histogram)
    if (first + r * 64 < n && (int64_t)pos < n) {
      kout[pos] = key[r];
      vout[pos] = val[r];
    }
  }
}

// Keys up to which the digits may be wide, and the widest ones' bits.
constexpr int64_t kWideMax = 1 << 20;
int widest(int64_t n) { return n <= kWideMax ? 10 : 8; }

}  // namespace

int64_t scan_tmp_words(int64_t n) { return (n + kTile - 1) / kTile + 1; }

hipError_t exclusive_scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* tmp,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t m = (n + kTile - 1) / kTile;
  hipLaunchKernelGGL(k_chunk_sums, dim3((unsigned)m), dim3(kBlock), 0, s, in, n, tmp);
  if (m <= kSelfParts) {
    hipLaunchKernelGGL(k_scan_apply<true>, dim3((unsigned)m), dim3(kBlock), 0, s, in, out, n,
                       (const uint32_t*)tmp);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(kBlock), 0, s, tmp, m);
  hipLaunchKernelGGL(k_scan_apply<false>, dim3((unsigned)m), dim3(kBlock), 0, s, in, out, n,
                     (const uint32_t*)tmp);
  return hipGetLastError();
}

// (Never less for more keys: up to kWideMax of them take wide digits, so a
// workspace made for a larger set has the room of the widest digits too.)
int64_t radix_tmp_words(int64_t n) {
  auto words = [](int64_t keys) { return ((keys + kTile - 1) / kTile) << widest(keys); };
  const int64_t most = n <= kWideMax ? words(n) : std::max(words(n), words(kWideMax));
  return most + scan_tmp_words(most);
}

hipError_t radix_sort_pairs(uint32_t* keys_a, uint32_t* vals_a, uint32_t* keys_b,
                            uint32_t* vals_b, int64_t n, int key_bits, uint32_t* tmp,
                            hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nblk = (n + kTile - 1) / kTile;
  const int passes = (key_bits + widest(n) - 1) / widest(n);
  const int need = passes > 0 ? (key_bits + passes - 1) / passes : 0;
  const int nb = need <= 8 ? 8 : need;  // bits a pass: 8, 9 or 10
  uint32_t* hist = tmp;
  uint32_t* stmp = tmp + (nblk << nb);
  uint32_t *ki = keys_a, *vi = vals_a, *ko = keys_b, *vo = vals_b;
  auto pass = [&](auto nb_t, int shift) -> hipError_t {
    constexpr int NB = decltype(nb_t)::value;
    hipLaunchKernelGGL(k_radix_hist<NB>, dim3((unsigned)nblk), dim3(kBlock), 0, s,
                       (const uint32_t*)ki, n, shift, nblk, hist);
    const hipError_t e = exclusive_scan_u32(hist, hist, nblk << NB, stmp, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_radix_scatter<NB>, dim3((unsigned)nblk), dim3(kBlock), 0, s,
                       (const uint32_t*)ki, (const uint32_t*)vi, ko, vo, n, shift, nblk,
                       (const uint32_t*)hist);
    return hipSuccess;
  };
  for (int p = 0; p < passes; ++p) {
    const int shift = p * nb;
    const hipError_t e = nb == 8 ? pass(std::integral_constant<int, 8>(), shift)
                         : nb == 9 ? pass(std::integral_constant<int, 9>(), shift)
                                   : pass(std::integral_constant<int, 10>(), shift);
    if (e != hipSuccess) return e;
    uint32_t* t1 = ki; ki = ko; ko = t1;
    uint32_t* t2 = vi; vi = vo; vo = t2;
  }
  if (passes & 1) {
    hipError_t e = hipMemcpyAsync(keys_a, ki, n * 4, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(vals_a, vi, n * 4, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

}  // namespace crk
