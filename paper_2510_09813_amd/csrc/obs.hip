// Outputs of an evolved state: occupations <n_i> and bitstring samples.
//
// Occupations: <n_i> = sum_b |psi_b|^2 b_p / sum_b |psi_b|^2 with p = n-1-i, FP64.  A
// workgroup owns 2^C contiguous amplitudes (C = min(n, 12)): thread-index bits and the
// register-loop bits are accumulated locally, bits above C are constant per workgroup and
// resolved in the second stage from the workgroup index.
//
// Sampling: shot s draws u_s from a SplitMix64 stream (Steele, Lea & Flood 2014; the Weyl
// increment 0x9E3779B97F4A7C15 and the variant-13 finaliser) seeded with `seed`, and returns
// the smallest b with CDF(b) > u_s * CDF(last); without such a b (rounding), the largest b
// with nonzero probability.  CDF is evaluated as a prefix sum in three levels: per-block
// sums of |psi|^2 (FP64), one exclusive scan over the blocks, then a scan inside the
// selected block.
#include <mutex>

#include "device_common.h"

namespace rsv {
namespace {

constexpr int kChunkBits = 12;
constexpr int kOccStride = 1 + kChunkBits;  // per chunk: total, then one sum per low bit

template <class R>
__device__ __forceinline__ double prob(const Cx<R>& v) {
  return norm_add(0.0, (double)v.x, (double)v.y);
}

// partial[slot * nchunk + chunk] (slot-major, so that the second stage's loads are coalesced).
template <class R>
__global__ __launch_bounds__(kBlock) void occ_partial_kernel(const Cx<R>* __restrict__ x,
                                                             const int cbits,
                                                             double* __restrict__ partial) {
  __shared__ double red[4];
  const uint32_t tid = threadIdx.x;
  const uint32_t chunk = 1u << cbits;
  const size_t base = (size_t)blockIdx.x << cbits;
  double tot = 0.0, reg[4] = {0.0, 0.0, 0.0, 0.0};
  for (int s = 0; s < 16; ++s) {
    const uint32_t e = tid + kBlock * s;
    if (e >= chunk) break;
    const double p = prob<R>(x[base + e]);
    tot += p;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((s >> q) & 1) reg[q] += p;
  }
  double* out = partial + blockIdx.x;
  const size_t nchunk = gridDim.x;
  const double t_all = block_sum_256(tot, red);
  if (tid == 0) out[0] = t_all;
  for (int p = 0; p < 8; ++p) {
    const double t = block_sum_256(((tid >> p) & 1) ? tot : 0.0, red);
    if (tid == 0) out[(1 + p) * nchunk] = t;
  }
  for (int q = 0; q < 4; ++q) {
    const double t = block_sum_256(reg[q], red);
    if (tid == 0) out[(9 + q) * nchunk] = t;
  }
}

// Second stage, one workgroup per output (0: the total, 1 + p: bit p): thread t sums chunks t,
// t + 256, ... (four independent chains), then a fixed tree.  One workgroup that looped over
// the outputs took 174 us at 25 atoms and 0.69 ms at 27, longer than the pass over the state (now
// 12 us at 25).
__global__ __launch_bounds__(kBlock) void occ_finalize_kernel(const double* __restrict__ partial,
                                                              const int64_t nchunk,
                                                              const int cbits,
                                                              double* __restrict__ out) {
  __shared__ double red[4];
  const int p = (int)blockIdx.x - 1;
  const double* c = partial + (p >= 0 && p < cbits ? (int64_t)(1 + p) * nchunk : 0);
  const int sh = p - cbits;  // >= 0: the total of the chunks whose index bit sh is set
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t ch = threadIdx.x; ch < nchunk; ch += 4 * kBlock) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t w = ch + j * kBlock;
      if (w < nchunk && (sh < 0 || ((w >> sh) & 1))) acc[j] += c[w];
    }
  }
  const double t = block_sum_256((acc[0] + acc[1]) + (acc[2] + acc[3]), red);
  if (threadIdx.x == 0) out[blockIdx.x] = t;
}

// --------------------------------------------------------------------------- correlations
// <n_i n_j> numerators.  Per chunk of 2^C amplitudes the low C bits vary and the bits above
// are constant, so a chunk contributes its total T, its single-bit sums S_p (p < C) and its
// pair sums P_pq (p < q < C); pairs involving high bits follow from T and S_p and the chunk
// index.  Thread t holds 2^SB amplitudes e = t + 256 s: bits 0..7 of e are t's, the SB others
// s's (C = 8 + SB).  Each thread keeps its total, its sums over the s bits and over pairs of s
// bits; the chunk's values are then sums over threads in a fixed order, a loop of 256 LDS reads
// per value.  That loop bounds the kernel on chunks of 2^12 (187 us at 25 atoms complex128, 2.9
// TB/s), so from 20 atoms on, where they still fill the chip, chunks of 2^14 run it a quarter
// as often (146 us, 3.7 TB/s).  (On 2^15 the 29 sums per thread take 59 KB of LDS: two workgroups per CU.)
template <int SB>
struct Corr {
  static constexpr int C = 8 + SB, NV = 1 + SB + SB * (SB - 1) / 2;
  static constexpr int kSlots = 1 + C + C * (C - 1) / 2;
  static __device__ __forceinline__ int pair_slot(int p, int q) {  // p < q < C
    return 1 + C + p * C - p * (p + 1) / 2 + (q - p - 1);
  }
  static constexpr __host__ __device__ int s_pair(int a, int b) {  // a < b < SB
    return 1 + SB + a * SB - a * (a + 1) / 2 + (b - a - 1);
  }
};

// partial[slot * nchunk + chunk]
template <class R, int SB>
__global__ __launch_bounds__(kBlock) void corr_partial_kernel(const Cx<R>* __restrict__ x,
                                                              const int cbits,
                                                              double* __restrict__ partial) {
  using G = Corr<SB>;
  __shared__ double th[G::NV][kBlock];
  const uint32_t tid = threadIdx.x;
  const uint32_t chunk = 1u << cbits;
  const size_t base = (size_t)blockIdx.x << cbits;
  double v[G::NV];
#pragma unroll
  for (int j = 0; j < G::NV; ++j) v[j] = 0.0;
  // 16 amplitudes at a time: their four s bits first, then the group's sums join the others
  for (uint32_t g = 0; g < (1u << (SB - 4)); ++g) {
    if (tid + kBlock * 16 * g >= chunk) break;
    double w[Corr<4>::NV];
#pragma unroll
    for (int j = 0; j < Corr<4>::NV; ++j) w[j] = 0.0;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const uint32_t e = tid + kBlock * (16 * g + s);
      const double p = e < chunk ? prob<R>(x[base + e]) : 0.0;
      w[0] += p;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if ((s >> q) & 1) w[1 + q] += p;
#pragma unroll
        for (int r = q + 1; r < 4; ++r)
          if (((s >> q) & 1) && ((s >> r) & 1)) w[Corr<4>::s_pair(q, r)] += p;
      }
    }
    v[0] += w[0];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[1 + q] += w[1 + q];
#pragma unroll
      for (int r = q + 1; r < 4; ++r) v[G::s_pair(q, r)] += w[Corr<4>::s_pair(q, r)];
    }
#pragma unroll
    for (int r = 4; r < SB; ++r) {
      if (!((g >> (r - 4)) & 1)) continue;
      v[1 + r] += w[0];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[G::s_pair(q, r)] += w[1 + q];
#pragma unroll
      for (int q = 4; q < r; ++q)
        if ((g >> (q - 4)) & 1) v[G::s_pair(q, r)] += w[0];
    }
  }
#pragma unroll
  for (int j = 0; j < G::NV; ++j) th[j][tid] = v[j];
  __syncthreads();
  if (tid < G::kSlots) {
    // which per-thread value, and which thread bits must be set, for slot tid
    int src = 0;
    uint32_t need = 0;
    const int slot = (int)tid;
    if (slot > G::C) {  // pair p < q
      int p = 0, q = 1;
      for (int a = 0; a < G::C; ++a)
        for (int b = a + 1; b < G::C; ++b)
          if (G::pair_slot(a, b) == slot) p = a, q = b;
      if (q < 8) need = (1u << p) | (1u << q);
      else if (p < 8) need = 1u << p, src = 1 + (q - 8);
      else src = G::s_pair(p - 8, q - 8);
    } else if (slot > 8) {  // single bit of s
      src = slot - 8;
    } else if (slot > 0) {  // single bit of t
      need = 1u << (slot - 1);
    }
    double acc = 0.0;
#pragma unroll 8
    for (uint32_t t = 0; t < kBlock; ++t) {
      const double a = th[src][t];
      acc += (t & need) == need ? a : 0.0;
    }
    partial[(size_t)slot * gridDim.x + blockIdx.x] = acc;
  }
}

// out[0] = total; out[1 + p * n + q] (p <= q, bit positions) = sum |x_b|^2 b_p b_q.  One
// workgroup per output; thread t sums chunks t, t + 256, ... then a fixed tree.
template <int SB>
__global__ __launch_bounds__(kBlock) void corr_finalize_kernel(const double* __restrict__ partial,
                                                               const int64_t nchunk, const int n,
                                                               const int cbits,
                                                               double* __restrict__ out) {
  __shared__ double red[4];
  int p = -1, q = -1;  // workgroup 0: the total
  if (blockIdx.x > 0) {
    int w = (int)blockIdx.x - 1;
    for (int a = 0; a < n && p < 0; ++a)
      for (int b = a; b < n; ++b, --w)
        if (w == 0) {
          p = a, q = b;
          break;
        }
  }
  // the slot to sum, and the chunk-index bits that must be set
  int slot = 0;
  int64_t need = 0;
  if (p >= 0 && q < cbits) {
    slot = p == q ? 1 + p : Corr<SB>::pair_slot(p, q);
  } else if (p >= 0) {
    need = int64_t(1) << (q - cbits);
    if (p < cbits) slot = 1 + p;
    else need |= int64_t(1) << (p - cbits);
  }
  const double* c = partial + (int64_t)slot * nchunk;
  double acc = 0.0;
  for (int64_t ch = threadIdx.x; ch < nchunk; ch += kBlock)
    if ((ch & need) == need) acc += c[ch];
  const double t = block_sum_256(acc, red);
  if (threadIdx.x == 0) {
    if (p < 0) out[0] = t;
    else out[1 + p * n + q] = t;
  }
}

template <int SB>
hipError_t correlations_sb(int prec, int n, const void* x, double* scratch, double** out_dev,
                           hipStream_t s) {
  const int cbits = n < Corr<SB>::C ? n : Corr<SB>::C;
  const uint32_t nchunk = 1u << (n - cbits);
  double* out = scratch + (size_t)nchunk * Corr<SB>::kSlots;
  if (prec == kC128)
    hipLaunchKernelGGL((corr_partial_kernel<double, SB>), dim3(nchunk), dim3(kBlock), 0, s,
                       (const double2*)x, cbits, scratch);
  else
    hipLaunchKernelGGL((corr_partial_kernel<float, SB>), dim3(nchunk), dim3(kBlock), 0, s,
                       (const float2*)x, cbits, scratch);
  hipLaunchKernelGGL(corr_finalize_kernel<SB>, dim3(1 + n * (n + 1) / 2), dim3(kBlock), 0, s,
                     scratch, (int64_t)nchunk, n, cbits, out);
  *out_dev = out;
  return hipGetLastError();
}

constexpr int kCorrWideAtoms = 20;  // 2^14-amplitude chunks from here on

// ------------------------------------------------------------------------------- sampling
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t s) {
  uint64_t z = seed + (s + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// LDS position of probability e of a chunk: one word of padding per 16, so that a thread's 16
// consecutive values and its neighbours' start in different banks.
__device__ __forceinline__ uint32_t padded(uint32_t e) { return e + (e >> 4); }
constexpr int kPaddedChunk = (1 << kChunkBits) + (1 << (kChunkBits - 4));

// Exclusive prefix of tsum[0..count) on top of `run`, in thread order (thread 0; 16 values at a
// time through registers, so that the adds do not wait for the LDS); returns the end.
__device__ __forceinline__ double serial_scan(double* tsum, double run, int count = kBlock) {
  for (int t0 = 0; t0 < count; t0 += 16) {
    double v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = tsum[t0 + j];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const double w = v[j];
      v[j] = run;
      run += w;
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) tsum[t0 + j] = v[j];
  }
  return run;
}

// Sum of |x|^2 per chunk.  Thread t adds amplitudes 16 t .. 16 t + 15, the order of the in-block
// scan of sample_kernel; they reach it through LDS, because loads of 16 consecutive
// amplitudes per lane use a sixteenth of each cache line they touch (25 atoms complex128: 565
// us that way, 0.95 TB/s; now 101 us, 5.3 TB/s).
template <class R>
__global__ __launch_bounds__(kBlock) void block_prob_kernel(const Cx<R>* __restrict__ x,
                                                            const int cbits,
                                                            double* __restrict__ bsum) {
  __shared__ double red[4];
  __shared__ double pr[kPaddedChunk];
  const uint32_t chunk = 1u << cbits;
  const size_t base = (size_t)blockIdx.x << cbits;
#pragma unroll
  for (uint32_t j = 0; j < 16; ++j) {
    const uint32_t e = threadIdx.x + kBlock * j;
    pr[padded(e)] = e < chunk ? prob<R>(x[base + e]) : 0.0;
  }
  __syncthreads();
  double acc = 0.0;
#pragma unroll
  for (uint32_t j = 0; j < 16; ++j) acc += pr[padded(threadIdx.x * 16 + j)];
  const double t = block_sum_256(acc, red);
  if (threadIdx.x == 0) bsum[blockIdx.x] = t;
}

// Exclusive scan of nb block sums into pre[0..nb], pre[nb] = total.  One workgroup; thread t
// owns a contiguous range, read eight values at a time.
__global__ __launch_bounds__(kBlock) void block_scan_kernel(const double* __restrict__ bsum,
                                                            const int64_t nb,
                                                            double* __restrict__ pre) {
  __shared__ double tsum[kBlock];
  const int64_t per = (nb + kBlock - 1) / kBlock;
  const int64_t lo = (int64_t)threadIdx.x * per;
  const int64_t hi = lo + per < nb ? lo + per : nb;
  double acc = 0.0;
  int64_t i = lo;
  for (; i + 8 <= hi; i += 8) {
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = bsum[i + j];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc += v[j];
  }
  for (; i < hi; ++i) acc += bsum[i];
  tsum[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x == 0) pre[nb] = serial_scan(tsum, 0.0);
  __syncthreads();
  double run = tsum[threadIdx.x];
  i = lo;
  for (; i + 8 <= hi; i += 8) {
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = bsum[i + j];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      pre[i + j] = run;
      run += v[j];
    }
  }
  for (; i < hi; ++i) {
    pre[i] = run;
    run += bsum[i];
  }
}

// One workgroup per shot.  STAGED: the chunk's probabilities reach their threads through LDS (as in
// block_prob_kernel).  A state of up to 2^kDirectBits amplitudes, one chunk, is read as it is: its few
// lines stay in the caches, and without the staging's 35 KB and the search more than four workgroups
// share a CU: 200 000 shots of 3 / 11 atoms 0.49 / 1.06 ms, staged 1.58 / 1.88 (12 atoms staged 2.05,
// as it is 2.3).
constexpr int kDirectBits = 11;
template <class R, bool STAGED>
__global__ __launch_bounds__(kBlock) void sample_kernel(const Cx<R>* __restrict__ x,
                                                        const int cbits, const int64_t nb,
                                                        const double* __restrict__ pre,
                                                        const double* __restrict__ bsum,
                                                        const uint64_t seed,
                                                        uint64_t* __restrict__ idx) {
  __shared__ double tsum[kBlock];
  __shared__ double pr[STAGED ? kPaddedChunk : 1];
  __shared__ int64_t blk_sh;
  __shared__ int fallback_sh;
  __shared__ unsigned int cand, last_sh, hit;
  const uint32_t tid = threadIdx.x;
  const uint32_t chunk = 1u << cbits;
  const double u = (double)(splitmix64_at(seed, blockIdx.x) >> 11) * 0x1.0p-53;
  const double target = u * pre[nb];
  // smallest block whose inclusive prefix exceeds the target: the prefixes do not decrease, so
  // each round tests 256 spaced candidates of the open range and keeps the gap below the first
  // that does (one memory latency per factor of 256 where a bisection takes eight)
  int64_t lo = 0, hi = nb;  // answer in [lo, hi]; hi == nb means none
  if constexpr (!STAGED) lo = hi = pre[1] > target ? 0 : 1;  // a short chunk is the only one
  while (lo < hi) {
    if (tid == 0) hit = kBlock;
    __syncthreads();
    const int64_t step = (hi - lo + kBlock - 1) / kBlock;
    const int64_t c = lo + (int64_t)(tid + 1) * step - 1;  // the last block of gap tid
    if (c < hi && pre[c + 1] > target) atomicMin(&hit, tid);
    __syncthreads();
    const int64_t h = hit;
    __syncthreads();
    const int64_t glo = lo + h * step;  // the answer lies in gap h, or beyond the last full one
    if (h < kBlock) {
      hi = glo + step - 1;
      lo = glo;
    } else {
      const int64_t full = (hi - lo) / step;  // gaps whose last block was tested
      lo += full * step;
      if (step == 1) lo = hi;
    }
  }
  if (tid == 0) {
    int fb = 0;
    if (lo == nb) {  // no block: fall back to the last block with mass
      fb = 1;
      lo = nb - 1;
      while (lo > 0 && !(bsum[lo] > 0.0)) --lo;
    }
    blk_sh = lo;
    fallback_sh = fb;
    cand = 0xFFFFFFFFu;
    last_sh = 0u;
  }
  __syncthreads();
  const int64_t blk = blk_sh;
  const size_t base = (size_t)blk << cbits;
  if constexpr (STAGED) {
#pragma unroll
    for (uint32_t j = 0; j < 16; ++j) {
      const uint32_t e = tid + kBlock * j;
      pr[padded(e)] = e < chunk ? prob<R>(x[base + e]) : 0.0;
    }
    __syncthreads();
  }
  double p[16];
  double own = 0.0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint32_t e = tid * 16 + j;
    if constexpr (STAGED) p[j] = pr[padded(e)];
    else p[j] = e < chunk ? prob<R>(x[base + e]) : 0.0;
    own += p[j];
  }
  tsum[tid] = own;
  __syncthreads();
  // (threads beyond a short chunk hold no probability and need no prefix)
  if (tid == 0) serial_scan(tsum, pre[blk], STAGED ? kBlock : (int)((chunk + 15) / 16));
  __syncthreads();
  if (!fallback_sh) {
    double c = tsum[tid];
    for (int j = 0; j < 16; ++j) {
      c += p[j];
      if (c > target && p[j] > 0.0) {
        atomicMin(&cand, tid * 16 + j);
        break;
      }
    }
  }
  __syncthreads();
  const unsigned int found = cand;  // every thread reads before anyone writes last_sh
  if (found == 0xFFFFFFFFu) {       // rounding left no index: take the last one with mass
    for (int j = 15; j >= 0; --j) {
      if (p[j] > 0.0) {
        atomicMax(&last_sh, tid * 16 + j + 1);  // +1: zero means "no mass in this block"
        break;
      }
    }
    __syncthreads();
    if (tid == 0) idx[blockIdx.x] = (uint64_t)base + (last_sh > 0 ? last_sh - 1 : 0);
    return;
  }
  if (tid == 0) idx[blockIdx.x] = (uint64_t)base + found;
}

template <class R>
void launch_samples(const void* x, int cbits, int64_t nb, const double* pre, const double* bsum,
                    uint64_t seed, int64_t shots, uint64_t* idx, hipStream_t s) {
  if (cbits > kDirectBits)
    hipLaunchKernelGGL((sample_kernel<R, true>), dim3((uint32_t)shots), dim3(kBlock), 0, s,
                       (const Cx<R>*)x, cbits, nb, pre, bsum, seed, idx);
  else
    hipLaunchKernelGGL((sample_kernel<R, false>), dim3((uint32_t)shots), dim3(kBlock), 0, s,
                       (const Cx<R>*)x, cbits, nb, pre, bsum, seed, idx);
}

// Scratch of the allocation-free sampling entry point: the block sums and their exclusive
// scan for up to kMaxAtoms atoms, then the drawn indices of up to kStaticMaxShots shots
// (4.7 MB, held by every device the library runs on until the process ends).
constexpr int64_t kStaticBlocks = int64_t(1) << (kMaxAtoms - kChunkBits);
constexpr size_t kStaticIdxOffset = (size_t)(2 * kStaticBlocks + 1 + 31) / 32 * 32;  // doubles
constexpr size_t kStaticDoubles = kStaticIdxOffset + kStaticMaxShots;
static __device__ __align__(256) double scratch[kStaticDoubles];

}  // namespace

int static_sample_scratch(int device, void** out) {
  // The array's host-side name is not a device address: its address on each device comes
  // from the runtime, once per device, with that device current.
  static std::mutex mu;
  static void* addr[64] = {};
  if (device < 0 || device >= 64) return -1;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return -1;
    addr[device] = p;
  }
  *out = addr[device];
  return 0;
}

size_t static_sample_idx_offset_bytes() { return kStaticIdxOffset * sizeof(double); }

int64_t occ_num_partials(int n) {
  const int cbits = n < kChunkBits ? n : kChunkBits;
  return (int64_t(1) << (n - cbits)) * kOccStride;
}

hipError_t occupations(int prec, int n, const void* x, double* partial, double* out,
                       hipStream_t s) {
  const int cbits = n < kChunkBits ? n : kChunkBits;
  const uint32_t nchunk = 1u << (n - cbits);
  if (prec == kC128)
    hipLaunchKernelGGL(occ_partial_kernel<double>, dim3(nchunk), dim3(kBlock), 0, s,
                       (const double2*)x, cbits, partial);
  else
    hipLaunchKernelGGL(occ_partial_kernel<float>, dim3(nchunk), dim3(kBlock), 0, s,
                       (const float2*)x, cbits, partial);
  hipLaunchKernelGGL(occ_finalize_kernel, dim3(n + 1), dim3(kBlock), 0, s, partial,
                     (int64_t)nchunk, cbits, out);
  return hipGetLastError();
}

int64_t corr_scratch_doubles(int n) {
  const bool wide = n >= kCorrWideAtoms;
  const int C = wide ? Corr<6>::C : Corr<4>::C;
  const int cbits = n < C ? n : C;
  return (int64_t(1) << (n - cbits)) * (wide ? Corr<6>::kSlots : Corr<4>::kSlots) + 1 +
         (int64_t)n * n;
}

hipError_t correlations(int prec, int n, const void* x, double* scratch, double** out_dev,
                        hipStream_t s) {
  return n >= kCorrWideAtoms ? correlations_sb<6>(prec, n, x, scratch, out_dev, s)
                             : correlations_sb<4>(prec, n, x, scratch, out_dev, s);
}

int64_t sample_scratch_doubles(int n) {
  const int cbits = n < kChunkBits ? n : kChunkBits;
  const int64_t nb = int64_t(1) << (n - cbits);
  return 2 * nb + 1;
}

hipError_t sample(int prec, int n, const void* x, uint64_t seed, int shots, double* scratch,
                  uint64_t* idx, hipStream_t s) {
  const int cbits = n < kChunkBits ? n : kChunkBits;
  const int64_t nb = int64_t(1) << (n - cbits);
  double* bsum = scratch;
  double* pre = scratch + nb;
  if (prec == kC128)
    hipLaunchKernelGGL(block_prob_kernel<double>, dim3((uint32_t)nb), dim3(kBlock), 0, s,
                       (const double2*)x, cbits, bsum);
  else
    hipLaunchKernelGGL(block_prob_kernel<float>, dim3((uint32_t)nb), dim3(kBlock), 0, s,
                       (const float2*)x, cbits, bsum);
  hipLaunchKernelGGL(block_scan_kernel, dim3(1), dim3(kBlock), 0, s, bsum, nb, pre);
  if (shots > 0) {
    if (prec == kC128) launch_samples<double>(x, cbits, nb, pre, bsum, seed, shots, idx, s);
    else launch_samples<float>(x, cbits, nb, pre, bsum, seed, shots, idx, s);
  }
  return hipGetLastError();
}

}  // namespace rsv
