// Gram-Schmidt kernels of the Arnoldi process (see arnoldi.h): the inner products of a new vector
// with the whole basis, and its update.
//
// Both are streams over the basis (HBM-bound for density matrices of 11 atoms and more,
// launch-bound for small ones).  The Gram-Schmidt coefficients never leave the device: the update
// takes them from the inner products in device memory, so a run of iterations is queued without a
// host round trip.  For vectors of up to 2^kSmallBits elements every workgroup sums the (at most
// kSmallParts) partial sums it needs itself, which makes an iteration two launches besides the
// operator; longer vectors take a second-stage launch each (2048 partials per value).
//
// y = s_j Op u_j is not orthogonalised as it is: for a skew-Hermitian operator it holds
// -beta_{j-1} v_{j-1} (the Lanczos coupling), usually its largest part, and where the next beta
// is smaller its removal cancels digits, so that the criterion for a second pass was met in
// every second iteration (12 atoms: 12 of 28) by that one known component.  So both kernels
// work on y1 = y + beta_{j-1} v_{j-1}; the inner products then measure what is left, the
// coefficient of v_{j-1} is the sum of both parts, and the criterion compares with |y1|.  For
// another operator the guess is merely a poor one: the result is the same, with more second passes.
// With `shift` (the gradients' operator -i H, whose mean energy is far from zero) the diagonal
// entry of the iteration before is taken out along u_j in the same way.
//
// Measured, with the host part of arnoldi.cpp, against inner products and coefficients that went
// through the host, a second pass by |y| and the whole exponential of H_m at every dimension: a
// Lindblad step of 12 atoms (28 vectors of 256 MiB) 109 -> 72 ms (35 ms with the Hermitian forms
// below), 20 steps of 6 atoms (12 vectors of 64 KiB each) 26 -> 5.5 ms.
#include <type_traits>

#include "arnoldi.h"
#include "device_common.h"
#include "herm_tile.h"

namespace rsv {
namespace {

template <class R>
__device__ __forceinline__ const Cx<R>* basis_vec(const ArnoldiStep& a, int i) {
  return i == 0 ? (const Cx<R>*)a.v0 : (const Cx<R>*)a.base + (size_t)i * a.stride;
}

// Sum of p[0..n), n <= kSmallParts, by every wave for itself (fixed order, uniform).
__device__ __forceinline__ double wave_parts(const double* p, int n) {
  const int lane = threadIdx.x & 63;
  double v = lane < n ? p[lane] : 0.0;
#pragma unroll
  for (int k = 64; k < kSmallParts; k += 64) v += lane + k < n ? p[lane + k] : 0.0;
  return wave_total(v);
}

struct Scales {
  double f, g;    // y1 = f w + g u_{j-1} + (hr + i hi) u_j
  double hr, hi;
};

// The coefficients of y1, with |u_j|^2 from its partial sums where they are not summed yet.
__device__ __forceinline__ Scales scales(const ArnoldiStep& a, double n2) {
  if (a.again) return Scales{1.0, 0.0, 0.0, 0.0};
  const double s = 1.0 / sqrt(n2);
  const bool sh = a.shift && a.j > 0;
  return Scales{s, a.j > 0 ? sqrt(n2) / sqrt(a.nrm2[a.j - 1]) : 0.0,
                sh ? -s * a.diag[2 * a.j - 2] : 0.0, sh ? -s * a.diag[2 * a.j - 1] : 0.0};
}

// Partial inner products <u_i, y1> (i <= j) and <y1, y1> (i = j + 1) of group blockIdx.y.
template <class R>
__global__ __launch_bounds__(kBlock) void arnoldi_dots_kernel(const ArnoldiStep a) {
  constexpr int G = kArnoldiGroup;
  __shared__ double red[16][2 * G];  // per row of 16 lanes
  double n2;
  if (!a.again && a.nparts > 0) {
    n2 = wave_parts(a.npart, a.nparts);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) a.nrm2[a.j] = n2;
  } else {
    n2 = a.nrm2[a.j];
  }
  const Scales sc = scales(a, n2);
  const Cx<R>* w = (const Cx<R>*)a.w;
  const Cx<R>* prev = sc.g != 0.0 ? basis_vec<R>(a, a.j - 1) : nullptr;
  const Cx<R>* own = sc.hr != 0.0 || sc.hi != 0.0 ? basis_vec<R>(a, a.j) : nullptr;
  const int i0 = blockIdx.y * G, total = a.j + 2;
  const Cx<R>* x[G];
#pragma unroll
  for (int g = 0; g < G; ++g) x[g] = i0 + g <= a.j ? basis_vec<R>(a, i0 + g) : nullptr;
  double acc[2 * G];
#pragma unroll
  for (int q = 0; q < 2 * G; ++q) acc[q] = 0.0;
  const size_t stride = (size_t)gridDim.x * kBlock;
  // U elements at a time, their loads in flight together
  auto elements = [&](size_t e0, auto ux) {
    constexpr int U = decltype(ux)::value;
    double yr[U], yi[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const size_t e = e0 + q * stride;
      const Cx<R> we = w[e];
      yr[q] = sc.f * (double)we.x;
      yi[q] = sc.f * (double)we.y;
      if (prev) {
        const Cx<R> pe = prev[e];
        yr[q] += sc.g * (double)pe.x;
        yi[q] += sc.g * (double)pe.y;
      }
      if (own) {
        const Cx<R> oe = own[e];
        yr[q] += sc.hr * (double)oe.x - sc.hi * (double)oe.y;
        yi[q] += sc.hr * (double)oe.y + sc.hi * (double)oe.x;
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (x[g]) {
        Cx<R> xe[U];
#pragma unroll
        for (int q = 0; q < U; ++q) xe[q] = x[g][e0 + q * stride];
#pragma unroll
        for (int q = 0; q < U; ++q) {
          acc[2 * g] += (double)xe[q].x * yr[q] + (double)xe[q].y * yi[q];
          acc[2 * g + 1] += (double)xe[q].x * yi[q] - (double)xe[q].y * yr[q];
        }
      } else if (i0 + g == a.j + 1) {
#pragma unroll
        for (int q = 0; q < U; ++q) acc[2 * g] += yr[q] * yr[q] + yi[q] * yi[q];
      }
    }
  };
  size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
  for (; e + stride < a.count; e += 2 * stride) elements(e, std::integral_constant<int, 2>());
  for (; e < a.count; e += stride) elements(e, std::integral_constant<int, 1>());
  // (DPP adds inside rows of 16 lanes: a shuffle tree over the wave for 16 values costs more than
  // the loads at these sizes)
#pragma unroll
  for (int q = 0; q < 2 * G; ++q) {
    const double v = row_reduce(acc[q], OpAdd());
    if ((threadIdx.x & 15) == 0) red[threadIdx.x >> 4][q] = v;
  }
  __syncthreads();
  if (threadIdx.x < 2 * G && i0 + (int)(threadIdx.x >> 1) < total) {
    const int q = threadIdx.x;
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) v += red[r][q];
    a.part[(size_t)(2 * i0 + q) * gridDim.x + blockIdx.x] = v;
  }
}

// u_{j+1} = y1 - sum_i v_i <v_i, y1>, rounded once, and the partials of |u_{j+1}|^2 (again: in
// place on u_{j+1}, with the inner products of the second pass).
template <class R>
__global__ __launch_bounds__(kBlock) void arnoldi_update_kernel(const ArnoldiStep a) {
  __shared__ double cr[kMaxKrylov + 2], ci[kMaxKrylov + 2], red[4];
  const int rows = 2 * (a.j + 2), tid = threadIdx.x;
  if (a.dparts > 0) {
    // sum the partial inner products: eight lanes per value, every load of a lane in flight (one
    // wave per value took a memory latency for each of its turns)
    static_assert(kSmallParts % 128 == 0, "turns of 16 partials per lane");
    for (int r0 = 0; r0 < rows; r0 += kBlock / 8) {
      const int r = r0 + (tid >> 3), l = tid & 7;
      const double* q = a.part + (size_t)(r < rows ? r : 0) * a.dparts;
      double t = 0.0;
      for (int p0 = l; p0 < a.dparts; p0 += 128) {
        double v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = p0 + 8 * k < a.dparts ? q[p0 + 8 * k] : 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += v[k];
      }
      t += dpp<kDppXor1>(t);
      t += dpp<kDppXor2>(t);
      t += dpp<kDppHalfMirror>(t);
      if (l == 0 && r < rows) ((r & 1) ? ci : cr)[r >> 1] = t;
    }
    __syncthreads();
    if (blockIdx.x == 0 && tid < kBlock)
      for (int r = tid; r < rows; r += kBlock) a.dots[r] = (r & 1) ? ci[r >> 1] : cr[r >> 1];
  } else {
    for (int r = tid; r < rows; r += kBlock) ((r & 1) ? ci : cr)[r >> 1] = a.dots[r];
    __syncthreads();
  }
  const Scales sc = scales(a, a.nrm2[a.j]);
  if (!a.again && a.shift && blockIdx.x == 0 && tid == 0) {
    // h_jj = <v_j, y>: what the inner product measured and what was taken out before it
    a.diag[2 * a.j] = sc.f * cr[a.j] + (a.j > 0 ? a.diag[2 * a.j - 2] : 0.0);
    a.diag[2 * a.j + 1] = sc.f * ci[a.j] + (a.j > 0 ? a.diag[2 * a.j - 1] : 0.0);
  }
  __syncthreads();
  if (tid <= a.j) {
    const double s2 = 1.0 / a.nrm2[tid];  // v_i = u_i / |u_i|
    cr[tid] = -s2 * cr[tid] + (tid == a.j - 1 ? sc.g : tid == a.j ? sc.hr : 0.0);
    ci[tid] = -s2 * ci[tid] + (tid == a.j ? sc.hi : 0.0);
  }
  __syncthreads();
  const Cx<R>* w = (const Cx<R>*)a.w;
  Cx<R>* out = (Cx<R>*)a.base + (size_t)(a.j + 1) * a.stride;
  double acc = 0.0;
  const size_t stride = (size_t)gridDim.x * kBlock;
  auto elements = [&](size_t e0, auto ux) {
    constexpr int U = decltype(ux)::value;
    double re[U], im[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const Cx<R> we = w[e0 + q * stride], x0 = ((const Cx<R>*)a.v0)[e0 + q * stride];
      re[q] = sc.f * (double)we.x + (cr[0] * (double)x0.x - ci[0] * (double)x0.y);
      im[q] = sc.f * (double)we.y + (cr[0] * (double)x0.y + ci[0] * (double)x0.x);
    }
    const Cx<R>* x = (const Cx<R>*)a.base + a.stride + e0;
#pragma unroll 4
    for (int i = 1; i <= a.j; ++i, x += a.stride) {
      Cx<R> xe[U];
#pragma unroll
      for (int q = 0; q < U; ++q) xe[q] = x[q * stride];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        re[q] += cr[i] * (double)xe[q].x - ci[i] * (double)xe[q].y;
        im[q] += cr[i] * (double)xe[q].y + ci[i] * (double)xe[q].x;
      }
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      Cx<R> r;
      r.x = (R)re[q];
      r.y = (R)im[q];
      out[e0 + q * stride] = r;
      acc = norm_add(acc, (double)r.x, (double)r.y);
    }
  };
  size_t e = (size_t)blockIdx.x * kBlock + tid;
  for (; e + stride < a.count; e += 2 * stride) elements(e, std::integral_constant<int, 2>());
  for (; e < a.count; e += stride) elements(e, std::integral_constant<int, 1>());
  const double t = block_sum_256(acc, red);
  if (tid == 0) a.npart_out[blockIdx.x] = t;
}

// ---------------------------------------------------------------------- Hermitian matrices
// The Liouvillian maps Hermitian matrices to Hermitian matrices, so from a Hermitian density
// matrix every Krylov vector is one, and the inner product of two is real and follows from one
// triangle.  These forms of the two kernels read the upper triangle's tiles only: half the bytes of
// the basis, which bound both.  The update writes both triangles, because the operator reads whole
// rows and columns.  Means over a step of 12 atoms complex128 (28 vectors of 256 MiB): inner
// products 855 -> 394 us, update 905 -> 490 us, both at 4.2 to 5.1 TB/s in the last iterations;
// with the operator's half (527 -> 245 us) the step went from 72 to 35 ms.
template <class R>
__global__ __launch_bounds__(kBlock) void herm_dots_kernel(const ArnoldiStep a, const uint32_t tiles) {
  constexpr int G = kHermGroup;
  __shared__ double red[16][G];
  const Scales sc = scales(a, a.nrm2[a.j]);
  const Cx<R>* w = (const Cx<R>*)a.w;
  const Cx<R>* prev = sc.g != 0.0 ? basis_vec<R>(a, a.j - 1) : nullptr;
  const int i0 = blockIdx.y * G, total = a.j + 2;
  double acc[G];
#pragma unroll
  for (int q = 0; q < G; ++q) acc[q] = 0.0;
  const uint32_t row0 = threadIdx.x >> 5, col = threadIdx.x & 31;
  const uint32_t b0 = xcd_remap(blockIdx.x, gridDim.x);
  for (uint32_t t = b0; t < tiles; t += gridDim.x) {
    const HermTile h = herm_tile(t, a.herm, true);
    const size_t e0 = h.base + ((size_t)row0 << a.herm) + col;
    double yr[kTileElems], yi[kTileElems];
#pragma unroll
    for (int q = 0; q < kTileElems; ++q) {
      const size_t e = e0 + ((size_t)(kTileRows * q) << a.herm);
      const Cx<R> we = w[e];
      const double wt = herm_weight(h, row0 + kTileRows * q, col);
      yr[q] = sc.f * (double)we.x;
      yi[q] = sc.f * (double)we.y;
      if (prev) {
        const Cx<R> pe = prev[e];
        yr[q] += sc.g * (double)pe.x;
        yi[q] += sc.g * (double)pe.y;
      }
      if (i0 + G >= total && i0 < total) {  // this group holds <y1, y1>
        const int self = a.j + 1 - i0;
#pragma unroll
        for (int g = 0; g < G; ++g)
          if (g == self) acc[g] += wt * (yr[q] * yr[q] + yi[q] * yi[q]);
      }
      yr[q] *= wt;
      yi[q] *= wt;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (i0 + g > a.j) continue;
      const Cx<R>* x = basis_vec<R>(a, i0 + g) + e0;
      Cx<R> xe[kTileElems];
#pragma unroll
      for (int q = 0; q < kTileElems; ++q) xe[q] = x[(size_t)(kTileRows * q) << a.herm];
#pragma unroll
      for (int q = 0; q < kTileElems; ++q) acc[g] += (double)xe[q].x * yr[q] + (double)xe[q].y * yi[q];
    }
  }
#pragma unroll
  for (int q = 0; q < G; ++q) {
    const double v = row_reduce(acc[q], OpAdd());
    if ((threadIdx.x & 15) == 0) red[threadIdx.x >> 4][q] = v;
  }
  __syncthreads();
  if (threadIdx.x < G && i0 + (int)threadIdx.x < total) {
    double v = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) v += red[r][threadIdx.x];
    a.part[(size_t)(i0 + threadIdx.x) * gridDim.x + blockIdx.x] = v;
  }
}

template <class R>
__global__ __launch_bounds__(kBlock) void herm_update_kernel(const ArnoldiStep a, const uint32_t tiles) {
  __shared__ double cr[kMaxKrylov + 2], red[4];
  __shared__ Cx<R> lds[kTileSide][kTileSide + 1];
  const int tid = threadIdx.x;
  const Scales sc = scales(a, a.nrm2[a.j]);
  if (tid <= a.j) cr[tid] = -a.dots[tid] / a.nrm2[tid] + (tid == a.j - 1 ? sc.g : 0.0);
  __syncthreads();
  const Cx<R>* w = (const Cx<R>*)a.w;
  Cx<R>* out = (Cx<R>*)a.base + (size_t)(a.j + 1) * a.stride;
  const uint32_t row0 = tid >> 5, col = tid & 31;
  const uint32_t b0 = xcd_remap(blockIdx.x, gridDim.x);
  double acc = 0.0;
  for (uint32_t t = b0; t < tiles; t += gridDim.x) {
    const HermTile h = herm_tile(t, a.herm, true);
    const size_t e0 = h.base + ((size_t)row0 << a.herm) + col;
    double re[kTileElems], im[kTileElems];
#pragma unroll
    for (int q = 0; q < kTileElems; ++q) {
      const size_t e = e0 + ((size_t)(kTileRows * q) << a.herm);
      const Cx<R> we = w[e], x0 = ((const Cx<R>*)a.v0)[e];
      re[q] = sc.f * (double)we.x + cr[0] * (double)x0.x;
      im[q] = sc.f * (double)we.y + cr[0] * (double)x0.y;
    }
    const Cx<R>* x = (const Cx<R>*)a.base + a.stride + e0;
#pragma unroll 2
    for (int i = 1; i <= a.j; ++i, x += a.stride) {
      const double c = cr[i];
      Cx<R> xe[kTileElems];
#pragma unroll
      for (int q = 0; q < kTileElems; ++q) xe[q] = x[(size_t)(kTileRows * q) << a.herm];
#pragma unroll
      for (int q = 0; q < kTileElems; ++q) {
        re[q] += c * (double)xe[q].x;
        im[q] += c * (double)xe[q].y;
      }
    }
    Cx<R> r[kTileElems];
#pragma unroll
    for (int q = 0; q < kTileElems; ++q) {
      const uint32_t row = row0 + kTileRows * q;
      r[q].x = (R)re[q];
      r[q].y = h.R == h.C && row == col ? (R)0 : (R)im[q];
      lds[row][col] = r[q];
      acc += herm_weight(h, row, col) * norm_add(0.0, (double)r[q].x, (double)r[q].y);
    }
    __syncthreads();
    // the conjugate transpose: into the mirrored tile, or the lower half of a diagonal one
    const size_t m0 = ((size_t)(h.C * kTileSide + row0) << a.herm) + h.R * kTileSide + col;
#pragma unroll
    for (int q = 0; q < kTileElems; ++q) {
      const uint32_t row = row0 + kTileRows * q;
      const Cx<R> tr = lds[col][row], cj = {tr.x, -tr.y};
      const size_t e = e0 + ((size_t)(kTileRows * q) << a.herm);
      if (h.R != h.C) {
        out[e] = r[q];
        out[m0 + ((size_t)(kTileRows * q) << a.herm)] = cj;
      } else {
        const bool own = col >= row;
        out[e] = Cx<R>{own ? r[q].x : cj.x, own ? r[q].y : cj.y};
      }
    }
    __syncthreads();
  }
  const double t = block_sum_256(acc, red);
  if (tid == 0) a.npart_out[blockIdx.x] = t;
}

// |u_j|^2 of a small vector for the host, in the order in which the other kernels sum it: the
// coefficients do not depend on where a run of iterations ends.
__global__ __launch_bounds__(64) void arnoldi_norm_kernel(const double* npart, int parts, double* out) {
  const double v = wave_parts(npart, parts);
  if (threadIdx.x == 0) *out = v;
}

// Partials of |x - x^+|^2 and |x|^2 (write = 0), or x <- (x + x^+) / 2 (write = 1).
template <class R>
__global__ __launch_bounds__(kBlock) void hermitise_kernel(Cx<R>* __restrict__ x, const int n,
                                                           const uint32_t tiles, const int write,
                                                           double* __restrict__ part) {
  __shared__ Cx<R> lds[kTileSide][kTileSide + 1];
  __shared__ double red[4];
  const uint32_t tid = threadIdx.x, row0 = tid >> 5, col = tid & 31;
  double diff = 0.0, all = 0.0;
  for (uint32_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const HermTile h = herm_tile(t, n, true);
    const size_t e0 = h.base + ((size_t)row0 << n) + col;
    const size_t m0 = ((size_t)(h.C * kTileSide + row0) << n) + h.R * kTileSide + col;
    Cx<R> v[kTileElems];
#pragma unroll
    for (int q = 0; q < kTileElems; ++q) {
      v[q] = x[e0 + ((size_t)(kTileRows * q) << n)];
      lds[row0 + kTileRows * q][col] = x[m0 + ((size_t)(kTileRows * q) << n)];
    }
    __syncthreads();
    Cx<R> s[kTileElems];
#pragma unroll
    for (int q = 0; q < kTileElems; ++q) {
      const uint32_t row = row0 + kTileRows * q;
      const Cx<R> o = lds[col][row];  // the mirrored element
      const double wt = herm_weight(h, row, col);
      const double dx = (double)v[q].x - (double)o.x, dy = (double)v[q].y + (double)o.y;
      diff += wt * (dx * dx + dy * dy);
      all += 0.5 * wt * ((double)v[q].x * (double)v[q].x + (double)v[q].y * (double)v[q].y +
                         (double)o.x * (double)o.x + (double)o.y * (double)o.y);
      s[q].x = (R)(0.5 * ((double)v[q].x + (double)o.x));
      s[q].y = (R)(0.5 * ((double)v[q].y - (double)o.y));
    }
    __syncthreads();
    if (write) {
#pragma unroll
      for (int q = 0; q < kTileElems; ++q) {
        x[e0 + ((size_t)(kTileRows * q) << n)] = s[q];
        lds[row0 + kTileRows * q][col] = s[q];
      }
      __syncthreads();
      if (h.R != h.C) {
#pragma unroll
        for (int q = 0; q < kTileElems; ++q) {
          const Cx<R> o = lds[col][row0 + kTileRows * q];
          x[m0 + ((size_t)(kTileRows * q) << n)] = Cx<R>{o.x, -o.y};
        }
      }
      __syncthreads();
    }
  }
  if (!write) {
    const double a = block_sum_256(diff, red);
    const double b = block_sum_256(all, red);
    if (tid == 0) {
      part[blockIdx.x] = a;
      part[gridDim.x + blockIdx.x] = b;
    }
  }
}

}  // namespace

int arnoldi_parts(size_t count) {
  if (count <= (size_t(1) << kSmallBits)) {
    // 256 elements per workgroup and more, 4 to kSmallParts of them: the gradients' 2^17 elements
    // take 10.1 + 9.5 us (update, inner products) on 256 workgroups, 13.0 + 11.9 on 128 and 12.4 +
    // 11.0 on 512, whose partial sums every workgroup of the update reads
    size_t g = count / 256;
    return (int)(g < 4 ? 4 : g > kSmallParts ? kSmallParts : g);
  }
  return (int)stream_grid(count, 8);
}

hipError_t arnoldi_dots(int prec, const ArnoldiStep& a, hipStream_t s) {
  if (a.herm) {
    const dim3 g(arnoldi_parts(a.count), (a.j + 2 + kHermGroup - 1) / kHermGroup);
    if (prec == kC128)
      hipLaunchKernelGGL(herm_dots_kernel<double>, g, dim3(kBlock), 0, s, a, herm_tiles(a.herm, true));
    else
      hipLaunchKernelGGL(herm_dots_kernel<float>, g, dim3(kBlock), 0, s, a, herm_tiles(a.herm, true));
    return hipGetLastError();
  }
  const dim3 grid(arnoldi_parts(a.count), (a.j + 2 + kArnoldiGroup - 1) / kArnoldiGroup);
  if (prec == kC128)
    hipLaunchKernelGGL(arnoldi_dots_kernel<double>, grid, dim3(kBlock), 0, s, a);
  else
    hipLaunchKernelGGL(arnoldi_dots_kernel<float>, grid, dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t arnoldi_update(int prec, const ArnoldiStep& a, hipStream_t s) {
  const dim3 grid(arnoldi_parts(a.count));
  if (a.herm) {
    if (prec == kC128)
      hipLaunchKernelGGL(herm_update_kernel<double>, grid, dim3(kBlock), 0, s, a, herm_tiles(a.herm, true));
    else
      hipLaunchKernelGGL(herm_update_kernel<float>, grid, dim3(kBlock), 0, s, a, herm_tiles(a.herm, true));
    return hipGetLastError();
  }
  if (prec == kC128)
    hipLaunchKernelGGL(arnoldi_update_kernel<double>, grid, dim3(kBlock), 0, s, a);
  else
    hipLaunchKernelGGL(arnoldi_update_kernel<float>, grid, dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t arnoldi_norm(const double* npart, int parts, double* out, hipStream_t s) {
  hipLaunchKernelGGL(arnoldi_norm_kernel, dim3(1), dim3(64), 0, s, npart, parts, out);
  return hipGetLastError();
}

hipError_t hermitise(int prec, int n, void* x, bool write, double* part, hipStream_t s) {
  const dim3 grid(arnoldi_parts(size_t(1) << (2 * n)));
  if (prec == kC128)
    hipLaunchKernelGGL(hermitise_kernel<double>, grid, dim3(kBlock), 0, s, (double2*)x, n,
                       herm_tiles(n, true), write ? 1 : 0, part);
  else
    hipLaunchKernelGGL(hermitise_kernel<float>, grid, dim3(kBlock), 0, s, (float2*)x, n,
                       herm_tiles(n, true), write ? 1 : 0, part);
  return hipGetLastError();
}

}  // namespace rsv
