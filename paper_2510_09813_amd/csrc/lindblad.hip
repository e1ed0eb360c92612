// Liouvillian of the Lindblad master equation (Sec. III.A: open-system dynamics by the full
// master equation, evolved with a Krylov method) on the vectorised density matrix.
//
//   d rho / dt = L rho = -i [H_k, rho] + sum_i (L_i rho L_i^+ - 1/2 {L_i^+ L_i, rho})
//
// with H_k the Hamiltonian of eq. (3) for step k and, per atom, relaxation of the Rydberg
// level L_i = sqrt(gamma_r) |0><1|_i and dephasing L_i = sqrt(2 gamma_phi) n_i (coherences of
// one atom decay at gamma_phi).  rho (2^n x 2^n) is stored row-major as a vector of 4^n
// amplitudes, index (r << n) | c, so the row's bits are the high n bits of the index and the
// column's the low n: bit p of r or c is atom n-1-p as in the state vector.  Element (r, c):
//
//   (L rho)_rc = [-i (D_r - D_c) - sum_p (gamma_r (r_p + c_p) / 2 + gamma_phi (r_p xor c_p))] rho_rc
//              + sum_p [ -i h(r_p) rho_{r^p, c}  +  i h(1 - c_p) rho_{r, c^p} ]
//              + gamma_r sum_{p: r_p = c_p = 0} rho_{r|p, c|p}
//
// where D_x = E_x - sum_p delta_p x_p is H's diagonal (E_x the interaction energy of pattern
// x), h(1) = <1|h_p|0> = Omega_p/2 e^{-i phi_p} and h(0) = <0|h_p|1>.  Every element needs
// 3n + 1 inputs; arithmetic is FP64, results are stored in the storage precision, and the
// 4^n vector is at most 4 GiB (n <= 14).  Up to 9 atoms (4 MiB, one L2) one thread per element
// gathers its inputs through the cache; from 10 atoms on, tiles of 32 x 32 go through LDS.
#include "device_common.h"
#include "herm_tile.h"
#include "lindblad.h"

namespace rsv {
namespace {

template <class R, int N>
__global__ __launch_bounds__(kBlock) void liouvillian_kernel(const LindbladCoef c,
                                                             const double* __restrict__ e,
                                                             const Cx<R>* __restrict__ x,
                                                             Cx<R>* __restrict__ y) {
  constexpr int n = N;
  const uint64_t count = uint64_t(1) << (2 * n);
  const uint32_t cmask = (1u << n) - 1u;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < count; idx += stride) {
    const uint32_t r = (uint32_t)(idx >> n), col = (uint32_t)idx & cmask;
    double dr = e[r], dc = e[col], loss = 0.0;
#pragma unroll
    for (int p = 0; p < n; ++p) {
      const uint32_t rp = (r >> p) & 1u, cp = (col >> p) & 1u;
      dr -= rp ? c.delta[p] : 0.0;
      dc -= cp ? c.delta[p] : 0.0;
      loss += 0.5 * c.gamma_r * (double)(rp + cp) + ((rp ^ cp) ? c.gamma_phi : 0.0);
    }
    const Cx<R> v = x[idx];
    // (-i (dr - dc) - loss) * v
    double are = -loss * (double)v.x + (dr - dc) * (double)v.y;
    double aim = -loss * (double)v.y - (dr - dc) * (double)v.x;
#pragma unroll
    for (int p = 0; p < n; ++p) {
      const uint32_t rp = (r >> p) & 1u, cp = (col >> p) & 1u;
      // row flip: -i h(r_p) rho_{r^p, c}
      const Cx<R> a = x[idx ^ (uint64_t(1) << (n + p))];
      const double hr = rp ? c.up_re[p] : c.dn_re[p], hi = rp ? c.up_im[p] : c.dn_im[p];
      // -i (hr + i hi)(a) = (hi a.x + hr a.y) + i (hi a.y - hr a.x)
      are += hi * (double)a.x + hr * (double)a.y;
      aim += hi * (double)a.y - hr * (double)a.x;
      // column flip: +i h(1 - c_p) rho_{r, c^p}
      const Cx<R> b = x[idx ^ (uint64_t(1) << p)];
      const double gr = cp ? c.dn_re[p] : c.up_re[p], gi = cp ? c.dn_im[p] : c.up_im[p];
      // i (gr + i gi)(b) = (-gi b.x - gr b.y) + i (gr b.x - gi b.y)
      are += -gi * (double)b.x - gr * (double)b.y;
      aim += gr * (double)b.x - gi * (double)b.y;
      // relaxation feeds (0, 0) of atom p from (1, 1)
      if (c.gamma_r != 0.0 && !rp && !cp) {
        const Cx<R> q = x[idx | (uint64_t(1) << (n + p)) | (uint64_t(1) << p)];
        are += c.gamma_r * (double)q.x;
        aim += c.gamma_r * (double)q.y;
      }
    }
    Cx<R> o;
    o.x = (R)are;
    o.y = (R)aim;
    y[idx] = o;
  }
}

// The same operator on tiles of 32 x 32 elements, one per 256-thread workgroup, four elements per
// thread.  The flips of the five lowest bits of row and column read the tile in LDS, those of the
// bits above read the neighbouring tiles at the thread's own places (512-byte runs; in row-major
// order of the tiles on one XCD the column flips hit its L2, the row flips the last-level cache).
// The diagonal comes from D of the tile's 32 rows and 32 columns and from popcounts.  REAL: a
// global drive without phase, where the neighbours are summed first and the coupling applied once.
// 12 atoms: 245 us for the upper triangle in complex128 (14 neighbours an element from the caches,
// 7.7 TB/s), 458 us for all of it and 206 us in complex64; the one-thread-per-element form above,
// which forms D and the loss bit by bit and reads all 2n neighbours through the caches, took 535
// and 399 us.  13 atoms: 2.15 and 1.02 ms, against 2.88 and 1.90 ms on runs of 4096 elements.  10
// atoms, the smallest: 23 and 17 us against 29 and 26.  The p loops stay rolled: unrolled, their
// loads took 256 registers and one wave per SIMD.
constexpr int kTileAtoms = 10;

template <class R, int N, bool REAL>
__global__ __launch_bounds__(kBlock, 4) void liouvillian_tile_kernel(const LindbladCoef c,
                                                                  const double* __restrict__ e,
                                                                  const Cx<R>* __restrict__ x,
                                                                  Cx<R>* __restrict__ y,
                                                                  const int upper) {
  using C = Cx<R>;
  __shared__ C tile[kTileSide][kTileSide + 1];
  __shared__ double dd[2][kTileSide];  // D of the rows, of the columns
  const uint32_t tid = threadIdx.x, row0 = tid >> 5, col = tid & 31;
  const HermTile h = herm_tile(xcd_remap(blockIdx.x, gridDim.x), N, upper != 0);
  const uint32_t r0 = h.R * kTileSide, c0 = h.C * kTileSide;
  const C* xt = x + h.base + ((size_t)row0 << N) + col;
#pragma unroll
  for (int q = 0; q < kTileElems; ++q) tile[row0 + kTileRows * q][col] = xt[(size_t)(kTileRows * q) << N];
  double are[kTileElems], aim[kTileElems];
  // REAL: the sum over p of rho_{r^p, c} - rho_{r, c^p}; else the drive's terms themselves
#pragma unroll
  for (int q = 0; q < kTileElems; ++q) are[q] = aim[q] = 0.0;
  // -i h(r_p) rho_{r^p, c} and +i h(1 - c_p) rho_{r, c^p}
  auto row_flip = [&](int q, int p, bool bit, const C& a) {
    if (REAL) {
      are[q] += (double)a.x;
      aim[q] += (double)a.y;
    } else {
      const double hr = bit ? c.up_re[p] : c.dn_re[p], hi = bit ? c.up_im[p] : c.dn_im[p];
      are[q] += hi * (double)a.x + hr * (double)a.y;
      aim[q] += hi * (double)a.y - hr * (double)a.x;
    }
  };
  auto col_flip = [&](int q, int p, bool bit, const C& b) {
    if (REAL) {
      are[q] -= (double)b.x;
      aim[q] -= (double)b.y;
    } else {
      const double gr = bit ? c.dn_re[p] : c.up_re[p], gi = bit ? c.dn_im[p] : c.up_im[p];
      are[q] += -gi * (double)b.x - gr * (double)b.y;
      aim[q] += gr * (double)b.x - gi * (double)b.y;
    }
  };
#pragma unroll 1
  for (int p = 5; p < N; ++p) {
    // (signed distances: the neighbour's tile lies 2^p rows or columns away)
    const bool rb = (r0 >> p) & 1u, cb = (c0 >> p) & 1u;
    const C* xr = xt + (rb ? -((int64_t)1 << (N + p)) : (int64_t)1 << (N + p));
    const C* xc = xt + (cb ? -((int64_t)1 << p) : (int64_t)1 << p);
    C a[kTileElems], b[kTileElems];
#pragma unroll
    for (int q = 0; q < kTileElems; ++q) {
      a[q] = xr[(size_t)(kTileRows * q) << N];
      b[q] = xc[(size_t)(kTileRows * q) << N];
    }
#pragma unroll
    for (int q = 0; q < kTileElems; ++q) {
      row_flip(q, p, rb, a[q]);
      col_flip(q, p, cb, b[q]);
    }
  }
  // relaxation feeds (0, 0) of atom p from (1, 1)
  double fre[kTileElems], fim[kTileElems];
#pragma unroll
  for (int q = 0; q < kTileElems; ++q) fre[q] = fim[q] = 0.0;
  if (c.gamma_r != 0.0) {
#pragma unroll 1
    for (int p = 5; p < N; ++p) {
      if (((r0 | c0) >> p) & 1u) continue;
      const C* xs = xt + ((size_t)1 << (N + p)) + ((size_t)1 << p);
#pragma unroll
      for (int q = 0; q < kTileElems; ++q) {
        const C a = xs[(size_t)(kTileRows * q) << N];
        fre[q] += (double)a.x;
        fim[q] += (double)a.y;
      }
    }
  }
  if (tid < 2 * kTileSide) {
    const uint32_t k = (tid < kTileSide ? r0 : c0) + (tid & 31);
    double d = e[k];
#pragma unroll
    for (int p = 0; p < N; ++p) d -= (k >> p) & 1u ? c.delta[p] : 0.0;
    dd[tid >> 5][tid & 31] = d;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kTileElems; ++q) {
    const uint32_t row = row0 + kTileRows * q;
#pragma unroll 1
    for (int p = 0; p < 5; ++p) {
      row_flip(q, p, (row >> p) & 1u, tile[row ^ (1u << p)][col]);
      col_flip(q, p, (col >> p) & 1u, tile[row][col ^ (1u << p)]);
      if (c.gamma_r != 0.0) {
        const C a = tile[row | (1u << p)][col | (1u << p)];
        const bool on = !(((row | col) >> p) & 1u);
        fre[q] += on ? (double)a.x : 0.0;
        fim[q] += on ? (double)a.y : 0.0;
      }
    }
    const C v = tile[row][col];
    const double diff = dd[0][row] - dd[1][col];
    const uint32_t r = r0 + row, k = c0 + col;
    const double loss = 0.5 * c.gamma_r * (double)(__popc(r) + __popc(k)) + c.gamma_phi * (double)__popc(r ^ k);
    double ore, oim;
    if (REAL) {  // -i h S
      ore = c.up_re[0] * aim[q];
      oim = -c.up_re[0] * are[q];
    } else {
      ore = are[q];
      oim = aim[q];
    }
    ore += c.gamma_r * fre[q] - loss * (double)v.x + diff * (double)v.y;
    oim += c.gamma_r * fim[q] - loss * (double)v.y - diff * (double)v.x;
    y[h.base + ((size_t)row << N) + col] = C{(R)ore, (R)oim};
  }
}

// Diagonal of rho: out[r] = Re rho_rr (FP64), r < 2^n.
template <class R>
__global__ __launch_bounds__(kBlock) void rho_diag_kernel(const Cx<R>* __restrict__ x, const int n,
                                                         double* __restrict__ out) {
  const uint32_t dim = 1u << n;
  for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < dim; r += gridDim.x * blockDim.x)
    out[r] = (double)x[((uint64_t)r << n) | r].x;
}

template <class R, int N>
void launch_liouvillian(const LindbladCoef& c, const double* e, const void* x, void* y, bool upper,
                        hipStream_t s) {
  if constexpr (N >= kTileAtoms) {
    bool real = true;  // one real coupling for every atom
    for (int p = 0; p < N; ++p)
      real = real && c.up_im[p] == 0.0 && c.up_re[p] == c.up_re[0];
    const dim3 grid(herm_tiles(N, upper));
    if (real)
      hipLaunchKernelGGL((liouvillian_tile_kernel<R, N, true>), grid, dim3(kBlock), 0, s, c, e,
                         (const Cx<R>*)x, (Cx<R>*)y, upper ? 1 : 0);
    else
      hipLaunchKernelGGL((liouvillian_tile_kernel<R, N, false>), grid, dim3(kBlock), 0, s, c, e,
                         (const Cx<R>*)x, (Cx<R>*)y, upper ? 1 : 0);
  } else {
    constexpr uint64_t count = uint64_t(1) << (2 * N);
    uint64_t g = (count + kBlock - 1) / kBlock;
    if (g > 8192) g = 8192;
    hipLaunchKernelGGL((liouvillian_kernel<R, N>), dim3((uint32_t)g), dim3(kBlock), 0, s, c, e,
                       (const Cx<R>*)x, (Cx<R>*)y);
  }
}

template <class R, int N = 1>
hipError_t liouvillian_r(const LindbladCoef& c, const double* e, const void* x, void* y, bool upper,
                         hipStream_t s) {
  if constexpr (N > kMaxLindbladAtoms) {
    return hipErrorInvalidValue;
  } else {
    if (c.n != N) return liouvillian_r<R, N + 1>(c, e, x, y, upper, s);
    if (upper && N < kTileAtoms) return hipErrorInvalidValue;
    launch_liouvillian<R, N>(c, e, x, y, upper, s);
    return hipGetLastError();
  }
}

}  // namespace

hipError_t liouvillian_apply(int prec, const LindbladCoef& c, const double* e, const void* x,
                             void* y, bool upper, hipStream_t s) {
  return prec == kC128 ? liouvillian_r<double>(c, e, x, y, upper, s)
                       : liouvillian_r<float>(c, e, x, y, upper, s);
}

hipError_t rho_diagonal(int prec, int n, const void* x, double* out, hipStream_t s) {
  const uint32_t dim = 1u << n;
  const uint32_t g = (dim + kBlock - 1) / kBlock;
  if (prec == kC128)
    hipLaunchKernelGGL(rho_diag_kernel<double>, dim3(g), dim3(kBlock), 0, s, (const double2*)x, n, out);
  else
    hipLaunchKernelGGL(rho_diag_kernel<float>, dim3(g), dim3(kBlock), 0, s, (const float2*)x, n, out);
  return hipGetLastError();
}

}  // namespace rsv
