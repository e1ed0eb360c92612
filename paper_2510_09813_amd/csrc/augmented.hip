// The block operator of the pulse gradients on an augmented vector [a | b] of 2 x 2^n amplitudes:
//   (a, b) -> -i (H a + V b, H b),
// V = dH/dOmega (the drive at unit amplitude with the step's phase) or dH/ddelta (-sum n), for a
// global drive.  Element-wise it needs the n neighbours of a_x and b_x: the eight lowest bits' from
// an LDS tile of 256, the others' through the cache, which holds vectors of this size.  One launch
// instead of three H psi (two or three launches each) and two combinations: 16 atoms complex128, 6 us
// instead of 45; bound by the cache's bandwidth on 2 (n - 8) loads of 16 bytes per element.
#include "augmented.h"
#include "device_common.h"

namespace rsv {
namespace {

template <class R>
__global__ __launch_bounds__(kBlock) void augmented_kernel(const AugmentedCoef c,
                                                           const double* __restrict__ e,
                                                           const Cx<R>* __restrict__ in,
                                                           Cx<R>* __restrict__ out) {
  using C = Cx<R>;
  __shared__ C tile[2][kBlock];
  const uint32_t tid = threadIdx.x, x = blockIdx.x * kBlock + tid;
  const size_t dim = size_t(1) << c.n;
  const bool live = x < dim;
  const C* b_in = in + dim;
  C a = {0, 0}, b = {0, 0};
  double ex = 0.0;
  if (live) {
    a = in[x];
    b = b_in[x];
    ex = e[x];
  }
  tile[0][tid] = a;
  tile[1][tid] = b;
  // sums over the neighbours: all of them, and those whose level here is 1
  C aa = {0, 0}, a1 = {0, 0}, ba = {0, 0}, b1 = {0, 0};
  auto add = [&](const C& na, const C& nb, bool bit) {
    aa.x += na.x;
    aa.y += na.y;
    ba.x += nb.x;
    ba.y += nb.y;
    if (bit) {
      a1.x += na.x;
      a1.y += na.y;
      b1.x += nb.x;
      b1.y += nb.y;
    }
  };
#pragma unroll 4
  for (int p = 8; p < c.n; ++p) {
    const uint32_t y = x ^ (1u << p);
    add(in[y], b_in[y], (x >> p) & 1u);
  }
  __syncthreads();
  const int low = c.n < 8 ? c.n : 8;
  for (int p = 0; p < low; ++p) add(tile[0][tid ^ (1u << p)], tile[1][tid ^ (1u << p)], (tid >> p) & 1u);
  if (!live) return;
  // <1|h|0> = u applies where the level is 1, its conjugate where it is 0
  auto drive = [](const C& all, const C& one, R ur, R ui) {
    const C zero = {all.x - one.x, all.y - one.y};
    return C{(ur * one.x - ui * one.y) + (ur * zero.x + ui * zero.y),
             (ur * one.y + ui * one.x) + (ur * zero.y - ui * zero.x)};
  };
  const R d = (R)(ex - c.delta * (double)__popc(x));
  const R ur = (R)c.up_re, ui = (R)c.up_im;
  C ha = drive(aa, a1, ur, ui), hb = drive(ba, b1, ur, ui);
  ha.x += d * a.x;
  ha.y += d * a.y;
  hb.x += d * b.x;
  hb.y += d * b.y;
  C vb;
  if (c.which == 0) {
    vb = drive(ba, b1, (R)c.v_re, (R)c.v_im);
  } else {
    const R k = (R)__popc(x);
    vb = C{-k * b.x, -k * b.y};
  }
  ha.x += vb.x;
  ha.y += vb.y;
  out[x] = C{ha.y, -ha.x};  // -i
  out[dim + x] = C{hb.y, -hb.x};
}

}  // namespace

hipError_t augmented_apply(int prec, const AugmentedCoef& c, const double* e, const void* in, void* out,
                           hipStream_t s) {
  const uint32_t grid = (uint32_t)(((size_t(1) << c.n) + kBlock - 1) / kBlock);
  if (prec == kC128)
    hipLaunchKernelGGL(augmented_kernel<double>, dim3(grid), dim3(kBlock), 0, s, c, e,
                       (const double2*)in, (double2*)out);
  else
    hipLaunchKernelGGL(augmented_kernel<float>, dim3(grid), dim3(kBlock), 0, s, c, e,
                       (const float2*)in, (float2*)out);
  return hipGetLastError();
}

}  // namespace rsv
