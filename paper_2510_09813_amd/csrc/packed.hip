// Evolution of small registers: one workgroup per job runs a whole time evolution (2^n
// amplitudes held by the workgroup) without host round trips.  The server packs many jobs into
// a launch; rsv_evolve and its device forms run their small registers the same way.
//
// Each step is the method of the host-driven path (Sec. III and III.A): midpoint parameters,
// the three-term Lanczos recurrence with FP64 scalars, the a-posteriori estimate
// beta_{m-1} |[exp(-i dt T_m) e_1]_{m-1}| |psi| <= tol, sub-steps on non-convergence, and
// psi <- |psi| sum_l y_l v_l.  Only the small exponential differs: instead of the host
// eigendecomposition, y = exp(-i tau T) e_1 is evaluated by one wave with the Chebyshev
// expansion
//   exp(-i a x) = J_0(a) + 2 sum_{k>=1} (-i)^k J_k(a) T_k(x),   x in [-1, 1],
// applied to X = (T - c)/r with c, r from Gershgorin bounds and a = tau r (Bessel coefficients
// by Miller's backward recurrence normalised with J_0 + 2 sum J_2k = 1), lane i holding row i of
// T (m <= 64).  The series is capped at kMaxBessel terms; a step whose tau r exceeds what that
// resolves is shortened (halved until it fits) before the estimate is tested, which only adds
// sub-steps.
//
// What bounds it is latency: a step is a chain of Krylov iterations, each a few hundred
// nanoseconds of LDS reads between two barriers.  So
//  * the workgroup holds the three vectors of the recurrence in registers (the Krylov basis is
//    only written, to the L2, and read back once per step by the thread that wrote it); the
//    level swaps of the thread-index bits read the LDS tile, the others are register moves;
//  * |u_k|^2 and <u_k, H u_k> are summed together (DPP adds inside a wave, one LDS exchange
//    between waves): two barriers per iteration;
//  * the estimate is first tested at the dimension where an a-priori value of it (`expected`)
//    comes within a factor 2^10 of the tolerance, and a test that fails says how far that value
//    is off, so the next test waits until the corrected one meets the tolerance.  All this
//    depends on T alone, so a run split at a step boundary takes the same dimensions as the
//    whole run; a dimension larger than the smallest one that meets the tolerance is as exact;
//  * sizes are compile-time constants, and a launch's threads fit its registers: 256 for up to
//    kPackSmallBits atoms (four or fewer amplitudes per thread, several jobs per CU), 512 or 1024
//    above.
// Measured on one MI355X: 100 steps of the 10-atom chain (27 iterations each, complex128) 5.0 ms,
// 66 ms by the host driver; 64 jobs of 6..13 atoms (complex64, 50..400 steps) 56 ms, 205 ms with
// runtime sizes, two reductions and an LDS read per swap.  Per iteration 0.6 us at 8 atoms, 1.6
// us at 10 (complex128), 5 us at 13 (complex64, the FP64 sums and conversions of 8192
// amplitudes on one CU).
#include "device_common.h"
#include "packed.h"

#include <cmath>
#include <cstring>

namespace rsv {
namespace {

constexpr int kMaxBessel = 512;
constexpr int kBesselPad = 16;  // Miller's start above the last term, and the loop's round-up

// exp(i x).  Not inlined: its range reduction would take registers from the whole kernel.
__device__ __attribute__((noinline)) double2 unit_phase(double x) {
  double s, c;
  sincos(x, &s, &c);
  return double2{c, s};
}

struct Shared {
  double alpha[kMaxKrylov + 1], beta[kMaxKrylov + 1], scale[kMaxKrylov + 1];
  double cre[kMaxKrylov], cim[kMaxKrylov];  // |psi| y_l s_l
  double bessel[kMaxBessel + kBesselPad];
  double2 red[16];                          // per wave (|u|^2, <u, H u>)
  double occ[16][kMaxPackBits + 1];
  double dl[kMaxPackBits];                  // detuning of bit p at the current step
  double est;
  double ba, binv, bscale;                  // the series in bessel: argument, 1 / a, normalisation
  int bk;                                   // and its terms
};

// Bessel coefficients of a series of argument a, by one wave, into sh (unnormalised; the factor
// that normalises them goes to sh.bscale).  Returns false where more than kMaxBessel terms are
// needed.
__device__ __forceinline__ bool bessel_series(Shared& sh, double a) {
  const int lane = threadIdx.x & 63;
  // terms: a + 8 a^(1/3) + 20 leaves a tail below 1e-15 for any a; for small a fewer do: J_k(a)
  // <= (a/2)^k / k! < (e a / 2k)^k, below e^-42 where k (ln(2k/a) - 1) >= 42 (Newton from above,
  // each iterate stays on the safe side of the convex function's root)
  const float fa = (float)fmin(a, 1e6);
  float kt = fa + 8.0f * __powf(fa, 0.33333334f) + 20.0f;
  if (kt > (float)(kMaxBessel - 1)) return false;
  {
    float k = kt;
#pragma unroll 1
    for (int it = 0; it < 6; ++it) {
      const float l = __logf(2.0f * k / fa);
      const float f = k * (l - 1.0f) - 42.0f;
      if (!(f > 0.0f && l > 0.1f)) break;
      k -= __fdividef(f, l);
    }
    kt = fminf(kt, fmaxf(k, 1.0f));
  }
  const int K = min((int)kt + 2, kMaxBessel - 1);
  // Miller's backward recurrence for J_K+8..J_0 (J_K is below the rounding of J_0, so a start
  // a few orders above it is enough), normalised by J_0 + 2 sum J_2k = 1
  const int M = K + 8;
  const double inv = 1.0 / a, two_over_a = 2.0 * inv;
  double jp = 0.0, j = 1e-250, norm = 0.0;
  if (lane < 8) sh.bessel[M + lane] = 0.0;  // read by the last group of the series' loop
#pragma unroll 2
  for (int k = M; k >= 1; --k) {
    if (lane == 0) sh.bessel[k] = j;
    norm += (k & 1) ? 0.0 : j;
    const double jm = fma(k * two_over_a, j, -jp);
    jp = j;
    j = jm;
    if (fabs(j) > 1e250) {  // rescale everything recurred so far (only where a is tiny)
      j *= 1e-250;
      jp *= 1e-250;
      norm *= 1e-250;
      if (lane == 0)
        for (int q = k; q <= M; ++q) sh.bessel[q] *= 1e-250;
    }
  }
  if (lane == 0) {
    sh.bessel[0] = j;
    sh.bscale = 2.0 / (2.0 * norm + j);
    sh.ba = a;
    sh.binv = inv;
    sh.bk = K;
  }
  // one wave: its LDS accesses are in order; keep the compiler from moving them
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return true;
}

// [exp(-i tau T_m) e_1] by one wave: lane i returns row i without the common phase factor
// exp(i phase); the return value is |row m - 1| (uniform), or -1 when tau times the spectral
// half-width of T_m needs more than kMaxBessel terms (the caller shortens tau).  The half-width
// is rounded up (by at most a quarter), so that most tests find the coefficients of the one
// before: Miller's recurrence costs as much as the series.
__device__ __forceinline__ double cheb_rows(Shared& sh, int m, double tau, double& yr, double& yi,
                                            double& phase) {
  const int lane = threadIdx.x & 63;
  const bool live = lane < m;
  const double al = live ? sh.alpha[lane] : 0.0;
  const double bl = live && lane > 0 ? sh.beta[lane - 1] : 0.0;
  const double br = live && lane + 1 < m ? sh.beta[lane] : 0.0;
  const double w = bl + br;
  const double lo = wave_reduce(live ? al - w : 1e300, OpMin());
  const double hi = wave_reduce(live ? al + w : -1e300, OpMax());
  const double c = 0.5 * (hi + lo);
  // a rounded up to three significant bits (at least 1/2)
  double a = fmax(0.5, 0.5 * tau * (hi - lo));
  {
    const uint64_t b = __builtin_bit_cast(uint64_t, a);
    a = __builtin_bit_cast(double, (b + ((uint64_t(1) << 50) - 1)) & ~((uint64_t(1) << 50) - 1));
  }
  phase = -tau * c;
  yr = yi = 0.0;
  if (!(sh.ba == a) && !bessel_series(sh, a)) return -1.0;
  const int K = sh.bk;
  // t_0 = e_1, t_1 = X e_1, t_{k+1} = 2 X t_k - t_{k-1}; the coefficients carry the factor 2
  const double s = 2.0 * tau * sh.binv;
  const double xa = live ? (al - c) * s : 0.0, xl = bl * s, xr = br * s;
  double t0 = lane == 0 ? 1.0 : 0.0;
  double t1 = 0.5 * fma(xa, t0, xl * dpp<kDppFromBelow>(t0));
  yr = 0.5 * sh.bessel[0] * t0;
  auto next = [&]() {
    const double below = dpp<kDppFromBelow>(t1), above = dpp<kDppFromAbove>(t1);
    const double t2 = fma(xr, above, fma(xl, below, fma(xa, t1, -t0)));
    t0 = t1;
    t1 = t2;
  };
#pragma unroll 1
  for (int k = 1; k <= K; k += 4) {  // (-i)^k: -i, -1, +i, +1
    const double b0 = sh.bessel[k], b1 = sh.bessel[k + 1], b2 = sh.bessel[k + 2], b3 = sh.bessel[k + 3];
    yi = fma(-b0, t1, yi);
    next();
    yr = fma(-b1, t1, yr);
    next();
    yi = fma(b2, t1, yi);
    next();
    yr = fma(b3, t1, yr);
    next();
  }
  yr *= sh.bscale;
  yi *= sh.bscale;
  const double er = lane_value(yr, m - 1), ei = lane_value(yi, m - 1);
  return sqrt(er * er + ei * ei);
}

// log2 of an a-priori value of the estimate beta |psi| |[exp(-i tau T_k) e_1]_{k-1}|: the
// component is at most prod (tau beta_j) / (k - 1)! (the leading term of the exponential; lead
// holds it times beta |psi|), and for a spectrum of half-width a / tau it falls below that by
// about exp(-a^2 / 4k) (J_k(a) against (a/2)^k / k!).  Gershgorin's half-width is up to twice the
// true one, so the first test (tight = false) takes that factor and later ones its fourth root.
__device__ __forceinline__ float expected(double lead, double a, int k, bool tight) {
  const float fa = (float)fmin(a, 1e6);
  return (float)__builtin_amdgcn_frexp_exp(lead) -
         (tight ? 0.0902f : 0.3607f) * fa * fa * __frcp_rn((float)k);
}

// ------------------------------------------------------------------------------- one job
// N atoms on 2^TB threads, A amplitudes each: the thread bits of the index are TB consecutive
// ones; the bits above (and, for complex64, bit 0, so that every access moves 16 bytes per lane)
// number the thread's own amplitudes.  MODE: kCoefReal (one real coupling for every atom) or
// kCoefSite (any other drive).
template <class R, int N, int TB, int MODE>
struct Runner {
  using C = Cx<R>;
  static constexpr int T = 1 << TB, W = T / 64;
  static constexpr int RB = N > TB ? N - TB : 0, A = 1 << RB;
  static constexpr int VB = sizeof(R) == 4 && RB > 0 ? 1 : 0;  // register bits below the thread bits
  static constexpr int LB = N < TB ? N : TB;  // bits of the index that are thread bits
  static constexpr uint32_t dim = 1u << N;

  // Index of amplitude s of thread tid; the slot bit of index bit p (-1: a thread bit).
  static __device__ __forceinline__ uint32_t pos(uint32_t tid, int s) {
    return (tid << VB) + (uint32_t)(s & ((1 << VB) - 1)) + ((uint32_t)(s >> VB) << (TB + VB));
  }
  static constexpr int slot_bit(int p) { return p < VB ? p : p >= TB + VB ? p - TB : -1; }

  // The thread index, opaque to the optimiser: without it every address and predicate derived
  // from the index is kept in a register across the whole kernel, and the vectors spill.
  static __device__ __forceinline__ uint32_t fresh(uint32_t tid) {
    asm volatile("" : "+v"(tid));
    return tid;
  }

  // Thread bits whose swap is a DPP move inside the wave rather than an LDS read: with complex64
  // it joins the add (bits 0, 1) or takes one move more (2, 3), where the LDS pipe takes 4 cycles
  // of the CU per wave and amplitude; complex128 needs four moves per amplitude against 8 cycles.
  static constexpr int DB = LB < (sizeof(R) == 4 ? 4 : 2) ? LB : (sizeof(R) == 4 ? 4 : 2);

  static __device__ __forceinline__ R moved(R v, int q) {
    switch (q) {
      case 0: return dpp<kDppXor1>(v);
      case 1: return dpp<kDppXor2>(v);
      case 2: return dpp<kDppXor3>(dpp<kDppHalfMirror>(v));
      default: return dpp<kDppHalfMirror>(dpp<kDppMirror>(v));
    }
  }

  // The amplitude with index bit p swapped (p < N known at compile time once unrolled).
  static __device__ __forceinline__ C neighbour(const C* tile, const C (&u)[A], uint32_t tid, int p,
                                                int s) {
    if (slot_bit(p) >= 0) return u[(s ^ (1 << (slot_bit(p) & 31))) & (A - 1)];
    const int q = p - VB;
    if (q < DB) return C{moved(u[s].x, q), moved(u[s].y, q)};
    return tile[pos(tid ^ (1u << q), s)];
  }

  // z = H u (u in the tile and in registers) and this thread's Re<u, z>
  static __device__ __forceinline__ double apply(const C* tile, const C (&u)[A], const R (&dg)[A],
                                                 const R* cf, uint32_t tid, C (&z)[A]) {
    if constexpr (MODE == kCoefReal) {
      // sum the neighbours, then apply the coupling once
#pragma unroll
      for (int s = 0; s < A; ++s) z[s] = C{0, 0};
#pragma unroll
      for (int p = 0; p < N; ++p) {
#pragma unroll
        for (int s = 0; s < A; ++s) {
          const C nb = neighbour(tile, u, tid, p, s);
          z[s].x += nb.x;
          z[s].y += nb.y;
        }
      }
      const R ur = cf[0];
#pragma unroll
      for (int s = 0; s < A; ++s)
        z[s] = C{dg[s] * u[s].x + ur * z[s].x, dg[s] * u[s].y + ur * z[s].y};
    } else {
#pragma unroll
      for (int s = 0; s < A; ++s) z[s] = C{dg[s] * u[s].x, dg[s] * u[s].y};
#pragma unroll
      for (int p = 0; p < N; ++p) {
        // <0|h|1> is the conjugate of <1|h|0>; a register bit's level is known per slot
        const R cr = cf[2 * p], ci1 = cf[2 * p + 1];
        const R ci = slot_bit(p) < 0 && !((tid >> (p - VB)) & 1u) ? -ci1 : ci1;
#pragma unroll
        for (int s = 0; s < A; ++s) {
          const C nb = neighbour(tile, u, tid, p, s);
          const R c = slot_bit(p) >= 0 && !((s >> (slot_bit(p) & 31)) & 1) ? -ci : ci;
          z[s].x += cr * nb.x - c * nb.y;
          z[s].y += cr * nb.y + c * nb.x;
        }
      }
    }
    double dot = 0.0;
#pragma unroll
    for (int s = 0; s < A; ++s)
      dot += (double)u[s].x * (double)z[s].x + (double)u[s].y * (double)z[s].y;
    return dot;
  }

  // Tile write, H, and both sums over the workgroup (uniform): the tile is free again after it.
  static __device__ __forceinline__ double2 sweep(Shared& sh, C* tile, const C (&u)[A],
                                                  const R (&dg)[A], const R* cf,
                                                  uint32_t tid0, bool live, C (&z)[A]) {
    const uint32_t tid = fresh(tid0);
#pragma unroll
    for (int s = 0; s < A; ++s) tile[pos(tid, s)] = u[s];
    double nn = 0.0;
#pragma unroll
    for (int s = 0; s < A; ++s) nn = norm_add(nn, (double)u[s].x, (double)u[s].y);
    __syncthreads();
    double dot = apply(tile, u, dg, cf, tid, z);
    if (!live) dot = 0.0;  // threads beyond the register hold zeros, and read zeros or rubbish
    nn = wave_total(nn);
    dot = wave_total(dot);
    if ((tid & 63u) == 0) sh.red[tid >> 6] = double2{nn, dot};
    __syncthreads();
    if constexpr (W <= 4) {
      double2 r = sh.red[0];
#pragma unroll
      for (int w = 1; w < W; ++w) {
        const double2 o = sh.red[w];
        r.x += o.x;
        r.y += o.y;
      }
      return r;
    } else {
      static_assert(W == 8 || W == 16, "every row of 16 lanes holds all waves' sums");
      double2 o = sh.red[tid & (W - 1)];
      o.x += dpp<kDppXor1>(o.x);
      o.y += dpp<kDppXor1>(o.y);
      o.x += dpp<kDppXor2>(o.x);
      o.y += dpp<kDppXor2>(o.y);
      o.x += dpp<kDppHalfMirror>(o.x);
      o.y += dpp<kDppHalfMirror>(o.y);
      if constexpr (W == 16) {
        o.x += dpp<kDppMirror>(o.x);
        o.y += dpp<kDppMirror>(o.y);
      }
      return double2{lane_value(o.x, 0), lane_value(o.y, 0)};
    }
  }

  static __device__ __forceinline__ void occupations(Shared& sh, const C (&u)[A], uint32_t tid,
                                                     double* dst) {
    tid = fresh(tid);
    double pr[A], tot = 0.0;
#pragma unroll
    for (int s = 0; s < A; ++s) {
      pr[s] = norm_add(0.0, (double)u[s].x, (double)u[s].y);
      tot += pr[s];
    }
#pragma unroll 1
    for (int p = -1; p < N; ++p) {  // -1: the total
      double v = tot;
      if (p >= 0) {
        v = 0.0;
#pragma unroll
        for (int s = 0; s < A; ++s) v += (pos(tid, s) >> p) & 1u ? pr[s] : 0.0;
      }
      v = wave_total(v);
      if ((tid & 63u) == 0) sh.occ[tid >> 6][1 + p] = v;
    }
    __syncthreads();
    if (tid <= (uint32_t)N) {
      double v = 0.0;
#pragma unroll 1
      for (int w = 0; w < W; ++w) v += sh.occ[w][tid];
      dst[tid] = v;
    }
    __syncthreads();
  }

  static __device__ __forceinline__ void run(const PackedJob& jb, const double* om, const double* de,
                                             const double* ph, bool has_phi, Shared& sh, C* tile,
                                             R* cf) {
    const uint32_t tid = threadIdx.x;
    const bool live = N >= TB || tid < dim;
    const bool wave0 = tid < 64;
    C* basis = (C*)jb.basis;
    int64_t iters = 0, kmax_used = 0, substeps = 0;
    int status = RSV_OK;
    if (jb.resume) {
      status = (int)jb.out[0];
      iters = (int64_t)jb.out[1];
      kmax_used = (int64_t)jb.out[2];
      substeps = (int64_t)jb.out[3];
      if (status != RSV_OK) return;  // (uniform)
    }
    C u[A];  // the newest Krylov vector; between steps the state
#pragma unroll
    for (int s = 0; s < A; ++s) {
      const uint32_t e = pos(tid, s);
      u[s] = C{0, 0};
      if (!live) continue;
      if (jb.psi0) u[s] = C{(R)jb.psi0[e].x, (R)jb.psi0[e].y};
      else if (jb.psi_in) u[s] = ((const C*)jb.psi_in)[e];
      else u[s] = C{(R)(e == 0 ? 1 : 0), 0};
    }
    {  // E_b, read back by this thread at each step
      double v[A];
#pragma unroll
      for (int s = 0; s < A; ++s) v[s] = 0.0;
#pragma unroll 1
      for (int p = 1; p < N; ++p) {
#pragma unroll 1
        for (int q = 0; q < p; ++q) {
          const double w = jb.ub[p * 32 + q];
#pragma unroll
          for (int s = 0; s < A; ++s) {
            const uint32_t e = pos(tid, s);
            v[s] += (e >> p) & (e >> q) & 1u ? w : 0.0;
          }
        }
      }
      if (live) {
#pragma unroll
        for (int s = 0; s < A; ++s) jb.diag[pos(tid, s)] = v[s];
      }
    }
    const float log2_tol = (float)__builtin_amdgcn_frexp_exp(jb.tol);
    if (tid == 0) sh.ba = -1.0;
    __syncthreads();  // every thread has read the previous launch's results from out

#pragma unroll 1
    for (int64_t step = 0; step < jb.n_steps && status == RSV_OK; ++step) {
      // coefficients of H_k by bit position p (atom n-1-p)
      if (tid < (uint32_t)N) {
        const size_t at = (jb.per_site ? (size_t)(N - 1 - tid) * jb.n_steps : 0) + step;
        const double h = 0.5 * om[at], f = has_phi ? ph[at] : 0.0;
        double re = h, im = 0.5 * f;
        if (!jb.direct) {
          const double2 w = unit_phase(f);
          re = h * w.x;
          im = -h * w.y;
        }
        cf[2 * tid] = (R)re;  // <1|h|0>
        cf[2 * tid + 1] = (R)im;
        sh.dl[tid] = de[at];
      }
      __syncthreads();
      R dg[A];  // diagonal of H_k
      {
        double v[A];
        const uint32_t t = fresh(tid);
#pragma unroll
        for (int s = 0; s < A; ++s) v[s] = live ? jb.diag[pos(t, s)] : 0.0;
        if (jb.per_site) {
#pragma unroll 1
          for (int p = 0; p < N; ++p) {
            const double d = sh.dl[p];
#pragma unroll
            for (int s = 0; s < A; ++s) v[s] -= (pos(t, s) >> p) & 1u ? d : 0.0;
          }
        } else {
          const double d = sh.dl[0];
#pragma unroll
          for (int s = 0; s < A; ++s) v[s] -= d * (double)__popc(pos(t, s));
        }
#pragma unroll
        for (int s = 0; s < A; ++s) dg[s] = (R)v[s];
      }

      double remaining = jb.tau;
#pragma unroll 1
      while (remaining > 0.0 && status == RSV_OK) {
        C prev[A], z[A];
#pragma unroll
        for (int s = 0; s < A; ++s) prev[s] = z[s] = C{0, 0};
        int m = 0;
        // target: the part of the step this basis must resolve; shortened while the
        // exponential of the growing T_m is too wide for one Chebyshev series
        double target = remaining, sub = remaining;
        double nrm = 0.0, lead = 0.0;         // |psi|, |psi| prod_{j<k} (tau beta_{j-1}) / (k-1)!
        double s1 = 0.0, s2 = 0.0;            // scales of u_{k-1} and u_{k-2}
        double glo = 1e300, ghi = -1e300, blast = 0.0;  // Gershgorin bounds of the rows before k-1
        double2 nd = {0.0, 0.0};              // |u|^2 and <u, H u> of the newest vector
        bool stop = false;
        float off = -10.0f;                   // log2 of the estimate over its a-priori value
        bool tested = false;
#pragma unroll 1
        for (int k = 0; !stop; ++k) {
          const double alpha = s1 * s1 * nd.y;  // alpha_{k-1}
          if (k > 0) {
            // u_k = s z - alpha s u_{k-1} - (s_{k-2}/s_{k-1}) u_{k-2}, rounded once
            const double ca = alpha * s1, cb = s2 * nd.x * s1;  // s2 / s1 = s2 |u_{k-1}|
#pragma unroll
            for (int s = 0; s < A; ++s) {
              const double re = s1 * (double)z[s].x - ca * (double)u[s].x - cb * (double)prev[s].x;
              const double im = s1 * (double)z[s].y - ca * (double)u[s].y - cb * (double)prev[s].y;
              prev[s] = u[s];
              u[s] = live ? C{(R)re, (R)im} : C{0, 0};
            }
          }
          if (k < jb.kmax && live) {
            const uint32_t t = fresh(tid);
            C* b = basis + (size_t)k * dim;
#pragma unroll
            for (int s = 0; s < A; ++s) b[pos(t, s)] = u[s];
          }
          // z_k = H u_k and |u_k|^2 together: z_k is not needed where this dimension resolves
          // the step, but its sum shares the exchange of |u_k|^2
          nd = sweep(sh, tile, u, dg, cf, tid, live, z);
          ++iters;
          if (k == 0) {
            nrm = sqrt(nd.x);
            if (!(nrm > 0.0) || !isfinite(nrm)) {
              status = RSV_ENUMERIC;
              break;
            }
            s1 = rsqrt(nd.x);
            lead = nrm;
            if (tid == 0) sh.scale[0] = s1;
            continue;
          }
          if (tid == 0) sh.alpha[k - 1] = alpha;
          if (!isfinite(nd.x) || !isfinite(alpha)) {
            status = RSV_ENUMERIC;
            break;
          }
          const double sk = rsqrt(nd.x);
          const double bk = nd.x > 0.0 ? nd.x * sk : 0.0;  // |u_k|
          m = k;
          const bool last = k == jb.kmax || bk == 0.0;
          // the last row of T_k couples upwards only
          const double half = 0.5 * (fmax(ghi, alpha + blast) - fmin(glo, alpha - blast));
          const float guess = expected(lead * bk, target * half, k, tested);
          if (last || !(guess + off > log2_tol)) {
            // phase 0: the target, shortened while it is too wide; then, where this basis is the
            // last and does not resolve it, the longest part that it does: 1 the first dyadic
            // fraction that converges, 2 ten bisections above it, 3 the exponential of the result
            int phase = 0, cnt = 0;
            double tq = target, bad = target;
#pragma unroll 1
            for (;;) {
              if (wave0) {
                double yr, yi, ang;
                const double e = cheb_rows(sh, m, tq, yr, yi, ang);
                if (tid == 0) sh.est = e;
                if ((int)tid < m && e >= 0.0 && bk * e * nrm <= jb.tol) {
                  const double2 w = unit_phase(ang);
                  const double sc = nrm * sh.scale[tid];
                  sh.cre[tid] = sc * (w.x * yr - w.y * yi);
                  sh.cim[tid] = jb.dir * sc * (w.x * yi + w.y * yr);
                }
              }
              __syncthreads();
              const double est = sh.est;  // < 0: too wide
              __syncthreads();
              // (met also at beta = 0, an invariant subspace)
              const bool ok = est >= 0.0 && bk * est * nrm <= jb.tol;
              if (phase == 0) {
                if (est < 0.0 && ++cnt <= 64) {
                  lead = ldexp(lead, 1 - k);  // target^(k-1) is a factor of it
                  tq = target *= 0.5;
                  continue;
                }
                if (ok) {
                  sub = target;
                  stop = true;
                  break;
                }
                if (est >= 0.0 && !last) {
                  off = (float)__builtin_amdgcn_frexp_exp(bk * est * nrm) -
                        expected(lead * bk, target * half, k, true) - 2.0f;
                  tested = true;
                  break;
                }
                if (est < 0.0 || jb.max_depth < 1) {
                  status = RSV_ENOTCONV;
                  break;
                }
                phase = cnt = 1;
                bad = target;
                tq = ldexp(target, -1);
              } else if (phase == 1) {
                if (ok) {
                  sub = tq;
                  phase = 2;
                  cnt = 0;
                  tq = 0.5 * (sub + bad);
                } else {
                  bad = tq;
                  if (++cnt > jb.max_depth) {
                    status = RSV_ENOTCONV;
                    break;
                  }
                  tq = ldexp(target, -cnt);
                }
              } else if (phase == 2) {
                if (ok) sub = tq;
                else bad = tq;
                if (++cnt < 10) {
                  tq = 0.5 * (sub + bad);
                } else {
                  phase = 3;
                  tq = sub;
                }
              } else {
                stop = true;
                break;
              }
            }
            if (stop || status != RSV_OK) break;
          }
          s2 = s1;
          s1 = sk;
          if (tid == 0) {
            sh.beta[k - 1] = bk;
            sh.scale[k] = s1;
          }
          lead *= target * bk * (double)__frcp_rn((float)k);
          glo = fmin(glo, alpha - blast - bk);
          ghi = fmax(ghi, alpha + blast + bk);
          blast = bk;
        }
        if (status != RSV_OK) break;
        kmax_used = kmax_used > m ? kmax_used : (int64_t)m;
        // psi <- |psi| sum_l y_l s_l u_l over this thread's own amplitudes
        double re[A], im[A];
#pragma unroll
        for (int s = 0; s < A; ++s) re[s] = im[s] = 0.0;
        if (live) {
          const uint32_t t = fresh(tid);
          const C* b = basis;
          // several vectors' loads in flight: the basis of a large job lives beyond the L2
          constexpr int G = A >= 16 ? 4 : 32 / A > 8 ? 8 : 32 / A;
          int l = 0;
#pragma unroll 1
          for (; l + G <= m; l += G, b += (size_t)G * dim) {
            C x[G][A];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
              for (int s = 0; s < A; ++s) x[g][s] = b[(size_t)g * dim + pos(t, s)];
#pragma unroll
            for (int g = 0; g < G; ++g) {
              const double cr = sh.cre[l + g], ci = sh.cim[l + g];
#pragma unroll
              for (int s = 0; s < A; ++s) {
                re[s] += cr * (double)x[g][s].x - ci * (double)x[g][s].y;
                im[s] += cr * (double)x[g][s].y + ci * (double)x[g][s].x;
              }
            }
          }
#pragma unroll 1
          for (; l < m; ++l, b += dim) {
            const double cr = sh.cre[l], ci = sh.cim[l];
#pragma unroll
            for (int s = 0; s < A; ++s) {
              const C x = b[pos(t, s)];
              re[s] += cr * (double)x.x - ci * (double)x.y;
              im[s] += cr * (double)x.y + ci * (double)x.x;
            }
          }
        }
#pragma unroll
        for (int s = 0; s < A; ++s) u[s] = C{(R)re[s], (R)im[s]};
        __syncthreads();  // the coefficients are read before the next run writes its own
        if (sub == remaining) {
          remaining = 0.0;
        } else {
          remaining -= sub;
          ++substeps;
        }
      }
      const int64_t done = jb.obs_first + step + 1;
      if (status == RSV_OK && jb.obs && done % jb.obs_every == 0)
        occupations(sh, u, tid, jb.obs + (done / jb.obs_every - 1) * (N + 1));
    }
    // final state, occupations (FP64), bookkeeping
    if (status == RSV_OK && live) {
#pragma unroll
      for (int s = 0; s < A; ++s) {
        const uint32_t e = pos(tid, s);
        if (jb.psi_out) ((C*)jb.psi_out)[e] = u[s];
        if (jb.state) jb.state[e] = double2{(double)u[s].x, (double)u[s].y};
      }
    }
    occupations(sh, u, tid, jb.out + kPackOccOffset - 1);
    if (tid == 0) {
      jb.out[4] = jb.out[kPackOccOffset - 1];
      jb.out[0] = status;
      jb.out[1] = (double)iters;
      jb.out[2] = (double)kmax_used;
      jb.out[3] = (double)substeps;
    }
  }
};

// The sizes of one launch: 2^TB threads, NLO..NHI atoms.
template <class R, int TB, int NLO, int NHI>
__device__ __forceinline__ void dispatch(const PackedJob& jb, const double* om, const double* de,
                                         const double* ph, bool has_phi, Shared& sh, Cx<R>* tile,
                                         R* cf) {
  if constexpr (NLO <= NHI) {
    if (jb.n == NLO && jb.real) Runner<R, NLO, TB, kCoefReal>::run(jb, om, de, ph, has_phi, sh, tile, cf);
    else if (jb.n == NLO) Runner<R, NLO, TB, kCoefSite>::run(jb, om, de, ph, has_phi, sh, tile, cf);
    else dispatch<R, TB, NLO + 1, NHI>(jb, om, de, ph, has_phi, sh, tile, cf);
  }
}

template <class R> constexpr int max_bits() { return sizeof(R) == 8 ? 12 : 13; }
constexpr int kSmallThreadBits = 8;
// 13 atoms complex64: 36 Mcycles for a 115-step job on 1024 threads, 38 on 512; 12 atoms
// complex128 spills its vectors on 1024.
template <class R> constexpr int large_thread_bits() { return sizeof(R) == 8 ? 9 : 10; }

template <class R, bool LARGE>
__global__ __launch_bounds__(1 << (LARGE ? large_thread_bits<R>() : kSmallThreadBits)) void packed_kernel(const PackedJob* __restrict__ jobs) {
  constexpr int HB = LARGE ? max_bits<R>() : kPackSmallBits;
  __shared__ __align__(16) Cx<R> tile[1 << HB];
  __shared__ Shared sh;
  __shared__ R cf[2 * kMaxPackBits];
  const PackedJob& jb = jobs[blockIdx.x];
  if constexpr (LARGE)
    dispatch<R, large_thread_bits<R>(), kPackSmallBits + 1, HB>(jb, jb.omega, jb.delta, jb.phi, jb.phi != nullptr, sh, tile, cf);
  else
    dispatch<R, kSmallThreadBits, 1, HB>(jb, jb.omega, jb.delta, jb.phi, jb.phi != nullptr, sh, tile, cf);
}

struct SmallArgs {
  PackedJob job;
  int with_phi;
  double mid[kMidValues];
};
static_assert(sizeof(SmallArgs) <= 4096, "kernel argument size");

template <class R, int N, int TB, int MODE>
__global__ __launch_bounds__(1 << TB) void small_kernel(const SmallArgs a) {
  __shared__ __align__(16) Cx<R> tile[N < TB ? (1 << TB) : (1 << N)];
  __shared__ Shared sh;
  __shared__ R cf[2 * kMaxPackBits];
  __shared__ double mid[kMidValues];
  for (int i = threadIdx.x; i < kMidValues; i += 1 << TB) mid[i] = a.mid[i];
  __syncthreads();
  const int cnt = (int)a.job.n_steps * (a.job.per_site ? N : 1);
  Runner<R, N, TB, MODE>::run(a.job, mid, mid + cnt, mid + 2 * cnt, a.with_phi != 0, sh, tile, cf);
}

template <class R, int N>
hipError_t small_launch(const SmallArgs& a, hipStream_t s) {
  if constexpr (N > max_bits<R>()) {
    return hipErrorInvalidValue;
  } else {
    if (a.job.n != N) return small_launch<R, N + 1>(a, s);
    constexpr int TB = N > 11 ? large_thread_bits<R>() : (N > kPackSmallBits ? 9 : (N < 6 ? 6 : (N < 8 ? N : 8)));
    if (a.job.real)
      hipLaunchKernelGGL((small_kernel<R, N, TB, kCoefReal>), dim3(1), dim3(1 << TB), 0, s, a);
    else
      hipLaunchKernelGGL((small_kernel<R, N, TB, kCoefSite>), dim3(1), dim3(1 << TB), 0, s, a);
    return hipGetLastError();
  }
}

template <class R>
hipError_t packed_r(const PackedJob* d_jobs, int n_small, int n_large, hipStream_t s_small,
                    hipStream_t s_large) {
  if (n_large > 0)
    hipLaunchKernelGGL((packed_kernel<R, true>), dim3(n_large), dim3(1 << large_thread_bits<R>()), 0, s_large, d_jobs + n_small);
  if (n_small > 0)
    hipLaunchKernelGGL((packed_kernel<R, false>), dim3(n_small), dim3(1 << kSmallThreadBits), 0, s_small, d_jobs);
  return hipGetLastError();
}

}  // namespace

int packed_max_atoms(int prec) { return prec == kC128 ? 12 : 13; }

bool packed_resolves(double tau, double half_width) {
  // T_m's diagonal lies in H's spectrum and its couplings are at most the half-width, so its
  // Gershgorin half-width is at most three times that
  const double a = 3.0 * tau * half_width;
  return a + 8.0 * std::cbrt(a) + 20.0 < kMaxBessel - 2;
}

hipError_t packed_evolve(int prec, const PackedJob* d_jobs, int n_small, int n_large,
                         hipStream_t s_small, hipStream_t s_large) {
  return prec == kC128 ? packed_r<double>(d_jobs, n_small, n_large, s_small, s_large)
                       : packed_r<float>(d_jobs, n_small, n_large, s_small, s_large);
}

hipError_t small_evolve(int prec, const PackedJob& job, const double* mid, bool with_phi,
                        hipStream_t s) {
  SmallArgs a;
  a.job = job;
  a.with_phi = with_phi ? 1 : 0;
  const int64_t cnt = job.n_steps * (job.per_site ? job.n : 1) * (with_phi ? 3 : 2);
  if (job.n_steps < 1 || cnt > kMidValues) return hipErrorInvalidValue;
  std::memcpy(a.mid, mid, (size_t)cnt * sizeof(double));
  std::memset(a.mid + cnt, 0, (kMidValues - (size_t)cnt) * sizeof(double));
  return prec == kC128 ? small_launch<double, 1>(a, s) : small_launch<float, 1>(a, s);
}

}  // namespace rsv
