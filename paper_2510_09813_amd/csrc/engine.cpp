// Host engine of librsv: memory, registers, the time stepper and the Lanczos driver.
//
// Stepper (Sec. III): step k holds the pulse at its midpoint sample value and advances psi
// by exp(-i H_k dt) (eq. 6).  Lanczos driver (Sec. III.A): each iteration is one H sweep
// whose first pass also forms the next Krylov vector from the three-term recurrence (alpha
// read from device memory) and whose last pass returns <u, H u>.  After a run of iterations
// one device-to-host copy brings their (alpha_{k-1}, beta_{k-1}^2) to the host, which evaluates
// the exponential of the tridiagonal T_k in FP64 and stops when the a-posteriori estimate
// beta_{k-1} |[exp(-i dt T_k) e_1]_k| |psi| is at most tol.  Then
// psi_{k+1} = |psi_k| sum_l y_l v_l (one combine sweep, which also returns |psi_{k+1}|^2).
//
// Registers that fit one workgroup (packed_max_atoms) run whole calls on the device instead, by
// the kernel of packed jobs: see evolve_small.
#include "engine.h"

#include "krylov_course.h"
#include "packed.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>

namespace rsv {

namespace {
thread_local std::string g_err;

bool finite_all(const double* p, size_t n) {
  for (size_t i = 0; i < n; ++i)
    if (!std::isfinite(p[i])) return false;
  return true;
}

constexpr size_t kScalarBytes = 4096;
// Most partials that every workgroup of the forming pass sums for itself.  At most one norm
// partial per thread, so that the sum's order is also finalize_sum's.
constexpr int64_t kFusedParts = 1024;
constexpr size_t kGranule = 256;
inline size_t round_up(size_t b) { return (b + kGranule - 1) / kGranule * kGranule; }
}  // namespace

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

const char* last_error() { return g_err.c_str(); }

// ------------------------------------------------------------------------------ memory
bool DeviceMem::get(size_t bytes, void** p) const {
  if (hipMalloc(p, bytes) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}
void DeviceMem::put(void* p) const { (void)hipFree(p); }
void DeviceMem::wait() const { (void)hipDeviceSynchronize(); }
bool DeviceMem::half_free() const {
  size_t free_b = 0, total_b = 0;
  return hipMemGetInfo(&free_b, &total_b) == hipSuccess && free_b >= total_b / 2;
}
void DeviceMem::reclaim() const { DeviceAllocator::trim_device(owner->device(), owner); }

namespace {
std::mutex g_allocators_mu;
DeviceAllocator* g_allocators = nullptr;
}  // namespace

DeviceAllocator::DeviceAllocator(int device, size_t budget, size_t device_bytes)
    : device_(device), budget_(budget), pool_(budget, device_bytes / 32, DeviceMem{this}) {
  std::lock_guard<std::mutex> lk(g_allocators_mu);
  next_ = g_allocators;
  if (next_) next_->prev_ = this;
  g_allocators = this;
}

DeviceAllocator::~DeviceAllocator() {
  {
    std::lock_guard<std::mutex> lk(g_allocators_mu);
    if (next_) next_->prev_ = prev_;
    (prev_ ? prev_->next_ : g_allocators) = next_;
  }
  while (n_pinned_ > 0) (void)hipHostFree(pinned_[--n_pinned_]);
}

void DeviceAllocator::trim_device(int device, const DeviceAllocator* except) {
  std::lock_guard<std::mutex> lk(g_allocators_mu);
  for (DeviceAllocator* a = g_allocators; a; a = a->next_)
    if (a != except && a->device_ == device) (void)a->trim();
}

int DeviceAllocator::status(ScratchPool<DeviceMem>::Status st, size_t bytes) const {
  if (st == ScratchPool<DeviceMem>::kOverBudget)
    return fail(RSV_ENOMEM, "HBM budget exceeded: %zu in use + %zu requested > %zu budget", in_use(),
                bytes, budget_);
  if (st == ScratchPool<DeviceMem>::kNoMemory)
    return fail(RSV_ENOMEM, "hipMalloc(%zu) failed: out of memory", bytes);
  return RSV_OK;
}

double* DeviceAllocator::pinned_take() {
  {
    std::lock_guard<std::mutex> lk(mu_);
    if (n_pinned_ > 0) return pinned_[--n_pinned_];
  }
  double* h = nullptr;
  if (hipHostMalloc((void**)&h, kPinnedDoubles * sizeof(double), hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return h;
}

void DeviceAllocator::pinned_give(double* h) {
  if (!h) return;
  {
    std::lock_guard<std::mutex> lk(mu_);
    if (n_pinned_ < kKeepPinned) {
      pinned_[n_pinned_++] = h;
      return;
    }
  }
  (void)hipHostFree(h);
}

ArenaAllocator::~ArenaAllocator() {
  if (base_) (void)hipFree(base_);
}

int ArenaAllocator::init(size_t bytes) {
  bytes = round_up(bytes);
  hipError_t e = hipMalloc((void**)&base_, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    base_ = nullptr;
    return fail(RSV_ENOMEM, "arena hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
  }
  std::lock_guard<std::mutex> lk(mu_);
  ff_.reset(bytes);
  return RSV_OK;
}

int ArenaAllocator::alloc(size_t bytes, void** p) {
  *p = nullptr;
  bytes = round_up(bytes ? bytes : 1);
  std::lock_guard<std::mutex> lk(mu_);
  size_t off = 0;
  if (!ff_.take(bytes, &off))
    return fail(RSV_ENOMEM, "arena has no free block of %zu bytes (%zu of %zu in use)", bytes,
                ff_.used(), ff_.size());
  *p = base_ + off;
  return RSV_OK;
}

void ArenaAllocator::release(void* p, size_t bytes) {
  if (!p) return;
  bytes = round_up(bytes ? bytes : 1);
  std::lock_guard<std::mutex> lk(mu_);
  ff_.give((size_t)((char*)p - base_), bytes);
}

size_t ArenaAllocator::in_use() const {
  std::lock_guard<std::mutex> lk(mu_);
  return ff_.used();
}

size_t vec_bytes(int n, int prec) { return (size_t(1) << n) * amp_bytes(prec); }

size_t partial_doubles(int n, int prec) {
  int64_t a = sweep_num_partials(prec, n), b = vec_num_partials(prec, n);
  int64_t c = occ_num_partials(n), d = sample_scratch_doubles(n);
  // the two partial arrays are adjacent: together they hold a group of re-orthogonalisation
  // inner products (2 kDotGroup rows of vec_num_partials)
  const int64_t e = (int64_t)kDotGroup * b;
  // and the norm partials of two iterations where the forming pass sums them
  const int64_t f = a <= kFusedParts ? 2 * a : a;
  return (size_t)std::max(std::max(std::max(f, b), std::max(c, d)), e);
}

size_t workspace_bytes(int n, int kmax, int prec) {
  return (size_t)(kmax + 3) * vec_bytes(n, prec) + 2 * round_up(partial_doubles(n, prec) * 8) +
         kScalarBytes;
}

size_t register_bytes(int n, int prec) {
  return 32 * 32 * 8 + round_up(diag_table_doubles(prec, n) * 8);
}

int check_state_args(int n, int prec) {
  if (n < 1 || n > kMaxAtoms) return fail(RSV_EINVAL, "n_atoms must be in 1..%d", kMaxAtoms);
  if (prec != kC128 && prec != kC64) return fail(RSV_EINVAL, "unknown precision %d", prec);
  return RSV_OK;
}

// ------------------------------------------------------------------------------ pulses
int check_pulses(const rsv_pulses* pl, int n) {
  if (!pl || !pl->omega || !pl->delta) return fail(RSV_EINVAL, "pulses: omega and delta required");
  if (pl->n_samples < 1) return fail(RSV_EINVAL, "pulses: n_samples must be >= 1");
  if (pl->per_site != 0 && pl->per_site != 1) return fail(RSV_EINVAL, "pulses: per_site is 0 or 1");
  const size_t cnt = (size_t)pl->n_samples * (pl->per_site ? (size_t)n : 1);
  if (!finite_all(pl->omega, cnt) || !finite_all(pl->delta, cnt) ||
      (pl->phi && !finite_all(pl->phi, cnt)))
    return fail(RSV_EINVAL, "pulses: non-finite sample");
  return RSV_OK;
}

// Midpoint value of step k (Sec. III): mean of the samples at floor(m) and ceil(m),
// m = (k + 1/2) dt in ns.
static double midpoint(const double* x, int64_t k, int dt_ns) {
  const int64_t twice = (2 * k + 1) * (int64_t)dt_ns;  // 2m, an integer
  const int64_t lo = twice / 2, hi = (twice + 1) / 2;
  return 0.5 * (x[lo] + x[hi]);
}

void step_midpoints(const double* x, int64_t first, int64_t count, int dt_ns, double* out) {
  for (int64_t j = 0; j < count; ++j) out[j] = midpoint(x, first + j, dt_ns);
}

StepCoef step_coef(const rsv_pulses* pl, int n, int64_t k, int dt_ns) {
  StepCoef c;
  std::memset(&c, 0, sizeof c);
  c.n = n;
  double om[kMaxAtoms], de[kMaxAtoms], ph[kMaxAtoms];
  for (int i = 0; i < n; ++i) {
    const size_t off = pl->per_site ? (size_t)i * pl->n_samples : 0;
    om[i] = midpoint(pl->omega + off, k, dt_ns);
    de[i] = midpoint(pl->delta + off, k, dt_ns);
    ph[i] = pl->phi ? midpoint(pl->phi + off, k, dt_ns) : 0.0;
  }
  bool uniform = true;
  for (int i = 1; i < n; ++i)
    uniform = uniform && om[i] == om[0] && de[i] == de[0] && ph[i] == ph[0];
  c.mode = !uniform ? kCoefSite : (ph[0] == 0.0 ? kCoefReal : kCoefUniform);
  for (int i = 0; i < n; ++i) {
    const int p = n - 1 - i;  // atom i is bit n-1-i
    const double h = 0.5 * om[i];
    c.up_re[p] = h * std::cos(ph[i]);
    c.up_im[p] = -h * std::sin(ph[i]);
    c.dn_re[p] = h * std::cos(ph[i]);
    c.dn_im[p] = h * std::sin(ph[i]);
    c.delta[p] = de[i];
  }
  return c;
}

int check_opts(const rsv_evolve_opts* o, const rsv_pulses* pl, int64_t* first, int64_t* count) {
  if (!o) return fail(RSV_EINVAL, "opts is NULL");
  if (o->dt_ns < 1) return fail(RSV_EINVAL, "dt_ns must be >= 1");
  if ((pl->n_samples - 1) % o->dt_ns != 0)
    return fail(RSV_EINVAL, "pulse duration %lld ns is not a multiple of dt = %d ns",
                (long long)(pl->n_samples - 1), o->dt_ns);
  if (!(o->tol > 0.0) || !std::isfinite(o->tol)) return fail(RSV_EINVAL, "tol must be > 0");
  if (o->kmax < 2 || o->kmax > kMaxKrylov) return fail(RSV_EINVAL, "kmax must be in 2..64");
  if (o->max_substep_depth < 0 || o->max_substep_depth > 40)
    return fail(RSV_EINVAL, "max_substep_depth must be in 0..40");
  if (o->reorth != 0 && o->reorth != 1) return fail(RSV_EINVAL, "reorth must be 0 or 1");
  const int64_t K = (pl->n_samples - 1) / o->dt_ns;
  if (o->first_step < 0 || o->first_step > K) return fail(RSV_EINVAL, "first_step out of range");
  const int64_t cnt = o->n_steps < 0 ? K - o->first_step : o->n_steps;
  if (o->first_step + cnt > K) return fail(RSV_EINVAL, "steps beyond the end of the pulse");
  *first = o->first_step;
  *count = cnt;
  return RSV_OK;
}

// ------------------------------------------------------------------------------ register
int build_interactions(int n, const double* xyz, double c6, double* ub) {
  if (!std::isfinite(c6)) return fail(RSV_EINVAL, "C6 not finite");
  if (!finite_all(xyz, (size_t)3 * n)) return fail(RSV_EINVAL, "positions not finite");
  std::memset(ub, 0, 32 * 32 * sizeof(double));
  for (int i = 0; i < n; ++i) {
    for (int j = 0; j < i; ++j) {
      const double dx = xyz[3 * i] - xyz[3 * j], dy = xyz[3 * i + 1] - xyz[3 * j + 1],
                   dz = xyz[3 * i + 2] - xyz[3 * j + 2];
      const double r2 = dx * dx + dy * dy + dz * dz;
      if (r2 == 0.0) return fail(RSV_EINVAL, "atoms %d and %d coincide", j, i);
      const double u = c6 / (r2 * r2 * r2);
      const int p = n - 1 - i, q = n - 1 - j;
      ub[p * 32 + q] = ub[q * 32 + p] = u;
    }
  }
  return RSV_OK;
}

int register_create(rsv_ctx* ctx, Allocator* alloc, int n, const double* xyz, double c6,
                    int prec, hipStream_t stream, double* h_scal, rsv_register** out) {
  *out = nullptr;
  if (!ctx || !xyz) return fail(RSV_EINVAL, "NULL argument");
  RSV_TRY(check_state_args(n, prec));
  double ub[32 * 32];
  RSV_TRY(build_interactions(n, xyz, c6, ub));
  HIP_TRY(hipSetDevice(ctx->device));
  rsv_register* r = new (std::nothrow) rsv_register();
  if (!r) return fail(RSV_ENOMEM, "host allocation failed");
  r->ctx = ctx;
  r->alloc = alloc;
  r->n = n;
  r->prec = prec;
  r->c6 = c6;
  for (int p = 1; p < n; ++p)
    for (int q = 0; q < p; ++q) r->u_abs += std::fabs(ub[p * 32 + q]);
  if (h_scal) {
    r->h_scal = h_scal;
  } else {
    hipError_t e = hipHostMalloc((void**)&r->h_scal, 512 * sizeof(double), hipHostMallocDefault);
    if (e != hipSuccess) {
      delete r;
      return fail(RSV_EDEVICE, "hipHostMalloc failed: %s", hipGetErrorString(e));
    }
    r->own_h_scal = true;
  }
  void* p = nullptr;
  const int rc = alloc->alloc(register_bytes(n, prec), &p);
  if (rc != RSV_OK) {
    register_destroy(r, stream);
    return rc;
  }
  r->bytes = register_bytes(n, prec);
  r->d_ub = (double*)p;
  r->d_dtab = (double*)((char*)p + 32 * 32 * 8);
  // the host array must outlive the asynchronous copy: synchronise before returning
  hipError_t e = hipMemcpyAsync(r->d_ub, ub, sizeof ub, hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = diag_tables_build(prec, n, r->d_ub, r->d_dtab, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    register_destroy(r, stream);
    return fail(RSV_EDEVICE, "interaction diagonal: %s", hipGetErrorString(e));
  }
  *out = r;
  return RSV_OK;
}

static void workspace_release(rsv_register* reg) {
  Workspace& ws = reg->ws;
  if (ws.block) reg->alloc->release(ws.block, ws.bytes);
  ws = Workspace{};
}

void register_destroy(rsv_register* reg, hipStream_t stream) {
  if (!reg) return;
  (void)hipSetDevice(reg->ctx->device);
  (void)hipStreamSynchronize(stream);
  workspace_release(reg);
  if (reg->d_hbuf) reg->alloc->release(reg->d_hbuf, vec_bytes(reg->n, reg->prec));
  if (reg->d_efull) reg->alloc->release(reg->d_efull, (size_t(1) << reg->n) * sizeof(double));
  if (reg->d_ub) reg->alloc->release(reg->d_ub, reg->bytes);
  if (reg->own_h_scal && reg->h_scal) (void)hipHostFree(reg->h_scal);
  if (reg->h_arnoldi) (void)hipHostFree(reg->h_arnoldi);
  delete reg;
}

int workspace_acquire(rsv_register* reg, int kmax) {
  Workspace& ws = reg->ws;
  if (ws.block && ws.kmax == kmax) return RSV_OK;
  workspace_release(reg);
  const size_t vb = vec_bytes(reg->n, reg->prec);
  const size_t pb = round_up(partial_doubles(reg->n, reg->prec) * 8);
  const size_t bytes = workspace_bytes(reg->n, kmax, reg->prec);
  void* block = nullptr;
  RSV_TRY(reg->alloc->alloc(bytes, &block));
  ws.block = block;
  ws.bytes = bytes;
  ws.kmax = kmax;
  char* p = (char*)block;
  ws.basis.resize(kmax + 1);
  for (int i = 0; i <= kmax; ++i) ws.basis[i] = p + (size_t)i * vb;
  ws.z = p + (size_t)(kmax + 1) * vb;
  ws.t = p + (size_t)(kmax + 2) * vb;
  ws.pnorm = (double*)(p + (size_t)(kmax + 3) * vb);
  ws.pnorm2 = ws.pnorm + sweep_num_partials(reg->prec, reg->n);
  ws.pdot = (double*)(p + (size_t)(kmax + 3) * vb + pb);
  ws.dscal = (double*)(p + (size_t)(kmax + 3) * vb + 2 * pb);
  return RSV_OK;
}

// The register's 2^N interaction energies in FP64, built on first use and kept.
int register_energies(rsv_register* reg, hipStream_t s, const double** out) {
  if (!reg->d_efull) {
    void* p = nullptr;
    RSV_TRY(reg->alloc->alloc((size_t(1) << reg->n) * sizeof(double), &p));
    const hipError_t e = diag_build(kC128, reg->n, reg->d_ub, p, s);
    if (e != hipSuccess) {
      reg->alloc->release(p, (size_t(1) << reg->n) * sizeof(double));
      return fail(RSV_EDEVICE, "interaction energies: %s", hipGetErrorString(e));
    }
    reg->d_efull = (double*)p;
  }
  *out = reg->d_efull;
  return RSV_OK;
}

// ------------------------------------------------------------------------------ Lanczos
namespace {

// Device scalars: slot 2k holds |u_k|^2, slot 2k+1 holds Re<u_k, H u_k>; kNormSlot |psi|^2;
// from kDotSlot, Re and Im <u_l, u_k> of the re-orthogonalisation (2 kMaxKrylov values).
constexpr int kNormSlot = 2 * kMaxKrylov + 4;
constexpr int kDotSlot = 256;
static_assert(kDotSlot + 2 * kMaxKrylov <= (int)(kScalarBytes / 8), "device scalar block");

struct Lanczos {
  rsv_register* reg;
  hipStream_t s;
  rsv_stats* st;
  double norm2 = 0.0;  // |psi|^2 of the state the last step began with
  double alpha[kMaxKrylov + 1], beta[kMaxKrylov + 1], scale[kMaxKrylov + 1];
  double yre[kMaxKrylov], yim[kMaxKrylov];
  std::vector<double> work;
  double* occ_partial = nullptr;  // fused occupation sums of an observed step's combination
  double dir = 1.0;               // -1: exp(+i tau H), the step backwards in time
  // dimensions of the previous step's runs (its sub-steps): how many iterations to queue first
  static constexpr int kHints = 8;
  int hint[kHints] = {};
};

// Device scalar slots [first_slot, first_slot + count) through the same slots of h_scal.
int fetch_scalars(Lanczos& L, int first_slot, int count, double* out) {
  double* h = L.reg->h_scal + first_slot;
  HIP_TRY(hipMemcpyAsync(h, L.reg->ws.dscal + first_slot, count * sizeof(double),
                         hipMemcpyDeviceToHost, L.s));
  HIP_TRY(hipStreamSynchronize(L.s));
  for (int i = 0; i < count; ++i) out[i] = h[i];
  return RSV_OK;
}

// Full re-orthogonalisation of the new vector u_k (classical Gram-Schmidt with FP64 inner
// products): u_k <- u_k - sum_{l<k} v_l <v_l, u_k>, v_l = s_l u_l.  The result goes to a
// fresh buffer that becomes basis[k] (the old one becomes the high-pass partial t, which
// the caller recomputes).  b2 is |u_k|^2 before on entry and after on return.
int reorthogonalise(Lanczos& L, int k, double* b2) {
  rsv_register* reg = L.reg;
  Workspace& ws = reg->ws;
  const int n = reg->n, prec = reg->prec;
  const int64_t nw = vec_num_partials(prec, n);
  for (int l0 = 0; l0 < k; l0 += kDotGroup) {
    DotGroup d{};
    d.g = std::min(kDotGroup, k - l0);
    for (int g = 0; g < d.g; ++g) d.x[g] = ws.basis[l0 + g];
    HIP_TRY(multi_dot(prec, n, d, ws.basis[k], ws.pnorm, L.s));
    HIP_TRY(finalize_rows(ws.pnorm, dot_num_partials(n), 2 * d.g, ws.dscal + kDotSlot + 2 * l0, L.s));
  }
  double dots[2 * kMaxKrylov];
  RSV_TRY(fetch_scalars(L, kDotSlot, 2 * k, dots));
  CombineCoef cc;
  std::memset(&cc, 0, sizeof cc);
  cc.m = k + 1;
  cc.re[0] = 1.0;
  cc.x[0] = ws.basis[k];
  double loss = 0.0;
  for (int l = 0; l < k; ++l) {
    const double sl = L.scale[l];
    if (!std::isfinite(dots[2 * l]) || !std::isfinite(dots[2 * l + 1]))
      return fail(RSV_ENUMERIC, "re-orthogonalisation inner product not finite");
    cc.re[l + 1] = -sl * sl * dots[2 * l];
    cc.im[l + 1] = -sl * sl * dots[2 * l + 1];
    cc.x[l + 1] = ws.basis[l];
    loss = std::max(loss, sl * std::hypot(dots[2 * l], dots[2 * l + 1]));
  }
  if (*b2 > 0.0) L.st->ortho_loss = std::max(L.st->ortho_loss, loss / std::sqrt(*b2));
  HIP_TRY(krylov_combine(prec, n, cc, ws.t, ws.pnorm, L.s));
  HIP_TRY(finalize_sum(ws.pnorm, nw, ws.dscal + 2 * k, L.s));
  std::swap(ws.basis[k], ws.t);
  RSV_TRY(fetch_scalars(L, 2 * k, 1, b2));
  return RSV_OK;
}

// y = exp(-i h T_m) e_1 (into L.yre, L.yim) and |y_{m-1}| for the current T_m.
int small_exponential(Lanczos& L, int m, double h, double* last) {
  if (tridiag_expm_series(m, L.alpha, L.beta, h, L.yre, L.yim, L.work.data()) != 0)
    return fail(RSV_ENUMERIC, "tridiagonal eigensolver failed (m = %d)", m);
  *last = std::hypot(L.yre[m - 1], L.yim[m - 1]);
  return RSV_OK;
}

// psi <- exp(-i tau H) psi with psi in basis[0] (|psi|^2 = dscal[kNormSlot]).
//
// Krylov vectors are kept unnormalised: v_k = s_k u_k with s_0 = 1/|psi| and
// s_k = 1/beta_{k-1}.  Sweep k >= 1 forms
//   u_k = s_{k-1} z_{k-1} - s_{k-1}^3 <u_{k-1}, z_{k-1}> u_{k-1} - (s_{k-2}/s_{k-1}) u_{k-2}
// (= H v_{k-1} - alpha_{k-1} v_{k-1} - beta_{k-2} v_{k-2}) in its first pass, from scalars in
// device memory, stores it and returns the partials of |u_k|^2 = beta_{k-1}^2; the later passes
// compute z_k = H u_k.  Iterations are queued several at a time (as many as the previous step took,
// or as the a-priori course of the estimate suggests) and their scalars fetched together; the
// host then goes through the dimensions in order and takes the smallest that meets the tolerance
// (reorth: one iteration at a time, since the host forms its coefficients).  With obs set, the
// combination that completes the step also writes the occupation sums of the new state to obs
// (device, n + 1 doubles).
int propagate(Lanczos& L, const StepCoef& c, double tau, double tol, int kmax, int max_depth,
              bool reorth, double* obs = nullptr) {
  rsv_register* reg = L.reg;
  Workspace& ws = reg->ws;
  const int n = reg->n, prec = reg->prec;
  const int64_t np_norm = sweep_norm_partials(prec, n), np_dot = sweep_dot_partials(prec, n);
  const bool single = sweep_passes(prec, n) == 1;
  // few enough partials: the forming pass sums them (the two norms alternate between buffers,
  // since its workgroups read one while they write the other)
  const bool fused = !single && !reorth && np_dot <= kFusedParts && np_norm <= kFusedParts;
  auto norm_parts = [&](int k) { return fused && (k & 1) ? ws.pnorm2 : ws.pnorm; };
  // an iteration too many costs large vectors (from about 40 us per iteration) more than a round trip
  const bool large = vec_bytes(n, prec) >= (size_t(16) << 20);
  const double hbytes = (double)(size_t(1) << n) * (prec == kC128 ? 40.0 : 20.0);
  const double log2_tol = std::log2(tol);
  double remaining = tau;
  for (int run = 0; remaining > 0.0; ++run) {
    int& hint = L.hint[run < Lanczos::kHints ? run : Lanczos::kHints - 1];
    // sweep 0: z_0 = H u_0 and <u_0, z_0>
    {
      const SweepIn in{ws.basis[0], nullptr, nullptr, 1.0, 0.0, 0.0, nullptr, 0.0};
      const SweepOut so{nullptr, nullptr, ws.pdot};
      HIP_TRY(hpsi_sweep(prec, n, c, reg->d_dtab, in, ws.z, ws.t, so, kAllPasses, L.s));
      if (!fused) HIP_TRY(finalize_sum(ws.pdot, np_dot, ws.dscal + 1, L.s));
      L.st->krylov_iters += 1;
      L.st->bytes_hpsi += hbytes;
    }
    // device address of |u_k|^2 (|psi|^2 for k = 0): the forming pass takes s_k from it
    auto dev_norm = [&](int k) { return ws.dscal + (k == 0 ? kNormSlot : 2 * k); };
    // u_k from z_{k-1}, u_{k-1}, u_{k-2} with device-side coefficients, and |u_k|^2
    auto form = [&](int k) -> int {
      SweepIn in{ws.z, ws.basis[k - 1], k >= 2 ? ws.basis[k - 2] : nullptr, 0.0, 0.0, 0.0,
                 ws.dscal + (2 * (k - 1) + 1), 0.0};
      in.nrm1 = dev_norm(k - 1);
      in.nrm2 = k >= 2 ? dev_norm(k - 2) : nullptr;
      if (fused) {
        in.part_dot = ws.pdot;
        in.n_dot = (int)np_dot;
        in.part_nrm = norm_parts(k - 1);
        in.n_nrm = k >= 2 ? (int)np_norm : 0;
      }
      const SweepOut so{ws.basis[k], norm_parts(k), ws.pdot};
      // single-pass sizes compute z_k in the same pass; otherwise only the forming pass
      HIP_TRY(hpsi_sweep(prec, n, c, reg->d_dtab, in, ws.z, ws.t, so, kFirstPass, L.s));
      if (!fused) HIP_TRY(finalize_sum(ws.pnorm, np_norm, ws.dscal + 2 * k, L.s));
      if (single) HIP_TRY(finalize_sum(ws.pdot, np_dot, ws.dscal + 2 * k + 1, L.s));
      return RSV_OK;
    };
    // z_k = H u_k: the remaining passes, or all of them when u_k was re-orthogonalised
    // after the forming pass
    auto later = [&](int k) -> int {
      L.st->krylov_iters += 1;
      L.st->bytes_hpsi += hbytes;
      if (single && !reorth) return RSV_OK;
      const SweepIn in2{ws.basis[k], nullptr, nullptr, 1.0, 0.0, 0.0, nullptr, 0.0};
      const SweepOut so2{nullptr, nullptr, ws.pdot};
      HIP_TRY(hpsi_sweep(prec, n, c, reg->d_dtab, in2, ws.z, ws.t, so2,
                         reorth ? kAllPasses : kLaterPasses, L.s));
      if (!fused) HIP_TRY(finalize_sum(ws.pdot, np_dot, ws.dscal + 2 * k + 1, L.s));
      return RSV_OK;
    };
    int m = 0;  // dimensions gone through
    double nrm = 0.0, sub = remaining;
    bool done = false;
    int next = reorth ? 1 : KrylovCourse::first(hint, large);
    KrylovCourse course;
    double bks[kMaxKrylov + 1];  // |u_k|
    while (!done) {
      const int upto = std::min(kmax, m + std::max(1, next));
      for (int k = m + 1; k <= upto; ++k) {
        if (k > 1) RSV_TRY(later(k - 1));
        RSV_TRY(form(k));
      }
      if (fused) HIP_TRY(finalize_sum(norm_parts(upto), np_norm, ws.dscal + 2 * upto, L.s));
      double scal[kNormSlot + 1];
      RSV_TRY(fetch_scalars(L, 0, kNormSlot + 1, scal));
      if (m == 0) {
        L.norm2 = scal[kNormSlot];
        nrm = std::sqrt(L.norm2);
        if (!(nrm > 0.0) || !std::isfinite(nrm)) return fail(RSV_ENUMERIC, "state norm is %g", nrm);
        L.scale[0] = 1.0 / nrm;
        course.start(remaining, nrm, large);
      }
      for (int k = m + 1; k <= upto && !done; ++k) {
        double ab[2] = {scal[2 * k - 1], scal[2 * k]};  // <u_{k-1}, z_{k-1}>, |u_k|^2
        if (!std::isfinite(ab[0]) || !std::isfinite(ab[1]))
          return fail(RSV_ENUMERIC, "Lanczos coefficient not finite at iteration %d", k);
        const double sk1 = L.scale[k - 1];
        L.alpha[k - 1] = sk1 * sk1 * ab[0];
        if (reorth) {
          RSV_TRY(reorthogonalise(L, k, &ab[1]));
          if (!std::isfinite(ab[1]))
            return fail(RSV_ENUMERIC, "Lanczos coefficient not finite at iteration %d", k);
        }
        const double bk = std::sqrt(std::max(ab[1], 0.0));  // beta_{k-1}
        bks[k] = bk;
        L.beta[k - 1] = bk;
        L.scale[k] = 1.0 / bk;
        m = k;
        course.add(L.alpha[k - 1], bk);
        if (k < kmax && bk != 0.0 && !course.due(log2_tol)) continue;
        double ylast = 0.0;
        RSV_TRY(small_exponential(L, m, remaining, &ylast));
        if (bk * ylast * nrm <= tol || bk == 0.0) {
          // a smaller dimension may do: the tests begin near the tolerance, not before it
          while (m > 1) {
            RSV_TRY(small_exponential(L, m - 1, remaining, &ylast));
            if (!(bks[m - 1] * ylast * nrm <= tol)) break;
            --m;
          }
          done = true;
          break;
        }
        course.found(bk * ylast * nrm, log2_tol);
        if (k == kmax) {
          // Not converged: advance by the longest part of the step that this basis already
          // resolves (same H_k, so the split is exact), then restart from the new state.
          // The first dyadic fraction that converges brackets it; bisection refines it.
          bool ok = false;
          double bad = remaining;
          for (int d = 1; d <= max_depth && !ok; ++d) {
            sub = std::ldexp(remaining, -d);
            RSV_TRY(small_exponential(L, m, sub, &ylast));
            ok = bk * ylast * nrm <= tol;
            if (!ok) bad = sub;
          }
          if (!ok) return fail(RSV_ENOTCONV, "Krylov exponential not converged with kmax = %d", kmax);
          for (int it = 0; it < 10; ++it) {
            const double mid = 0.5 * (sub + bad);
            RSV_TRY(small_exponential(L, m, mid, &ylast));
            if (bk * ylast * nrm <= tol) sub = mid;
            else bad = mid;
          }
          L.st->substeps += 1;
          done = true;
        }
      }
      if (!done) next = reorth ? 1 : course.ahead(log2_tol, kmax - m);
    }
    hint = m;
    L.st->krylov_max = std::max<int64_t>(L.st->krylov_max, m);
    double ylast = 0.0;
    RSV_TRY(small_exponential(L, m, L.dir * sub, &ylast));
    CombineCoef cc;
    std::memset(&cc, 0, sizeof cc);
    cc.m = m;
    for (int l = 0; l < m; ++l) {
      cc.re[l] = nrm * L.yre[l] * L.scale[l];
      cc.im[l] = nrm * L.yim[l] * L.scale[l];
      cc.x[l] = ws.basis[l];
    }
    if (obs && sub == remaining)
      HIP_TRY(krylov_combine_occ(prec, n, cc, ws.z, ws.pnorm, L.occ_partial, obs, L.s));
    else
      HIP_TRY(krylov_combine(prec, n, cc, ws.z, ws.pnorm, L.s));
    HIP_TRY(finalize_sum(ws.pnorm, vec_num_partials(prec, n), ws.dscal + kNormSlot, L.s));
    std::swap(ws.basis[0], ws.z);
    remaining = (sub == remaining) ? 0.0 : remaining - sub;
  }
  return RSV_OK;
}

}  // namespace

namespace {

// Device memory borrowed from an allocator for the duration of one call.
struct Borrowed {
  Allocator* a = nullptr;
  void* p = nullptr;
  size_t bytes = 0;
  hipStream_t s = nullptr;
  ~Borrowed() {
    if (p) {
      const bool idle = hipStreamSynchronize(s) == hipSuccess;
      a->give_back(p, bytes, idle);
    }
  }
};

}  // namespace

// Whether calls on this register run on one workgroup: it fits, nothing asks for the host driver
// (re-orthogonalisation does), and every step's exponential fits the device's series (else the
// device would sub-step where the host's eigendecomposition need not, or give up where it would
// not).  A step there costs its iterations' latency on the chip (about 1 us each at 10 atoms),
// on the host driver five API calls per iteration (20 us).
static bool small_route(const rsv_register* reg, double tau, double max_drive, double max_detuning) {
  return reg->n <= packed_max_atoms(reg->prec) &&
         packed_resolves(tau, 0.5 * (reg->u_abs + max_detuning + max_drive));
}

// `count` steps in launches of as many as the kernel arguments hold.
struct SmallRun {
  rsv_register* reg;
  double tau, tol, dir;
  int kmax, max_depth, per_site, direct;
  bool with_phi;  // direct: whether any coupling has an imaginary part
};

// values(k, c, dst): omega, delta (and phi) of steps k..k+c-1, sites x c values each, to dst.
template <class Values>
static int run_small(const SmallRun& r, const Values& values, int64_t count, void* d_psi, double* obs,
                     int64_t obs_every, hipStream_t s, rsv_stats* st, double* norm2) {
  rsv_register* reg = r.reg;
  RSV_TRY(workspace_acquire(reg, r.kmax));
  Workspace& ws = reg->ws;
  const int n = reg->n, prec = reg->prec;
  const size_t vb = vec_bytes(n, prec);
  const int64_t sites = r.per_site ? n : 1;
  const int64_t per = kMidValues / (sites * (r.with_phi ? 3 : 2));
  char* blk = (char*)ws.block;  // kmax + 1 basis vectors, then two more
  PackedJob jb{};
  jb.n = n;
  jb.kmax = r.kmax;
  jb.max_depth = r.max_depth;
  jb.per_site = r.per_site;
  jb.real = !r.per_site && !r.with_phi;
  jb.direct = r.direct;
  jb.dir = r.dir;
  jb.tau = r.tau;
  jb.tol = r.tol;
  jb.ub = reg->d_ub;
  jb.diag = (double*)(blk + (size_t)(r.kmax + 1) * vb);  // 8 bytes per amplitude at least
  void* carry = blk + (size_t)(r.kmax + 2) * vb;         // the state between launches
  jb.basis = blk;
  jb.out = ws.dscal;
  jb.obs = obs;
  jb.obs_every = obs_every;
  double mid[kMidValues];
  for (int64_t k = 0; k < count; k += per) {
    const int64_t c = std::min(per, count - k);
    values(k, c, mid);
    jb.n_steps = c;
    jb.resume = k > 0;
    jb.obs_first = k;
    jb.psi_in = k == 0 ? d_psi : carry;
    jb.psi_out = k + c == count ? d_psi : carry;
    HIP_TRY(small_evolve(prec, jb, mid, r.with_phi, s));
  }
  double* h = reg->h_scal;
  HIP_TRY(hipMemcpyAsync(h, ws.dscal, 8 * sizeof(double), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  const int status = (int)h[0];
  st->krylov_iters += (int64_t)h[1];
  st->krylov_max = std::max<int64_t>(st->krylov_max, (int64_t)h[2]);
  st->substeps += (int64_t)h[3];
  st->bytes_hpsi += h[1] * (double)(size_t(1) << n) * (prec == kC128 ? 40.0 : 20.0);
  *norm2 = h[4];
  if (status == RSV_ENOTCONV)
    return fail(RSV_ENOTCONV, "Krylov exponential not converged with kmax = %d", r.kmax);
  if (status != RSV_OK) {
    if (!(h[4] > 0.0) || !std::isfinite(h[4]))
      return fail(RSV_ENUMERIC, "state norm is %g", std::sqrt(h[4]));
    return fail(RSV_ENUMERIC, "Lanczos coefficient not finite");
  }
  return RSV_OK;
}

// evolve on one workgroup.  *taken = false: the call takes the host driver.  (Allocates nothing on
// the host, whatever the number of steps.)
static int evolve_small(rsv_register* reg, const rsv_pulses* pl, const rsv_evolve_opts* o,
                        int64_t first, int64_t count, void* d_psi, double* obs_dev, int obs_every,
                        hipStream_t s, rsv_stats* st, double* norm2, bool* taken) {
  const int n = reg->n;
  const double tau = o->dt_ns * 1e-3;
  const int64_t rows = pl->per_site ? n : 1;
  *taken = false;
  if (count < 1 || o->reorth || n > packed_max_atoms(reg->prec)) return RSV_OK;
  // the widest step, 64 at a time
  double drive = 0.0, detuning = 0.0;
  for (int64_t k = 0; k < count; k += 64) {
    const int64_t c = std::min<int64_t>(64, count - k);
    double a[64] = {}, d[64] = {}, x[64];
    for (int64_t i = 0; i < rows; ++i) {
      step_midpoints(pl->omega + i * pl->n_samples, first + k, c, o->dt_ns, x);
      for (int64_t j = 0; j < c; ++j) a[j] += std::fabs(x[j]);
      step_midpoints(pl->delta + i * pl->n_samples, first + k, c, o->dt_ns, x);
      for (int64_t j = 0; j < c; ++j) d[j] += std::fabs(x[j]);
    }
    for (int64_t j = 0; j < c; ++j) {
      drive = std::max(drive, a[j] * (double)(n / rows));
      detuning = std::max(detuning, d[j] * (double)(n / rows));
    }
  }
  if (!small_route(reg, tau, drive, detuning)) return RSV_OK;
  *taken = true;
  const SmallRun r{reg, tau, o->tol, 1.0, o->kmax, o->max_substep_depth, pl->per_site, 0,
                   pl->phi != nullptr};
  const auto values = [&](int64_t k, int64_t c, double* dst) {
    for (const double* x : {pl->omega, pl->delta, pl->phi}) {
      if (!x) continue;
      for (int64_t i = 0; i < rows; ++i, dst += c)
        step_midpoints(x + i * pl->n_samples, first + k, c, o->dt_ns, dst);
    }
  };
  return run_small(r, values, count, d_psi, obs_dev, obs_every, s, st, norm2);
}

int evolve(rsv_register* reg, const rsv_pulses* pl, const rsv_evolve_opts* o, void* d_psi,
           hipStream_t s, rsv_stats* st, int obs_every, double* obs_out) {
  if (!reg) return fail(RSV_EINVAL, "register is NULL");
  if (!d_psi) return fail(RSV_EINVAL, "state pointer is NULL");
  RSV_TRY(check_pulses(pl, reg->n));
  int64_t first = 0, count = 0;
  RSV_TRY(check_opts(o, pl, &first, &count));
  if (obs_out && obs_every < 1) return fail(RSV_EINVAL, "observation interval must be >= 1");
  const int64_t n_obs = obs_out ? count / obs_every : 0;
  const auto t0 = std::chrono::steady_clock::now();
  HIP_TRY(hipSetDevice(reg->ctx->device));
  RSV_TRY(workspace_acquire(reg, o->kmax));
  Workspace& ws = reg->ws;
  const int n = reg->n, prec = reg->prec;
  const size_t vb = vec_bytes(n, prec);
  // observed steps: fused occupation partials, then n + 1 sums per observation
  Borrowed ob;
  double* obs_dev = nullptr;
  if (n_obs > 0) {
    const size_t part = (size_t)combine_occ_partial_doubles(n);
    ob.a = reg->alloc;
    ob.s = s;
    ob.bytes = (part + (size_t)n_obs * (n + 1)) * sizeof(double);
    RSV_TRY(reg->alloc->borrow(ob.bytes, &ob.p));
    obs_dev = (double*)ob.p + part;
  }
  double norm2 = 0.0;
  bool small = false;
  RSV_TRY(evolve_small(reg, pl, o, first, count, d_psi, obs_dev, obs_every, s, st, &norm2, &small));
  if (small) {
    st->steps += count;
  } else {
    HIP_TRY(hipMemcpyAsync(ws.basis[0], d_psi, vb, hipMemcpyDeviceToDevice, s));
    HIP_TRY(norm2_partial(prec, n, ws.basis[0], ws.pnorm, s));
    HIP_TRY(finalize_sum(ws.pnorm, vec_num_partials(prec, n), ws.dscal + kNormSlot, s));
    Lanczos L;
    L.occ_partial = (double*)ob.p;
    L.reg = reg;
    L.s = s;
    L.st = st;
    std::memset(L.alpha, 0, sizeof L.alpha);
    std::memset(L.beta, 0, sizeof L.beta);
    std::memset(L.scale, 0, sizeof L.scale);
    L.work.assign(tridiag_work_doubles(kMaxKrylov), 0.0);
    const double tau = o->dt_ns * 1e-3;  // us
    for (int64_t k = first; k < first + count; ++k) {
      const StepCoef c = step_coef(pl, n, k, o->dt_ns);
      const int64_t j = k - first + 1;  // steps done after this one
      double* slot = (n_obs > 0 && j % obs_every == 0) ? obs_dev + (j / obs_every - 1) * (n + 1)
                                                        : nullptr;
      RSV_TRY(propagate(L, c, tau, o->tol, o->kmax, o->max_substep_depth, o->reorth != 0, slot));
      st->steps += 1;
    }
    HIP_TRY(hipMemcpyAsync(d_psi, ws.basis[0], vb, hipMemcpyDeviceToDevice, s));
    RSV_TRY(fetch_scalars(L, kNormSlot, 1, &norm2));
  }
  if (n_obs > 0) {
    std::vector<double> h((size_t)n_obs * (n + 1));
    HIP_TRY(hipMemcpy(h.data(), obs_dev, h.size() * sizeof(double), hipMemcpyDeviceToHost));
    for (int64_t r = 0; r < n_obs; ++r) {
      const double* v = h.data() + r * (n + 1);
      if (!(v[0] > 0.0)) return fail(RSV_ENUMERIC, "observed state has zero norm");
      for (int i = 0; i < n; ++i) obs_out[r * n + i] = v[1 + (n - 1 - i)] / v[0];
    }
  }
  st->norm_final = std::sqrt(norm2);
  st->seconds += std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  return RSV_OK;
}

int krylov_exp(rsv_register* reg, const StepCoef& c, double tau, double dir, double tol,
               int kmax, int max_depth, void* d_psi, hipStream_t s, rsv_stats* st) {
  if (!reg || !d_psi) return fail(RSV_EINVAL, "NULL argument");
  HIP_TRY(hipSetDevice(reg->ctx->device));
  const int n = reg->n, prec = reg->prec;
  double drive = 0.0, detuning = 0.0, v[3 * kMaxAtoms];  // by atom: bit p is atom n-1-p
  const int sites = c.mode == kCoefSite ? n : 1;
  for (int p = 0; p < sites; ++p) {
    const int i = sites - 1 - p;
    v[i] = 2.0 * c.up_re[p];
    v[sites + i] = c.delta[p];
    v[2 * sites + i] = 2.0 * c.up_im[p];
    drive += std::hypot(v[i], v[2 * sites + i]) * (n / sites);
    detuning += std::fabs(c.delta[p]) * (n / sites);
  }
  if (small_route(reg, tau, drive, detuning)) {
    const bool phi = c.mode != kCoefReal;
    const SmallRun r{reg, tau, tol, dir < 0 ? -1.0 : 1.0, kmax, max_depth, sites > 1 ? 1 : 0, 1, phi};
    double norm2 = 1.0;
    const auto values = [&](int64_t, int64_t, double* dst) {
      std::memcpy(dst, v, (size_t)sites * (phi ? 3 : 2) * sizeof(double));
    };
    const int rc = run_small(r, values, 1, d_psi, nullptr, 1, s, st, &norm2);
    return norm2 == 0.0 ? RSV_OK : rc;  // exp(...) 0 = 0
  }
  RSV_TRY(workspace_acquire(reg, kmax));
  Workspace& ws = reg->ws;
  const size_t vb = vec_bytes(n, prec);
  HIP_TRY(hipMemcpyAsync(ws.basis[0], d_psi, vb, hipMemcpyDeviceToDevice, s));
  HIP_TRY(norm2_partial(prec, n, ws.basis[0], ws.pnorm, s));
  HIP_TRY(finalize_sum(ws.pnorm, vec_num_partials(prec, n), ws.dscal + kNormSlot, s));
  Lanczos L;
  L.reg = reg;
  L.s = s;
  L.st = st;
  L.dir = dir < 0 ? -1.0 : 1.0;
  std::memset(L.alpha, 0, sizeof L.alpha);
  std::memset(L.beta, 0, sizeof L.beta);
  std::memset(L.scale, 0, sizeof L.scale);
  L.work.assign(tridiag_work_doubles(kMaxKrylov), 0.0);
  RSV_TRY(fetch_scalars(L, kNormSlot, 1, &L.norm2));
  if (L.norm2 == 0.0) return RSV_OK;  // exp(...) 0 = 0
  RSV_TRY(propagate(L, c, tau, tol, kmax, max_depth, false));
  HIP_TRY(hipMemcpyAsync(d_psi, ws.basis[0], vb, hipMemcpyDeviceToDevice, s));
  HIP_TRY(hipStreamSynchronize(s));
  return RSV_OK;
}

// ------------------------------------------------------------------------------ outputs
size_t occupation_scratch_bytes(int n) { return round_up((size_t)(occ_num_partials(n) + 64) * 8); }

size_t sample_scratch_bytes(int n, int shots) {
  return round_up((size_t)sample_scratch_doubles(n) * 8) + round_up((size_t)shots * 8);
}

int occupations_with(int n, int prec, const void* d_psi, void* d_scratch, double* h_tmp,
                     double* out, hipStream_t s) {
  double* part = (double*)d_scratch;
  double* res = part + occ_num_partials(n);
  HIP_TRY(occupations(prec, n, d_psi, part, res, s));
  HIP_TRY(hipMemcpyAsync(h_tmp, res, (n + 1) * sizeof(double), hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (!(h_tmp[0] > 0.0)) return fail(RSV_ENUMERIC, "state has zero norm");
  for (int i = 0; i < n; ++i) out[i] = h_tmp[1 + (n - 1 - i)] / h_tmp[0];
  return RSV_OK;
}

int sample_with(int n, int prec, const void* d_psi, uint64_t seed, int shots, void* d_scratch,
                uint64_t* out, hipStream_t s) {
  if (shots <= 0) return RSV_OK;
  double* scratch = (double*)d_scratch;
  uint64_t* d_idx = (uint64_t*)((char*)d_scratch + round_up((size_t)sample_scratch_doubles(n) * 8));
  HIP_TRY(sample(prec, n, d_psi, seed, shots, scratch, d_idx, s));
  HIP_TRY(hipMemcpyAsync(out, d_idx, (size_t)shots * 8, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  return RSV_OK;
}

}  // namespace rsv
