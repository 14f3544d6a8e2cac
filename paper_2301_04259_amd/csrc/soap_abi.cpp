// C ABI of libsoap (declarations and documentation in include/soap.h).
//
// This file holds argument validation, the context and its device workspace,
// host <-> device staging and the order of kernel launches.  All arithmetic of
// the method runs in the kernels of geom.hip, weights.hip, apply.hip and
// ccf.hip.
#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "soap_internal.hpp"

#define SOAP_API extern "C" __attribute__((visibility("default")))

namespace {

thread_local std::string g_init_err;

void setf(std::string& dst, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  dst = buf;
}

#define ARG_CHECK(cond, ...)        \
  do {                              \
    if (!(cond)) {                  \
      setf(err, __VA_ARGS__);       \
      return SOAP_ERR_ARG;          \
    }                               \
  } while (0)

#define HIP_TRY(expr)                                                                  \
  do {                                                                                 \
    hipError_t e_ = (expr);                                                            \
    if (e_ != hipSuccess) {                                                            \
      const bool oom_ = e_ == hipErrorOutOfMemory || e_ == hipErrorMemoryAllocation;  \
      setf(c->err, "%s failed: %s%s", #expr, hipGetErrorString(e_), oom_ ? soap::dev_cap_note() : ""); \
      return oom_ ? SOAP_ERR_OOM : SOAP_ERR_HIP;                                        \
    }                                                                                  \
  } while (0)

bool is_finite(double x) { return std::isfinite(x); }

template <typename T>
bool all_finite_host(const void* p, size_t n) {
  const T* a = static_cast<const T*>(p);
  for (size_t i = 0; i < n; ++i)
    if (!std::isfinite((double)a[i])) return false;
  return true;
}

soap_status validate_desc(const soap_star_desc* d, std::string& err) {
  ARG_CHECK(d != nullptr, "desc is NULL");
  ARG_CHECK(d->n_grid >= 2 && d->n_grid <= soap::MAX_GRID, "n_grid must be in [2, %d], got %d", soap::MAX_GRID,
            d->n_grid);
  ARG_CHECK(d->n_mu >= 1 && d->n_mu <= soap::MAX_MU, "n_mu must be in [1, %d], got %d", soap::MAX_MU, d->n_mu);
  ARG_CHECK(d->n_pix >= 8 && d->n_pix <= (int64_t(1) << 30), "n_pix must be in [8, 2^30], got %lld",
            (long long)d->n_pix);
  ARG_CHECK(d->precision == SOAP_PREC_FP32 || d->precision == SOAP_PREC_FP64, "unknown precision %d",
            d->precision);
  ARG_CHECK(d->contrast_mode == SOAP_CONTRAST_SCALAR || d->contrast_mode == SOAP_CONTRAST_PLANCK ||
                d->contrast_mode == SOAP_CONTRAST_ARRAY,
            "unknown contrast_mode %d", d->contrast_mode);
  ARG_CHECK(is_finite(d->vsini_kms) && std::fabs(d->vsini_kms) < 0.1 * soap::C_KMS, "vsini_kms out of range");
  ARG_CHECK(is_finite(d->incl_deg) && d->incl_deg >= 0.0 && d->incl_deg <= 180.0, "incl_deg must be in [0, 180]");
  ARG_CHECK(is_finite(d->ld_u1) && is_finite(d->ld_u2), "limb-darkening coefficients must be finite");
  ARG_CHECK(is_finite(d->diff_rot) && std::fabs(d->diff_rot) < 1.0, "diff_rot must be in (-1, 1)");
  ARG_CHECK(is_finite(d->ln_lambda0), "ln_lambda0 must be finite");
  ARG_CHECK(is_finite(d->dln_lambda) && d->dln_lambda > 0.0 && d->dln_lambda < 1.0, "dln_lambda must be in (0, 1)");
  ARG_CHECK(d->mu_bins != nullptr, "mu_bins is NULL");
  for (int b = 0; b < d->n_mu; ++b) {
    ARG_CHECK(is_finite(d->mu_bins[b]) && d->mu_bins[b] > 0.0 && d->mu_bins[b] <= 1.0,
              "mu_bins[%d] must be in (0, 1]", b);
    if (b) ARG_CHECK(d->mu_bins[b] < d->mu_bins[b - 1], "mu_bins must be strictly decreasing");
  }
  ARG_CHECK(d->spectra[SOAP_QUIET] != nullptr, "spectra[SOAP_QUIET] is NULL");
  if (!d->spectra_on_device) {
    const size_t n = (size_t)d->n_mu * (size_t)d->n_pix;
    for (int t = 0; t < 3; ++t) {
      if (!d->spectra[t]) continue;
      bool ok = (d->precision == SOAP_PREC_FP32) ? all_finite_host<float>(d->spectra[t], n)
                                                 : all_finite_host<double>(d->spectra[t], n);
      ARG_CHECK(ok, "spectra[%d] holds a non-finite value", t);
    }
  }
  if (d->contrast_mode == SOAP_CONTRAST_ARRAY) {
    ARG_CHECK(d->contrast[SOAP_QUIET] == nullptr, "contrast[SOAP_QUIET] must be NULL");
    for (int t = 1; t < 3; ++t) {
      ARG_CHECK(!d->spectra[t] || d->contrast[t], "contrast[%d] is required with spectra[%d]", t, t);
      if (d->contrast[t] && !d->spectra_on_device) {
        const size_t n = (size_t)d->n_mu * (size_t)d->n_pix;
        bool ok = (d->precision == SOAP_PREC_FP32) ? all_finite_host<float>(d->contrast[t], n)
                                                   : all_finite_host<double>(d->contrast[t], n);
        ARG_CHECK(ok, "contrast[%d] holds a non-finite value", t);
      }
    }
  } else {
    for (int t = 0; t < 3; ++t) ARG_CHECK(d->contrast[t] == nullptr, "contrast[%d] must be NULL outside ARRAY mode", t);
  }
  if (d->contrast_mode == SOAP_CONTRAST_PLANCK) {
    ARG_CHECK(is_finite(d->teff_k) && d->teff_k > 100.0, "teff_k must be > 100 K");
    ARG_CHECK(is_finite(d->dt_spot_k) && d->teff_k - d->dt_spot_k > 100.0, "spot temperature must be > 100 K");
    for (int b = 0; b < d->n_mu; ++b) {
      double mu = d->mu_bins[b];
      double dt = d->dt_fac_coef[0] + d->dt_fac_coef[1] * mu + d->dt_fac_coef[2] * mu * mu;
      ARG_CHECK(is_finite(dt) && d->teff_k + dt > 100.0, "facula temperature must be > 100 K");
    }
  }
  return SOAP_OK;
}

bool is_oom(hipError_t e) { return e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation; }

void free_ws(soap::Workspace& w) {
  if (w.ptr) (void)soap::dev_free(w.ptr);
  w.ptr = nullptr;
  w.bytes = 0;
}

void free_tables(soap_ctx::Prep& S) {
  free_ws(S.mem);
  std::fill(std::begin(S.at), std::end(S.at), 0);
  S.used = S.built = false;
}

// frees every table set but the last call's, which soap_profile_read reads;
// whether there was one to free
bool free_spare_tables(soap_ctx* c) {
  bool any = false;
  for (int i = 0; i < soap_ctx::NPREP; ++i) any = any || (i != c->last_prep && c->prep[i].mem.ptr);
  if (!any || hipStreamSynchronize(c->stream) != hipSuccess) return false;
  for (int i = 0; i < soap_ctx::NPREP; ++i)
    if (i != c->last_prep) free_tables(c->prep[i]);
  return true;
}

}  // namespace

soap::StreamShare::~StreamShare() {
  if (side) (void)hipStreamDestroy(side);
}

hipError_t soap::dev_malloc_for(soap_ctx* const* ctxs, int n, void** p, size_t bytes) {
  hipError_t e = soap::dev_malloc(p, bytes);
  if (!is_oom(e)) return e;
  (void)hipGetLastError();
  bool freed = false;
  for (int i = 0; i < n; ++i) freed = free_spare_tables(ctxs[i]) || freed;
  return freed ? soap::dev_malloc(p, bytes) : e;
}

namespace {

hipError_t grow(soap_ctx* c, soap::Workspace& w, size_t bytes) {
  if (w.bytes >= bytes) return hipSuccess;
  if (w.ptr) {
    hipError_t e = soap::dev_free(w.ptr);
    if (e != hipSuccess) return e;
    w.ptr = nullptr;
    w.bytes = 0;
  }
  size_t want = std::max<size_t>(bytes, 256);
  hipError_t e = soap::dev_malloc_for(&c, 1, &w.ptr, want);
  if (e == hipSuccess) w.bytes = want;
  return e;
}

// the record of a stream, made by its first context
std::shared_ptr<soap::StreamShare> share_of(int device, hipStream_t stream) {
  static std::mutex mu;
  static auto* all = new std::vector<std::weak_ptr<soap::StreamShare>>;
  std::lock_guard<std::mutex> lk(mu);
  std::shared_ptr<soap::StreamShare> found;
  size_t n = 0;
  for (auto& w : *all) {
    auto s = w.lock();
    if (!s) continue;
    if (s->device == device && s->stream == stream) found = s;
    (*all)[n++] = w;
  }
  all->resize(n);
  if (!found) {
    found = std::make_shared<soap::StreamShare>();
    found->device = device;
    found->stream = stream;
    all->push_back(found);
  }
  return found;
}

constexpr size_t PIN_BYTES = soap_ctx::PIN_WORD + soap_ctx::NSLOT * soap_ctx::PIN_SLOT + soap_ctx::PIN_STAGE;

// the context's block of pinned memory
hipError_t ensure_pin(soap_ctx* c) {
  if (c->pin) return hipSuccess;
  const hipError_t e =
      hipHostMalloc(reinterpret_cast<void**>(&c->pin), PIN_BYTES, hipHostMallocMapped | hipHostMallocCoherent);
  if (e != hipSuccess) return e;
  c->started = reinterpret_cast<unsigned*>(c->pin);
  *c->started = c->call_seq;
  for (int k = 0; k < soap_ctx::NSLOT; ++k) {
    c->slot[k] = c->pin + soap_ctx::PIN_WORD + k * soap_ctx::PIN_SLOT;
    c->slot_bytes[k] = soap_ctx::PIN_SLOT;
  }
  c->pinned = c->pin + soap_ctx::PIN_WORD + soap_ctx::NSLOT * soap_ctx::PIN_SLOT;
  c->pinned_bytes = soap_ctx::PIN_STAGE;
  return hipSuccess;
}

bool in_pin(const soap_ctx* c, const void* p) {
  const uintptr_t q = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(c->pin);
  return b && q >= b && q < b + PIN_BYTES;
}

// gives back an allocation of its own, not a part of the block
hipError_t free_pinned(const soap_ctx* c, void* p) { return !p || in_pin(c, p) ? hipSuccess : hipHostFree(p); }

void destroy_ctx(soap_ctx* c) {
  if (!c) return;
  if (c->hip_used) {
    // (table kernels of the side stream are waited for on this stream)
    (void)hipStreamSynchronize(c->stream);
  }
  if (c->share) {
    std::lock_guard<std::mutex> lk(c->share->mu);
    for (auto* call : {&c->share->last, &c->share->before})
      if (call->started == c->started) call->started = nullptr;
  }
  void* bufs[] = {c->d_mu, c->d_col_c, c->d_col_w, c->d_colW, c->d_Kq, c->d_Kq_fx, c->d_rows};
  for (void* p : bufs)
    if (p) (void)soap::dev_free(p);
  soap::Workspace* ws[] = {&c->ws_flux, &c->ws_ccf, &c->ws_ccfout, &c->ws_rv, &c->ws_mask, &c->ws_specin,
                           &c->ws_lsf, &c->ws_sg};
  for (auto* w : ws) free_ws(*w);
  for (auto& S : c->prep) {
    free_tables(S);
    if (S.done) (void)hipEventDestroy(S.done);
  }
  for (auto& p : c->pending) {
    (void)hipEventDestroy(p.a);
    (void)hipEventDestroy(p.b);
  }
  for (void* p : c->slot) (void)free_pinned(c, p);
  (void)free_pinned(c, c->pinned);
  if (c->pin) (void)hipHostFree(c->pin);
  if (c->pinned_done) (void)hipEventDestroy(c->pinned_done);
  delete c;
}

// copies n_rows rows of P samples (host or device) into padded device rows
// starting at dst; host rows go through pinned memory, so the copy is one
// DMA from memory that stays valid until it has completed
hipError_t upload_rows(soap_ctx* c, void* dst, const void* src, int n_rows, bool on_device) {
  const size_t row_bytes = (size_t)c->Pstride * c->esize;
  const size_t src_bytes = (size_t)c->P * c->esize * n_rows;
  void* pinned = nullptr;
  if (!on_device) {
    hipError_t e = hipHostMalloc(&pinned, src_bytes, hipHostMallocDefault);
    if (e != hipSuccess) return e;
    std::memcpy(pinned, src, src_bytes);
    src = pinned;
  }
  hipError_t ce = hipMemcpy2DAsync(dst, row_bytes, src, (size_t)c->P * c->esize, (size_t)c->P * c->esize, n_rows,
                                   on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, c->stream);
  if (pinned) {
    const hipError_t se = hipStreamSynchronize(c->stream);
    (void)hipHostFree(pinned);
    if (ce == hipSuccess) ce = se;
  }
  return ce;
}

// whether `bytes` at p lie in one allocation on the context's device: rows that
// a kernel may copy (others go through the runtime's copy, which checks them)
bool on_this_device(const soap_ctx* c, const void* p, size_t bytes) {
  hipPointerAttribute_t at;
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (hipPointerGetAttributes(&at, p) != hipSuccess || at.type != hipMemoryTypeDevice || at.device != c->device ||
      hipMemGetAddressRange(&base, &size, const_cast<void*>(p)) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const size_t off = static_cast<const unsigned char*>(p) - static_cast<const unsigned char*>(base);
  return off <= size && bytes <= size - off;
}

// sum over the visible cells of (2/N)^2 |I(mu)|: bounds every tap and
// column sum of the fixed-point accumulators.  One eighth of the disk stands
// for all of it (all 300 x 300 cells took 230 us of a context's opening, 30 so).
double disk_weight(int N, double u1, double u2) {
  const double area = (2.0 / N) * (2.0 / N);
  double tot = 0.0;
  for (int i = N / 2; i < N; ++i) {  // the middle column of an odd grid, and those past it
    const double x = soap::cell_coord(i, N);
    const double nx = 2 * i + 1 == N ? 1.0 : 2.0;
    for (int k = i; k < N; ++k) {
      const double y = soap::cell_coord(k, N);
      const double r2 = x * x + y * y;
      if (!(r2 < 1.0)) break;
      const double cells = nx * (2 * k + 1 == N ? 1.0 : 2.0) * (i == k ? 1.0 : 2.0);
      tot += cells * area * std::fabs(soap::limb_dark(std::sqrt(1.0 - r2), u1, u2));
    }
  }
  return tot;
}

using soap::FX_RANGE;

soap_status init_impl(const soap_star_desc* d, soap_ctx* c) {
  c->N = d->n_grid;
  c->B = d->n_mu;
  c->P = d->n_pix;
  c->vsini = d->vsini_kms;
  c->incl = d->incl_deg;
  c->u1 = d->ld_u1;
  c->u2 = d->ld_u2;
  c->ln0 = d->ln_lambda0;
  c->dln = d->dln_lambda;
  c->diff_rot = d->diff_rot;
  c->sin_i = std::sin(c->incl * soap::DEG);
  c->cos_i = std::cos(c->incl * soap::DEG);
  c->prec = d->precision;
  c->cmode = d->contrast_mode;
  c->teff = d->teff_k;
  c->dt_spot = d->dt_spot_k;
  for (int i = 0; i < 3; ++i) c->dt_fac[i] = d->dt_fac_coef[i];
  c->mu_bins.assign(d->mu_bins, d->mu_bins + d->n_mu);
  c->esize = (c->prec == SOAP_PREC_FP32) ? sizeof(float) : sizeof(double);

  // tap offset range: a bound on the column shifts |s| <= atanh(|vsini| x_max / c) / dln
  // with one offset of margin on each side, so rounding of the device's
  // own shift can never leave the table
  // (differential rotation scales a cell's velocity by 1 + diff_rot sin^2,
  // at most max(1, 1 + diff_rot) in size)
  const double xmax = 1.0 - 1.0 / c->N;
  const double vscale = std::max(1.0, 1.0 + c->diff_rot);
  const double smax = std::atanh(std::fabs(c->vsini) * xmax * vscale / soap::C_KMS) / c->dln;
  c->jmin = -(int)std::floor(smax) - 2;
  c->jmax = (int)std::ceil(smax) + 1;
  c->J = c->jmax - c->jmin + 1;
  std::string& err = c->err;
  ARG_CHECK(c->J <= 64, "rotation shift of %.1f pixels exceeds the supported 30 pixels", smax);
  c->disk_weight = disk_weight(c->N, c->u1, c->u2);
  if (!(c->disk_weight < FX_RANGE)) {
    setf(c->err, "limb darkening gives a disk weight of %.3f, beyond the fixed-point range of the tap sums (%.2f)",
         c->disk_weight, FX_RANGE);
    return SOAP_ERR_UNSUPPORTED;
  }
  ARG_CHECK(c->P >= 2 * (int64_t)c->J + 4, "n_pix must be at least 2 * (max shift + 3) + 4");
  if (c->diff_rot != 0.0 && 3 * c->B * c->J > soap::DR_TAB_MAX) {
    setf(c->err, "differential rotation supports n_mu x shift range up to %d, got %d x %d", soap::DR_TAB_MAX / 3,
         c->B, c->J);
    return SOAP_ERR_UNSUPPORTED;
  }
  const size_t gj_bytes = (size_t)3 * c->B * c->J * sizeof(double) + 192 * sizeof(int);
  if (gj_bytes > 60 * 1024) {
    setf(c->err, "n_mu x shift range too large for the per-phase tap table (%zu bytes)", gj_bytes);
    return SOAP_ERR_UNSUPPORTED;
  }

  c->hip_used = true;
  HIP_TRY(hipGetDevice(&c->device));
  c->share = share_of(c->device, c->stream);
  // the allocation-free entry point's scratch on this device (its status is
  // kept and reported by that entry point)
  (void)soap::scratch_setup(c->device);
  c->n_tiles = (int)((c->P + soap::APPLY_TILE_MAX - 1) / soap::APPLY_TILE_MAX);
  // padded rows: PAD_FRONT samples before pixel 0, and past the last tile
  // enough room for the widest window the apply kernel reads
  const int64_t tail = (int64_t)c->n_tiles * soap::APPLY_TILE_MAX + 2 * soap::MAX_J + 64;
  c->Pstride = ((soap::PAD_FRONT + tail + 63) / 64) * 64;
  const size_t row_bytes = (size_t)c->Pstride * c->esize;
  const bool on_dev = d->spectra_on_device != 0;
  // flags of non-finite values: [0] in rows, [1] in the quiet spectrum; read
  // back with a blocking copy once the stream is idle
  struct Flags {
    int* p = nullptr;
    ~Flags() {
      if (p) (void)soap::dev_free(p);
    }
  } flags;
  HIP_TRY(soap::dev_malloc((void**)&flags.p, 2 * sizeof(int)));
  HIP_TRY(hipMemsetAsync(flags.p, 0, 2 * sizeof(int), c->stream));
  // one allocation for all padded rows and the quiet spectrum (each large one
  // costs 12 us to make and 12 to give back)
  int n_rows = 0;
  for (int t = 0; t < 3; ++t) n_rows += d->spectra[t] ? c->B : 0;
  if (c->cmode == SOAP_CONTRAST_PLANCK) c->con_rows = c->B + 1;  // one spot row for every bin, one facula row per bin
  if (c->cmode == SOAP_CONTRAST_ARRAY) c->con_rows = 2 * c->B;   // the caller's rows: spot [B], then facula [B]
  const size_t q_bytes = sizeof(double) * c->n_tiles * soap::APPLY_TILE_MAX;
  HIP_TRY(soap::dev_malloc(&c->d_rows, row_bytes * (n_rows + c->con_rows) + q_bytes));
  unsigned char* rows = static_cast<unsigned char*>(c->d_rows);
  c->d_Q = reinterpret_cast<double*>(rows);
  rows += q_bytes;
  const void* fill_src[3];
  void* fill_base[3];
  int n_fill = 0;
  bool filled[3] = {false, false, false};
  for (int t = 0; t < 3; ++t) {
    if (!d->spectra[t]) continue;
    c->d_spec_base[t] = rows;
    rows += row_bytes * c->B;
    c->d_spec[t] = static_cast<unsigned char*>(c->d_spec_base[t]) + soap::PAD_FRONT * c->esize;
    filled[t] = on_dev && on_this_device(c, d->spectra[t], (size_t)c->P * c->esize * c->B);
    if (filled[t]) {
      fill_src[n_fill] = d->spectra[t];
      fill_base[n_fill++] = c->d_spec_base[t];
    } else {
      HIP_TRY(upload_rows(c, c->d_spec[t], d->spectra[t], c->B, on_dev));
      HIP_TRY(soap::launch_pad_rows(c, c->d_spec_base[t], c->B));
    }
    c->has_type[t] = true;
  }
  if (n_fill) HIP_TRY(soap::launch_fill_rows(c, fill_src, fill_base, n_fill, c->B, flags.p));
  HIP_TRY(soap::dev_malloc((void**)&c->d_mu, sizeof(double) * c->B));
  HIP_TRY(soap::dev_malloc((void**)&c->d_col_c, sizeof(int) * c->N));
  HIP_TRY(soap::dev_malloc((void**)&c->d_col_w, sizeof(double) * c->N));
  HIP_TRY(soap::dev_malloc((void**)&c->d_colW, sizeof(double) * c->N * c->B));
  HIP_TRY(soap::dev_malloc((void**)&c->d_Kq, sizeof(double) * c->B * c->J));
  if (c->diff_rot != 0.0) {
    HIP_TRY(soap::dev_malloc((void**)&c->d_Kq_fx, sizeof(unsigned long long) * c->B * c->J));
    HIP_TRY(hipMemsetAsync(c->d_Kq_fx, 0, sizeof(unsigned long long) * c->B * c->J, c->stream));
  }
  if (c->cmode == SOAP_CONTRAST_PLANCK) {
    c->d_con_base = rows;
    c->d_con_spot = static_cast<unsigned char*>(c->d_con_base) + soap::PAD_FRONT * c->esize;
    c->d_con_fac = static_cast<unsigned char*>(c->d_con_spot) + row_bytes;
    c->con_spot_stride = 0;
  } else if (c->cmode == SOAP_CONTRAST_ARRAY) {
    // a type without spectra keeps rows of zeros (never read)
    c->d_con_base = rows;
    c->d_con_spot = static_cast<unsigned char*>(c->d_con_base) + soap::PAD_FRONT * c->esize;
    c->d_con_fac = static_cast<unsigned char*>(c->d_con_spot) + row_bytes * c->B;
    c->con_spot_stride = c->Pstride;
    for (int t = 1; t < 3; ++t) {
      void* dst = t == SOAP_SPOT ? c->d_con_spot : c->d_con_fac;
      if (d->contrast[t]) HIP_TRY(upload_rows(c, dst, d->contrast[t], c->B, on_dev));
      else HIP_TRY(hipMemsetAsync(dst, 0, row_bytes * c->B - soap::PAD_FRONT * c->esize, c->stream));
    }
  }
  HIP_TRY(hipEventCreateWithFlags(&c->pinned_done, hipEventDisableTiming));
  HIP_TRY(soap::launch_geom(c));
  if (c->cmode == SOAP_CONTRAST_PLANCK) HIP_TRY(soap::launch_contrast(c));
  if (c->cmode == SOAP_CONTRAST_ARRAY) HIP_TRY(soap::launch_pad_rows(c, c->d_con_base, c->con_rows));
  HIP_TRY(soap::launch_quiet(c));
  // the device copies must be finite: device inputs were not checked on the
  // host, and a host input that was finite there yet is not here means the
  // upload went wrong
  int h_flag[2] = {0, 0};
  for (int t = 0; t < 3; ++t)
    if (c->d_spec_base[t] && !filled[t])
      HIP_TRY(soap::launch_check_finite(c, c->d_spec_base[t], c->B, false, flags.p));
  if (c->d_con_base) HIP_TRY(soap::launch_check_finite(c, c->d_con_base, c->con_rows, false, flags.p));
  HIP_TRY(soap::launch_check_finite(c, nullptr, 0, true, flags.p + 1));
  // host arrays (mu bins, spectra) may be released once the call returns
  HIP_TRY(hipStreamSynchronize(c->stream));
  HIP_TRY(hipMemcpy(h_flag, flags.p, sizeof h_flag, hipMemcpyDeviceToHost));
  if (h_flag[0] || h_flag[1]) {
    const char* what = h_flag[0] ? "the device copy of the local spectra or contrast arrays"
                                 : "the quiet integrated spectrum";
    if (on_dev) {
      setf(c->err, "%s holds a non-finite value (device inputs)", what);
      return SOAP_ERR_ARG;
    }
    setf(c->err, "%s holds a non-finite value although the host inputs are finite: the upload failed", what);
    return SOAP_ERR_HIP;
  }
  return SOAP_OK;
}

// copy a small host block to device memory through pinned staging; the host
// waits for the previous staging copy before overwriting the buffer
soap_status stage_to_device(soap_ctx* c, const void* src, size_t bytes, void* dst) {
  HIP_TRY(ensure_pin(c));
  HIP_TRY(hipEventSynchronize(c->pinned_done));
  if (c->pinned_bytes < bytes) {
    HIP_TRY(free_pinned(c, c->pinned));
    c->pinned = nullptr;
    c->pinned_bytes = 0;
    HIP_TRY(hipHostMalloc(&c->pinned, bytes, hipHostMallocDefault));
    c->pinned_bytes = bytes;
  }
  std::memcpy(c->pinned, src, bytes);
  HIP_TRY(hipMemcpyAsync(dst, c->pinned, bytes, hipMemcpyHostToDevice, c->stream));
  HIP_TRY(hipEventRecord(c->pinned_done, c->stream));
  return SOAP_OK;
}

const char* const kStageName[] = {"soap:weights", "soap:compact", "soap:apply", "soap:ccf", "soap:fit", "soap:lsf"};

// Brackets one stage with events on the context stream when profiling is on,
// and always with a roctx range named after the stage (the host-side span of
// its enqueue, seen by a marker trace).
struct StageTimer {
  soap_ctx* c;
  int stage;
  hipStream_t st;
  hipEvent_t a = nullptr;
  bool open = true;
  StageTimer(soap_ctx* c_, int s, hipStream_t st_ = nullptr) : c(c_), stage(s), st(st_ ? st_ : c_->stream) {
    roctxRangePushA(kStageName[s]);
    if (c->prof && hipEventCreate(&a) == hipSuccess) (void)hipEventRecord(a, st);
  }
  ~StageTimer() {
    if (open) roctxRangePop();
  }
  void done() {
    if (open) roctxRangePop();
    open = false;
    if (!a) return;
    hipEvent_t b = nullptr;
    if (hipEventCreate(&b) == hipSuccess && hipEventRecord(b, st) == hipSuccess) {
      c->pending.push_back({stage, a, b});
    } else {
      (void)hipEventDestroy(a);
      if (b) (void)hipEventDestroy(b);
    }
    a = nullptr;
  }
};

enum { ST_WEIGHTS = 0, ST_COMPACT = 1, ST_APPLY = 2, ST_CCF = 3, ST_GFIT = 4, ST_LSF = 5 };

}  // namespace

SOAP_API int32_t soap_abi_version(void) { return SOAP_ABI_VERSION; }

SOAP_API uint64_t soap_device_bytes(void) { return soap::dev_bytes_held(); }

SOAP_API const char* soap_status_string(soap_status s) {
  switch (s) {
    case SOAP_OK: return "SOAP_OK";
    case SOAP_ERR_ARG: return "SOAP_ERR_ARG";
    case SOAP_ERR_OOM: return "SOAP_ERR_OOM";
    case SOAP_ERR_HIP: return "SOAP_ERR_HIP";
    case SOAP_ERR_STATE: return "SOAP_ERR_STATE";
    case SOAP_ERR_NOCONV: return "SOAP_ERR_NOCONV";
    case SOAP_ERR_UNSUPPORTED: return "SOAP_ERR_UNSUPPORTED";
  }
  return "unknown soap_status";
}

SOAP_API const char* soap_last_error(const soap_ctx* c) {
  if (!c) return g_init_err.c_str();
  return c->err.c_str();
}

SOAP_API soap_status soap_grid_init(const soap_star_desc* desc, void* hip_stream, soap_ctx** out) {
  if (!out) {
    g_init_err = "out is NULL";
    return SOAP_ERR_ARG;
  }
  *out = nullptr;
  {
    std::string err;
    soap_status st = validate_desc(desc, err);
    if (st != SOAP_OK) {
      g_init_err = err;
      return st;
    }
  }
  soap_ctx* c = new (std::nothrow) soap_ctx();
  if (!c) {
    g_init_err = "host allocation of the context failed";
    return SOAP_ERR_OOM;
  }
  c->stream = static_cast<hipStream_t>(hip_stream);
  soap_status st = init_impl(desc, c);
  if (st != SOAP_OK) {
    g_init_err = c->err;
    destroy_ctx(c);
    return st;
  }
  *out = c;
  return SOAP_OK;
}

SOAP_API soap_status soap_quiet_spectrum(soap_ctx* c, void* out, int32_t out_on_device) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(out != nullptr, "out is NULL");
  const size_t bytes = (size_t)c->P * c->esize;
  void* dst = out;
  if (!out_on_device) {
    HIP_TRY(grow(c, c->ws_flux, bytes));
    dst = c->ws_flux.ptr;
  }
  if (c->prec == SOAP_PREC_FP64)
    HIP_TRY(hipMemcpyAsync(dst, c->d_Q, bytes, hipMemcpyDeviceToDevice, c->stream));
  else
    HIP_TRY(soap::launch_q_convert(c, dst));
  if (!out_on_device) {
    HIP_TRY(hipStreamSynchronize(c->stream));
    HIP_TRY(hipMemcpy(out, dst, bytes, hipMemcpyDeviceToHost));
  }
  return SOAP_OK;
}

namespace {

// Waits until the apply kernel of call `seq` has begun: whatever was enqueued
// before it is done.  The kernel writes its call's number to a host word; an
// event would put a marker between the kernels of the stream, 5 to 10 us each.
// An idle stream ends the wait too (a call whose apply was never launched).
hipError_t wait_started(soap_ctx* c, unsigned seq) {
  auto passed = [&] { return (int)(__atomic_load_n(c->started, __ATOMIC_ACQUIRE) - seq) >= 0; };
  for (;;) {
    const auto t0 = std::chrono::steady_clock::now();
    do {
      for (int i = 0; i < 32; ++i) {
        if (passed()) return hipSuccess;
        __builtin_ia32_pause();
      }
    } while (std::chrono::steady_clock::now() - t0 < std::chrono::milliseconds(2));
    const hipError_t e = hipStreamQuery(c->stream);
    if (e != hipErrorNotReady) return e;
  }
}

// Sizes of the parts of a call's tables
struct TableSizes {
  size_t bytes[soap::TAB_N];
};

bool tables_fit(const soap_ctx::Prep& S, const TableSizes& z) {
  for (int i = 0; i < soap::TAB_N; ++i)
    if (S.at[i + 1] - S.at[i] < z.bytes[i]) return false;
  return S.mem.ptr != nullptr;
}

// Makes the tables of an idle set hold z, and every part what it held unless
// `least`; a set that cannot keeps none of them.  One allocation: 15 us for a
// new context's 100-phase set, six of its parts' sizes up to 80 (a new chunk
// of the runtime's pool).
hipError_t grow_tables(soap_ctx::Prep& S, const TableSizes& z, bool least) {
  size_t at[soap::TAB_N + 1] = {0};
  for (int i = 0; i < soap::TAB_N; ++i) {
    const size_t part = std::max(z.bytes[i], least ? 0 : S.at[i + 1] - S.at[i]);
    at[i + 1] = at[i] + 256 * std::max<size_t>(1, (part + 255) / 256);
  }
  free_tables(S);
  const hipError_t e = soap::dev_malloc(&S.mem.ptr, at[soap::TAB_N]);
  if (e != hipSuccess) return e;
  S.mem.bytes = at[soap::TAB_N];
  std::copy(std::begin(at), std::end(at), std::begin(S.at));
  S.kfx_dirty = true;
  return hipSuccess;
}

// the side stream when the caller is ahead of the device, else null.  (One
// pending call is enough for a context's own series: 63.9 us a pass in FP64 with
// differential rotation against 66.5 with two; contexts in turn whose passes
// take the host longer than the device are a call ahead now and then, and gain
// nothing then: three small FP64 series 43.3 us a pass with one, 42.0 with two.)
hipError_t side_if_ahead(soap_ctx* c, hipStream_t* side) {
  soap::StreamShare& sh = *c->share;
  std::lock_guard<std::mutex> lk(sh.mu);
  auto begun = [](const soap::StreamShare::Call& k) {
    return (int)(__atomic_load_n(k.started, __ATOMIC_ACQUIRE) - k.seq) >= 0;
  };
  bool ahead;
  if (sh.last.started) {
    ahead = !begun(sh.last) && (sh.last.started == c->started || !sh.before.started || !begun(sh.before));
  } else {
    const hipError_t e = hipStreamQuery(c->stream);
    ahead = e == hipErrorNotReady;
    if (e != hipSuccess) (void)hipGetLastError();
  }
  if (!ahead) return hipSuccess;
  if (!sh.side) {
    const hipError_t e = hipStreamCreateWithFlags(&sh.side, hipStreamNonBlocking);
    if (e != hipSuccess) return e;
  }
  *side = sh.side;
  return hipSuccess;
}

// The table set of the next call, and the stream of its table kernels.  On the
// context stream any set will do: the stream keeps the order.  When the caller
// is ahead of the device (the apply of the context's last call has not begun,
// or, when another context came after it, those of the stream's last two calls
// have not; before the stream's first call, the stream is busy) the table
// kernels, short and far from filling the chip, run beside what is pending
// instead: a 100-phase series enqueued over and over takes 76 us a call so, 100
// on one stream.  They take the set that was used longest ago, whose apply is
// over once a later one has begun.
// Otherwise the second queue only adds its hand-over and host time: the same
// series with a wait after each call, 133 us with the second queue, 112 us on
// one stream.
// Memory for the side stream's sets is spare: a call that cannot have it runs
// on the context stream.
hipError_t choose_prep(soap_ctx* c, const TableSizes& z, int* sidx, hipStream_t* st) {
  hipError_t e;
  if ((e = ensure_pin(c)) != hipSuccess) return e;
  *st = c->stream;
  hipStream_t side = nullptr;
  if ((e = side_if_ahead(c, &side)) != hipSuccess) return e;
  if (side) {
    size_t all = 0;
    for (size_t b : z.bytes) all += b;
    const int n = all <= soap::PREP_SMALL ? soap_ctx::NPREP : 2;
    int k = 0;  // the first unused set, else the one used longest ago
    for (int i = 1; i < n && c->prep[k].used; ++i)
      if (!c->prep[i].used || (int)(c->prep[k].seq - c->prep[i].seq) > 0) k = i;
    soap_ctx::Prep& S = c->prep[k];
    if (S.used && (e = wait_started(c, S.seq + 1)) != hipSuccess) return e;
    if (!S.done && (e = hipEventCreateWithFlags(&S.done, hipEventDisableTiming)) != hipSuccess) return e;
    if (tables_fit(S, z) || (e = grow_tables(S, z, false)) == hipSuccess) {
      *sidx = k;
      *st = side;
      return hipSuccess;
    }
    if (!is_oom(e)) return e;
    (void)hipGetLastError();
  }
  for (int i = 0; i < soap_ctx::NPREP; ++i)
    if (tables_fit(c->prep[i], z)) {
      *sidx = i;
      return hipSuccess;
    }
  soap_ctx::Prep& S = c->prep[c->last_prep];
  *sidx = c->last_prep;
  // buffers in use are replaced only with the stream idle
  if (S.used && (e = hipStreamSynchronize(c->stream)) != hipSuccess) return e;
  if ((e = grow_tables(S, z, false)) == hipSuccess || !is_oom(e)) return e;
  (void)hipGetLastError();
  (void)free_spare_tables(c);
  return grow_tables(S, z, true);
}

// Shared body of soap_active_spectra and soap_active_spectra_jobs.  With
// pj_host == NULL every phase uses regions[0 .. n_regions); otherwise phase
// p uses pj_host[p] = (first region, count).  Arguments are validated.
soap_status active_impl(soap_ctx* c, const soap_region* regions, int32_t n_regions, int max_reg,
                        const int2* pj_host, const double* phases, int32_t n_phases, int32_t effect, void* flux,
                        int32_t flux_on_device) {
  // a captured call would replay from a parameter slot that later calls rewrite
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  HIP_TRY(hipStreamIsCapturing(c->stream, &cap));
  if (cap != hipStreamCaptureStatusNone) {
    setf(c->err, "the context's stream is being captured: synthesis calls cannot be replayed (use a batch)");
    return SOAP_ERR_HIP;
  }
  // per-call plan: paired tables when every active weight equals its
  // removal weight (chromatic contrast, the convective effect, or unit
  // scalar contrasts); otherwise split tables with explicit removal rows
  soap::Plan pl;
  pl.n_ph = n_phases;
  pl.effect = effect;
  bool unit = true;
  for (int r = 0; r < n_regions; ++r) unit = unit && regions[r].contrast == 1.0;
  pl.paired = (c->cmode != SOAP_CONTRAST_SCALAR || effect == SOAP_EFFECT_BCONV || unit) ? 1 : 0;
  if (!pl.paired) {
    // split tables scale the active rows by the region contrasts
    double cmax = 1.0;
    for (int r = 0; r < n_regions; ++r) cmax = std::max(cmax, regions[r].contrast);
    if (!(c->disk_weight * cmax < FX_RANGE)) {
      setf(c->err, "disk weight %.3f x contrast %.3f reaches the fixed-point range of the tap sums (%.2f)",
           c->disk_weight, cmax, FX_RANGE);
      return SOAP_ERR_UNSUPPORTED;
    }
  }
  pl.G = (pl.paired ? 2 : 3) * c->B;
  pl.n_slabs = (c->N + soap::SLAB_COLS - 1) / soap::SLAB_COLS;
  pl.pc = c->pc ? c->pc : soap::auto_pc(c->prec == SOAP_PREC_FP32, c->P, n_phases, pj_host != nullptr);
  pl.n_chunks = (n_phases + pl.pc - 1) / pl.pc;
  pl.vg_cap = pl.G * ((c->J + soap::APPLY_JW - 1) / soap::APPLY_JW);
  const size_t GJ = (size_t)pl.G * c->J;

  // parameter block (regions then phases) in the next pinned slot; the
  // weights kernel reads it in place
  const size_t n_reg_slots = std::max<size_t>(soap::MAX_REGIONS, (size_t)n_regions);
  const size_t reg_bytes = 256 * ((sizeof(soap::Region) * n_reg_slots + 255) / 256);
  const size_t ph_bytes = 256 * ((sizeof(double) * n_phases + 255) / 256);
  const size_t par_bytes = reg_bytes + ph_bytes + (pj_host ? sizeof(int2) * n_phases : 0);
  const size_t reg_dev = reg_bytes;
  const size_t pj_dev = 256 * ((sizeof(int2) * (size_t)n_phases + 255) / 256);
  const size_t cen_dev = 256 * ((sizeof(double4) * (size_t)n_phases * std::max(1, max_reg) + 255) / 256);
  const size_t par_dev = reg_dev + pj_dev + cen_dev + sizeof(int4) * (size_t)n_phases;
  const size_t kfx_bytes = sizeof(unsigned long long) * (size_t)n_phases * GJ;
  const size_t k_bytes = sizeof(double) * (size_t)n_phases * GJ;
  const size_t m_bytes = sizeof(unsigned long long) * (size_t)n_phases * pl.G;
  const size_t vg_bytes = (size_t)soap::win_bytes(pl.pc, (int)c->esize) * pl.n_chunks * pl.vg_cap;
  const size_t nvg_bytes = sizeof(int) * (size_t)pl.n_chunks;
  // the outputs' workspaces first: making room for them may take table sets
  const size_t out_bytes = (size_t)n_phases * c->P * c->esize;
  void* dflux = flux;
  if (!flux_on_device) {
    HIP_TRY(grow(c, c->ws_flux, out_bytes));
    dflux = c->ws_flux.ptr;
  }
  // with resolution lowering the synthesis goes to a workspace first
  void* dsyn = dflux;
  const bool lower = c->lsf_resolution > 0.0;
  if (lower && n_phases > soap::lsf_max_spectra(c->P)) {
    setf(c->err, "resolution lowering takes at most %lld spectra per call", (long long)soap::lsf_max_spectra(c->P));
    return SOAP_ERR_UNSUPPORTED;
  }
  if (lower) {
    if (c->ws_lsf.bytes < out_bytes) {
      HIP_TRY(hipStreamSynchronize(c->stream));
      HIP_TRY(grow(c, c->ws_lsf, out_bytes));
    }
    dsyn = c->ws_lsf.ptr;
  }
  const unsigned seq = c->call_seq + 1;
  int sidx = 0;
  hipStream_t st = nullptr;
  HIP_TRY(choose_prep(c, TableSizes{{par_dev, kfx_bytes, k_bytes, m_bytes, vg_bytes, nvg_bytes}}, &sidx, &st));
  soap_ctx::Prep& S = c->prep[sidx];
  const int k = (int)(seq % soap_ctx::NSLOT);
  HIP_TRY(wait_started(c, seq - soap_ctx::NSLOT));
  if (c->slot_bytes[k] < par_bytes) {
    HIP_TRY(free_pinned(c, c->slot[k]));
    c->slot[k] = nullptr;
    c->slot_bytes[k] = 0;
    HIP_TRY(hipHostMalloc(&c->slot[k], par_bytes, hipHostMallocMapped | hipHostMallocCoherent));
    c->slot_bytes[k] = par_bytes;
  }
  unsigned char* host = static_cast<unsigned char*>(c->slot[k]);
  soap::Region* hr = reinterpret_cast<soap::Region*>(host);
  for (int r = 0; r < n_regions; ++r) {
    hr[r].type = regions[r].type;
    hr[r].pad = 0;
    hr[r].lat_deg = regions[r].lat_deg;
    hr[r].lon_deg = regions[r].lon_deg;
    hr[r].radius = regions[r].radius;
    hr[r].contrast = regions[r].contrast;
  }
  std::memcpy(host + reg_bytes, phases, sizeof(double) * n_phases);
  if (pj_host) std::memcpy(host + reg_bytes + ph_bytes, pj_host, sizeof(int2) * n_phases);
  void* dev_view = nullptr;
  if (in_pin(c, c->slot[k])) {
    HIP_TRY(hipHostGetDevicePointer(&dev_view, c->pin, 0));
    dev_view = static_cast<unsigned char*>(dev_view) + (host - c->pin);
  } else {
    HIP_TRY(hipHostGetDevicePointer(&dev_view, c->slot[k], 0));
  }
  const unsigned char* dev_par = static_cast<const unsigned char*>(dev_view);
  const soap::Region* d_reg = reinterpret_cast<const soap::Region*>(dev_par);
  const double* d_ph = reinterpret_cast<const double*>(dev_par + reg_bytes);
  const int2* d_pj = pj_host ? reinterpret_cast<const int2*>(dev_par + reg_bytes + ph_bytes) : nullptr;

  soap::WeightsOut wo;
  unsigned char* par = S.part<unsigned char>(soap::TAB_PAR);
  wo.reg = reinterpret_cast<soap::Region*>(par);
  wo.pj = reinterpret_cast<int2*>(par + reg_dev);
  wo.cen = reinterpret_cast<double4*>(par + reg_dev + pj_dev);
  wo.box = reinterpret_cast<int4*>(par + reg_dev + pj_dev + cen_dev);
  wo.Kfx = S.part<unsigned long long>(soap::TAB_KFX);
  wo.K = S.part<double>(soap::TAB_K);
  wo.mask = S.part<unsigned long long>(soap::TAB_MASK);
  wo.wins = S.part<unsigned char>(soap::TAB_WIN);
  wo.nvg = S.part<int>(soap::TAB_NWIN);
  // a call that stops between its table kernels and its apply leaves nothing
  // running, so that its set, its slot and its number can be used again
  struct Idle {
    hipStream_t a, b;
    bool open = true;
    ~Idle() {
      if (!open) return;
      (void)hipStreamSynchronize(a);
      (void)hipStreamSynchronize(b);
    }
  } idle{st, c->stream};
  S.built = false;
  // every call that accumulates also clears the accumulators, so they are
  // zeroed only when new and after an interrupted call
  if (S.kfx_dirty)
    HIP_TRY(hipMemsetAsync(S.part(soap::TAB_KFX), 0, S.at[soap::TAB_KFX + 1] - S.at[soap::TAB_KFX], st));
  S.kfx_dirty = true;
  {
    StageTimer t(c, ST_WEIGHTS, st);
    HIP_TRY(soap::launch_weights(c, pl, d_reg, n_regions, std::max(1, max_reg), d_ph, d_pj, wo, st));
    t.done();
  }
  {
    StageTimer t(c, ST_COMPACT, st);
    HIP_TRY(soap::launch_finish(c, pl, wo, st));
    t.done();
  }
  S.kfx_dirty = false;
  if (st != c->stream) {
    HIP_TRY(hipEventRecord(S.done, st));
    HIP_TRY(hipStreamWaitEvent(c->stream, S.done, 0));
  }
  {
    StageTimer t(c, ST_APPLY);
    HIP_TRY(soap::launch_apply(c, pl, wo.wins, wo.nvg, dsyn, seq));
    t.done();
  }
  idle.open = false;
  c->call_seq = seq;
  {
    std::lock_guard<std::mutex> lk(c->share->mu);
    c->share->before = c->share->last;
    c->share->last = {c->started, seq};
  }
  S.seq = seq;
  S.used = S.built = true;
  c->last_prep = sidx;
  if (lower) {
    StageTimer t(c, ST_LSF);
    HIP_TRY(soap::launch_lsf(c, c->lsf, dsyn, dflux, n_phases, c->stream));
    t.done();
  }
  c->active_calls++;
  c->last_phases = n_phases;
  c->last_effect = effect;
  c->last_vg_cap = pl.vg_cap;
  c->last_pc = pl.pc;
  c->last_paired = pl.paired;
  c->last_mode = soap::apply_table_mode(c, pl);
  if (dflux != flux) {
    HIP_TRY(hipStreamSynchronize(c->stream));
    HIP_TRY(hipMemcpy(flux, dflux, out_bytes, hipMemcpyDeviceToHost));
  }
  return SOAP_OK;
}

soap_status check_region(soap_ctx* c, const soap_region& R, int r, int32_t effect) {
  std::string& err = c->err;
  ARG_CHECK(R.type == SOAP_SPOT || R.type == SOAP_FACULA, "regions[%d].type must be SOAP_SPOT or SOAP_FACULA", r);
  ARG_CHECK(is_finite(R.lat_deg) && R.lat_deg >= -90.0 && R.lat_deg <= 90.0, "regions[%d].lat_deg out of range", r);
  ARG_CHECK(is_finite(R.lon_deg), "regions[%d].lon_deg is not finite", r);
  ARG_CHECK(is_finite(R.radius) && R.radius > 0.0 && R.radius < 1.0, "regions[%d].radius must be in (0, 1)", r);
  ARG_CHECK(is_finite(R.contrast) && R.contrast > 0.0, "regions[%d].contrast must be > 0", r);
  if (effect != SOAP_EFFECT_FLUX)
    ARG_CHECK(c->has_type[R.type], "regions[%d] has type %d but the star has no spectra of that type", r, R.type);
  return SOAP_OK;
}

soap_status check_common(soap_ctx* c, const double* phases, int64_t n_phases, int32_t effect, void* flux) {
  std::string& err = c->err;
  ARG_CHECK(n_phases >= 1 && n_phases <= soap::MAX_PHASES, "n_phases must be in [1, %d]", soap::MAX_PHASES);
  ARG_CHECK(phases != nullptr, "phases is NULL");
  ARG_CHECK(effect == SOAP_EFFECT_TOT || effect == SOAP_EFFECT_FLUX || effect == SOAP_EFFECT_BCONV,
            "unknown effect %d", effect);
  ARG_CHECK(flux != nullptr, "flux is NULL");
  for (int64_t p = 0; p < n_phases; ++p) ARG_CHECK(is_finite(phases[p]), "phases[%lld] is not finite", (long long)p);
  return SOAP_OK;
}

}  // namespace

SOAP_API soap_status soap_active_spectra(soap_ctx* c, const soap_region* regions, int32_t n_regions,
                                         const double* phases, int32_t n_phases, int32_t effect, void* flux,
                                         int32_t flux_on_device) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(n_regions >= 0 && n_regions <= soap::MAX_REGIONS, "n_regions must be in [0, %d]", soap::MAX_REGIONS);
  ARG_CHECK(n_regions == 0 || regions != nullptr, "regions is NULL");
  soap_status st = check_common(c, phases, n_phases, effect, flux);
  if (st != SOAP_OK) return st;
  for (int r = 0; r < n_regions; ++r)
    if ((st = check_region(c, regions[r], r, effect)) != SOAP_OK) return st;
  return active_impl(c, regions, n_regions, n_regions, nullptr, phases, n_phases, effect, flux, flux_on_device);
}

SOAP_API soap_status soap_active_spectra_jobs(soap_ctx* c, const soap_region* regions,
                                              const int32_t* region_offsets, const double* phases,
                                              const int32_t* phase_offsets, int32_t n_jobs, int32_t effect,
                                              void* flux, int32_t flux_on_device) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(n_jobs >= 1 && n_jobs <= soap::MAX_PHASES, "n_jobs must be in [1, %d]", soap::MAX_PHASES);
  ARG_CHECK(region_offsets && phase_offsets, "offset arrays are NULL");
  ARG_CHECK(region_offsets[0] == 0 && phase_offsets[0] == 0, "offsets must start at 0");
  int max_reg = 0;
  for (int j = 0; j < n_jobs; ++j) {
    const int64_t nr = (int64_t)region_offsets[j + 1] - region_offsets[j];
    const int64_t np = (int64_t)phase_offsets[j + 1] - phase_offsets[j];
    ARG_CHECK(nr >= 0 && nr <= soap::MAX_REGIONS, "job %d has %lld regions (0 .. %d allowed)", j, (long long)nr,
              soap::MAX_REGIONS);
    ARG_CHECK(np >= 1, "job %d has no phases", j);
    max_reg = std::max(max_reg, (int)nr);
  }
  const int64_t n_regions = region_offsets[n_jobs], n_phases = phase_offsets[n_jobs];
  ARG_CHECK(n_regions <= (int64_t(1) << 22), "at most 2^22 regions in all");
  ARG_CHECK(n_regions == 0 || regions != nullptr, "regions is NULL");
  soap_status st = check_common(c, phases, n_phases, effect, flux);
  if (st != SOAP_OK) return st;
  for (int64_t r = 0; r < n_regions; ++r)
    if ((st = check_region(c, regions[r], (int)r, effect)) != SOAP_OK) return st;
  std::vector<int2> pj((size_t)n_phases);
  for (int j = 0; j < n_jobs; ++j)
    for (int p = phase_offsets[j]; p < phase_offsets[j + 1]; ++p)
      pj[p] = make_int2(region_offsets[j], region_offsets[j + 1] - region_offsets[j]);
  return active_impl(c, regions, (int32_t)n_regions, max_reg, pj.data(), phases, (int32_t)n_phases, effect, flux,
                     flux_on_device);
}

namespace {

bool law_ok(const soap_evolution& e) {
  if (!is_finite(e.t0_days) || !is_finite(e.size0_msh) || !(e.size0_msh > 0.0) || !(e.size0_msh < 1e6)) return false;
  switch (e.mode) {
    case SOAP_EVOLVE_NONE: return true;
    case SOAP_EVOLVE_LINEAR_GROWTH:
    case SOAP_EVOLVE_LINEAR_DECAY: return is_finite(e.rate_msh_day) && e.rate_msh_day >= 0.0;
    case SOAP_EVOLVE_ASYM_GAUSS:
      return is_finite(e.fwhm_days) && e.fwhm_days > 0.0 && is_finite(e.asym_per_day);
  }
  return false;
}

double law_size(const soap_evolution& e, double t) {
  const double d = t - e.t0_days;
  switch (e.mode) {
    case SOAP_EVOLVE_LINEAR_GROWTH: return d >= 0.0 ? e.size0_msh + e.rate_msh_day * d : e.size0_msh;
    case SOAP_EVOLVE_LINEAR_DECAY: return d >= 0.0 ? std::max(0.0, e.size0_msh - e.rate_msh_day * d) : e.size0_msh;
    case SOAP_EVOLVE_ASYM_GAUSS: {
      const double sigma = e.fwhm_days / (2.0 * std::sqrt(2.0 * std::log(2.0)));
      const double w = sigma * (1.0 + e.asym_per_day * d);
      return w > 0.0 ? e.size0_msh * std::exp(-(d * d) / (2.0 * w * w)) : 0.0;
    }
    default: return e.size0_msh;
  }
}

}  // namespace

SOAP_API double soap_evolution_size(const soap_evolution* law, double t_days) {
  if (!law || !law_ok(*law) || !is_finite(t_days)) return std::nan("");
  return law_size(*law, t_days);
}

SOAP_API soap_status soap_active_spectra_evolving(soap_ctx* c, const soap_region* regions,
                                                  const soap_evolution* laws, int32_t n_regions,
                                                  const double* phases, int32_t n_phases, double prot_days,
                                                  int32_t effect, void* flux, int32_t flux_on_device) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(n_regions >= 0 && n_regions <= soap::MAX_REGIONS, "n_regions must be in [0, %d]", soap::MAX_REGIONS);
  ARG_CHECK(n_regions == 0 || (regions != nullptr && laws != nullptr), "regions or laws is NULL");
  ARG_CHECK(is_finite(prot_days) && prot_days > 0.0, "prot_days must be > 0");
  soap_status st = check_common(c, phases, n_phases, effect, flux);
  if (st != SOAP_OK) return st;
  for (int r = 0; r < n_regions; ++r) {
    ARG_CHECK(law_ok(laws[r]), "laws[%d] is invalid (mode, size0 in (0, 1e6), rate >= 0, fwhm > 0)", r);
    soap_region probe = regions[r];
    probe.radius = 0.5;  // the radius comes from the law
    if ((st = check_region(c, probe, r, effect)) != SOAP_OK) return st;
  }
  // per-phase region lists: the regions of non-zero size with their radii
  std::vector<soap_region> flat;
  flat.reserve((size_t)n_regions * n_phases);
  std::vector<int2> pj((size_t)n_phases);
  int max_reg = 0;
  for (int p = 0; p < n_phases; ++p) {
    const double t = phases[p] * prot_days;
    const int first = (int)flat.size();
    for (int r = 0; r < n_regions; ++r) {
      const double a = law_size(laws[r], t);
      if (!(a > 0.0)) continue;
      const double f = std::min(1.0, a * 1e-6);
      soap_region g = regions[r];
      g.radius = std::sqrt(f * (2.0 - f));
      ARG_CHECK(g.radius < 1.0, "region %d reaches the whole hemisphere at phase %d", r, p);
      flat.push_back(g);
    }
    pj[p] = make_int2(first, (int)flat.size() - first);
    max_reg = std::max(max_reg, pj[p].y);
  }
  ARG_CHECK(flat.size() <= (size_t(1) << 22), "at most 2^22 regions over all phases");
  return active_impl(c, flat.empty() ? regions : flat.data(), (int32_t)flat.size(), max_reg, pj.data(), phases,
                     n_phases, effect, flux, flux_on_device);
}

SOAP_API soap_status soap_set_instrument(soap_ctx* c, double resolution) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(is_finite(resolution) && resolution >= 0.0, "resolution must be >= 0");
  if (resolution == 0.0) {
    c->lsf_resolution = 0.0;
    return SOAP_OK;
  }
  soap::LsfPlan pl;
  if (!soap::lsf_plan(resolution, c->dln, &pl)) {
    setf(c->err, "resolution %.6g gives a line-spread function wider than %d pixels each side", resolution,
         soap::LSF_KMAX);
    return SOAP_ERR_UNSUPPORTED;
  }
  c->lsf = pl;
  c->lsf_resolution = resolution;
  return SOAP_OK;
}

SOAP_API soap_status soap_instrument_lsf(soap_ctx* c, const void* in, void* out, int64_t n_spec, double resolution,
                                         int32_t on_device) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(in != nullptr && out != nullptr, "in or out is NULL");
  ARG_CHECK(n_spec >= 1 && n_spec <= soap::lsf_max_spectra(c->P), "n_spec must be in [1, %lld]",
            (long long)soap::lsf_max_spectra(c->P));
  ARG_CHECK(is_finite(resolution) && resolution > 0.0, "resolution must be > 0");
  const size_t bytes = (size_t)n_spec * c->P * c->esize;
  const uintptr_t a = reinterpret_cast<uintptr_t>(in), b = reinterpret_cast<uintptr_t>(out);
  ARG_CHECK(a + bytes <= b || b + bytes <= a, "in and out overlap");
  soap::LsfPlan pl;
  if (!soap::lsf_plan(resolution, c->dln, &pl)) {
    setf(c->err, "resolution %.6g gives a line-spread function wider than %d pixels each side", resolution,
         soap::LSF_KMAX);
    return SOAP_ERR_UNSUPPORTED;
  }
  const void* din = in;
  void* dout = out;
  if (!on_device) {
    HIP_TRY(grow(c, c->ws_specin, bytes));
    soap_status st = stage_to_device(c, in, bytes, c->ws_specin.ptr);
    if (st != SOAP_OK) return st;
    din = c->ws_specin.ptr;
    HIP_TRY(grow(c, c->ws_lsf, bytes));
    dout = c->ws_lsf.ptr;
  }
  {
    StageTimer t(c, ST_LSF);
    HIP_TRY(soap::launch_lsf(c, pl, din, dout, n_spec, c->stream));
    t.done();
  }
  if (!on_device) {
    HIP_TRY(hipStreamSynchronize(c->stream));
    HIP_TRY(hipMemcpy(out, dout, bytes, hipMemcpyDeviceToHost));
  }
  return SOAP_OK;
}

namespace soap {

// Validates a mask for the context and uploads its CCF tables unless they are
// the cached ones (soap_ccf_rv, batches with a CCF stage).
soap_status ctx_set_mask(soap_ctx* c, const soap_mask* mask) {
  std::string& err = c->err;
  ARG_CHECK(mask != nullptr, "mask is NULL");
  ARG_CHECK(mask->n_lines >= 1 && mask->n_lines <= (int64_t(1) << 20), "mask.n_lines must be in [1, 2^20]");
  ARG_CHECK(mask->ln_lambda != nullptr && mask->weight != nullptr, "mask arrays are NULL");
  ARG_CHECK(mask->n_v >= 4 && mask->n_v <= 768, "mask.n_v must be in [4, 768]");
  ARG_CHECK(is_finite(mask->v0_kms) && is_finite(mask->dv_kms) && mask->dv_kms > 0.0, "mask velocity grid invalid");
  ARG_CHECK(is_finite(mask->half_width_kms) && mask->half_width_kms > 0.0, "mask.half_width_kms must be > 0");
  const double vlo = mask->v0_kms - mask->half_width_kms;
  const double vhi = mask->v0_kms + mask->dv_kms * (mask->n_v - 1) + mask->half_width_kms;
  ARG_CHECK(std::fabs(vlo) < 0.1 * soap::C_KMS && std::fabs(vhi) < 0.1 * soap::C_KMS,
            "mask velocity grid beyond 0.1 c");
  const double hole_px = 2.0 * std::atanh(mask->half_width_kms / soap::C_KMS) / c->dln;
  if (hole_px > 8.0) {
    setf(c->err, "mask holes of %.2f pixels exceed the supported 8 pixels", hole_px);
    return SOAP_ERR_UNSUPPORTED;
  }
  const double reach_px = (std::atanh(vhi / soap::C_KMS) - std::atanh(vlo / soap::C_KMS)) / c->dln;
  if (reach_px + 4.0 > soap::ccf_span_pixels(c->prec == SOAP_PREC_FP32)) {
    setf(c->err, "the velocity grid spans %.0f pixels, beyond the supported %d", reach_px,
         soap::ccf_span_pixels(c->prec == SOAP_PREC_FP32) - 4);
    return SOAP_ERR_UNSUPPORTED;
  }
  const int nl = (int)mask->n_lines;
  for (int l = 0; l < nl; ++l)
    ARG_CHECK(is_finite(mask->ln_lambda[l]) && is_finite(mask->weight[l]), "mask line %d is not finite", l);

  // mask upload when it differs from the cached one
  const bool same = soap::mask_is_cached(c, mask);
  if (!same) {
    c->mask_valid = false;
    c->mask_h = mask->half_width_kms;
    c->mask_v0 = mask->v0_kms;
    c->mask_dv = mask->dv_kms;
    c->mask_nv = mask->n_v;
    std::vector<unsigned char> blob;
    std::string terr;
    if (!soap::ccf_build_tables(c, mask->ln_lambda, mask->weight, nl, blob, terr)) {
      c->err = terr;
      return SOAP_ERR_UNSUPPORTED;
    }
    HIP_TRY(grow(c, c->ws_mask, blob.size()));
    c->mask_blob_bytes = blob.size();
    soap_status st = stage_to_device(c, blob.data(), blob.size(), c->ws_mask.ptr);
    if (st != SOAP_OK) return st;
    c->mask_lnl.assign(mask->ln_lambda, mask->ln_lambda + nl);
    c->mask_w.assign(mask->weight, mask->weight + nl);
    c->mask_valid = true;
  }

  return SOAP_OK;
}

}  // namespace soap

SOAP_API soap_status soap_ccf_rv(soap_ctx* c, const void* flux, int32_t flux_on_device, int64_t n_spec,
                                 const soap_mask* mask, double* ccf_out, int32_t ccf_on_device, soap_rv* rv_out,
                                 int32_t rv_on_device) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(flux != nullptr, "flux is NULL");
  ARG_CHECK(n_spec >= 1 && n_spec <= (int64_t(1) << 24), "n_spec must be in [1, 2^24]");
  {
    const soap_status ms = soap::ctx_set_mask(c, mask);
    if (ms != SOAP_OK) return ms;
  }
  const int nl = c->ccf_nl;  // the lines in the tables

  const void* dflux = flux;
  const size_t in_bytes = (size_t)n_spec * c->P * c->esize;
  if (!flux_on_device) {
    HIP_TRY(grow(c, c->ws_specin, in_bytes));
    // through the context's pinned staging, not an asynchronous copy from
    // pageable memory
    soap_status st = stage_to_device(c, flux, in_bytes, c->ws_specin.ptr);
    if (st != SOAP_OK) return st;
    dflux = c->ws_specin.ptr;
  }
  const int nlb = soap::ccf_line_blocks(nl);
  const size_t ccf_elems = (size_t)n_spec * c->mask_nv;
  HIP_TRY(grow(c, c->ws_ccf, c->esize * ccf_elems * nlb));
  double* dccf = (ccf_out && ccf_on_device) ? ccf_out : nullptr;
  if (!dccf) {
    HIP_TRY(grow(c, c->ws_ccfout, sizeof(double) * ccf_elems));
    dccf = static_cast<double*>(c->ws_ccfout.ptr);
  }
  {
    StageTimer t(c, ST_CCF);
    HIP_TRY(soap::launch_ccf(c, dflux, n_spec, nl, c->ws_ccf.ptr));
    t.done();
  }
  c->ccf_calls++;
  soap_rv* drv = nullptr;
  if (rv_out) {
    drv = rv_on_device ? rv_out : nullptr;
    if (!drv) {
      HIP_TRY(grow(c, c->ws_rv, sizeof(soap_rv) * (size_t)n_spec));
      drv = static_cast<soap_rv*>(c->ws_rv.ptr);
    }
  }
  {
    StageTimer t(c, ST_GFIT);
    HIP_TRY(soap::launch_ccf_fit(c, nl, c->ws_ccf.ptr, n_spec, dccf, drv));
    t.done();
  }
  // host outputs: blocking copies once the stream is idle
  const bool rv_host = rv_out && !rv_on_device, ccf_host = ccf_out && !ccf_on_device;
  if (rv_host || ccf_host || !flux_on_device) HIP_TRY(hipStreamSynchronize(c->stream));
  if (rv_host) HIP_TRY(hipMemcpy(rv_out, drv, sizeof(soap_rv) * n_spec, hipMemcpyDeviceToHost));
  if (ccf_host) HIP_TRY(hipMemcpy(ccf_out, dccf, sizeof(double) * ccf_elems, hipMemcpyDeviceToHost));
  return SOAP_OK;
}

SOAP_API soap_status soap_ccf_linear_rv(soap_ctx* c, const float* coef, int64_t n, int32_t k, const double* base,
                                        const double* basis, double* ccf_out, soap_rv* rv_out) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(coef && base && basis, "coef, base and basis must be device arrays");
  ARG_CHECK(n >= 1 && n <= (int64_t(1) << 24), "n must be in [1, 2^24]");
  ARG_CHECK(k >= 1 && k <= 4096, "k must be in [1, 4096]");
  if (!c->mask_valid) {
    setf(c->err, "no mask yet: call soap_ccf_rv with the mask first");
    return SOAP_ERR_STATE;
  }
  double* lin = ccf_out;
  if (!lin) {
    HIP_TRY(grow(c, c->ws_ccfout, sizeof(double) * (size_t)n * c->mask_nv));
    lin = static_cast<double*>(c->ws_ccfout.ptr);
  }
  // the fit reads each row into registers before writing it back, so the
  // linear CCF and the output may share storage
  HIP_TRY(soap::launch_ccf_linear_fit(c, coef, n, k, base, basis, lin, lin, rv_out));
  return SOAP_OK;
}

SOAP_API soap_status soap_surrogate_rv(soap_ctx* c, const float* coef, const float* members, int64_t n,
                                       int32_t n_ens, int32_t k, const double* base, const int32_t* base_index,
                                       int32_t n_base, const double* basis, double calib, double threshold_kms,
                                       soap_rv* rv_out, double* rv_kms, double* err_kms, int32_t* fallback) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(coef && members && base && basis && rv_kms && fallback, "a required device array is NULL");
  ARG_CHECK(n >= 1 && n <= (int64_t(1) << 24), "n must be in [1, 2^24]");
  ARG_CHECK(k >= 1 && k <= 4096, "k must be in [1, 4096]");
  ARG_CHECK(n_ens >= 2 && n_ens <= 16, "n_ens must be in [2, 16]");
  ARG_CHECK(is_finite(calib) && calib >= 0.0 && !std::isnan(threshold_kms), "calib or threshold invalid");
  if (!c->mask_valid) {
    setf(c->err, "no mask yet: call soap_ccf_rv with the mask first");
    return SOAP_ERR_STATE;
  }
  ARG_CHECK(!base_index || n_base >= 1, "n_base must be >= 1 with base_index");
  const size_t wb = soap::sg_rv_work_bytes(c, n);
  if (c->ws_sg.bytes < wb) {
    // the workspace is replaced only with the stream idle
    HIP_TRY(hipStreamSynchronize(c->stream));
    HIP_TRY(grow(c, c->ws_sg, wb));
  }
  HIP_TRY(soap::launch_sg_rv(c, coef, members, n, n_ens, k, base, base_index, n_base, basis, calib, threshold_kms,
                             rv_out, rv_kms, err_kms, fallback, c->ws_sg.ptr));
  return SOAP_OK;
}

SOAP_API soap_status soap_profile_enable(soap_ctx* c, int32_t on) {
  if (!c) return SOAP_ERR_ARG;
  HIP_TRY(hipStreamSynchronize(c->stream));
  for (auto& p : c->pending) {
    (void)hipEventDestroy(p.a);
    (void)hipEventDestroy(p.b);
  }
  c->pending.clear();
  for (double& v : c->stage_ms) v = 0.0;
  c->active_calls = c->ccf_calls = 0;
  c->prof = on != 0;
  return SOAP_OK;
}

SOAP_API soap_status soap_profile_read(soap_ctx* c, soap_profile* out) {
  if (!c) return SOAP_ERR_ARG;
  std::string& err = c->err;
  ARG_CHECK(out != nullptr, "out is NULL");
  HIP_TRY(hipStreamSynchronize(c->stream));
  for (auto& p : c->pending) {
    float ms = 0.f;
    hipError_t e = hipEventElapsedTime(&ms, p.a, p.b);
    (void)hipEventDestroy(p.a);
    (void)hipEventDestroy(p.b);
    if (e == hipSuccess) c->stage_ms[p.stage] += ms;
  }
  c->pending.clear();
  out->weights_ms = c->stage_ms[ST_WEIGHTS];
  out->compact_ms = c->stage_ms[ST_COMPACT];
  out->apply_ms = c->stage_ms[ST_APPLY];
  out->ccf_ms = c->stage_ms[ST_CCF];
  out->gfit_ms = c->stage_ms[ST_GFIT];
  out->lsf_ms = c->stage_ms[ST_LSF];
  out->active_calls = c->active_calls;
  out->ccf_calls = c->ccf_calls;
  out->src_arrays = out->con_arrays = 0;
  out->taps_nonzero = out->taps_offsets = out->fma_issued = 0;
  out->last_phases = c->last_phases;
  if (c->last_phases > 0 && c->prep[c->last_prep].built) {
    // distinct inputs the last apply walked, from its virtual-group lists
    const int n_chunks = (c->last_phases + c->last_pc - 1) / c->last_pc;
    const size_t wb = (size_t)soap::win_bytes(c->last_pc, (int)c->esize);
    std::vector<int> nvg(n_chunks);
    std::vector<unsigned char> vg((size_t)n_chunks * c->last_vg_cap * wb);
    const soap_ctx::Prep& S = c->prep[c->last_prep];
    HIP_TRY(hipMemcpy(nvg.data(), S.part(soap::TAB_NWIN), sizeof(int) * n_chunks, hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(vg.data(), S.part(soap::TAB_WIN), vg.size(), hipMemcpyDeviceToHost));
    std::vector<char> src(3 * c->B, 0), con(3 * c->B, 0);
    const bool per_pixel = c->cmode != SOAP_CONTRAST_SCALAR;
    const bool spot_rows = c->con_spot_stride != 0;  // one spot contrast row per bin
    for (int ch = 0; ch < n_chunks; ++ch)
      for (int v = 0; v < nvg[ch]; ++v) {
        soap::WinHead h;
        const unsigned char* rec = vg.data() + ((size_t)ch * c->last_vg_cap + v) * wb;
        std::memcpy(&h, rec, sizeof(h));
        {
          out->fma_issued += soap::window_fmas(h.gmask, c->last_pc, (int)c->esize, c->last_mode);
          for (int q = 0; q < soap::APPLY_JW; ++q) {
            bool any = false;
            for (int pp = 0; pp < c->last_pc; ++pp) {
              double tap;
              if (c->prec == SOAP_PREC_FP32) {
                float f;
                std::memcpy(&f, rec + soap::WIN_HEAD + sizeof(float) * soap::win_tap(q, pp, c->last_pc, 4), sizeof f);
                tap = f;
              } else {
                std::memcpy(&tap, rec + soap::WIN_HEAD + sizeof(double) * soap::win_tap(q, pp, c->last_pc, 8), sizeof tap);
              }
              if (tap != 0.0) {
                ++out->taps_nonzero;
                any = true;
              }
            }
            if (any) ++out->taps_offsets;
          }
        }
        const int t = h.t, b = h.b;
        if (t == 0) {
          src[b] = 1;
          continue;
        }
        if (c->last_paired) src[b] = 1;  // the implied quiet removal
        if (c->last_effect == SOAP_EFFECT_FLUX) src[b] = 1;
        else src[t * c->B + b] = 1;
        // spot contrast is one array for every bin, facula one per bin
        if (per_pixel && c->last_effect != SOAP_EFFECT_BCONV)
          con[(t == SOAP_SPOT && !spot_rows) ? SOAP_SPOT * c->B : t * c->B + b] = 1;
      }
    for (char x : src) out->src_arrays += x;
    for (char x : con) out->con_arrays += x;
  }
  return SOAP_OK;
}

SOAP_API soap_status soap_sync(soap_ctx* c) {
  if (!c) return SOAP_ERR_ARG;
  HIP_TRY(hipStreamSynchronize(c->stream));
  return SOAP_OK;
}

SOAP_API void soap_destroy(soap_ctx* c) { destroy_ctx(c); }
