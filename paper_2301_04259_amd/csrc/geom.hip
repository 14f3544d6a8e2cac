// Per-star kernels: disk-column Doppler shifts, chromatic contrast and the
// quiet integrated spectrum.
//
// Section 3.2 (Eqs. 5-11): on a log-uniform grid ln(lambda_m) = ln0 + m dln
// the relativistic factor of Eq. 6 is a translation by
// s = ln(1+f)/dln = atanh(beta)/dln pixels, the same for every pixel.  A disk
// column at x has beta = vsini x / c for all its cells (solid-body rotation),
// so the whole column shares one shift.  The bracketing index of Eqs. 9-10
// is n = m - ceil(s) and the interpolation factor of Eq. 11,
// (lambda_m - lambda'_n)/(lambda'_{n+1} - lambda'_n), evaluates exactly to
// w = expm1(u dln)/expm1(dln) with u = ceil(s) - s.  The shifted spectrum is
// S'_m = (1-w) S[m - c] + w S[m - c + 1] with the source index held inside
// [0, P-1] (end values held outside the shifted grid).
//
// Algorithm 1 (quiet disk): Q = sum over disk cells of A I(mu) S'_{q,bin}.
// Cells are summed per (column, mu bin) first ("column sums", FP32 + Kahan in
// the FP32 mode, FP64 otherwise, then one wave64 reduction in FP64), then the
// column sums are collapsed in FP64 onto integer offsets j:
//   K[b][j] = sum_{c_i = j} (1 - w_i) W[i][b] + sum_{c_i - 1 = j} w_i W[i][b]
// and Q[m] = sum_b sum_j K[b][j] S_{q,b}[clamp(m - j)], accumulated in FP64.
#include <type_traits>

#include "soap_internal.hpp"

namespace soap {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// column shifts, and the limb angles of the bins to device memory
struct MuBins {
  double v[MAX_MU];
};
__global__ void k_geom(int N, int B, MuBins mu, double vsini, double dln, double* __restrict__ mu_b,
                       int* __restrict__ col_c, double* __restrict__ col_w) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < B) mu_b[i] = mu.v[i];
  if (i >= N) return;
  double x = cell_coord(i, N);
  double beta = vsini * x / C_KMS;
  double s = atanh(beta) / dln;
  double c = ceil(s);
  double u = c - s;
  col_c[i] = (int)c;
  col_w[i] = expm1(u * dln) / expm1(dln);
}

// contrast arrays over whole padded rows: pad entries hold the end values
template <typename T>
__global__ void k_contrast(int64_t P, int64_t Pstride, int B, double ln0, double dln, double teff, double dts,
                           double f0, double f1, double f2, const double* __restrict__ mu_b,
                           T* __restrict__ con_spot, T* __restrict__ con_fac) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // index in the padded row
  if (i >= Pstride) return;
  int64_t m = i - PAD_FRONT;
  m = m < 0 ? 0 : (m >= P ? P - 1 : m);
  double lam = exp(ln0 + dln * (double)m) * 1e-10;
  double eref = expm1(C2_MK / (lam * teff));
  con_spot[i] = (T)(eref / expm1(C2_MK / (lam * (teff - dts))));
  for (int b = 0; b < B; ++b) {
    double mu = mu_b[b];
    double dt = f0 + f1 * mu + f2 * mu * mu;
    con_fac[(int64_t)b * Pstride + i] = (T)(eref / expm1(C2_MK / (lam * (teff + dt))));
  }
}

// Rows of P samples in device memory to padded rows (pads hold the row's first
// and last sample); flags a non-finite value.  One pass for the copy, the pads
// and the check: three types of 20 rows of 100000 floats took 24 us to copy,
// 18 to pad and 15 to check, 10 so.
struct FillSet {
  const void* src;
  void* base;  // padded rows
};
struct FillArgs {
  FillSet set[3];
};
template <typename T>
__global__ void __launch_bounds__(256) k_fill_rows(int64_t P, int64_t Pstride, FillArgs a, int* __restrict__ flag) {
  const T* src = static_cast<const T*>(a.set[blockIdx.z].src) + (int64_t)blockIdx.y * P;
  T* dst = static_cast<T*>(a.set[blockIdx.z].base) + (int64_t)blockIdx.y * Pstride;
  constexpr int U = 4;  // samples per thread, all loaded before the first is stored
  const int64_t i0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x;
  T v[U];
  bool bad = false;
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = src[min(max(i0 + 256 * u - PAD_FRONT, (int64_t)0), P - 1)];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t i = i0 + 256 * u;
    bad = bad || !isfinite((double)v[u]);
    if (i < Pstride) dst[i] = v[u];
  }
  if (bad) flag[0] = 1;
}

// fill the pads of every row with the row's first / last sample (thread t: pad
// sample t of PAD_FRONT + Pstride - P)
template <typename T>
__global__ void k_pad(int64_t P, int64_t Pstride, int rows, T* __restrict__ base) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = t < PAD_FRONT ? t : t + P;
  const int row = blockIdx.y;
  if (row >= rows || i >= Pstride) return;
  T* r = base + (int64_t)row * Pstride;
  r[i] = r[t < PAD_FRONT ? PAD_FRONT : PAD_FRONT + P - 1];
}

// flags a non-finite value in n samples (and optionally in Q)
template <typename T>
__global__ void k_check_finite(int64_t n, const T* __restrict__ base, int64_t nq, const double* __restrict__ Q,
                               int* __restrict__ flag) {
  bool bad = false;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    bad = bad || !isfinite((double)base[i]);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq; i += stride)
    bad = bad || !isfinite(Q[i]);
  if (bad) flag[0] = 1;
}

// W[i][b] = sum_{cells of column i in bin b} A I, one block per disk column.
// The cells' bins and weights are worked out once, in LDS; then a wave per bin
// sums them, each lane its cells in order (FP32 + Kahan or FP64), the lanes in
// FP64.  (One wave per column that worked them out again for every bin: 84 us
// at 300 columns and 20 bins, 5 so.)
constexpr int COLSUM_WAVES = 8;
template <bool KAHAN32>
__global__ void __launch_bounds__(64 * COLSUM_WAVES) k_quiet_colsum(int N, int B, double u1, double u2,
                                                                    const double* __restrict__ mu_b,
                                                                    double* __restrict__ colW) {
  using V = typename std::conditional<KAHAN32, float, double>::type;
  __shared__ V s_v[MAX_GRID];
  __shared__ signed char s_b[MAX_GRID];  // bin, or -1 off the disk
  __shared__ double s_mu[MAX_MU];
  const int i = blockIdx.x;
  const double x = cell_coord(i, N);
  const double area = (2.0 / N) * (2.0 / N);
  if ((int)threadIdx.x < B) s_mu[threadIdx.x] = mu_b[threadIdx.x];
  __syncthreads();
  for (int k = threadIdx.x; k < N; k += 64 * COLSUM_WAVES) {
    const double y = cell_coord(k, N);
    double r2;
    {
#pragma clang fp contract(off)
      r2 = x * x + y * y;
    }
    int b = -1;
    if (r2 < 1.0) {
      const double mu = sqrt(1.0 - r2);
      b = nearest_bin(mu, s_mu, B);
      const double ld = limb_dark(mu, u1, u2);
      s_v[k] = KAHAN32 ? (V)(area * ld) : (V)ld;
    }
    s_b[k] = (signed char)b;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  for (int b = threadIdx.x >> 6; b < B; b += COLSUM_WAVES) {
    double part;
    if constexpr (KAHAN32) {
      float s = 0.f, comp = 0.f;
      for (int k = lane; k < N; k += 64)
        if (s_b[k] == b) {
          const float yk = s_v[k] - comp;
          const float t = s + yk;
          comp = (t - s) - yk;
          s = t;
        }
      part = (double)s - (double)comp;
    } else {
      double s = 0.0;
      for (int k = lane; k < N; k += 64)
        if (s_b[k] == b) s += area * s_v[k];
      part = s;
    }
    const double tot = wave_sum(part);
    if (lane == 0) colW[(int64_t)i * B + b] = tot;
  }
}

// K[b][j] over columns in index order (FP64, deterministic), one block per bin:
// the columns pass through LDS, which also finds the first and last column of
// every offset (a serial walk over all columns from global memory: 67 us at
// 300 columns, 11 so)
constexpr int COLLAPSE_COLS = 1024;
__global__ void __launch_bounds__(256) k_quiet_collapse(int N, int B, int jmin, int J,
                                                        const int* __restrict__ col_c,
                                                        const double* __restrict__ col_w,
                                                        const double* __restrict__ colW, double* __restrict__ Kq) {
  __shared__ int s_c[COLLAPSE_COLS], s_lo[MAX_J], s_hi[MAX_J];
  __shared__ double s_w[COLLAPSE_COLS], s_W[COLLAPSE_COLS];
  const int b = blockIdx.x, t = threadIdx.x;
  double acc = 0.0;
  for (int i0 = 0; i0 < N; i0 += COLLAPSE_COLS) {
    const int n = min(COLLAPSE_COLS, N - i0);
    __syncthreads();
    if (t < J) {
      s_lo[t] = n;
      s_hi[t] = -1;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < COLLAPSE_COLS / 256; ++u) {
      const int i = t + 256 * u, ic = min(i, n - 1);
      const int c = col_c[i0 + ic];
      s_c[i] = c;
      s_w[i] = col_w[i0 + ic];
      s_W[i] = colW[(int64_t)(i0 + ic) * B + b];
      if (i < n)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int j = c - q - jmin;
          if (j >= 0 && j < J) {
            atomicMin(&s_lo[j], i);
            atomicMax(&s_hi[j], i);
          }
        }
    }
    __syncthreads();
    if (t < J) {
      const int j = jmin + t;
      for (int i = s_lo[t]; i <= s_hi[t]; ++i) {
        const int c = s_c[i];
        const double w = s_w[i], W = s_W[i];
        if (c == j) acc += (1.0 - w) * W;
        if (c - 1 == j) acc += w * W;
      }
    }
  }
  if (t < J) Kq[b * J + t] = acc;
}

// Differential rotation: quiet taps K[b][j] from per-cell shifts.  One wave
// per disk column; each visible cell splits A I(mu) onto its two offsets
// (Eq. 11) in an LDS table [B][J] of exact 64-bit fixed-point sums, which the
// wave adds to the global fixed-point table (order-free, so the totals repeat
// bit for bit).
__global__ void __launch_bounds__(64) k_quiet_dr(int N, int B, int J, int jmin, double u1, double u2,
                                                 double vsini, double diff_rot, double sin_i, double cos_i,
                                                 double dln, const double* __restrict__ mu_b,
                                                 unsigned long long* __restrict__ Kfx) {
  extern __shared__ unsigned long long s_q[];  // [B * J]
  const int i = blockIdx.x;
  const int lane = threadIdx.x;
  const int BJ = B * J;
  for (int e = lane; e < BJ; e += 64) s_q[e] = 0ull;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const double x = cell_coord(i, N);
  const double area = (2.0 / N) * (2.0 / N);
  for (int k = lane; k < N; k += 64) {
    const double y = cell_coord(k, N);
    double r2;
    {
#pragma clang fp contract(off)
      r2 = x * x + y * y;
    }
    if (!(r2 < 1.0)) continue;
    const double mu = sqrt(1.0 - r2);
    const int b = nearest_bin(mu, mu_b, B);
    int cc;
    double w;
    cell_shift(x, y, mu, vsini, diff_rot, sin_i, cos_i, dln, &cc, &w);
    const int ja = cc - jmin, jb = cc - 1 - jmin;
    if (jb < 0 || ja >= J) continue;  // unreachable: the offset range bounds every shift
    const double aw = area * limb_dark(mu, u1, u2);
    atomicAdd(&s_q[b * J + ja], (unsigned long long)__double2ll_rn((1.0 - w) * aw * FX_ONE));
    atomicAdd(&s_q[b * J + jb], (unsigned long long)__double2ll_rn(w * aw * FX_ONE));
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int e = lane; e < BJ; e += 64) {
    const unsigned long long v = s_q[e];
    if (v) atomicAdd(Kfx + e, v);
  }
}

__global__ void k_quiet_dr_convert(int n, const unsigned long long* __restrict__ Kfx, double* __restrict__ Kq) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) Kq[t] = (double)(long long)Kfx[t] * FX_INV;
}

// Q[m] = sum_b sum_j K[b][j] S_b[m - j] in order of b, then j.  A block first
// lists the runs of QR offsets that hold a bin's taps; then every thread adds
// run after run, the samples of the next two already on their way (the rows'
// pads stand for the ends).  A load per tap, each waited for, took 46 us at
// 100000 pixels, 20 bins; 21 so.
constexpr int QR = 8;
template <typename T>
__global__ void __launch_bounds__(256) k_quiet(int64_t P, int64_t Pstride, int64_t Qlen, int B, int jmin, int J,
                                               const double* __restrict__ Kq, const T* __restrict__ S,
                                               double* __restrict__ Q) {
  extern __shared__ double s_k[];  // [B][J] taps, QR zeros, then the runs
  __shared__ int s_n[MAX_MU + 1], s_lo[MAX_MU];
  int* s_run = reinterpret_cast<int*>(s_k + B * J + QR);  // first tap of each run: b J + j
  const int t = threadIdx.x;
  for (int e = t; e < B * J + QR; e += 256) s_k[e] = e < B * J ? Kq[e] : 0.0;
  __syncthreads();
  if (t < B) {
    int lo = J, hi = -1;
    for (int j = 0; j < J; ++j)
      if (s_k[t * J + j] != 0.0) {
        lo = min(lo, j);
        hi = j;
      }
    s_lo[t] = lo;
    s_n[t] = hi < lo ? 0 : (hi - lo) / QR + 1;
  }
  __syncthreads();
  if (t == 0) {
    int n = 0;
    for (int b = 0; b < B; ++b) {
      const int k = s_n[b];
      s_n[b] = n;
      n += k;
    }
    s_n[B] = n;
  }
  __syncthreads();
  if (t < B)
    for (int q = s_n[t]; q < s_n[t + 1]; ++q) s_run[q] = t * J + s_lo[t] + QR * (q - s_n[t]);
  __syncthreads();
  const int64_t m = (int64_t)blockIdx.x * 256 + t;
  const int n = s_n[B];
  const int64_t mc = min(m, P - 1);
  struct Set {
    T v[QR];
  };
  auto load = [&](Set& o, int q) {  // past the last run it is read again
    const int e = s_run[min(q, n - 1)], b = e / J, j = e - b * J;
    const T* row = S + (int64_t)b * Pstride + mc - (jmin + j);
#pragma unroll
    for (int u = 0; u < QR; ++u) o.v[u] = row[-u];  // offsets past the table read the pads or the row before
  };
  double acc = 0.0;
  constexpr int D = 3;
  if (n > 0) {
    Set o[D];
#pragma unroll
    for (int d = 0; d + 1 < D; ++d) load(o[d], d);
    for (int q0 = 0; q0 < n; q0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        load(o[(d + D - 1) % D], q0 + d + D - 1);
        if (q0 + d < n) {
          const int e = s_run[q0 + d], left = J - e % J;  // taps of the run's bin
#pragma unroll
          for (int u = 0; u < QR; ++u)
            if (u < left && s_k[e + u] != 0.0) acc += s_k[e + u] * (double)o[d].v[u];
        }
      }
    }
  }
  if (m < Qlen) Q[m] = m < P ? acc : 0.0;
}

template <typename T>
__global__ void k_q_convert(int64_t P, const double* __restrict__ Q, T* __restrict__ out) {
  int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m < P) out[m] = (T)Q[m];
}

hipError_t launch_geom(soap_ctx* c) {
  MuBins mu{};
  for (int b = 0; b < c->B; ++b) mu.v[b] = c->mu_bins[b];
  hipLaunchKernelGGL(k_geom, dim3((c->N + 255) / 256), dim3(256), 0, c->stream, c->N, c->B, mu, c->vsini, c->dln,
                     c->d_mu, c->d_col_c, c->d_col_w);
  return hipGetLastError();
}

hipError_t launch_contrast(soap_ctx* c) {
  dim3 grid((unsigned)((c->Pstride + 255) / 256));
  // the pointers address pixel 0; the kernel writes whole padded rows
  if (c->prec == SOAP_PREC_FP32)
    hipLaunchKernelGGL(k_contrast<float>, grid, dim3(256), 0, c->stream, c->P, c->Pstride, c->B, c->ln0, c->dln,
                       c->teff, c->dt_spot, c->dt_fac[0], c->dt_fac[1], c->dt_fac[2], c->d_mu,
                       (float*)c->d_con_spot - PAD_FRONT, (float*)c->d_con_fac - PAD_FRONT);
  else
    hipLaunchKernelGGL(k_contrast<double>, grid, dim3(256), 0, c->stream, c->P, c->Pstride, c->B, c->ln0, c->dln,
                       c->teff, c->dt_spot, c->dt_fac[0], c->dt_fac[1], c->dt_fac[2], c->d_mu,
                       (double*)c->d_con_spot - PAD_FRONT, (double*)c->d_con_fac - PAD_FRONT);
  return hipGetLastError();
}

hipError_t launch_pad_rows(soap_ctx* c, void* base, int rows) {
  if (!base || rows <= 0) return hipSuccess;
  dim3 grid((unsigned)((c->Pstride - c->P + 255) / 256), rows);
  if (c->prec == SOAP_PREC_FP32)
    hipLaunchKernelGGL(k_pad<float>, grid, dim3(256), 0, c->stream, c->P, c->Pstride, rows, (float*)base);
  else
    hipLaunchKernelGGL(k_pad<double>, grid, dim3(256), 0, c->stream, c->P, c->Pstride, rows, (double*)base);
  return hipGetLastError();
}

hipError_t launch_fill_rows(soap_ctx* c, const void* const* src, void* const* base, int n_sets, int rows,
                            int* d_flag) {
  FillArgs a{};
  for (int t = 0; t < n_sets; ++t) a.set[t] = FillSet{src[t], base[t]};
  const dim3 grid((unsigned)((c->Pstride + 1023) / 1024), rows, n_sets);
  if (c->prec == SOAP_PREC_FP32)
    hipLaunchKernelGGL(k_fill_rows<float>, grid, dim3(256), 0, c->stream, c->P, c->Pstride, a, d_flag);
  else
    hipLaunchKernelGGL(k_fill_rows<double>, grid, dim3(256), 0, c->stream, c->P, c->Pstride, a, d_flag);
  return hipGetLastError();
}

hipError_t launch_check_finite(soap_ctx* c, const void* base, int rows, bool with_q, int* d_flag) {
  const int64_t n = base ? (int64_t)rows * c->Pstride : 0;
  const int64_t nq = with_q ? (int64_t)c->n_tiles * APPLY_TILE_MAX : 0;
  if (n == 0 && nq == 0) return hipSuccess;
  const dim3 grid(1024), block(256);
  if (c->prec == SOAP_PREC_FP32)
    hipLaunchKernelGGL(k_check_finite<float>, grid, block, 0, c->stream, n, (const float*)base, nq, c->d_Q, d_flag);
  else
    hipLaunchKernelGGL(k_check_finite<double>, grid, block, 0, c->stream, n, (const double*)base, nq, c->d_Q,
                       d_flag);
  return hipGetLastError();
}

static hipError_t launch_quiet_sum(soap_ctx* c) {
  const int64_t qlen = (int64_t)c->n_tiles * APPLY_TILE_MAX;
  const dim3 grid((unsigned)((qlen + 255) / 256));
  const size_t lds = sizeof(double) * (c->B * c->J + QR) + sizeof(int) * c->B * ((c->J + QR - 1) / QR);
  if (c->prec == SOAP_PREC_FP32)
    hipLaunchKernelGGL(k_quiet<float>, grid, dim3(256), lds, c->stream, c->P, c->Pstride, qlen, c->B, c->jmin, c->J,
                       c->d_Kq, (const float*)c->d_spec[SOAP_QUIET], c->d_Q);
  else
    hipLaunchKernelGGL(k_quiet<double>, grid, dim3(256), lds, c->stream, c->P, c->Pstride, qlen, c->B, c->jmin, c->J,
                       c->d_Kq, (const double*)c->d_spec[SOAP_QUIET], c->d_Q);
  return hipGetLastError();
}

hipError_t launch_quiet(soap_ctx* c) {
  if (c->diff_rot != 0.0) {
    const int nt = c->B * c->J;
    hipLaunchKernelGGL(k_quiet_dr, dim3(c->N), dim3(64), (size_t)nt * sizeof(unsigned long long), c->stream, c->N,
                       c->B, c->J, c->jmin, c->u1, c->u2, c->vsini, c->diff_rot, c->sin_i, c->cos_i, c->dln, c->d_mu,
                       c->d_Kq_fx);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_quiet_dr_convert, dim3((nt + 255) / 256), dim3(256), 0, c->stream, nt, c->d_Kq_fx, c->d_Kq);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_quiet_sum(c);
  }
  if (c->prec == SOAP_PREC_FP32)
    hipLaunchKernelGGL(k_quiet_colsum<true>, dim3(c->N), dim3(64 * COLSUM_WAVES), 0, c->stream, c->N, c->B,
                       c->u1, c->u2, c->d_mu, c->d_colW);
  else
    hipLaunchKernelGGL(k_quiet_colsum<false>, dim3(c->N), dim3(64 * COLSUM_WAVES), 0, c->stream, c->N, c->B,
                       c->u1, c->u2, c->d_mu, c->d_colW);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_quiet_collapse, dim3(c->B), dim3(256), 0, c->stream, c->N, c->B, c->jmin, c->J, c->d_col_c,
                     c->d_col_w, c->d_colW, c->d_Kq);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_quiet_sum(c);
}

hipError_t launch_q_convert(soap_ctx* c, void* out) {
  dim3 grid((unsigned)((c->P + 255) / 256));
  hipLaunchKernelGGL(k_q_convert<float>, grid, dim3(256), 0, c->stream, c->P, c->d_Q, (float*)out);
  return hipGetLastError();
}

}  // namespace soap
