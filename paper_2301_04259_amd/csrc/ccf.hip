// CCF against a line mask and Gaussian fit of the CCF (section 4.1: RVs from
// cross-correlation with a line mask and the mean of a fitted Gaussian).
//
// CCF: pixel m is a constant-flux bin [m, m+1) in the pixel coordinate
// q = (ln(lambda) - ln0)/dln + 1/2.  Mask line l sits at u_l in that
// coordinate; at trial velocity v_k its hole spans [u_l + a_k^-, u_l + a_k^+]
// with a_k^+- = atanh((v_k +- h)/c)/dln (the ln of the Eq. 6 factor).
// CCF_k = sum_l w_l sum_m F_m * overlap(bin m, hole), existing pixels only.
// The line positions, the hole edges per velocity and the split of the mask
// into blocks of lines and batches of nearby lines are built on the host
// once per mask.  Layout: one block per (block of lines, block of SB
// spectra), one thread per velocity (two or three past 512); each thread keeps SB
// accumulators and reuses its hole geometry for every spectrum of the block.
// Partial sums per line block are added in a fixed order by the fit kernel,
// so results repeat bit for bit.
//
// Fit: one wave64 per CCF; damped Newton (Levenberg-Marquardt damping) in
// double on the unweighted least squares of c0 - a exp(-(v - mu)^2 /
// (2 sigma^2)); the gradient, J^T J and the second-derivative sums are wave
// reductions, the 4 x 4 damped system is solved by LDL^T in every lane.
// Start values: c0 = max, a = c0 - min, mu at the vertex of the parabola
// through the minimum and its neighbours, sigma from the half-depth width
// with the crossings interpolated between samples.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "soap_internal.hpp"
#include "wave.hpp"

namespace soap {

constexpr int CCF_LB = 32;        // mask lines per block (one partial CCF row each)
constexpr int CCF_SB = 8;         // spectra per block
constexpr int CCF_FEW = 2;        // and in calls of few blocks,
constexpr int CCF_AHEAD = 3;      // with this many batches of loads in flight
constexpr int CCF_FEW_WAVES = 640;  // few: blocks of CCF_SB with fewer waves than this in all
constexpr int CCF_THREADS = 512;  // most threads of a block: one per velocity, more velocities each past 512
constexpr int CCF_MIN_THREADS = 192;  // fewest: the block also stages the pixels
constexpr int CCF_NV_MAX = 768;   // velocities per grid
constexpr int CCF_STG_MAX = 512;  // widest staged span of a batch, in pixels
// a line's hole centre, in pixels, is kept within this margin of the grid:
// lines further out reach no pixel
constexpr double CCF_U_MARGIN = 4096.0;

int ccf_line_blocks(int n_lines) { return (n_lines + CCF_LB - 1) / CCF_LB; }
int ccf_span_pixels(bool) { return CCF_STG_MAX; }

namespace {

// Velocities of a thread past CCF_THREADS: two, and of float spectra three, whose
// weights in double cost as much as their products (768 velocities, FP32, 100
// spectra of 100003 pixels, 4000 lines and holes of 1.6 km/s: 163 us with two, 126
// with three, 154 with four; FP64, 700 spectra of 20000 pixels, 400 lines: 155, 177
// and 222).
template <typename T>
constexpr int CCF_MORE = sizeof(T) == 4 ? 3 : 2;
// most threads of a block of A velocities each
constexpr int ccf_max_threads(int a) { return a == 1 ? CCF_THREADS : 64 * ((CCF_NV_MAX + 64 * a - 1) / (64 * a)); }

// the spectra of a pixel, in pieces of at most 16 bytes
template <typename T, int SB>
struct Piece {
  static constexpr int N = 16 / (int)sizeof(T) < SB ? 16 / (int)sizeof(T) : SB;
  T x[N];
};

}  // namespace

// One block per (CCF_LB mask lines, CCF_SB spectra).  The block walks the
// batches of its lines (host-built: consecutive lines whose holes, at every
// trial velocity, stay inside a span of STG pixels).  A batch's span of the
// block's spectra is staged in LDS in planes of 16 bytes of spectra per pixel,
// so that one thread reads the SB values of a pixel with 16-byte loads and
// without bank conflicts (rows of all SB values had 2.4 conflict cycles per
// load: 76 us against 71 for 300 spectra of 150001 pixels, 3000 lines and 401
// velocities); two stage
// buffers alternate, the next PF batches' loads are in flight while one is
// used, and one barrier per batch separates them.  Pixels outside the
// spectrum are staged as zeros.  Each thread computes its holes' pixel
// overlaps once per line (in double: the hole edges come from differences of
// nearby pixel coordinates) and applies them to every staged spectrum with
// FMAs in the flux precision: a block's partial CCF sums at most 32 lines x
// a few pixels in FP32 for float spectra, and the partials of the line blocks
// are added in double by the fit kernel.
// Line block lb, spectrum block sb.
template <typename T, int A, int NPX, int STG, int SB, int PF>
__device__ __forceinline__ void ccf_block(int P, int64_t n_spec, const T* __restrict__ F,
                                          const double2* __restrict__ lines, const double2* __restrict__ edges,
                                          const int4* __restrict__ batches, const int* __restrict__ bfirst,
                                          int n_v, T* __restrict__ part, int lb, int sb) {
  constexpr int R = (STG + CCF_MIN_THREADS - 1) / CCF_MIN_THREADS;  // staged pixels per thread
  using Quad = Piece<T, SB>;
  constexpr int QN = Quad::N, NQ = SB / QN;
  static_assert(SB % QN == 0, "whole pieces");
  __shared__ __align__(16) Quad st[2][NQ][STG];
  __shared__ double2 s_line[CCF_LB];
  // the edges on their way to registers: past the first stage buffer, which
  // is filled meanwhile, or over both
  constexpr size_t ED = sizeof(double2) * (A == 1 ? CCF_THREADS : CCF_NV_MAX);
  constexpr bool OWN = sizeof(st) < ED, OVER = !OWN && sizeof(st[1]) < ED;
  __shared__ double2 s_own[OWN ? ED / sizeof(double2) : 1];
  double2* s_ed = OWN ? s_own : reinterpret_cast<double2*>(&st[OVER ? 0 : 1][0][0]);
  __shared__ int4 s_bat[PF == 1 ? 1 : CCF_LB];  // the block's batches, one line each or more: read ahead
  const int tid = threadIdx.x, nt = blockDim.x;
  const int64_t s0 = (int64_t)sb * SB;
  const int ns = (int)min<int64_t>(SB, n_spec - s0);
  const int b0 = bfirst[lb], b1 = bfirst[lb + 1];
  const int l0 = batches[b0].y;
  const int nl = batches[b1 - 1].z - l0;
  if (tid < nl) s_line[tid] = lines[l0 + tid];
  if (PF > 1 && tid < b1 - b0) s_bat[tid] = batches[b0 + tid];
  // lanes past the velocity grid repeat its last velocity (results dropped);
  // the edges go through LDS so that no global load is pending in the loop
#pragma unroll
  for (int a = 0; a < A; ++a) s_ed[tid + a * nt] = edges[min(tid + a * nt, n_v - 1)];
  __syncthreads();
  double alo[A], ahi[A];
  T acc[A][SB];
#pragma unroll
  for (int a = 0; a < A; ++a) {
    const double2 e = s_ed[tid + a * nt];
    alo[a] = e.x;
    ahi[a] = e.y;
#pragma unroll
    for (int s = 0; s < SB; ++s) acc[a][s] = T(0);
  }
  if constexpr (OVER) __syncthreads();
  T vals[PF][R][SB];
  // only the batch's read span (batches[bi].w <= STG pixels) is loaded and
  // staged: no hole of the batch reads past it
  const int nb = b1 - b0;
  auto bat = [&](int i) {  // batch i of the block (uniform)
    if constexpr (PF == 1) return batches[b0 + i];
    const int4 v = s_bat[i];
    return make_int4(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y),
                     __builtin_amdgcn_readfirstlane(v.z), __builtin_amdgcn_readfirstlane(v.w));
  };
  auto load = [&](int i, T (&v)[R][SB]) {
    if (i >= nb) return;
    const int4 B = bat(i);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (tid + r * nt < B.w) {
        const int m = min(max(B.x + tid + r * nt, 0), P - 1);
#pragma unroll
        for (int s = 0; s < SB; ++s) v[r][s] = F[(s0 + min(s, ns - 1)) * (int64_t)P + m];
      }
    }
  };
  auto put = [&](int i, const T (&v)[R][SB]) {
    if (i >= nb) return;
    const int4 B = bat(i);
    Quad(*sb)[STG] = st[i & 1];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int p = tid + r * nt;
      if (p < B.w) {
        const int m = B.x + p;
        const bool ok = m >= 0 && m < P;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          Quad x;
#pragma unroll
          for (int s = 0; s < QN; ++s) x.x[s] = ok ? v[r][q * QN + s] : T(0);
          sb[q][p] = x;
        }
      }
    }
  };
  load(0, vals[0]);
  put(0, vals[0]);
#pragma unroll
  for (int d = 0; d < PF; ++d) load(1 + d, vals[d]);
  __syncthreads();
  for (int n0 = 0; n0 < nb; n0 += PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d) {
      const int i = n0 + d;
      if (PF > 1 && i >= nb) break;
      const int4 B = bat(i);
      const Quad(*sb)[STG] = st[i & 1];
      for (int l = B.y; l < B.z; ++l) {
        const double2 mw = s_line[l - l0];
#pragma unroll
        for (int a = 0; a < A; ++a) {
          const double qlo = mw.x + alo[a];
          const double qhi = mw.x + ahi[a];
          const double fa = floor(qlo);
          const int i0 = (int)fa - B.x;
          double w[NPX];
          if constexpr (NPX == 2) {
            // a hole narrower than a pixel: the first pixel takes the part of
            // the hole below fa + 1, the second the rest
            const double e1 = fa + 1.0;
            w[0] = mw.y * (fmin(qhi, e1) - qlo);
            w[1] = mw.y * fmax(qhi - e1, 0.0);
          } else {
            // pixel px covers [fa + px, fa + px + 1); the first pixel's lower
            // edge is the hole's, pixels past the hole get weight zero
#pragma unroll
            for (int px = 0; px < NPX; ++px) {
              const double mlo = fa + (double)px;
              w[px] = mw.y * fmax(fmin(qhi, mlo + 1.0) - (px == 0 ? qlo : mlo), 0.0);
            }
          }
#pragma unroll
          for (int px = 0; px < NPX; ++px) {
            const T wp = (T)w[px];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              const Quad f = sb[q][i0 + px];
#pragma unroll
              for (int s = 0; s < QN; ++s) acc[a][q * QN + s] = fma(wp, f.x[s], acc[a][q * QN + s]);
            }
          }
        }
      }
      put(i + 1, vals[d]);
      load(i + 1 + PF, vals[d]);
      __syncthreads();
    }
  }
#pragma unroll
  for (int a = 0; a < A; ++a) {
    const int k = tid + a * nt;
    if (k >= n_v) break;
#pragma unroll
    for (int s = 0; s < SB; ++s)
      if (s < ns) part[((int64_t)lb * n_spec + s0 + s) * n_v + k] = acc[a][s];
  }
}

template <typename T, int A, int NPX, int STG, int SB, int PF>
__global__ void __launch_bounds__(ccf_max_threads(A)) k_ccf(int P, int64_t n_spec, const T* __restrict__ F,
                                                     const double2* __restrict__ lines,
                                                     const double2* __restrict__ edges,
                                                     const int4* __restrict__ batches,
                                                     const int* __restrict__ bfirst, int n_v,
                                                     T* __restrict__ part) {
  ccf_block<T, A, NPX, STG, SB, PF>(P, n_spec, F, lines, edges, batches, bfirst, n_v, part, blockIdx.x, blockIdx.y);
}

// Work-list form over many spectra sets with one mask layout: blk[b] =
// (set, line block, spectrum block).
template <typename T, int A, int NPX, int STG>
__global__ void __launch_bounds__(ccf_max_threads(A)) k_ccf_batch(const CcfBatchSet* __restrict__ sets,
                                                           const int4* __restrict__ blk, int n_v) {
  const int4 t = blk[blockIdx.x];
  const CcfBatchSet c = sets[t.x];
  const unsigned char* tb = c.tables;
  ccf_block<T, A, NPX, STG, CCF_SB, 1>(c.P, c.n_spec, static_cast<const T*>(c.flux), reinterpret_cast<const double2*>(tb),
                            reinterpret_cast<const double2*>(tb + c.off_edges),
                            reinterpret_cast<const int4*>(tb + c.off_batch),
                            reinterpret_cast<const int*>(tb + c.off_bfirst), n_v, static_cast<T*>(c.part), t.y, t.z);
}

// Host tables of one mask (section 4.1's CCF with the holes of Eq. 6),
// appended to blob with 16-byte-aligned sections: lines (u, w) double2[nl],
// hole edges (a^-, a^+) double2[n_v], batches int4 {first staged pixel,
// first line, end line, pixels read}, and per line block the index of its first batch
// (int[n_lb + 1]).  Batches hold consecutive lines whose reads, from the
// floor of the lowest hole edge to NPX pixels past the floor of the highest,
// fit a span of STG pixels.
bool ccf_build_tables(soap_ctx* c, const double* lnl, const double* wl, int nl, std::vector<unsigned char>& blob,
                      std::string& err) {
  const int nv = c->mask_nv;
  std::vector<double2> ln(nl), ed(nv);
  for (int l = 0; l < nl; ++l) {
    const double u = (lnl[l] - c->ln0) / c->dln + 0.5;
    ln[l] = make_double2(std::fmin(std::fmax(u, -CCF_U_MARGIN), (double)c->P + CCF_U_MARGIN), wl[l]);
  }
  double wmax = 0.0;
  for (int k = 0; k < nv; ++k) {
    const double vk = c->mask_v0 + c->mask_dv * k;
    ed[k] = make_double2(std::atanh((vk - c->mask_h) / C_KMS) / c->dln, std::atanh((vk + c->mask_h) / C_KMS) / c->dln);
    wmax = std::fmax(wmax, ed[k].y - ed[k].x);
  }
  const int npx = wmax < 1.0 ? 2 : (wmax < 2.0 ? 3 : (wmax < 4.0 ? 5 : 10));
  // the edges grow with k (atanh is increasing), so these bound every hole
  const double amin = ed[0].x, amax = ed[nv - 1].y;
  auto span_lo = [&](int l) { return (int)std::floor(ln[l].x + amin); };
  auto span_end = [&](int l) { return (int)std::floor(ln[l].x + amax) + npx; };
  // lines whose reads all fall outside the spectrum add exactly zero to
  // every velocity (their staged pixels are zeros): they are left out of the
  // tables (one is kept when none reaches the spectrum, so that there is a
  // line block)
  {
    int kept = 0;
    for (int l = 0; l < nl; ++l)
      if (span_end(l) > 0 && span_lo(l) < (int64_t)c->P) ln[kept++] = ln[l];
    if (kept == 0) kept = 1;
    nl = kept;
    ln.resize(nl);
  }
  c->ccf_nl = nl;
  int widest = 0;
  for (int l = 0; l < nl; ++l) widest = std::max(widest, span_end(l) - span_lo(l));
  if (widest > CCF_STG_MAX) {
    err = "the velocity grid and holes span " + std::to_string(widest) + " pixels, beyond the supported " +
          std::to_string(CCF_STG_MAX);
    return false;
  }
  const int stg = widest <= 256 ? 256 : CCF_STG_MAX;
  const int nlb = ccf_line_blocks(nl);
  std::vector<int4> bat;
  std::vector<int> bfirst(nlb + 1);
  for (int b = 0; b < nlb; ++b) {
    bfirst[b] = (int)bat.size();
    const int l0 = b * CCF_LB, l1 = std::min(nl, l0 + CCF_LB);
    int lo = span_lo(l0), hi = span_end(l0), beg = l0;
    for (int l = l0 + 1; l < l1; ++l) {
      const int nlo = std::min(lo, span_lo(l)), nhi = std::max(hi, span_end(l));
      if (nhi - nlo > stg) {
        bat.push_back(make_int4(lo, beg, l, hi - lo));
        lo = span_lo(l);
        hi = span_end(l);
        beg = l;
      } else {
        lo = nlo;
        hi = nhi;
      }
    }
    bat.push_back(make_int4(lo, beg, l1, hi - lo));
  }
  bfirst[nlb] = (int)bat.size();
  auto al16 = [](size_t v) { return (v + 15) & ~size_t(15); };
  const size_t o_ed = al16(sizeof(double2) * nl);
  const size_t o_bat = al16(o_ed + sizeof(double2) * nv);
  const size_t o_bf = al16(o_bat + sizeof(int4) * bat.size());
  blob.assign(al16(o_bf + sizeof(int) * bfirst.size()), 0);
  std::memcpy(blob.data(), ln.data(), sizeof(double2) * nl);
  std::memcpy(blob.data() + o_ed, ed.data(), sizeof(double2) * nv);
  std::memcpy(blob.data() + o_bat, bat.data(), sizeof(int4) * bat.size());
  std::memcpy(blob.data() + o_bf, bfirst.data(), sizeof(int) * bfirst.size());
  c->ccf_off_edges = o_ed;
  c->ccf_off_batch = o_bat;
  c->ccf_off_bfirst = o_bf;
  c->ccf_nbatch = (int)bat.size();
  c->ccf_npx = npx;
  c->ccf_stg = stg;
  c->mask_hole_px = wmax;
  return true;
}

namespace {

constexpr double FWHM_PER_SIGMA = 2.3548200450309493;  // 2 sqrt(2 ln 2)
constexpr int CCF_FIN_THREADS = 256;
constexpr int64_t CCF_FIT_WAVES_FROM = 512;  // spectra per call above which one wave fits each

// Sums of the fit at p = (c0, amp, mu, sigma), identical in every lane.  With
// q = (v - mu) / sigma, e = exp(-q^2 / 2) and r = c0 - amp e - y they are the
// sums over the samples of r^2, r, r e q^k (k = 0 .. 4), e q^k (k = 0 .. 2) and
// e^2 q^k (k = 0 .. 4): every entry of J^T r, J^T J and of the residual-weighted
// second derivatives is one or two of them, up to factors amp and sigma that
// gf_solve leaves out by scaling the centre and width (15 sums in one
// butterfly, where the 20 sums of the entries themselves took two).
enum { GF_RR, GF_R, GF_RE, GF_RE1, GF_RE2, GF_RE3, GF_RE4, GF_E, GF_E1, GF_E2, GF_EE, GF_EE1, GF_EE2, GF_EE3, GF_EE4,
       GF_N };  // GF_N: number of samples

template <int NPT>
__device__ __forceinline__ void gf_eval(const double (&y)[NPT], int n_v, double v0, double dv, const double p[4],
                                        double S[16]) {
  const int lane = threadIdx.x & 63;
  double v[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) v[q] = 0.0;
  const double is = 1.0 / p[3];
  // no branch per sample, so that the samples of a lane overlap: places past
  // the grid count as e = r = 0
#pragma unroll
  for (int t = 0; t < NPT; ++t) {
    const int i = lane + 64 * t;
    const bool in = i < n_v;
    const double q = (v0 + dv * i - p[2]) * is;
    const double q2 = q * q;
    const double ex = exp(-0.5 * q2);
    const double e = in ? ex : 0.0;
    const double r = in ? p[0] - p[1] * ex - y[t] : 0.0;
    const double e1 = e * q, e2 = e * q2, re2 = r * e2;
    v[GF_RR] = fma(r, r, v[GF_RR]);
    v[GF_R] += r;
    v[GF_RE] = fma(r, e, v[GF_RE]);
    v[GF_RE1] = fma(r, e1, v[GF_RE1]);
    v[GF_RE2] += re2;
    v[GF_RE3] = fma(re2, q, v[GF_RE3]);
    v[GF_RE4] = fma(re2, q2, v[GF_RE4]);
    v[GF_E] += e;
    v[GF_E1] += e1;
    v[GF_E2] += e2;
    v[GF_EE] = fma(e, e, v[GF_EE]);
    v[GF_EE1] = fma(e, e1, v[GF_EE1]);
    v[GF_EE2] = fma(e1, e1, v[GF_EE2]);
    v[GF_EE3] = fma(e1, e2, v[GF_EE3]);
    v[GF_EE4] = fma(e2, e2, v[GF_EE4]);
  }
  const double tv = butterfly16_rows(v, lane);
#pragma unroll
  for (int q = 0; q < 15; ++q) S[q] = read_lane(tv, q);
  S[GF_N] = (double)n_v;
}

// 1 / x to rounding error (two Newton steps on the hardware estimate) for the
// pivots of a small solve; not for x = 0, infinities or denormals
__device__ __forceinline__ double fast_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

// Solves (H + lam diag(J^T J)) x = b at p by L D L^T, H = J^T J (+ the
// second-derivative sums when newton is set), for the parameters (c0, amp, mu,
// sigma).  The system is formed for s = amp / sigma times the last two, whose
// model derivatives are then -e q and -e q^2; b and x are in those scaled
// parameters too (b = D^-1 b_p, x = D x_p with D = diag(1, 1, s, s)).  False
// when the matrix is not positive definite.
__device__ __forceinline__ bool gf_solve_scaled(const double S[16], const double p[4], bool newton, double lam,
                                                const double b[4], double x[4]) {
  double a01 = -S[GF_E], a02 = -S[GF_E1], a03 = -S[GF_E2], a12 = S[GF_EE1], a13 = S[GF_EE2], a23 = S[GF_EE3];
  double a11 = S[GF_EE], a22 = S[GF_EE2], a33 = S[GF_EE4];
  const double a00 = fma(lam, S[GF_N], S[GF_N]);
  const double d11 = lam * a11, d22 = lam * a22, d33 = lam * a33;
  if (newton) {
    const double ia = 1.0 / p[1];
    a12 = fma(-ia, S[GF_RE1], a12);
    a13 = fma(-ia, S[GF_RE2], a13);
    a22 = fma(-ia, S[GF_RE2] - S[GF_RE], a22);
    a23 = fma(-ia, S[GF_RE3] - 2.0 * S[GF_RE1], a23);
    a33 = fma(-ia, S[GF_RE4] - 3.0 * S[GF_RE2], a33);
  }
  a11 += d11;
  a22 += d22;
  a33 += d33;
  // pivots d0 .. d3, unit lower factor l
  const double r0 = fast_rcp(a00);
  const double l10 = a01 * r0, l20 = a02 * r0, l30 = a03 * r0;
  const double d1 = fma(-l10, a01, a11);
  const double m21 = fma(-l10, a02, a12), m31 = fma(-l10, a03, a13);
  const double r1 = fast_rcp(d1);
  const double l21 = m21 * r1, l31 = m31 * r1;
  const double d2 = fma(-l21, m21, fma(-l20, a02, a22));
  const double m32 = fma(-l21, m31, fma(-l20, a03, a23));
  const double r2 = fast_rcp(d2);
  const double l32 = m32 * r2;
  const double d3 = fma(-l32, m32, fma(-l31, m31, fma(-l30, a03, a33)));
  // every pivot positive and normal (false for NaN and infinities too)
  const double tiny = 2.2250738585072014e-308, huge = 1.7976931348623157e308;
  if (!(a00 >= tiny && d1 >= tiny && d2 >= tiny && d3 >= tiny && a00 <= huge && d1 <= huge && d2 <= huge &&
        d3 <= huge))
    return false;
  const double z0 = b[0];
  const double z1 = fma(-l10, z0, b[1]);
  const double z2 = fma(-l21, z1, fma(-l20, z0, b[2]));
  const double z3 = fma(-l32, z2, fma(-l31, z1, fma(-l30, z0, b[3])));
  x[3] = z3 * fast_rcp(d3);
  x[2] = fma(-l32, x[3], z2 * r2);
  x[1] = fma(-l31, x[3], fma(-l21, x[2], z1 * r1));
  x[0] = fma(-l30, x[3], fma(-l20, x[2], fma(-l10, x[1], z0 * r0)));
  return true;
}

// The step x = -(H + lam diag(J^T J))^-1 J^T r in the parameters themselves
__device__ __forceinline__ bool gf_solve(const double S[16], const double p[4], bool newton, double lam, double x[4]) {
  const double b[4] = {-S[GF_R], S[GF_RE], S[GF_RE1], S[GF_RE2]};
  if (!gf_solve_scaled(S, p, newton, lam, b, x)) return false;
  const double f = p[3] / p[1];
  x[2] *= f;
  x[3] *= f;
  return true;
}

// Gaussian fit of one CCF held by the calling wave (y[t] = CCF point
// lane + 64 t); returns the result record and leaves the parameters in p and
// the last sums (gf_eval) in S.  Damped Newton / Levenberg-Marquardt as
// described at k_ccf_fit.
template <int NPT>
__device__ soap_rv fit_wave(const double (&y)[NPT], int n_v, double v0, double dv, double p[4],
                            double S[16]) {
  const int lane = threadIdx.x & 63;
  // start values: max, first argmin, half-depth width.  The extremes are wave
  // reductions; sample positions come from ballots, samples by readlane.
  double ymax = -1e308, ymin = 1e308;
#pragma unroll
  for (int t = 0; t < NPT; ++t) {
    if (lane + 64 * t < n_v) {
      ymax = fmax(ymax, y[t]);
      ymin = fmin(ymin, y[t]);
    }
  }
  ymax = read_lane(wave_max_f64(ymax), 0);
  ymin = read_lane(-wave_max_f64(-ymin), 0);
  const double c0 = ymax;
  const double a0 = c0 - ymin;
  const double half = c0 - 0.5 * a0;
  int kmin = n_v, first = n_v, last = -1;
#pragma unroll
  for (int t = 0; t < NPT; ++t) {
    const bool in = lane + 64 * t < n_v;
    const unsigned long long at_min = __ballot(in && y[t] == ymin), low = __ballot(in && y[t] <= half);
    if (at_min && kmin == n_v) kmin = 64 * t + (int)__builtin_ctzll(at_min);
    if (low) {
      if (first == n_v) first = 64 * t + (int)__builtin_ctzll(low);
      last = 64 * t + 63 - (int)__builtin_clzll(low);
    }
  }
  // sample i of the CCF in every lane (i uniform, 0 <= i < n_v)
  auto at = [&](int i) {
    double v = read_lane(y[0], i & 63);
#pragma unroll
    for (int t = 1; t < NPT; ++t) {
      const double w = read_lane(y[t], i & 63);
      v = (i >> 6) == t ? w : v;
    }
    return v;
  };
  // half-depth crossings interpolated between samples, and the minimum's
  // position from the parabola through it and its neighbours
  double xl = first, xr = last;
  if (first > 0 && first < n_v) {
    const double ya = at(first - 1), yb = at(first);
    if (ya > yb) xl = (first - 1) + (ya - half) / (ya - yb);
  }
  if (last >= 0 && last + 1 < n_v) {
    const double ya = at(last), yb = at(last + 1);
    if (yb > ya) xr = last + (half - ya) / (yb - ya);
  }
  double kc = kmin;
  if (kmin > 0 && kmin + 1 < n_v) {
    const double ym = at(kmin - 1), y0 = at(kmin), yp = at(kmin + 1);
    const double den = ym - 2.0 * y0 + yp;
    if (den > 0.0) kc += fmin(fmax(0.5 * (ym - yp) / den, -0.5), 0.5);
  }
  const double width = (xr > xl) ? dv * (xr - xl) : dv;
  p[0] = c0;
  p[1] = a0;
  p[2] = v0 + dv * kc;
  p[3] = fmax(width, dv) / FWHM_PER_SIGMA;

  // every sample finite: max and min skip NaN, so test each one
  bool bad_sample = false;
#pragma unroll
  for (int t = 0; t < NPT; ++t) {
    const int i = lane + 64 * t;
    if (i < n_v && !isfinite(y[t])) bad_sample = true;
  }
  const bool any_bad = __ballot(bad_sample) != 0ull;

  soap_rv res;
  res.status = 0;
  if (any_bad || !(a0 > 1e-12 * fabs(c0)) || !isfinite(c0) || !isfinite(ymin)) {
    res.status = 2;
    res.iters = 0;
  } else {
    gf_eval(y, n_v, v0, dv, p, S);
    double lam = 1e-3;
    int it = 0, accepted = 0;
    res.status = 1;
    for (; it < 100; ++it) {
      double x[4];
      double Sn[16];
      bool ok = gf_solve(S, p, true, lam, x) || gf_solve(S, p, false, lam, x);
      bool tiny = false;
      if (ok) {
        const double sig = fabs(p[3]);
        tiny = fabs(x[0]) <= 1e-10 * fabs(p[0]) && fabs(x[1]) <= 1e-10 * fabs(p[1]) &&
               fabs(x[2]) <= 1e-10 * sig && fabs(x[3]) <= 1e-10 * sig;
        if (tiny) {
          // a step of rounding size: take it without another pass (chi2
          // stays that of the last evaluated point)
          for (int q = 0; q < 4; ++q) p[q] += x[q];
          res.status = 0;
          ++it;
          break;
        }
        double pn[4];
        for (int q = 0; q < 4; ++q) pn[q] = p[q] + x[q];
        gf_eval(y, n_v, v0, dv, pn, Sn);
        if (Sn[0] <= S[0]) {
          const double dchi = S[0] - Sn[0];
          for (int q = 0; q < 4; ++q) p[q] = pn[q];
          for (int q = 0; q < 16; ++q) S[q] = Sn[q];
          ++accepted;
          lam = (lam > 1e-9) ? lam * 0.1 : 0.0;
          const double sgn = fabs(p[3]);
          const bool floor_hit =
              dchi <= 1e-15 * S[0] && fabs(x[2]) <= 1e-9 * sgn && fabs(x[3]) <= 1e-9 * sgn;
          if (tiny || floor_hit) {
            res.status = 0;
            ++it;
            break;
          }
          continue;
        }
      }
      if (tiny) {  // a rounding-size step that does not lower chi^2
        res.status = 0;
        ++it;
        break;
      }
      lam = (lam > 0.0) ? lam * 10.0 : 1e-6;
      if (lam > 1e10) {
        // No damped step lowers chi^2.  That is the minimum at this
        // precision only when the point came from an accepted step and the
        // undamped Newton step there is of rounding size (at most 1e-7 of
        // each parameter's scale) or predicts a decrease of chi^2 / 2 below
        // 1e-12 of chi^2; otherwise (singular or non-finite sums, no step
        // ever accepted) the fit failed.
        bool conv = false;
        double xn[4];
        if (accepted > 0 && (gf_solve(S, p, true, 0.0, xn) || gf_solve(S, p, false, 0.0, xn))) {
          const double sg = fabs(p[3]);
          const bool small = fabs(xn[0]) <= 1e-7 * fabs(p[0]) && fabs(xn[1]) <= 1e-7 * fabs(p[1]) &&
                             fabs(xn[2]) <= 1e-7 * sg && fabs(xn[3]) <= 1e-7 * sg;
          // J^T r . x, with J = (1, -e, -s e q, -s e q^2), s = amp / sigma
          const double s = p[1] / p[3];
          const double dec =
              -0.5 * (S[GF_R] * xn[0] - S[GF_RE] * xn[1] - s * (S[GF_RE1] * xn[2] + S[GF_RE2] * xn[3]));
          conv = small || (isfinite(dec) && dec <= 1e-12 * S[0]);
        }
        res.status = conv ? 0 : 3;
        ++it;
        break;
      }
    }
    res.iters = it;
    res.chi2 = S[0];
  }
  res.rv_kms = p[2];
  res.sigma_kms = fabs(p[3]);
  res.fwhm_kms = FWHM_PER_SIGMA * fabs(p[3]);
  res.c0 = p[0];
  res.amp = p[1];
  if (res.status == 2) res.chi2 = 0.0;
  return res;
}

}  // namespace

// One block of four waves per spectrum.  The waves first add the line
// blocks' partial CCFs (wave w takes the line blocks lb = w mod 4, in
// order; the four partial sums are then added in wave order, so the result
// repeats bit for bit) and write the CCF.  With fit set, wave 0 then fits
// the Gaussian.
//
// Fit: damped Newton / Levenberg-Marquardt.  The step solves
// (H + lam diag(J^T J)) x = -J^T r with H the full Hessian of chi^2 / 2
// (J^T J plus the residual-weighted second derivatives; the CCF is not an
// exact Gaussian, so the residuals stay finite and Gauss-Newton alone
// converges only linearly) and falls back to H = J^T J where the full one
// is not positive definite.  A trial step is evaluated with all its sums,
// so an accepted step costs one pass over the CCF.  The fit has converged
// when a step moves every parameter by at most 1e-10 of its scale (sigma
// for the centre and width; at that size its chi^2 only reflects rounding,
// so it is taken without a pass), or when an accepted step no longer lowers
// chi^2 and moves the centre and width by at most 1e-9 sigma; a run of
// rejected steps that drives the damping past 1e10 means no downhill step
// exists at this precision, which is the minimum only when an earlier step
// was accepted and the undamped Newton step there is of rounding size
// (status 0); otherwise the fit failed (status 3).  A CCF with a non-finite
// sample or no depth is degenerate (status 2).
//
// Bound by the latency of the fit's chain: 100 spectra of 161 velocities and
// 125 partial rows take 13.5 us, about 5 of them for the sums and 1.2 an
// iteration (four on the headline).  As 20 sums in two butterflies with a
// Cholesky solve (square roots and divisions in the chain), extremes by
// shuffles and a branch per sample: 16.9 us; 4000 spectra, a wave each, 40.4
// and now 30.1 (170 registers instead of 195: three waves per SIMD); 300
// spectra of 401 velocities 43.0 and 30.4.
template <int NPT, typename PT>
__device__ __forceinline__ void fit_block(int n_lb, int64_t n_spec, int n_v, double v0, double dv,
                                          const PT* __restrict__ part, double* __restrict__ ccf, int fit,
                                          soap_rv* __restrict__ out, int64_t s) {
  __shared__ double s_sum[CCF_FIN_THREADS / 64][NPT * 64];
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  constexpr int NW = CCF_FIN_THREADS / 64;
  constexpr int RB = (NPT <= 3 ? 16 : (NPT <= 6 ? 8 : 4)) / (sizeof(PT) == 8 ? 2 : 1);  // rows in flight per wave
  {
    double acc[NPT];
#pragma unroll
    for (int t = 0; t < NPT; ++t) acc[t] = 0.0;
    for (int lb0 = wave; lb0 < n_lb; lb0 += RB * NW) {
      double v[RB][NPT];
      // every load is unconditional (indices clamped into the rows) and the
      // out-of-range values are zeroed after it: loads under a branch would
      // each be waited for before the next one is issued
      PT raw[RB][NPT];
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int lb = min(lb0 + u * NW, n_lb - 1);
        const PT* src = part + ((int64_t)lb * n_spec + s) * n_v;
#pragma unroll
        for (int t = 0; t < NPT; ++t) raw[u][t] = src[min(lane + 64 * t, n_v - 1)];
      }
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int lb = lb0 + u * NW;
#pragma unroll
        for (int t = 0; t < NPT; ++t) {
          const int i = lane + 64 * t;
          v[u][t] = (lb < n_lb && i < n_v) ? (double)raw[u][t] : 0.0;
        }
      }
#pragma unroll
      for (int u = 0; u < RB; ++u)
#pragma unroll
        for (int t = 0; t < NPT; ++t) acc[t] += v[u][t];
    }
#pragma unroll
    for (int t = 0; t < NPT; ++t) s_sum[wave][lane + 64 * t] = acc[t];
  }
  __syncthreads();
  if (wave != 0) return;
  double y[NPT];
#pragma unroll
  for (int t = 0; t < NPT; ++t) {
    const int i = lane + 64 * t;
    double a = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) a += s_sum[w][i];
    y[t] = a;
    if (i < n_v) ccf[s * n_v + i] = a;
  }
  if (!fit) return;
  double p[4], S[16];
  const soap_rv res = fit_wave(y, n_v, v0, dv, p, S);
  if (lane == 0) out[s] = res;
}

template <int NPT, typename PT>
__global__ void __launch_bounds__(CCF_FIN_THREADS) k_ccf_fit(int n_lb, int64_t n_spec, int n_v, double v0,
                                                             double dv, const PT* __restrict__ part,
                                                             double* __restrict__ ccf, int fit,
                                                             soap_rv* __restrict__ out) {
  fit_block<NPT, PT>(n_lb, n_spec, n_v, v0, dv, part, ccf, fit, out, blockIdx.x);
}

// One wave per spectrum: the same sums in the same order as fit_block's
// four waves (row lb goes to accumulator lb mod 4, rows ascending; the four
// accumulators are then added in order), so the CCF and the fit repeat
// fit_block's bit for bit; with every wave of a block fitting, four times as
// many fits are in flight.
template <int NPT, typename PT>
__device__ __forceinline__ void fit_one_wave(int n_lb, int64_t n_spec, int n_v, double v0, double dv,
                                             const PT* __restrict__ part, double* __restrict__ ccf, int fit,
                                             soap_rv* __restrict__ out, int64_t s) {
  const int lane = threadIdx.x & 63;
  constexpr int NW = CCF_FIN_THREADS / 64;  // fit_block's interleave of line blocks
  constexpr int RB = 2 * NW;                // rows in flight, a multiple of NW
  double acc[NW][NPT];
#pragma unroll
  for (int w = 0; w < NW; ++w)
#pragma unroll
    for (int t = 0; t < NPT; ++t) acc[w][t] = 0.0;
  for (int lb0 = 0; lb0 < n_lb; lb0 += RB) {
    // unconditional loads (indices clamped), out-of-range values zeroed after
    PT raw[RB][NPT];
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int lb = min(lb0 + u, n_lb - 1);
      const PT* src = part + ((int64_t)lb * n_spec + s) * n_v;
#pragma unroll
      for (int t = 0; t < NPT; ++t) raw[u][t] = src[min(lane + 64 * t, n_v - 1)];
    }
#pragma unroll
    for (int u = 0; u < RB; ++u)
#pragma unroll
      for (int t = 0; t < NPT; ++t) {
        const int i = lane + 64 * t;
        acc[u % NW][t] += (lb0 + u < n_lb && i < n_v) ? (double)raw[u][t] : 0.0;
      }
  }
  double y[NPT];
#pragma unroll
  for (int t = 0; t < NPT; ++t) {
    const int i = lane + 64 * t;
    double a = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) a += acc[w][t];
    y[t] = a;
    if (i < n_v) ccf[s * n_v + i] = a;
  }
  if (!fit) return;
  double p[4], S[16];
  const soap_rv res = fit_wave(y, n_v, v0, dv, p, S);
  if (lane == 0) out[s] = res;
}

// One wave per spectrum over one spectra set (calls with many spectra).
template <int NPT, typename PT>
__global__ void __launch_bounds__(CCF_FIN_THREADS) k_ccf_fit_waves(int n_lb, int64_t n_spec, int n_v, double v0,
                                                                   double dv, const PT* __restrict__ part,
                                                                   double* __restrict__ ccf, int fit,
                                                                   soap_rv* __restrict__ out) {
  const int64_t s = (int64_t)blockIdx.x * (CCF_FIN_THREADS / 64) + (threadIdx.x >> 6);
  if (s >= n_spec) return;  // whole waves
  fit_one_wave<NPT, PT>(n_lb, n_spec, n_v, v0, dv, part, ccf, fit, out, s);
}

// Work-list form, one wave per entry: blk[b] = (set, spectrum).
template <int NPT, typename PT>
__global__ void __launch_bounds__(CCF_FIN_THREADS) k_ccf_fit_batch(const CcfBatchSet* __restrict__ sets,
                                                                   const int2* __restrict__ blk, int n_blk, int n_v,
                                                                   double v0, double dv) {
  const int b = blockIdx.x * (CCF_FIN_THREADS / 64) + (threadIdx.x >> 6);
  if (b >= n_blk) return;  // whole waves
  const int2 t = blk[b];
  const CcfBatchSet c = sets[t.x];
  fit_one_wave<NPT, PT>(c.nlb, c.n_spec, n_v, v0, dv, static_cast<const PT*>(c.part), c.ccf, c.rv ? 1 : 0, c.rv,
                        t.y);
}

// Whole waves that hold the velocity grid, so that a grid is not rounded up to
// a fixed block: 401 velocities run on 448 lanes (300 spectra of 150001 pixels,
// 3000 lines: 103 us on 768 lanes, 71 so).
template <int A>
static unsigned ccf_threads(int n_v) {
  return (unsigned)std::max(CCF_MIN_THREADS, 64 * ((n_v + 64 * A - 1) / (64 * A)));
}

template <typename T, int A, int NPX, int STG>
static void launch_ccf_a(const CcfPlan& q, hipStream_t st, const void* d_flux, int64_t n_spec,
                         void* d_part) {
  const unsigned char* base = q.tables;
  const int nlb = ccf_line_blocks(q.n_lines);
  auto blocks = [&](int sb) { return dim3((unsigned)nlb, (unsigned)((n_spec + sb - 1) / sb)); };
  // Few blocks of CCF_SB spectra leave the chip idle, and each is a chain of
  // batches that wait for their loads: then blocks of CCF_FEW spectra with
  // CCF_AHEAD batches of loads in flight.  The line lies where the blocks' waves
  // would fill it (stage times with CCF_SB and so, FP32): 161 velocities, 3 waves
  // a block, 13 blocks 12.1 and 10.7 us, 125 12.4 and 11.6, 190 13.2 and 12.8, 250
  // 12.8 and 12.8, 375 13.9 and 15.1; 401 velocities, 7 waves, 13 blocks 12.6 and
  // 11.2, 75 13.8 and 12.4, 94 14.4 and 14.3, 125 13.3 and 13.7, 190 14.2 and 16.7.
  // FP64 gains more below it (125 blocks: 12.7 and 11.1, 14.6 and 13.9).
  const unsigned threads = ccf_threads<A>(q.nv);
  const bool few = (int64_t)nlb * blocks(CCF_SB).y * (threads / 64) < CCF_FEW_WAVES;
  auto* kernel = few ? &k_ccf<T, A, NPX, STG, CCF_FEW, CCF_AHEAD> : &k_ccf<T, A, NPX, STG, CCF_SB, 1>;
  hipLaunchKernelGGL(kernel, blocks(few ? CCF_FEW : CCF_SB), dim3(threads), 0, st, (int)q.P, n_spec,
                     static_cast<const T*>(d_flux), reinterpret_cast<const double2*>(base),
                     reinterpret_cast<const double2*>(base + q.off_edges),
                     reinterpret_cast<const int4*>(base + q.off_batch),
                     reinterpret_cast<const int*>(base + q.off_bfirst), q.nv, static_cast<T*>(d_part));
}

template <typename T, int NPX, int STG>
static void launch_ccf_n(const CcfPlan& q, hipStream_t st, const void* d_flux, int64_t n_spec,
                         void* d_part) {
  if (q.nv <= CCF_THREADS) launch_ccf_a<T, 1, NPX, STG>(q, st, d_flux, n_spec, d_part);
  else launch_ccf_a<T, CCF_MORE<T>, NPX, STG>(q, st, d_flux, n_spec, d_part);
}

template <typename T, int STG>
static void launch_ccf_s(const CcfPlan& q, hipStream_t st, const void* d_flux, int64_t n_spec,
                         void* d_part) {
  switch (q.npx) {
    case 2: launch_ccf_n<T, 2, STG>(q, st, d_flux, n_spec, d_part); break;
    case 3: launch_ccf_n<T, 3, STG>(q, st, d_flux, n_spec, d_part); break;
    case 5: launch_ccf_n<T, 5, STG>(q, st, d_flux, n_spec, d_part); break;
    default: launch_ccf_n<T, 10, STG>(q, st, d_flux, n_spec, d_part); break;
  }
}

template <typename T>
static void launch_ccf_t(const CcfPlan& q, hipStream_t st, const void* d_flux, int64_t n_spec,
                         void* d_part) {
  if (q.stg <= 256) launch_ccf_s<T, 256>(q, st, d_flux, n_spec, d_part);
  else launch_ccf_s<T, CCF_STG_MAX>(q, st, d_flux, n_spec, d_part);
}

CcfPlan ccf_plan(const soap_ctx* c, int n_lines, const void* tables) {
  CcfPlan q;
  q.tables = static_cast<const unsigned char*>(tables);
  q.off_edges = c->ccf_off_edges;
  q.off_batch = c->ccf_off_batch;
  q.off_bfirst = c->ccf_off_bfirst;
  q.npx = c->ccf_npx;
  q.stg = c->ccf_stg;
  q.nv = c->mask_nv;
  q.n_lines = n_lines;
  q.v0 = c->mask_v0;
  q.dv = c->mask_dv;
  q.fp32 = c->prec == SOAP_PREC_FP32;
  q.P = c->P;
  return q;
}

hipError_t launch_ccf_p(const CcfPlan& q, hipStream_t st, const void* d_flux, int64_t n_spec, void* d_part) {
  if (q.fp32) launch_ccf_t<float>(q, st, d_flux, n_spec, d_part);
  else launch_ccf_t<double>(q, st, d_flux, n_spec, d_part);
  return hipGetLastError();
}

hipError_t launch_ccf(soap_ctx* c, const void* d_flux, int64_t n_spec, int n_lines, void* d_part) {
  return launch_ccf_p(ccf_plan(c, n_lines, c->ws_mask.ptr), c->stream, d_flux, n_spec, d_part);
}

// the fit kernel for the mask's points per lane
template <typename PT>
static hipError_t launch_fit_npt(const CcfPlan& q, hipStream_t st, int nlb, int64_t n_spec, const PT* d_part,
                                 double* d_ccf, soap_rv* d_rv) {
  const int npt = (q.nv + 63) / 64;
  // up to CCF_FIT_WAVES_FROM spectra a block of four waves per spectrum
  // (partial sums spread over the block, every fit in flight at once);
  // beyond, a wave per spectrum (four fits in flight per block); both give
  // the same records bit for bit
  constexpr int kWaves = CCF_FIN_THREADS / 64;
  const bool waves = n_spec > CCF_FIT_WAVES_FROM;
  const unsigned grid = waves ? (unsigned)((n_spec + kWaves - 1) / kWaves) : (unsigned)n_spec;
#define FIT_CASE(N)                                                                                          \
  case N:                                                                                                    \
    if (waves)                                                                                               \
      hipLaunchKernelGGL((k_ccf_fit_waves<N, PT>), dim3(grid), dim3(CCF_FIN_THREADS), 0, st, nlb, n_spec, q.nv, \
                         q.v0, q.dv, d_part, d_ccf, d_rv ? 1 : 0, d_rv);                                     \
    else                                                                                                     \
      hipLaunchKernelGGL((k_ccf_fit<N, PT>), dim3(grid), dim3(CCF_FIN_THREADS), 0, st, nlb, n_spec, q.nv, q.v0, \
                         q.dv, d_part, d_ccf, d_rv ? 1 : 0, d_rv);                                           \
    break;
  switch (npt) {
    FIT_CASE(1) FIT_CASE(2) FIT_CASE(3) FIT_CASE(4) FIT_CASE(5) FIT_CASE(6)
    FIT_CASE(7) FIT_CASE(8) FIT_CASE(9) FIT_CASE(10) FIT_CASE(11) FIT_CASE(12)
    default: return hipErrorInvalidValue;
  }
#undef FIT_CASE
  return hipGetLastError();
}

hipError_t launch_ccf_fit_p(const CcfPlan& q, hipStream_t st, const void* d_part, int64_t n_spec, double* d_ccf,
                            soap_rv* d_rv) {
  const int nlb = ccf_line_blocks(q.n_lines);
  if (q.fp32) return launch_fit_npt(q, st, nlb, n_spec, static_cast<const float*>(d_part), d_ccf, d_rv);
  return launch_fit_npt(q, st, nlb, n_spec, static_cast<const double*>(d_part), d_ccf, d_rv);
}

hipError_t launch_ccf_fit(soap_ctx* c, int n_lines, const void* d_part, int64_t n_spec, double* d_ccf,
                          soap_rv* d_rv) {
  return launch_ccf_fit_p(ccf_plan(c, n_lines, c->ws_mask.ptr), c->stream, d_part, n_spec, d_ccf, d_rv);
}

// ---- work-list CCF + fit over many spectra sets ------------------------------

bool ccf_same_layout(const CcfPlan& a, const CcfPlan& b) {
  return a.fp32 == b.fp32 && a.npx == b.npx && (a.stg <= 256) == (b.stg <= 256) && a.nv == b.nv && a.v0 == b.v0 &&
         a.dv == b.dv;
}

namespace {

size_t al256c(size_t b) { return 256 * ((b + 255) / 256); }

template <typename T, int A, int NPX, int STG>
void launch_ccf_batch_a(const CcfBatch& cb, hipStream_t st) {
  hipLaunchKernelGGL((k_ccf_batch<T, A, NPX, STG>), dim3((unsigned)cb.n_ccf_blocks),
                     dim3(ccf_threads<A>(cb.shape.nv)), 0, st, cb.sets, cb.ccf_blk, cb.shape.nv);
}

template <typename T, int NPX, int STG>
void launch_ccf_batch_n(const CcfBatch& cb, hipStream_t st) {
  if (cb.shape.nv <= CCF_THREADS) launch_ccf_batch_a<T, 1, NPX, STG>(cb, st);
  else launch_ccf_batch_a<T, CCF_MORE<T>, NPX, STG>(cb, st);
}

template <typename T, int STG>
void launch_ccf_batch_s(const CcfBatch& cb, hipStream_t st) {
  switch (cb.shape.npx) {
    case 2: launch_ccf_batch_n<T, 2, STG>(cb, st); break;
    case 3: launch_ccf_batch_n<T, 3, STG>(cb, st); break;
    case 5: launch_ccf_batch_n<T, 5, STG>(cb, st); break;
    default: launch_ccf_batch_n<T, 10, STG>(cb, st); break;
  }
}

template <typename T>
void launch_ccf_batch_t(const CcfBatch& cb, hipStream_t st) {
  if (cb.shape.stg <= 256) launch_ccf_batch_s<T, 256>(cb, st);
  else launch_ccf_batch_s<T, CCF_STG_MAX>(cb, st);
}

template <typename PT>
hipError_t launch_fit_batch_pt(const CcfBatch& cb, hipStream_t st) {
  const int npt = (cb.shape.nv + 63) / 64;
  constexpr int kWaves = CCF_FIN_THREADS / 64;  // one spectrum per wave
  const unsigned grid = (unsigned)((cb.n_fit_blocks + kWaves - 1) / kWaves);
#define FITB_CASE(N)                                                                                           \
  case N:                                                                                                      \
    hipLaunchKernelGGL((k_ccf_fit_batch<N, PT>), dim3(grid), dim3(CCF_FIN_THREADS), 0, st, cb.sets, cb.fit_blk, \
                       cb.n_fit_blocks, cb.shape.nv, cb.shape.v0, cb.shape.dv);                                 \
    break;
  switch (npt) {
    FITB_CASE(1) FITB_CASE(2) FITB_CASE(3) FITB_CASE(4) FITB_CASE(5) FITB_CASE(6)
    FITB_CASE(7) FITB_CASE(8) FITB_CASE(9) FITB_CASE(10) FITB_CASE(11) FITB_CASE(12)
    default: return hipErrorInvalidValue;
  }
#undef FITB_CASE
  return hipGetLastError();
}

}  // namespace

size_t ccf_batch_bytes(const CcfPlan* plans, const int64_t* n_spec, int n) {
  size_t ccf_blocks = 0, fit_blocks = 0;
  for (int i = 0; i < n; ++i) {
    ccf_blocks += (size_t)ccf_line_blocks(plans[i].n_lines) * (size_t)((n_spec[i] + CCF_SB - 1) / CCF_SB);
    fit_blocks += (size_t)n_spec[i];
  }
  return al256c(sizeof(CcfBatchSet) * n) + al256c(sizeof(int4) * ccf_blocks) + al256c(sizeof(int2) * fit_blocks);
}

hipError_t ccf_batch_upload(const CcfPlan* plans, const CcfBatchSet* sets, int n, void* d_buf, CcfBatch* cb) {
  if (n < 1) return hipErrorInvalidValue;
  std::vector<CcfBatchSet> hs(sets, sets + n);
  std::vector<int4> cblk;
  std::vector<int2> fblk;
  for (int i = 0; i < n; ++i) {
    if (!ccf_same_layout(plans[i], plans[0]) || sets[i].n_spec < 1 || sets[i].n_spec > (int64_t(1) << 24))
      return hipErrorInvalidValue;
    const CcfPlan& q = plans[i];
    CcfBatchSet& h = hs[i];
    h.P = (int)q.P;
    h.nlb = ccf_line_blocks(q.n_lines);
    h.tables = q.tables;
    h.off_edges = q.off_edges;
    h.off_batch = q.off_batch;
    h.off_bfirst = q.off_bfirst;
    const int nsb = (int)((h.n_spec + CCF_SB - 1) / CCF_SB);
    for (int lb = 0; lb < h.nlb; ++lb)
      for (int sb = 0; sb < nsb; ++sb) cblk.push_back(make_int4(i, lb, sb, 0));
    for (int64_t sp = 0; sp < h.n_spec; ++sp) fblk.push_back(make_int2(i, (int)sp));
  }
  unsigned char* base = static_cast<unsigned char*>(d_buf);
  cb->shape = plans[0];
  cb->n_sets = n;
  cb->n_ccf_blocks = (int)cblk.size();
  cb->n_fit_blocks = (int)fblk.size();
  cb->sets = reinterpret_cast<CcfBatchSet*>(base);
  size_t used = al256c(sizeof(CcfBatchSet) * n);
  cb->ccf_blk = reinterpret_cast<int4*>(base + used);
  used += al256c(sizeof(int4) * cblk.size());
  cb->fit_blk = reinterpret_cast<int2*>(base + used);
  hipError_t e = hipMemcpy(cb->sets, hs.data(), sizeof(CcfBatchSet) * n, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(cb->ccf_blk, cblk.data(), sizeof(int4) * cblk.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(cb->fit_blk, fblk.data(), sizeof(int2) * fblk.size(), hipMemcpyHostToDevice);
  return e;
}

hipError_t ccf_batch_launch(const CcfBatch& cb, hipStream_t st) {
  if (cb.n_ccf_blocks <= 0) return hipSuccess;
  if (cb.shape.fp32) launch_ccf_batch_t<float>(cb, st);
  else launch_ccf_batch_t<double>(cb, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return cb.shape.fp32 ? launch_fit_batch_pt<float>(cb, st) : launch_fit_batch_pt<double>(cb, st);
}

// ccf[i][v] = base[v] + sum_k coef[i][k] basis[k][v] (double, increasing k):
// the CCF of a spectrum written in a basis, by linearity.  One block per row.
__global__ void __launch_bounds__(256) k_ccf_linear(int64_t n, int k, int n_v, const float* __restrict__ coef,
                                                    const double* __restrict__ base,
                                                    const double* __restrict__ basis, double* __restrict__ ccf) {
  __shared__ double s_c[256];
  const int64_t i = blockIdx.x;
  for (int v0 = 0; v0 < n_v; v0 += 256) {
    const int v = v0 + threadIdx.x;
    double a = v < n_v ? base[v] : 0.0;
    for (int k0 = 0; k0 < k; k0 += 256) {
      __syncthreads();
      if (k0 + (int)threadIdx.x < k) s_c[threadIdx.x] = (double)coef[i * k + k0 + threadIdx.x];
      __syncthreads();
      const int kn = min(256, k - k0);
      if (v < n_v)
        for (int j = 0; j < kn; ++j) a = fma(s_c[j], basis[(int64_t)(k0 + j) * n_v + v], a);
    }
    if (v < n_v) ccf[i * n_v + v] = a;
  }
}

constexpr int SG_MAX_ENS = 16;

// Surrogate RVs and their gate in three launches:
//   k_sg_lin: CCF of the ensemble-mean prediction by linearity, base (the
//     sample's row base[base_idx[i]] when base_idx is given) + sum_k
//     coef[i][k] basis[k];
//   k_sg_fit: its Gaussian fit (fit_wave), one wave per sample (issue-bound:
//     88 us per 1e4 samples with the fit's former 20 sums, 62 now), and the RV
//     sensitivity g = J H^-1 e_mu at the fit: the fitted parameters move by
//     dp = H^-1 J^T dy for a CCF change dy (H the Hessian of chi^2 / 2 at the
//     fit, J the model Jacobian), so dRV = g . dy;
//   k_sg_spread: each member's RV change dRV_e = sum_k h_k (y_e,k - coef_k)
//     with h = basis g (dy_e = sum_k (y_e,k - coef_k) basis[k]); err = calib x
//     the sample standard deviation of the dRV_e; fallback when err is not
//     below thr or the fit did not converge.
// The first and the last are matrix products in double, on the matrix cores
// (v_mfma_f64_16x16x4_f64: lane l holds A(l % 16, l / 16) and B(l / 16, l % 16)
// and ends with C(l / 16 + 4 r, l % 16), r < 4; the four terms are added in
// order).  k_sg_lin takes its components in order, so its sums are those of
// k_ccf_linear; k_sg_spread takes velocities 4 (l / 16) + s of 16 in step s, so
// that a lane's operands are contiguous.  A block of SG_W waves takes 16 samples, each wave its share of
// the columns.  Bound by the first-level cache, so the samples' operands pass
// through LDS and the basis is read 16 bytes a lane.
// 10000 samples, 128 components, 161 velocities: 19 and 26 us, against
// 42 and 52 as vector FMAs with 4 samples a wave.  Every sum of a sample keeps
// one fixed order.
constexpr int SG_W = 4;
constexpr int SG_KC = 128;  // components per LDS pass of k_sg_lin
constexpr int SG_VC = 192;  // velocities per LDS pass of k_sg_spread, at most
// row length of its LDS: whole groups of 16 velocities, and two against bank conflicts
__host__ __device__ constexpr int sg_spread_ld(int n_v) { return (n_v < SG_VC ? (n_v + 15) & ~15 : SG_VC) + 2; }
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

// NPT column tiles per wave: SG_W NPT 16 = 64 NPT columns
template <int NPT>
__global__ void __launch_bounds__(64 * SG_W, NPT <= 3 ? 3 : 1) k_sg_lin(int64_t n, int k, int n_v, const float* __restrict__ coef,
                                                      const double* __restrict__ base,
                                                      const int* __restrict__ base_idx, int n_base,
                                                      const double* __restrict__ basis, double* __restrict__ Y,
                                                      int* __restrict__ flag) {
  __shared__ float s_a[16][SG_KC + 4];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = l & 15, g = l >> 4;
  const int64_t i0 = (int64_t)blockIdx.x * 16;
  // The wave's columns: pairs of tiles take every other one of 32, so that a
  // lane loads two at once, an odd last tile takes 16.  Loads are
  // unconditional, with indices clamped into the rows (columns past the grid
  // and samples past n compute values that are never stored): a load under a
  // branch is waited for before the next one is issued.  A sample whose star
  // row does not exist reads row 0 and is flagged.
  constexpr int PAIRS = NPT / 2;
  constexpr bool ODD = NPT % 2;
  int col[NPT];
#pragma unroll
  for (int t = 0; t < NPT; ++t) col[t] = 16 * NPT * w + (t < 2 * PAIRS ? 32 * (t / 2) + 2 * c + t % 2 : 16 * t + c);
  struct Set {
    f64x2u p[4][PAIRS > 0 ? PAIRS : 1];
    double b[4];
  };
  auto load = [&](Set& o, int k0) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double* bj = basis + (int64_t)min(k0 + 4 * s + g, k - 1) * n_v;
#pragma unroll
      for (int q = 0; q < PAIRS; ++q) o.p[s][q] = *reinterpret_cast<const f64x2u*>(bj + min(col[2 * q], n_v - 2));
      if constexpr (ODD) o.b[s] = bj[min(col[NPT - 1], n_v - 1)];
    }
  };
  auto column = [&](const Set& o, int s, int t) {  // a pair that starts in the last column has it as its second
    if (t < 2 * PAIRS) return t % 2 || col[t] == n_v - 1 ? o.p[s][t / 2][1] : o.p[s][t / 2][0];
    return o.b[s];
  };
  constexpr int D = NPT <= 4 ? 3 : 2;  // groups in flight
  Set o[D];
#pragma unroll
  for (int d = 0; d + 1 < D; ++d) load(o[d], 16 * d);
  // the sums start at the samples' base rows; every row index is loaded before
  // the first is used, and every base value has arrived before the loop (which
  // would wait for all its loads in each turn otherwise)
  int brow[4] = {0, 0, 0, 0};
  if (base_idx) {
#pragma unroll
    for (int r = 0; r < 4; ++r) brow[r] = base_idx[min(i0 + g + 4 * r, n - 1)];
  }
  f64x4 acc[NPT];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double* b = base + (int64_t)(brow[r] >= 0 && brow[r] < n_base ? brow[r] : 0) * n_v;
#pragma unroll
    for (int t = 0; t < NPT; ++t) acc[t][r] = b[min(col[t], n_v - 1)];
  }
#pragma unroll
  for (int t = 0; t < NPT; ++t) asm volatile("" : "+v"(acc[t]));
  for (int kc = 0; kc < k; kc += SG_KC) {  // the coefficients pass through LDS
    const int kn = min(SG_KC, k - kc);
    if (kc) {
      __syncthreads();
#pragma unroll
      for (int d = 0; d + 1 < D; ++d) load(o[d], kc + 16 * d);
    }
    constexpr int U = 16 * SG_KC / (64 * SG_W);
    float x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = threadIdx.x + 64 * SG_W * u;
      x[u] = coef[min(i0 + t / SG_KC, n - 1) * k + kc + min(t % SG_KC, kn - 1)];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = threadIdx.x + 64 * SG_W * u;
      s_a[t / SG_KC][t % SG_KC] = t % SG_KC < kn ? x[u] : 0.f;  // rows past k add zero
    }
    __syncthreads();
    for (int k0 = 0; k0 < kn; k0 += 16 * D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        load(o[(d + D - 1) % D], kc + k0 + 16 * (d + D - 1));
        if (k0 + 16 * d >= kn) continue;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double a = (double)s_a[c][k0 + 16 * d + 4 * s + g];
#pragma unroll
          for (int t = 0; t < NPT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, column(o[d], s, t), acc[t], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t i = i0 + g + 4 * r;
    if (w == 0 && c == 0 && i < n) flag[i] = brow[r] >= 0 && brow[r] < n_base ? 0 : 1;
#pragma unroll
    for (int t = 0; t < NPT; ++t)
      if (i < n && col[t] < n_v) Y[i * n_v + col[t]] = acc[t][r];
  }
}

// flag[i] on entry: 1 when the sample has no star row; on exit: 1 when it
// has no surrogate RV (no row, or the fit or its sensitivity failed).
template <int NPT>
__global__ void __launch_bounds__(64) k_sg_fit(int64_t n, int n_v, double v0, double dv,
                                               const double* __restrict__ Y, int* __restrict__ flag,
                                               soap_rv* __restrict__ out, double* __restrict__ rv_kms,
                                               double* __restrict__ G) {
  const int64_t i = blockIdx.x;
  const int lane = threadIdx.x;
  const bool row_ok = flag[i] == 0;
  double y[NPT];
#pragma unroll
  for (int t = 0; t < NPT; ++t) y[t] = Y[i * n_v + min(lane + 64 * t, n_v - 1)];
  double p[4], S[16];
  soap_rv res = fit_wave(y, n_v, v0, dv, p, S);
  bool bad = res.status != 0 || !row_ok;
  double z[4] = {0.0, 0.0, 0.0, 0.0};
  if (!bad) {
    // z = H^-1 e_mu (full Hessian; J^T J where that is not positive definite),
    // for the scaled centre and width (z[2], z[3] times amp / sigma)
    const double b[4] = {0.0, 0.0, p[3] / p[1], 0.0};
    if (!(gf_solve_scaled(S, p, true, 0.0, b, z) || gf_solve_scaled(S, p, false, 0.0, b, z))) bad = true;
  }
  const double is = 1.0 / p[3];
#pragma unroll
  for (int t = 0; t < NPT; ++t) {
    const int v = lane + 64 * t;
    if (v < n_v) {
      const double q = (v0 + dv * v - p[2]) * is;
      const double e = exp(-0.5 * q * q);
      G[i * n_v + v] = bad ? 0.0 : z[0] - e * (z[1] + q * (z[2] + q * z[3]));
    }
  }
  if (lane == 0) {
    if (!row_ok) {
      res = soap_rv{};
      res.status = 2;
    }
    if (out) out[i] = res;
    rv_kms[i] = row_ok ? res.rv_kms : 0.0;
    flag[i] = bad ? 1 : 0;
  }
}

// EB: members, rounded up; W waves per block, 32 components each at a time.  In
// calls of many blocks with few components fewer waves per block, and LDS for the
// velocities there are, so that more blocks are in flight: 8 members, 32
// components, 41 velocities, 20000 samples 99 us with four waves and room for 192
// velocities, 41 so.
template <int EB, int W>
__global__ void __launch_bounds__(64 * W) k_sg_spread(int64_t n, int k, int E, int n_v,
                                                         const float* __restrict__ coef,
                                                         const float* __restrict__ members,
                                                         const double* __restrict__ basis,
                                                         const double* __restrict__ G, const int* __restrict__ flag,
                                                         double calib, double thr, double* __restrict__ err_kms,
                                                         int* __restrict__ fallback) {
  constexpr int NT = 2;
  __shared__ double s_dr[W][16][EB];
  extern __shared__ __align__(16) double s_g[];  // [16][ld]
  const int ld = sg_spread_ld(n_v);
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int c = l & 15, g = l >> 4;
  const int64_t i0 = (int64_t)blockIdx.x * 16;
  double dr[4][EB];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int e = 0; e < EB; ++e) dr[r][e] = 0.0;
  // h_k = sum_v basis[k][v] g_v, then dRV_e = sum_k h_k (y_e,k - coef_k)
  for (int kb = 0; kb < k; kb += 16 * NT * W) {
    const int k0 = kb + 16 * NT * w;
    // waves past k only stage
    const bool mine = k0 < k;
    const double* bp[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) bp[t] = basis + (int64_t)min(k0 + 16 * t + c, k - 1) * n_v;
    f64x4 h[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) h[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    struct Set {
      f64x2u b[NT][2];
    };
    auto load = [&](Set& o, int v) {  // the lane's four velocities of a group of 16
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int t = 0; t < NT; ++t) o.b[t][q] = *reinterpret_cast<const f64x2u*>(bp[t] + v + 4 * g + 2 * q);
    };
    auto multiply = [&](const Set& o, int v) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f64x2 a = *reinterpret_cast<const f64x2*>(&s_g[c * ld + v + 4 * g + 2 * q]);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int t = 0; t < NT; ++t)
            h[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], o.b[t][q][x], h[t], 0, 0, 0);
      }
    };
    for (int vc = 0; vc < n_v; vc += SG_VC) {  // the sensitivities pass through LDS, zeros past the grid
      const int vn = min(SG_VC, n_v - vc), whole = vn & ~15;
      constexpr int D = 3;  // groups in flight; past the last whole one it is read again
      Set o[D];
      if (mine && whole) {
#pragma unroll
        for (int d = 0; d + 1 < D; ++d) load(o[d], vc + min(16 * d, whole - 16));
      }
      if ((kb == 0 && vc == 0) || n_v > SG_VC) {
        if (kb || vc) __syncthreads();
        constexpr int TR = 4 * W, U = SG_VC / TR;  // threads per sample's row
        const int row = threadIdx.x / TR, col = threadIdx.x % TR, wide = (vn + 15) & ~15;
        const double* gr = G + min(i0 + row, n - 1) * n_v + vc;
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += 12) {
          double x[12];  // all loads before the first is waited for
#pragma unroll
          for (int u = 0; u < 12; ++u)
            if (TR * (u0 + u) < vn) x[u] = gr[min(col + TR * (u0 + u), vn - 1)];
#pragma unroll
          for (int u = 0; u < 12; ++u) {
            const int v = col + TR * (u0 + u);
            if (v < wide) s_g[row * ld + v] = v < vn ? x[u] : 0.0;
          }
        }
        __syncthreads();
      }
      if (!mine) continue;
      for (int v = 0; v < whole; v += 16 * D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          load(o[(d + D - 1) % D], vc + min(v + 16 * (d + D - 1), whole - 16));
          if (v + 16 * d < whole) multiply(o[d], v + 16 * d);
        }
      }
      if (whole < vn) {
        Set e;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int v = whole + 4 * g + x;
#pragma unroll
          for (int t = 0; t < NT; ++t) e.b[t][x >> 1][x & 1] = v < vn ? bp[t][vc + min(v, vn - 1)] : 0.0;
        }
        multiply(e, whole);
      }
    }
    if (!mine) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t i = min(i0 + g + 4 * r, n - 1);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int kc = min(k0 + 16 * t + c, k - 1);
        const double hk = k0 + 16 * t + c < k ? h[t][r] : 0.0;
        const double cm = (double)coef[i * k + kc];
#pragma unroll
        for (int e = 0; e < EB; ++e) {
          const double ye = (double)members[((int64_t)min(e, E - 1) * n + i) * k + kc];
          dr[r][e] += hk * (ye - cm);
        }
      }
    }
  }
  // sums over the 16 lanes of a sample's components, then over the waves
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      double x = dr[r][e];
      x += dpp_f64<DPP_PAIR>(x);
      x += dpp_f64<DPP_QUAD>(x);
      x += dpp_f64<DPP_HALF_MIRROR>(x);
      x += dpp_f64<DPP_MIRROR>(x);
      if (c == 0) s_dr[w][g + 4 * r][e] = x;
    }
  __syncthreads();
  const int s = threadIdx.x;
  if (s >= 16 || i0 + s >= n) return;
  const bool bad = flag[i0 + s] != 0;
  double err = 0.0;
  if (!bad) {
    double d[EB], m = 0.0;
#pragma unroll
    for (int e = 0; e < EB; ++e) {
      if constexpr (W == 4) d[e] = (s_dr[0][s][e] + s_dr[1][s][e]) + (s_dr[2][s][e] + s_dr[3][s][e]);
      else if constexpr (W == 2) d[e] = s_dr[0][s][e] + s_dr[1][s][e];
      else d[e] = s_dr[0][s][e];
      if (e < E) m += d[e];
    }
    m /= (double)E;
    double var = 0.0;
#pragma unroll
    for (int e = 0; e < EB; ++e)
      if (e < E) var += (d[e] - m) * (d[e] - m);
    err = calib * sqrt(var / (double)(E - 1));
  }
  if (err_kms) err_kms[i0 + s] = bad ? INFINITY : err;
  fallback[i0 + s] = (bad || !(err < thr)) ? 1 : 0;
}

namespace {

template <int NPT>
void launch_sg_rv_n(soap_ctx* c, const float* d_coef, const float* d_members, int64_t n, int E, int k,
                    const double* d_base, const int* d_base_idx, int n_base, const double* d_basis, double calib,
                    double thr, soap_rv* d_rv, double* d_rv_kms, double* d_err, int* d_fallback, double* Y,
                    double* G, int* flag) {
  const dim3 grid((unsigned)((n + 15) / 16)), block(64 * SG_W);
  const int nb = d_base_idx ? n_base : 1;
  hipLaunchKernelGGL((k_sg_lin<NPT>), grid, block, 0, c->stream, n, k, c->mask_nv, d_coef, d_base,
                     d_base_idx, nb, d_basis, Y, flag);
  hipLaunchKernelGGL((k_sg_fit<NPT>), dim3((unsigned)n), dim3(64), 0, c->stream, n, c->mask_nv, c->mask_v0,
                     c->mask_dv, Y, flag, d_rv, d_rv_kms, G);
  const size_t lds = sizeof(double) * 16 * sg_spread_ld(c->mask_nv);
  auto spread = [&](auto eb) {
    constexpr int EB = decltype(eb)::value;
    // Up to a block per CU the waves past the components still stage (call times
    // with one, two and four waves, 32 components, 401 velocities, us: 960 samples
    // of 2 members 53, 52 and 48; 6000 of 2 100, 96 and 98; 6000 of 8 123, 119 and
    // 139).  One wave pays past two blocks per CU of more than four members: 12000
    // of 8 170, 192 and 206; 20000 of 2 231, 226 and 230.
    const int w = k > 64 || grid.x <= 256 ? 4 : (k > 32 || EB <= 4 || grid.x <= 512 ? 2 : 1);
    auto* kernel = w == 1 ? &k_sg_spread<EB, 1> : (w == 2 ? &k_sg_spread<EB, 2> : &k_sg_spread<EB, 4>);
    hipLaunchKernelGGL(kernel, grid, dim3(64 * w), lds, c->stream, n, k, E, c->mask_nv, d_coef, d_members, d_basis, G,
                       flag, calib, thr, d_err, d_fallback);
  };
  if (E <= 4) spread(std::integral_constant<int, 4>());
  else if (E <= 8) spread(std::integral_constant<int, 8>());
  else spread(std::integral_constant<int, SG_MAX_ENS>());
}

}  // namespace

hipError_t launch_sg_rv(soap_ctx* c, const float* d_coef, const float* d_members, int64_t n, int E, int k,
                        const double* d_base, const int* d_base_idx, int n_base, const double* d_basis,
                        double calib, double thr, soap_rv* d_rv, double* d_rv_kms, double* d_err,
                        int* d_fallback, void* d_work) {
  if (E < 2 || E > SG_MAX_ENS) return hipErrorInvalidValue;
  const int npt = (c->mask_nv + 63) / 64;
  double* Y = static_cast<double*>(d_work);
  double* G = Y + (size_t)n * c->mask_nv;
  int* flag = reinterpret_cast<int*>(G + (size_t)n * c->mask_nv);
#define SG_CASE(N)                                                                                              \
  case N:                                                                                                       \
    launch_sg_rv_n<N>(c, d_coef, d_members, n, E, k, d_base, d_base_idx, n_base, d_basis, calib, thr, d_rv,     \
                      d_rv_kms, d_err, d_fallback, Y, G, flag);                                                 \
    break;
  switch (npt) {
    SG_CASE(1) SG_CASE(2) SG_CASE(3) SG_CASE(4) SG_CASE(5) SG_CASE(6)
    SG_CASE(7) SG_CASE(8) SG_CASE(9) SG_CASE(10) SG_CASE(11) SG_CASE(12)
    default: return hipErrorInvalidValue;
  }
#undef SG_CASE
  return hipGetLastError();
}

size_t sg_rv_work_bytes(const soap_ctx* c, int64_t n) {
  return sizeof(double) * 2 * (size_t)n * c->mask_nv + sizeof(int) * (size_t)n;
}

hipError_t launch_ccf_linear_fit(soap_ctx* c, const float* d_coef, int64_t n, int k, const double* d_base,
                                 const double* d_basis, double* d_lin, double* d_ccf, soap_rv* d_rv) {
  hipLaunchKernelGGL(k_ccf_linear, dim3((unsigned)n), dim3(256), 0, c->stream, n, k, c->mask_nv, d_coef, d_base,
                     d_basis, d_lin);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the rows are complete CCFs: one "block of lines" for the fit kernel
  return launch_fit_npt(ccf_plan(c, 1, c->ws_mask.ptr), c->stream, 1, n, d_lin, d_ccf, d_rv);
}



}  // namespace soap
