// Learned surrogate of the disk-integrated spectrum: a small MLP that maps
// the active-region and star parameters of one spectrum to the PCA
// coefficients of its difference from the quiet spectrum (Eqs. 1-4 give the
// spectrum the network stands in for), with its training and inference
// kernels.
//
// Network per ensemble member: x[n_in] -> SiLU(x W1 + b1)[H] ->
// SiLU(. W2 + b2)[H] -> . W3 + b3 [n_out].  Parameters are FP32 masters;
// the matrix products run on BF16 copies with MFMA (v_mfma_f32_16x16x32_bf16,
// FP32 accumulate): the whole network per block of rows where its activations
// fit in LDS, else a kernel per layer.  Training minimises the
// mean squared error over the batch and outputs with Adam (bias-corrected
// moments, FP32).  Every kernel has a fixed order of operations, so results
// repeat bit for bit.
//
// The PCA projection coef = (d - mean) V of spectra differences onto a basis
// is an FP32 product on the matrix cores (K = pixels, large).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "surrogate_internal.hpp"
#include "wave.hpp"

namespace soap {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

__device__ __forceinline__ float silu_grad(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

}  // namespace

// C[M][N] = op(A)[M][K] op(B)[K][N] for every ensemble member (grid z), BF16
// in, FP32 accumulate.  op(A)(i, k) = TA ? A[k lda + i] : A[i lda + k];
// op(B)(k, j) = TB ? B[j ldb + k] : B[k ldb + j].  M, N multiples of 16, K a
// multiple of 32, lda and ldb multiples of 8 (16-byte rows of 8 elements).
// A block of four waves computes a 64 x 64 tile of C, each wave a 32 x 32
// quarter as 2 x 2 MFMA tiles of 16 x 16 (v_mfma_f32_16x16x32_bf16: lane l
// holds A(l % 16, 8 (l / 16) + e) and B(8 (l / 16) + e, l % 16), e < 8, and
// ends with C(4 (l / 16) + r, l % 16), r < 4).  Per K step of 32 the block
// stages the 64 x 32 slices of op(A) and op(B)^T in LDS with 16-byte global
// loads (one per thread and operand), so every lane reads its 8 operands as
// one 16-byte LDS read; rows past M or N read a clamped row and are not
// stored.  Each output adds its K steps in order, as one MFMA chain.
constexpr int MM_T = 64;        // block tile
constexpr int MM_LDK = 32 + 8;  // LDS row of 32 k values, padded against bank conflicts

template <bool TA, bool TB, int EPI>
__global__ void __launch_bounds__(256) k_mm_bf16(int M, int N, int K, const __bf16* __restrict__ A, int lda,
                                                 int64_t sA, const __bf16* __restrict__ B, int ldb, int64_t sB,
                                                 const float* __restrict__ bias, int64_t sBias, float* __restrict__ Cf,
                                                 int ldc, int64_t sC, __bf16* __restrict__ Cb, int64_t sCb,
                                                 const float* __restrict__ Z, int64_t sZ) {
  __shared__ __align__(16) __bf16 As[MM_T][MM_LDK];  // op(A) rows i, k contiguous
  __shared__ __align__(16) __bf16 Bs[MM_T][MM_LDK];  // op(B) columns j, k contiguous
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  const int i0 = blockIdx.y * MM_T, j0 = blockIdx.x * MM_T;
  const int e_ = blockIdx.z;
  A += e_ * sA;
  B += e_ * sB;
  // staging: thread t moves 8 elements of each operand per K step
  //   k-contiguous source: row t / 4 of the tile, k = 8 (t % 4) .. + 8
  //   row-contiguous source: k = t / 8, rows 8 (t % 8) .. + 8
  const int r_kc = t >> 2, k_kc = 8 * (t & 3);
  const int k_rc = t >> 3, r_rc = 8 * (t & 7);
  const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
  f32x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < K; k0 += 32) {
    if (k0) __syncthreads();  // every wave is done with the previous slices
    if constexpr (!TA) {
      const int i = min(i0 + r_kc, M - 1);
      *reinterpret_cast<bf16x8*>(&As[r_kc][k_kc]) =
          *reinterpret_cast<const bf16x8*>(A + (int64_t)i * lda + k0 + k_kc);
    } else {
      const int i = min(i0 + r_rc, M - 8);  // M is a multiple of 16, so the 8 rows stay in range
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(A + (int64_t)(k0 + k_rc) * lda + i);
#pragma unroll
      for (int e = 0; e < 8; ++e) As[i - i0 + e < MM_T ? i - i0 + e : MM_T - 1][k_rc] = v[e];
    }
    if constexpr (TB) {
      const int j = min(j0 + r_kc, N - 1);
      *reinterpret_cast<bf16x8*>(&Bs[r_kc][k_kc]) =
          *reinterpret_cast<const bf16x8*>(B + (int64_t)j * ldb + k0 + k_kc);
    } else {
      const int j = min(j0 + r_rc, N - 8);
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(B + (int64_t)(k0 + k_rc) * ldb + j);
#pragma unroll
      for (int e = 0; e < 8; ++e) Bs[j - j0 + e < MM_T ? j - j0 + e : MM_T - 1][k_rc] = v[e];
    }
    __syncthreads();
    bf16x8 av[2], bv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) av[a] = *reinterpret_cast<const bf16x8*>(&As[wm + 16 * a + (l & 15)][8 * (l >> 4)]);
#pragma unroll
    for (int b = 0; b < 2; ++b) bv[b] = *reinterpret_cast<const bf16x8*>(&Bs[wn + 16 * b + (l & 15)][8 * (l >> 4)]);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[a], bv[b], acc[a][b], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int j = j0 + wn + 16 * b + (l & 15);
      if (j >= N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + wm + 16 * a + 4 * (l >> 4) + r;
        if (i >= M) continue;
        const int64_t o = (int64_t)i * ldc + j;
        const float v = acc[a][b][r];
        if constexpr (EPI == MM_HIDDEN) {  // z = v + b, keep z, emit SiLU(z) in BF16
          const float z = v + bias[e_ * sBias + j];
          Cf[e_ * sC + o] = z;
          Cb[e_ * sCb + o] = (__bf16)silu(z);
        } else if constexpr (EPI == MM_OUTPUT) {  // y = v + b
          Cf[e_ * sC + o] = v + bias[e_ * sBias + j];
        } else if constexpr (EPI == MM_DHIDDEN) {  // dz = v SiLU'(z), in FP32 and BF16
          const float dz = v * silu_grad(Z[e_ * sZ + o]);
          Cf[e_ * sC + o] = dz;
          Cb[e_ * sCb + o] = (__bf16)dz;
        } else {  // MM_PLAIN: weight gradient
          Cf[e_ * sC + o] = v;
        }
      }
    }
}

// x[B][n_in] (FP32) -> X[B][K0] (BF16, zero padded)
__global__ void k_pack_input(int B, int n_in, int K0, const float* __restrict__ x, __bf16* __restrict__ X) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)B * K0) return;
  const int i = (int)(t / K0), k = (int)(t - (int64_t)i * K0);
  X[t] = (__bf16)(k < n_in ? x[(int64_t)i * n_in + k] : 0.f);
}

// Squared error per (member, row) and dY = 2 (y - t) / (B n_out) in BF16: one
// wave per row (lanes over outputs, fixed-order wave sum), four rows a block
__global__ void __launch_bounds__(256) k_mse(int B, int n_out, const float* __restrict__ Y,
                                             const float* __restrict__ T, __bf16* __restrict__ dY,
                                             float* __restrict__ row_se) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int e = blockIdx.y;
  if (i >= B) return;  // whole wave
  const float sc = 2.0f / ((float)B * (float)n_out);
  const float* y = Y + ((int64_t)e * B + i) * n_out;
  const float* t = T + (int64_t)i * n_out;
  __bf16* d = dY + ((int64_t)e * B + i) * n_out;
  float se = 0.f;
  for (int j = lane; j < n_out; j += 64) {
    const float df = y[j] - t[j];
    se = fmaf(df, df, se);
    d[j] = (__bf16)(sc * df);
  }
  const double tot = wave_sum_f64((double)se);
  if (lane == 0) row_se[(int64_t)e * B + i] = (float)tot;
}

// one member's loss = sum of row_se / (B n_out), rows added in order by one
// block of 256 threads (strided partials, then a fixed tree)
__device__ __forceinline__ void loss_block(int B, int n_out, const float* __restrict__ row_se,
                                           float* __restrict__ loss, int e) {
  __shared__ float s[256];
  float a = 0.f;
  for (int i = threadIdx.x; i < B; i += 256) a += row_se[(int64_t)e * B + i];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[e] = s[0] / ((float)B * (float)n_out);
}

__global__ void __launch_bounds__(256) k_loss_sum(int B, int n_out, const float* __restrict__ row_se,
                                                  float* __restrict__ loss) {
  loss_block(B, n_out, row_se, loss, blockIdx.x);
}

// db[j] = sum_i D[i][j] per member, in two fixed-order stages: partial sums
// over chunks of SG_COLSUM_ROWS rows (block: 64 columns x 4 row phases,
// combined in phase order), then the chunks in order
__global__ void __launch_bounds__(256) k_colsum_part(int B, int N, const float* __restrict__ D, int64_t sD,
                                                     float* __restrict__ part) {
  __shared__ float s[4][64];
  const int col = blockIdx.x * 64 + (threadIdx.x & 63);
  const int g = threadIdx.x >> 6;
  const int c = blockIdx.y, e = blockIdx.z;
  const int r0 = c * SG_COLSUM_ROWS, r1 = min(B, r0 + SG_COLSUM_ROWS);
  float a = 0.f;
  if (col < N)
    for (int i = r0 + g; i < r1; i += 4) a += D[e * sD + (int64_t)i * N + col];
  s[g][threadIdx.x & 63] = a;
  __syncthreads();
  if (g == 0 && col < N) {
    const int l = threadIdx.x;
    part[((int64_t)e * gridDim.y + c) * N + col] = ((s[0][l] + s[1][l]) + s[2][l]) + s[3][l];
  }
}

__global__ void k_colsum_final(int n_chunks, int N, const float* __restrict__ part, float* __restrict__ db,
                               int64_t sdb) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int e = blockIdx.y;
  if (j >= N) return;
  float a = 0.f;
  for (int c = 0; c < n_chunks; ++c) a += part[((int64_t)e * n_chunks + c) * N + j];
  db[e * sdb + j] = a;
}

// dY (BF16) -> FP32 copy for the output-bias gradient
__global__ void k_bf16_to_f32(int64_t n, const __bf16* __restrict__ a, float* __restrict__ b) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) b[t] = (float)a[t];
}

struct AdamArgs {
  float lr, b1, b2, eps, c1, c2;
};

// the parameter after its Adam step (the contractions written out, so that every
// kernel rounds alike)
__device__ __forceinline__ float adam(const AdamArgs& a, float g, float p, float* m_, float* v_) {
  const float m = fmaf(1.0f - a.b1, g, a.b1 * *m_);
  const float v = fmaf((1.0f - a.b2) * g, g, a.b2 * *v_);
  *m_ = m;
  *v_ = v;
  const float mh = m / a.c1, vh = v / a.c2;
  return p - a.lr * mh / (sqrtf(vh) + a.eps);
}

// Fragment order of a BF16 matrix X[row][k] (rows a multiple of 16, K of 32):
// the 16 x 32 pieces that one MFMA reads, each in lane order (1 KiB that a wave
// loads as 16 bytes per lane), k steps of a row tile after one another.
__device__ __forceinline__ int64_t frag(int row, int64_t k, int64_t K) {
  return (int64_t)(row >> 4) * 16 * K + (k >> 5) * 512 + ((row & 15) + 16 * ((k >> 3) & 3)) * 8 + (k & 7);
}

// Eight rows of one column of a weight matrix, the unit of the BF16 copies (16
// bytes of the transposed one), or one bias.  Units of a network: the matrices'
// by row group and column, then the biases.
struct ParamUnit {
  int64_t at, step;  // first parameter, distance to the next row's
  int n;             // rows (1: a bias)
  int64_t bt;        // place of its eight in the transposed copy (-1: a bias)
  int64_t base;      // the matrix, its first row and column there, and its width
  int i, j, cols;
};
__host__ __device__ inline int64_t param_units(int H, int O) {
  return ((int64_t)SG_K0 * H + (int64_t)H * H + (int64_t)H * O) / 8 + 2 * H + O;
}
__device__ __forceinline__ ParamUnit param_unit(int64_t t, const SgLayout& L, int H, int O) {
  const int64_t per = param_units(H, O), e = t / per, m = e * L.n_params;
  int64_t u = t - e * per;
  const int rows[3] = {SG_K0, H, H}, cols[3] = {H, H, O};
  const int64_t at[3] = {L.W1, L.W2, L.W3};
#pragma unroll
  for (int w = 0; w < 3; ++w) {
    const int64_t n = (int64_t)rows[w] * cols[w] / 8;
    if (u < n) {
      const int i = 8 * (int)(u / cols[w]), j = (int)(u % cols[w]);
      const int64_t base = m + at[w];
      return ParamUnit{base + (int64_t)i * cols[w] + j, cols[w], 8, base + frag(j, i, rows[w]), base, i, j, cols[w]};
    }
    u -= n;
  }
  const int64_t b = u < H ? L.b1 + u : u < 2 * H ? L.b2 + (u - H) : L.b3 + (u - 2 * H);
  return ParamUnit{m + b, 0, 1, -1, 0, 0, 0, 0};
}
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8p;

// The BF16 copies of a unit's weights: transposed in fragment order (the row
// kernel's forward products), and in fragment order (bfrag) or as they lie
__device__ __forceinline__ void put_bf16(const ParamUnit& q, int bfrag, const float (&v)[8], __bf16* __restrict__ b,
                                         __bf16* __restrict__ bt) {
  if (q.bt < 0) return;  // biases are read in FP32
  bf16x8p x;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    x[r] = (__bf16)v[r];
    b[bfrag ? q.base + frag(q.i + r, q.j, q.cols) : q.at + r * q.step] = x[r];
  }
  if (bt) *reinterpret_cast<bf16x8p*>(bt + q.bt) = x;
}

// Adam on the FP32 masters (all members), then the BF16 copies.  (A thread per
// parameter wrote the transposed copy 2 bytes at a time: 59 us for 4 networks of
// 1536 hidden units and 32 outputs, 47 so; 41 without that copy, which
// networks that never use it are spared: bt null.)
__global__ void k_adam(int64_t n, AdamArgs a, SgLayout L, int H, int O, int bfrag, float* __restrict__ P,
                       const float* __restrict__ G, float* __restrict__ Mm, float* __restrict__ Vm,
                       __bf16* __restrict__ Pb, __bf16* __restrict__ PbT) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const ParamUnit q = param_unit(t, L, H, O);
  float g[8], p[8], m[8], v[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int64_t o = q.at + min(r, q.n - 1) * q.step;
    g[r] = G[o];
    p[r] = P[o];
    m[r] = Mm[o];
    v[r] = Vm[o];
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    p[r] = adam(a, g[r], p[r], &m[r], &v[r]);
    if (r < q.n) {
      const int64_t o = q.at + r * q.step;
      P[o] = p[r];
      Mm[o] = m[r];
      Vm[o] = v[r];
    }
  }
  put_bf16(q, bfrag, p, Pb, PbT);
}

__global__ void k_f32_to_bf16(int64_t n, SgLayout L, int H, int O, int bfrag, const float* __restrict__ a,
                              __bf16* __restrict__ b, __bf16* __restrict__ bt) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const ParamUnit q = param_unit(t, L, H, O);
  if (q.bt < 0) return;
  float v[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = a[q.at + r * q.step];
  put_bf16(q, bfrag, v, b, bt);
}

// ---- row kernels: a network in one launch, its gradients in another ----------
//
// Everything but the weight gradients is local to a row of the batch: the three
// layers, the output error and the two back-propagated layers.  A block takes
// 16 MT rows of one member through all of them, activations in LDS, weights
// read from L2 as the MFMA's B operand, whole cache lines in fragment order.
// What the weight gradients need goes out transposed in the same order, so that
// k_sg_grads reads both operands straight into registers; it also updates the
// parameters.
// Every output is one MFMA chain over k in steps of 32, as in the general
// kernels, and the column sums keep their order.
// Bound by launches and latency at the usual sizes: a step of batch 512, hidden
// 256, 128 outputs and 4 members takes 17 us of rows (about 3.5 of them before the
// first product, 2 a layer, of those 1.5 of VALU work on two waves' SiLUs) and 12
// of gradients, 31 us in all against 139 as 20 launches; batch 4096, 96 against
// 460.  Row-major weights (64-byte pieces at power-of-two strides) took 26 and
// 27 us, eight waves a block 19.
// Waves per block: 16 in training, 8 in inference; 2 in inference of many rows
// where every layer's columns fit in two waves' tiles (the others would idle: 8
// networks of 32 hidden units, 20000 rows, 43 us with 8 waves, 25 so).  Of
// few rows the waves past the columns still help to stage them: below
// SR_NARROW_ROWS rows of all networks 8 waves (2048 rows of 8 networks 12.4 us
// by 13.4 with 2).
constexpr int SR_TRAIN = 16, SR_INFER = 8, SR_NARROW = 2;
constexpr int SR_NARROW_COLS = SR_NARROW * 2 * 16, SR_NARROW_ROWS = 49152;
constexpr int SR_MT = 2;  // row tiles per block of large inference batches

namespace {

struct SgRows {
  int B, n_in, H, O;
  SgLayout L;
  const float* x;
  const float* target;
  const float* P;
  const __bf16 *Pb, *PbT;
  float* Y;  // inference: [E][B][O]
  // training
  __bf16 *XT, *H1T, *H2T, *dYT, *dZ2T, *dZ1T;  // [E][width][B] (XT: one for all members)
  float *dYf, *dZ2f, *dZ1f;                    // [E][B][width]
  float* row_se;                               // [E][B]
};

// bytes of LDS of a block of R rows
size_t sg_rows_lds(int R, int H, int O, bool train) {
  size_t b = 2 * ((size_t)R * (SG_K0 + 8) + 2 * (size_t)R * (H + 8)) + 4 * (size_t)(2 * H + O);
  if (train) b += 2 * (size_t)R * (O + 8) + 4 * (2 * (size_t)R * (H + 4) + (size_t)R * (O + 4));
  return b;
}

typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;

// Barrier for data that passes through LDS: unlike __syncthreads it does not
// wait for the global loads and stores in flight, the next layer's weights
// among them.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A wave's weights of NT column tiles over SR_S k steps (past K the last step
// is read again and not used)
constexpr int SR_S = 8;
template <int NT>
struct RowsB {
  bf16x8 v[SR_S][NT];
};

template <int NT>
__device__ __forceinline__ void rows_load(RowsB<NT>& o, const __bf16* __restrict__ Bf, int K, int t, int k0) {
  const __bf16* bp = Bf + (int64_t)t * 16 * K + 8 * (threadIdx.x & 63);
#pragma unroll
  for (int s = 0; s < SR_S; ++s)
#pragma unroll
    for (int n = 0; n < NT; ++n)
      o.v[s][n] = *reinterpret_cast<const bf16x8*>(bp + n * 16 * K + 16 * min(k0 + 32 * s, K - 32));
}

// the first weights that rows_mm uses: loaded one layer ahead, so that their
// latency is spent under the layer before (waves past N load tile 0)
template <int NT>
__device__ __forceinline__ void rows_first(RowsB<NT>& o, const __bf16* Bf, int K, int N) {
  const int t = NT * __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  rows_load(o, Bf, K, 16 * t < N ? t : 0, 0);
}

// out[16 MT][N] = As[16 MT][K] B[N][K]^T for the block's rows, B in fragment
// order, NT column
// tiles at a time per wave of W (N is a multiple of 32).  next() runs after the
// wave's last product, before its results are stored: loads that it issues don't
// queue behind those stores.  ep(row, column, values of
// rows row .. row + 3).
template <int MT, int NT, int W, bool PRE, typename NEXT, typename EP>
__device__ __forceinline__ void rows_mm(RowsB<NT>& first, const __bf16* As, int lda, const __bf16* __restrict__ Bf, int K,
                                        int N, NEXT&& next, EP&& ep) {
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int c = l & 15, q = 4 * (l >> 4);
  const __bf16* ap = As + c * lda + 2 * q;
  if (16 * NT * w >= N) next();
  for (int t = NT * w; 16 * t < N; t += NT * W) {
    f32x4 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < K; k0 += 32 * SR_S) {
      if (!PRE || t != NT * w || k0) rows_load(first, Bf, K, t, k0);
#pragma unroll
      for (int s = 0; s < SR_S; ++s) {
        if (k0 + 32 * s >= K) break;
        bf16x8 av[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) av[m] = *reinterpret_cast<const bf16x8*>(ap + m * 16 * lda + k0 + 32 * s);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int n = 0; n < NT; ++n)
            acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[m], first.v[s][n], acc[m][n], 0, 0, 0);
      }
    }
    if (16 * (t + NT * W) >= N) next();
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < NT; ++n) ep(16 * m + q, 16 * (t + n) + c, acc[m][n]);
  }
}

}  // namespace

template <int MT, bool TRAIN, int W>
__global__ void __launch_bounds__(64 * W, MT == 1 ? 1 : 4) k_sg_rows(SgRows a) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int R = 16 * MT;
  constexpr int NT = TRAIN ? 1 : 2;  // column tiles at a time per wave
  constexpr bool PRE = MT == 1;
  const int H = a.H, O = a.O, B = a.B, e = blockIdx.y;
  const int ldx = SG_K0 + 8, ldh = H + 8, ldo = O + 8, ldz = H + 4, ldd = O + 4;
  __bf16* Xs = reinterpret_cast<__bf16*>(lds);
  __bf16* H1s = Xs + R * ldx;
  __bf16* H2s = H1s + R * ldh;
  float* bias = reinterpret_cast<float*>(H2s + R * ldh);   // b1, b2, b3
  __bf16* dYs = reinterpret_cast<__bf16*>(bias + 2 * H + O);  // training only, as are the next three
  float* Z1 = reinterpret_cast<float*>(dYs + R * ldo);
  float* Z2 = Z1 + R * ldz;
  float* Df = Z2 + R * ldz;                               // the targets, then the errors
  __bf16* dZ2s = H1s;                                    // layer 2 is done with H1 by then
  const int64_t r0 = (int64_t)blockIdx.x * R;
  const float* P = a.P + e * a.L.n_params;
  const __bf16* Pb = a.Pb + e * a.L.n_params;
  const __bf16* PbT = a.PbT + e * a.L.n_params;
  RowsB<NT> wa, wb;
  auto first = [](RowsB<NT>& o, const __bf16* Bf, int K, int N) {
    return [&, Bf, K, N] {
      if (PRE && N) rows_first(o, Bf, K, N);
    };
  };
  first(wa, PbT + a.L.W1, SG_K0, H)();
  first(wb, PbT + a.L.W2, H, H)();
  // the inputs, zero padded to one k step; rows past the batch repeat its last
  for (int t = threadIdx.x; t < R * SG_K0; t += 64 * W) {
    const int i = t / SG_K0, k = t - i * SG_K0;
    const int64_t row = min(r0 + i, (int64_t)B - 1);
    Xs[i * ldx + k] = (__bf16)(k < a.n_in ? a.x[row * a.n_in + k] : 0.f);
  }
  for (int t = threadIdx.x; t < 2 * H + O; t += 64 * W)
    bias[t] = P[t < H ? a.L.b1 + t : t < 2 * H ? a.L.b2 + t - H : a.L.b3 + t - 2 * H];
  if constexpr (TRAIN)
    for (int t = threadIdx.x; t < R * O; t += 64 * W) {
      const int i = t / O, j = t - i * O;
      Df[i * ldd + j] = a.target[(r0 + i) * O + j];
    }
  lds_barrier();
  if constexpr (TRAIN) {
    if (e == 0)
      for (int t = threadIdx.x; t < R * SG_K0; t += 64 * W) {
        const int k = t / R, i = t - k * R;
        a.XT[frag(k, r0 + i, B)] = Xs[i * ldx + k];
      }
  }
  auto column = [&](__bf16* T, int width, int col, int row, bf16x4 v) {  // rows row .. row + 3 of a transposed matrix
    *reinterpret_cast<bf16x4*>(T + (int64_t)e * width * B + frag(col, r0 + row, B)) = v;
  };
  auto hidden = [&](const float* bv, float* Z, __bf16* Hs, __bf16* HT) {
    return [=](int row, int col, f32x4 v) {
      const float b = bv[col];
      bf16x4 h;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float z = v[r] + b;
        h[r] = (__bf16)silu(z);
        Hs[(row + r) * ldh + col] = h[r];
        if constexpr (TRAIN) Z[(row + r) * ldz + col] = z;
      }
      if constexpr (TRAIN) column(HT, H, col, row, h);
    };
  };
  rows_mm<MT, NT, W, PRE>(wa, Xs, ldx, PbT + a.L.W1, SG_K0, H, first(wa, PbT + a.L.W3, H, O), hidden(bias, Z1, H1s, a.H1T));
  lds_barrier();
  rows_mm<MT, NT, W, PRE>(wb, H1s, ldh, PbT + a.L.W2, H, H, first(wb, Pb + a.L.W3, O, TRAIN ? H : 0), hidden(bias + H, Z2, H2s, a.H2T));
  lds_barrier();
  const float* b3 = bias + 2 * H;
  if constexpr (!TRAIN) {
    rows_mm<MT, NT, W, PRE>(wa, H2s, ldh, PbT + a.L.W3, H, O, [] {}, [=](int row, int col, f32x4 v) {
      if (r0 + __builtin_amdgcn_readfirstlane(row & ~15) >= B) return;  // uniform: the batch is a multiple of 16
      const float b = b3[col];
      float* y = a.Y + ((int64_t)e * B + r0 + row) * O + col;
#pragma unroll
      for (int r = 0; r < 4; ++r) y[(int64_t)r * O] = v[r] + b;
    });
  } else {
    const float sc = 2.0f / ((float)B * (float)O);
    rows_mm<MT, NT, W, PRE>(wa, H2s, ldh, PbT + a.L.W3, H, O, first(wa, Pb + a.L.W2, H, H), [=](int row, int col, f32x4 v) {
      const float b = b3[col];
      bf16x4 d;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float y = v[r] + b;
        const float df = y - Df[(row + r) * ldd + col];
        d[r] = (__bf16)(sc * df);
        Df[(row + r) * ldd + col] = df;
        dYs[(row + r) * ldo + col] = d[r];
        a.dYf[((int64_t)e * B + r0 + row + r) * O + col] = (float)d[r];
      }
      column(a.dYT, O, col, row, d);
    });
    lds_barrier();
    // squared error of each row, one wave per row
    for (int i = threadIdx.x >> 6; i < R; i += W) {
      const int lane = threadIdx.x & 63;
      float se = 0.f;
      for (int j = lane; j < O; j += 64) {
        const float df = Df[i * ldd + j];
        se = fmaf(df, df, se);
      }
      const double tot = wave_sum_f64((double)se);
      if (lane == 0) a.row_se[(int64_t)e * B + r0 + i] = (float)tot;
    }
    // dZ2 = (dY W3^T) SiLU'(Z2), dZ1 = (dZ2 W2^T) SiLU'(Z1)
    rows_mm<MT, NT, W, PRE>(wb, dYs, ldo, Pb + a.L.W3, O, H, [] {}, [=](int row, int col, f32x4 v) {
      bf16x4 d;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float dz = v[r] * silu_grad(Z2[(row + r) * ldz + col]);
        d[r] = (__bf16)dz;
        dZ2s[(row + r) * ldh + col] = d[r];
        a.dZ2f[((int64_t)e * B + r0 + row + r) * H + col] = dz;
      }
      column(a.dZ2T, H, col, row, d);
    });
    lds_barrier();
    rows_mm<MT, NT, W, PRE>(wa, dZ2s, ldh, Pb + a.L.W2, H, H, [] {}, [=](int row, int col, f32x4 v) {
      bf16x4 d;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float dz = v[r] * silu_grad(Z1[(row + r) * ldz + col]);
        d[r] = (__bf16)dz;
        a.dZ1f[((int64_t)e * B + r0 + row + r) * H + col] = dz;
      }
      column(a.dZ1T, H, col, row, d);
    });
  }
}

namespace {

struct SgGrads {
  int B, H, O;
  SgLayout L;
  const __bf16 *XT, *H1T, *H2T, *dYT, *dZ2T, *dZ1T;
  const float *dYf, *dZ2f, *dZ1f, *row_se;
  float *P, *G, *M, *V, *loss;
  __bf16 *Pb, *PbT;
  AdamArgs adam;
  int blk_w, blk_b;  // blocks of weight tiles, then of bias columns, then one for the loss
};

constexpr int SG_S = 4, SG_D = 3;  // weight gradients: k steps per set, sets in flight
// bias columns of one block
constexpr int SG_BIAS_COLS = 16;

// Sum over rows of 16 columns of D[B][N] and the bias update.  Rows are taken
// in chunks of SG_COLSUM_ROWS, a chunk in four interleaved phases: lane 16 g + j
// adds phase g of column j, a wave per chunk; phases, then chunks, in order.
__device__ __forceinline__ void bias_step(const SgGrads& a, int e, const float* __restrict__ D, int N, int col0,
                                          int64_t off) {
  __shared__ float s_part[4][SG_BIAS_COLS];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = l & 15, g = l >> 4;
  const int n_chunks = (a.B + SG_COLSUM_ROWS - 1) / SG_COLSUM_ROWS;
  const float* src = D + (int64_t)e * a.B * N + col0 + j;
  const int64_t o = e * a.L.n_params + off + col0 + j;
  const float p_ = a.P[o];  // the optimiser state, loaded ahead of the sums
  float m_ = a.M[o], v_ = a.V[o], sum = 0.f;
  for (int c0 = 0; c0 < n_chunks; c0 += 4) {
    const int r0 = (c0 + w) * SG_COLSUM_ROWS, r1 = min(a.B, r0 + SG_COLSUM_ROWS);
    float p = 0.f;
    constexpr int U = SG_COLSUM_ROWS / 4;
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = src[(int64_t)min(r0 + g + 4 * u, a.B - 1) * N];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r0 + g + 4 * u < r1) p += v[u];
    const float p0 = __shfl(p, j, 64), p1 = __shfl(p, j + 16, 64), p2 = __shfl(p, j + 32, 64),
                p3 = __shfl(p, j + 48, 64);
    if (l < SG_BIAS_COLS) s_part[w][j] = ((p0 + p1) + p2) + p3;
    __syncthreads();
    for (int c = 0; c < min(4, n_chunks - c0); ++c) sum += s_part[c][j];
    __syncthreads();
  }
  if (threadIdx.x >= SG_BIAS_COLS) return;
  a.P[o] = adam(a.adam, sum, p_, &m_, &v_);
  a.M[o] = m_;
  a.V[o] = v_;
  a.G[o] = sum;
}

}  // namespace

// Weight gradients dW[i][j] = sum_b AT[i][b] DT[j][b] and the parameters'
// Adam step.  A wave makes a 16 x 32 tile, all operands in registers (8 k steps
// of 16-byte loads in flight); bias columns and the loss have blocks of their
// own in the same launch.
__global__ void __launch_bounds__(256) k_sg_grads(SgGrads a) {
  const int e = blockIdx.y, H = a.H, O = a.O, B = a.B;
  int b = blockIdx.x;
  if (b >= a.blk_w) {
    b -= a.blk_w;
    if (b < a.blk_b) {
      const int nh = H / SG_BIAS_COLS;
      if (b < nh) bias_step(a, e, a.dZ1f, H, b * SG_BIAS_COLS, a.L.b1);
      else if (b < 2 * nh) bias_step(a, e, a.dZ2f, H, (b - nh) * SG_BIAS_COLS, a.L.b2);
      else bias_step(a, e, a.dYf, O, (b - 2 * nh) * SG_BIAS_COLS, a.L.b3);
    } else {
      loss_block(B, O, a.row_se, a.loss, e);
    }
    return;
  }
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int t = 4 * b + w;  // wave tile: W2, then W3, then W1
  const int n2 = (H / 16) * (H / 32), n3 = (H / 16) * (O / 32), n1 = (SG_K0 / 16) * (H / 32);
  const __bf16 *AT, *DT;
  int M, N;
  int64_t off;
  if (t < n2) {
    AT = a.H1T + (int64_t)e * H * B, DT = a.dZ2T + (int64_t)e * H * B, M = H, N = H, off = a.L.W2;
  } else if (t < n2 + n3) {
    t -= n2;
    AT = a.H2T + (int64_t)e * H * B, DT = a.dYT + (int64_t)e * O * B, M = H, N = O, off = a.L.W3;
  } else if (t < n2 + n3 + n1) {
    t -= n2 + n3;
    AT = a.XT, DT = a.dZ1T + (int64_t)e * H * B, M = SG_K0, N = H, off = a.L.W1;
  } else {
    return;
  }
  const int i0 = 16 * (t / (N / 32)), j0 = 32 * (t % (N / 32));
  const int c = l & 15, q = 4 * (l >> 4);
  const __bf16* ap = AT + (int64_t)i0 * B + 8 * l;
  const __bf16* dp = DT + (int64_t)j0 * B + 8 * l;
  // the optimiser state of the tile, loaded before the product
  const int64_t base = e * a.L.n_params + off;
  float p_[2][4], m_[2][4], v_[2][4];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t o = base + (int64_t)(i0 + q + r) * N + j0 + 16 * n + c;
      p_[n][r] = a.P[o];
      m_[n][r] = a.M[o];
      v_[n][r] = a.V[o];
    }
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  // a ring of SG_D sets of SG_S k steps (past the batch the last step again)
  struct Set {
    bf16x8 a[SG_S], d[SG_S][2];
  };
  auto load = [&](Set& o, int k0) {
#pragma unroll
    for (int s = 0; s < SG_S; ++s) {
      const int64_t k = 16 * (int64_t)min(k0 + 32 * s, B - 32);
      o.a[s] = *reinterpret_cast<const bf16x8*>(ap + k);
      o.d[s][0] = *reinterpret_cast<const bf16x8*>(dp + k);
      o.d[s][1] = *reinterpret_cast<const bf16x8*>(dp + (int64_t)16 * B + k);
    }
  };
  Set o[SG_D];
#pragma unroll
  for (int d = 0; d + 1 < SG_D; ++d) load(o[d], 32 * SG_S * d);
  for (int k0 = 0; k0 < B; k0 += 32 * SG_S * SG_D) {
#pragma unroll
    for (int d = 0; d < SG_D; ++d) {
      load(o[(d + SG_D - 1) % SG_D], k0 + 32 * SG_S * (d + SG_D - 1));
#pragma unroll
      for (int s = 0; s < SG_S; ++s) {
        if (k0 + 32 * (SG_S * d + s) >= B) break;
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o[d].a[s], o[d].d[s][0], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o[d].a[s], o[d].d[s][1], acc[1], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int j = j0 + 16 * n + c;
    bf16x4 pb;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t o = base + (int64_t)(i0 + q + r) * N + j;
      const float p = adam(a.adam, acc[n][r], p_[n][r], &m_[n][r], &v_[n][r]);
      pb[r] = (__bf16)p;
      a.G[o] = acc[n][r];
      a.M[o] = m_[n][r];
      a.V[o] = v_[n][r];
      a.P[o] = p;
      a.Pb[base + frag(i0 + q + r, j, N)] = pb[r];
    }
    *reinterpret_cast<bf16x4*>(a.PbT + base + frag(j, i0 + q, M)) = pb;
  }
}

// ensemble mean of the outputs (members added in order)
__global__ void k_ens_mean(int64_t n, int E, const float* __restrict__ Y, float* __restrict__ mean) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  float m = 0.f;
  for (int e = 0; e < E; ++e) m += Y[(int64_t)e * n + t];
  mean[t] = m / (float)E;
}

// per sample: RV of the mean prediction, calib x sample standard deviation
// of the members' RVs, and the fallback flag
__global__ void k_gate(int64_t n, int E, double calib, double thr, const soap_rv* __restrict__ rv,
                       double* __restrict__ rv_kms, double* __restrict__ err_kms, int* __restrict__ fallback) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  bool bad = rv[i].status != 0;
  double m = 0.0;
  for (int e = 0; e < E; ++e) {
    const soap_rv& r = rv[(1 + e) * n + i];
    bad = bad || r.status != 0;
    m += r.rv_kms;
  }
  m /= (double)E;
  double v = 0.0;
  for (int e = 0; e < E; ++e) {
    const double d = rv[(1 + e) * n + i].rv_kms - m;
    v += d * d;
  }
  const double err = calib * sqrt(v / (double)(E - 1));
  rv_kms[i] = rv[i].rv_kms;
  if (err_kms) err_kms[i] = err;
  fallback[i] = (bad || !(err < thr)) ? 1 : 0;
}

// Network inputs of one sample from its raw description r = (lat, lon,
// radius, contrast, phase, T_eff, inclination, v sin i) in degrees, R*, K
// and km/s: the spot latitude scaled to +-60 deg, the sine and cosine of
// its rotated longitude, its centre on the sky (x, y, z; y up the projected
// axis, z towards the observer), and the scalar parameters centred and
// scaled over their sampled ranges, then a constant 1.
__global__ void __launch_bounds__(256) k_features(int64_t n, const double* __restrict__ raw, float* __restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double* r = raw + i * SG_RAW;
  constexpr double D2R = 3.14159265358979323846 / 180.0;
  const double lat = r[0] * D2R;
  const double th = (r[1] + 360.0 * r[4]) * D2R;
  const double inc = r[6] * D2R;
  const double cl = cos(lat), sl = sin(lat), st = sin(th), ct = cos(th), si = sin(inc), ci = cos(inc);
  float* o = x + i * SG_FEATURES;
  o[0] = (float)(lat / (60.0 * D2R));
  o[1] = (float)st;
  o[2] = (float)ct;
  o[3] = (float)(cl * st);
  o[4] = (float)(sl * si - cl * ct * ci);
  o[5] = (float)(sl * ci + cl * ct * si);
  o[6] = (float)((r[2] - 0.055) / 0.045);
  o[7] = (float)((r[3] - 0.6) / 0.3);
  o[8] = (float)((r[5] - 5500.0) / 1000.0);
  o[9] = (float)((r[6] - 60.0) / 30.0);
  o[10] = (float)((r[7] - 3.0) / 2.0);
  o[11] = 1.0f;
}

// coef[n][k] = sum_p (D[n][p] - mean[p]) V[p][k] (mean row mean_idx[n] when
// given), FP32 on the matrix cores (v_mfma_f32_16x16x4_f32).  A block of PCA_W
// waves makes a tile of 16 MT rows x 64 components; the waves split the pixels
// (16 at a time, in turn, so a block reads its rows in contiguous stretches)
// and their partial tiles are added in wave order through LDS, so results
// repeat bit for bit.  Lane l holds, for row l % 16, the four pixels
// 4 (l / 16) + s of a step's 16 (one 16-byte load; MFMA s takes pixel s of
// every lane) and, for each of those pixels, the components 4 (l % 16) + c
// (one 16-byte load of a row of V; component tile c).
// Bound by the FP32 matrix rate (16 MFMAs of 32 cycles per step and wave) and
// the loads of V from L2 (every row tile reads its 64 columns of V).  2048
// rows x 20000 pixels x 128 components: 126 us (83 TFLOP/s; a large FP32
// matrix product reaches 149), against 4.85 ms as 64 x 64 tiles on 64 blocks
// with vector FMAs; 8192 rows: 482 us.  Sixteen waves per block take 139 us,
// two steps in flight 125 us, and a step that subtracts the mean as it loads
// (so that every load is waited for at once) 209 us.
constexpr int PCA_W = 8;   // waves per block
constexpr int PCA_N = 64;   // components per block
constexpr int PCA_D = 3;   // steps of 16 pixels in flight per wave

typedef float pca_f4 __attribute__((ext_vector_type(4), aligned(4)));  // any element alignment

// C4 (k at least 4): 16-byte loads from the rows of V; a lane that would pass k
// takes the last four components, and keeps those that are its own.
// SPLIT: the waves of a block split the pixels of one row tile; else (many rows of
// few pixels, where a wave had two or three steps and the block its sums to add:
// 100000 rows, 161 pixels, 256 components 286 us) each takes a tile of its own,
// and all pixels of it, 129 us.  There 16-row tiles are as fast as 32 or faster
// while D fits in the 256 MiB cache.
template <int MT, bool C4, bool SPLIT>
__global__ void __launch_bounds__(64 * PCA_W) k_pca_project(int n, int P, int k, const float* __restrict__ D,
                                                            int64_t ldd, const float* __restrict__ mean,
                                                            const int* __restrict__ mean_idx, int n_mean,
                                                            const float* __restrict__ V, float* __restrict__ coef) {
  __shared__ float s_part[PCA_W / 2][16 * MT][PCA_N + 4];
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // rows on x: up to 2^25 / 16 blocks
  const int64_t r0 = (SPLIT ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * PCA_W + w) * 16 * MT;
  const int c0 = blockIdx.y * PCA_N;
  constexpr int NW = SPLIT ? PCA_W : 1;  // waves of a row tile
  const int first = SPLIT ? w : 0;
  if (r0 >= n) return;  // never when SPLIT
  const int lk = 4 * (l >> 4), lc = c0 + 4 * (l & 15);
  const int cl = C4 ? min(lc, k - 4) : lc;  // the lane's first component
  const bool own = !C4 || cl == lc;         // all four are its own
  const float* drow[MT];
  const float* mrow[MT];
#pragma unroll
  for (int a = 0; a < MT; ++a) {
    const int64_t row = min(r0 + 16 * a + (l & 15), (int64_t)n - 1);  // rows past n are not stored
    const int mi = mean_idx ? mean_idx[row] : 0;
    drow[a] = D + row * ldd + lk;
    mrow[a] = lk + mean + (int64_t)(mi >= 0 && mi < n_mean ? mi : 0) * P;  // no such centre: NaN at the store
  }
  unsigned vo[4];  // the lane's part of its offsets in V
#pragma unroll
  for (int c = 0; c < 4; ++c) vo[c] = (unsigned)lk * k + min(cl + c, k - 1);
  f32x4 acc[MT][4];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[a][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Loads keep their raw values until they are used, PCA_D - 1 steps later, and
  // are unconditional (past the wave's last whole step they repeat it), so
  // that nothing waits for them early.
  struct Step {
    pca_f4 d[MT], m[MT], v[4];  // v[s][c]: pixel s, component c
  };
  auto load = [&](Step& o, int p) {
#pragma unroll
    for (int a = 0; a < MT; ++a) {
      o.d[a] = *reinterpret_cast<const pca_f4*>(drow[a] + p);
      o.m[a] = *reinterpret_cast<const pca_f4*>(mrow[a] + p);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const float* vr = V + (int64_t)(p + s) * k;
      if constexpr (C4) {
        o.v[s] = *reinterpret_cast<const pca_f4*>(vr + vo[0]);
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) o.v[s][c] = vr[vo[c]];
      }
    }
  };
  auto multiply = [&](const Step& o, f32x4 (&to)[MT][4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          to[a][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.d[a][s] - o.m[a][s], o.v[s][c], to[a][c], 0, 0, 0);
  };
  auto add = [&](f32x4 (&to)[MT][4], const f32x4 (&x)[MT][4]) {
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c) to[a][c] += x[a][c];
  };
  // A wave that has all pixels of its tile would round more in one chain than
  // the split's eight do (2.3e-8 against 1.0e-8 of outputs of 0.1 for 161 pixels,
  // 5.1e-8 against 1.9e-8 for 800): each step's products are a sum of their own
  // there, and PCA_D of those are added before they go to the tile's
  // (0.94e-8 and 1.1e-8).
  auto take = [&](const Step& o, f32x4 (&to)[MT][4]) {
    if constexpr (SPLIT) {
      multiply(o, acc);
    } else {
      f32x4 x[MT][4] = {};
      multiply(o, x);
      add(to, x);
    }
  };
  // whole steps of 16 pixels: step i of the wave starts at pixel 16 (first + NW i)
  const int steps = P / 16;
  const int mine = (steps - first + NW - 1) / NW;
  // past them, a tile's only wave takes the last 16 pixels, if there are as many,
  // and leaves out those that it has had: loads without a branch or a wait
  const bool rest16 = !SPLIT && P % 16 && P > 16;
  Step tail;
  if (rest16) load(tail, P - 16);
  if (mine > 0) {
    Step o[PCA_D];
    auto at = [&](int i) { return 16 * (first + NW * min(i, mine - 1)); };
#pragma unroll
    for (int d = 0; d + 1 < PCA_D; ++d) load(o[d], at(d));
    for (int i0 = 0; i0 < mine; i0 += PCA_D) {
      f32x4 group[MT][4] = {};
#pragma unroll
      for (int d = 0; d < PCA_D; ++d) {
        load(o[(d + PCA_D - 1) % PCA_D], at(i0 + d + PCA_D - 1));
        if (i0 + d < mine) take(o[d], group);
      }
      if constexpr (!SPLIT) add(acc, group);
    }
  }
  if (rest16) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool in = lk + s >= 16 - P % 16;
#pragma unroll
      for (int a = 0; a < MT; ++a) {
        tail.d[a][s] = in ? tail.d[a][s] : 0.f;
        tail.m[a][s] = in ? tail.m[a][s] : 0.f;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) tail.v[s][c] = in ? tail.v[s][c] : 0.f;
    }
    take(tail, acc);
  } else if (P % 16 && first == steps % NW) {  // the rest, by the wave whose turn it is: pixels past P are zeros
    Step o;
    const int p = 16 * steps;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool in = p + lk + s < P;
#pragma unroll
      for (int a = 0; a < MT; ++a) {
        o.d[a][s] = in ? drow[a][p + s] : 0.f;
        o.m[a][s] = in ? mrow[a][p + s] : 0.f;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) o.v[s][c] = in ? V[(int64_t)(p + s) * k + vo[c]] : 0.f;
    }
    take(o, acc);
  }
  // partial tiles: lane l ends with row 4 (l / 16) + r, component 4 (l % 16) + c.
  if constexpr (!SPLIT) {
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = r0 + 16 * a + 4 * (l >> 4) + r;
        if (row >= n) continue;
        const int mi = mean_idx ? mean_idx[row] : 0;
        const bool bad = mi < 0 || mi >= n_mean;
        pca_f4 v;
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = bad ? __builtin_nanf("") : acc[a][c][r];
        float* o = coef + row * k + cl;
        if (C4 && own) {
          *reinterpret_cast<pca_f4*>(o) = v;
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (cl + c >= lc && cl + c < k) o[c] = v[c];
        }
      }
    return;
  }
  // The upper half of the waves hands its tiles to the lower half, which adds
  // them to its own; then every output adds the PCA_W / 2 sums in order.
  auto put = [&](int slot) {
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) s_part[slot][16 * a + 4 * (l >> 4) + r][4 * (l & 15) + c] = acc[a][c][r];
  };
  if (w >= PCA_W / 2) put(w - PCA_W / 2);
  __syncthreads();
  if (w < PCA_W / 2) {
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c][r] += s_part[w][16 * a + 4 * (l >> 4) + r][4 * (l & 15) + c];
    put(w);  // each lane rewrites the slots it has just read
  }
  __syncthreads();
  for (int t = threadIdx.x; t < 16 * MT * PCA_N; t += 64 * PCA_W) {
    const int i = t / PCA_N, j = t - i * PCA_N;
    const int past = C4 ? max(c0 + (j & ~3) + 4 - k, 0) : 0;  // components of the lane's four that lie before its own
    const int at = min(j + past, PCA_N - 1);                  // (past k: not stored)
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < PCA_W / 2; ++q) v += s_part[q][i][at];
    const int64_t row = r0 + i;
    if (row >= n || c0 + j >= k) continue;
    const int mi = mean_idx ? mean_idx[row] : 0;
    coef[row * k + c0 + j] = (mi < 0 || mi >= n_mean) ? __builtin_nanf("") : v;
  }
}

// ---- launchers -------------------------------------------------------------

namespace {

template <bool TA, bool TB, int EPI>
hipError_t mm(hipStream_t st, int E, int M, int N, int K, const __bf16* A, int lda, int64_t sA, const __bf16* B,
              int ldb, int64_t sB, const float* bias, int64_t sBias, float* Cf, int ldc, int64_t sC, __bf16* Cb,
              int64_t sCb, const float* Z, int64_t sZ) {
  if (M % 16 || N % 16 || K % 32 || lda % 8 || ldb % 8) return hipErrorInvalidValue;
  dim3 grid((N + MM_T - 1) / MM_T, (M + MM_T - 1) / MM_T, E);
  hipLaunchKernelGGL((k_mm_bf16<TA, TB, EPI>), grid, dim3(256), 0, st, M, N, K, A, lda, sA, B, ldb, sB, bias,
                     sBias, Cf, ldc, sC, Cb, sCb, Z, sZ);
  return hipGetLastError();
}

inline dim3 blocks(int64_t n, int t = 256) { return dim3((unsigned)((n + t - 1) / t)); }

hipError_t colsum(hipStream_t st, int E, int B, int N, const float* D, int64_t sD, float* part, float* db,
                  int64_t sdb) {
  const int nc = (B + SG_COLSUM_ROWS - 1) / SG_COLSUM_ROWS;
  hipLaunchKernelGGL(k_colsum_part, dim3((N + 63) / 64, nc, E), dim3(256), 0, st, B, N, D, sD, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_colsum_final, dim3((N + 255) / 256, E), dim3(256), 0, st, nc, N, part, db, sdb);
  return hipGetLastError();
}

}  // namespace

#define SG_TRY(x)                              \
  do {                                         \
    hipError_t e_ = (x);                       \
    if (e_ != hipSuccess) return e_;           \
  } while (0)

hipError_t sg_forward(soap_surrogate* s, const float* x, int B) {
  const SgLayout& L = s->lay;
  const int E = s->n_ens, H = s->hidden;
  hipStream_t st = s->stream;
  hipLaunchKernelGGL(k_pack_input, blocks((int64_t)B * SG_K0), dim3(256), 0, st, B, s->n_in, SG_K0, x, s->X);
  SG_TRY(hipGetLastError());
  const int64_t sP = L.n_params;
  // layer 1: K0 -> H
  SG_TRY((mm<false, false, MM_HIDDEN>(st, E, B, H, SG_K0, s->X, SG_K0, 0, s->Pb + L.W1, H, sP, s->P + L.b1, sP,
                                      s->Z1, H, (int64_t)B * H, s->H1, (int64_t)B * H, nullptr, 0)));
  // layer 2: H -> H
  SG_TRY((mm<false, false, MM_HIDDEN>(st, E, B, H, H, s->H1, H, (int64_t)B * H, s->Pb + L.W2, H, sP, s->P + L.b2,
                                      sP, s->Z2, H, (int64_t)B * H, s->H2, (int64_t)B * H, nullptr, 0)));
  // layer 3: H -> n_out
  SG_TRY((mm<false, false, MM_OUTPUT>(st, E, B, s->n_out, H, s->H2, H, (int64_t)B * H, s->Pb + L.W3, s->n_out, sP,
                                      s->P + L.b3, sP, s->Y, s->n_out, (int64_t)B * s->n_out, nullptr, 0, nullptr,
                                      0)));
  return hipSuccess;
}

hipError_t sg_backward(soap_surrogate* s, const float* target, int B) {
  const SgLayout& L = s->lay;
  const int E = s->n_ens, H = s->hidden, O = s->n_out;
  hipStream_t st = s->stream;
  const int64_t sP = L.n_params, sBH = (int64_t)B * H, sBO = (int64_t)B * O;
  hipLaunchKernelGGL(k_mse, dim3((B + 3) / 4, E), dim3(256), 0, st, B, O, s->Y, target, s->dY, s->row_se);
  SG_TRY(hipGetLastError());
  hipLaunchKernelGGL(k_loss_sum, dim3(E), dim3(256), 0, st, B, O, s->row_se, s->loss);
  SG_TRY(hipGetLastError());
  // output layer: dW3 = H2^T dY, db3 = colsum dY
  SG_TRY((mm<true, false, MM_PLAIN>(st, E, H, O, B, s->H2, H, sBH, s->dY, O, sBO, nullptr, 0, s->G + L.W3, O, sP,
                                    nullptr, 0, nullptr, 0)));
  hipLaunchKernelGGL(k_bf16_to_f32, blocks((int64_t)E * B * O), dim3(256), 0, st, (int64_t)E * B * O, s->dY,
                     s->dYf);
  SG_TRY(hipGetLastError());
  SG_TRY(colsum(st, E, B, O, s->dYf, sBO, s->colpart, s->G + L.b3, sP));
  // dZ2 = (dY W3^T) SiLU'(Z2); dW2 = H1^T dZ2; db2 = colsum dZ2
  SG_TRY((mm<false, true, MM_DHIDDEN>(st, E, B, H, O, s->dY, O, sBO, s->Pb + L.W3, O, sP, nullptr, 0, s->dZf, H, sBH,
                                      s->dZb, sBH, s->Z2, sBH)));
  SG_TRY((mm<true, false, MM_PLAIN>(st, E, H, H, B, s->H1, H, sBH, s->dZb, H, sBH, nullptr, 0, s->G + L.W2, H, sP,
                                    nullptr, 0, nullptr, 0)));
  SG_TRY(colsum(st, E, B, H, s->dZf, sBH, s->colpart, s->G + L.b2, sP));
  // dZ1 = (dZ2 W2^T) SiLU'(Z1); dW1 = X^T dZ1; db1 = colsum dZ1
  SG_TRY((mm<false, true, MM_DHIDDEN>(st, E, B, H, H, s->dZb, H, sBH, s->Pb + L.W2, H, sP, nullptr, 0, s->dZf2, H,
                                      sBH, s->dZb2, sBH, s->Z1, sBH)));
  SG_TRY((mm<true, false, MM_PLAIN>(st, E, SG_K0, H, B, s->X, SG_K0, 0, s->dZb2, H, sBH, nullptr, 0, s->G + L.W1, H,
                                    sP, nullptr, 0, nullptr, 0)));
  return colsum(st, E, B, H, s->dZf2, sBH, s->colpart, s->G + L.b1, sP);
}

namespace {

// the next step's constants
AdamArgs next_adam(soap_surrogate* s, float lr) {
  s->step += 1;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  return AdamArgs{lr, b1, b2, eps, 1.0f - powf(b1, (float)s->step), 1.0f - powf(b2, (float)s->step)};
}

template <int MT, bool TRAIN, int W>
hipError_t launch_rows(soap_surrogate* s, const SgRows& a) {
  const size_t lds = sg_rows_lds(16 * MT, a.H, a.O, TRAIN);
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_sg_rows<MT, TRAIN, W>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_sg_rows<MT, TRAIN, W>), dim3((unsigned)((a.B + 16 * MT - 1) / (16 * MT)), s->n_ens),
                     dim3(64 * W), lds, s->stream, a);
  return hipGetLastError();
}

constexpr size_t SR_LDS = 160 * 1024;  // of a compute unit

SgRows rows_args(soap_surrogate* s, const float* x, int B) {
  SgRows a{};
  a.B = B;
  a.n_in = s->n_in;
  a.H = s->hidden;
  a.O = s->n_out;
  a.L = s->lay;
  a.x = x;
  a.P = s->P;
  a.Pb = s->Pb;
  a.PbT = s->PbT;
  return a;
}

}  // namespace

// networks past about 740 (training) or 2200 (inference) hidden units keep the
// general kernels
bool sg_rows_fit(int hidden, int n_out, bool train) { return sg_rows_lds(16, hidden, n_out, train) <= SR_LDS; }

// In inference a block walks all weights for its 16 rows, which for few rows of
// very wide networks takes longer than the general kernels, whose blocks spread
// the columns over the chip.  By the rows of all networks, row kernel and general
// kernels in us: 1792 hidden units, 64 rows 81 and 77, 256 rows of 4 networks 82
// and 90; 2048 units, 64 rows 102 and 84, 512 rows 98 and 92, 960 rows of 4
// 109 and 105; 2176 units, 960 rows of 4 123 and 135.  (1696 units: 80 and 84 at 64 rows, 79 and 76 at 16.)
bool sg_rows_predict(const soap_surrogate* s, int B) {
  const int few = s->hidden < 1792 ? 0 : s->hidden < 2048 ? 240 : 960;
  return sg_rows_fit(s->hidden, s->n_out, false) && (int64_t)B * s->n_ens >= few;
}

// 32 rows a block when that leaves every compute unit two blocks, since each
// block reads all weights (10000 rows, hidden 256, 128 outputs, 4 members: 34 us
// against 56 with 16 rows and their weights loaded ahead, 36 without, 38 with 48
// or 64 rows; three launches of the general kernels 66); else 16, to fill the
// chip, and there the weights' latency counts
hipError_t sg_rows_forward(soap_surrogate* s, const float* x, int B, float* Y) {
  SgRows a = rows_args(s, x, B);
  a.Y = Y;
  const bool wide = (int64_t)B * s->n_ens >= 16 * SR_MT * 512 && 2 * sg_rows_lds(16 * SR_MT, a.H, a.O, false) <= SR_LDS;
  if (a.H <= SR_NARROW_COLS && a.O <= SR_NARROW_COLS && (int64_t)B * s->n_ens >= SR_NARROW_ROWS)
    return launch_rows<SR_MT, false, SR_NARROW>(s, a);
  return wide ? launch_rows<SR_MT, false, SR_INFER>(s, a) : launch_rows<1, false, SR_INFER>(s, a);
}

hipError_t sg_rows_step(soap_surrogate* s, const float* x, const float* target, int B, float lr) {
  SgRows a = rows_args(s, x, B);
  a.target = target;
  a.XT = s->XT;
  a.H1T = s->H1T;
  a.H2T = s->H2T;
  a.dYT = s->dYT;
  a.dZ2T = s->dZ2T;
  a.dZ1T = s->dZ1T;
  a.dYf = s->dYf;
  a.dZ2f = s->dZf;
  a.dZ1f = s->dZf2;
  a.row_se = s->row_se;
  SG_TRY((launch_rows<1, true, SR_TRAIN>(s, a)));
  const int H = a.H, O = a.O;
  SgGrads g{};
  g.B = B;
  g.H = H;
  g.O = O;
  g.L = s->lay;
  g.XT = s->XT;
  g.H1T = s->H1T;
  g.H2T = s->H2T;
  g.dYT = s->dYT;
  g.dZ2T = s->dZ2T;
  g.dZ1T = s->dZ1T;
  g.dYf = s->dYf;
  g.dZ2f = s->dZf;
  g.dZ1f = s->dZf2;
  g.row_se = s->row_se;
  g.P = s->P;
  g.G = s->G;
  g.M = s->M;
  g.V = s->V;
  g.loss = s->loss;
  g.Pb = s->Pb;
  g.PbT = s->PbT;
  g.adam = next_adam(s, lr);
  const int tiles = (H / 16) * (H / 32) + (H / 16) * (O / 32) + (SG_K0 / 16) * (H / 32);
  g.blk_w = (tiles + 3) / 4;
  g.blk_b = (2 * H + O) / SG_BIAS_COLS;
  hipLaunchKernelGGL(k_sg_grads, dim3((unsigned)(g.blk_w + g.blk_b + 1), s->n_ens), dim3(256), 0, s->stream, g);
  return hipGetLastError();
}

hipError_t sg_adam(soap_surrogate* s, float lr) {
  const AdamArgs a = next_adam(s, lr);
  const int64_t n = s->n_ens * param_units(s->hidden, s->n_out);
  hipLaunchKernelGGL(k_adam, blocks(n), dim3(256), 0, s->stream, n, a, s->lay, s->hidden, s->n_out,
                     sg_rows_fit(s->hidden, s->n_out, true) ? 1 : 0, s->P, s->G, s->M, s->V, s->Pb,
                     sg_rows_fit(s->hidden, s->n_out, false) ? s->PbT : nullptr);
  return hipGetLastError();
}

hipError_t sg_sync_bf16(soap_surrogate* s) {
  const int64_t n = s->n_ens * param_units(s->hidden, s->n_out);
  hipLaunchKernelGGL(k_f32_to_bf16, blocks(n), dim3(256), 0, s->stream, n, s->lay, s->hidden, s->n_out,
                     sg_rows_fit(s->hidden, s->n_out, true) ? 1 : 0, s->P, s->Pb,
                     sg_rows_fit(s->hidden, s->n_out, false) ? s->PbT : nullptr);
  return hipGetLastError();
}

hipError_t sg_ens_mean(soap_surrogate* s, int B, const float* Y, float* mean) {
  const int64_t n = (int64_t)B * s->n_out;
  hipLaunchKernelGGL(k_ens_mean, blocks(n), dim3(256), 0, s->stream, n, s->n_ens, Y, mean);
  return hipGetLastError();
}

hipError_t sg_gate(hipStream_t st, const soap_rv* rv, int64_t n, int E, double calib, double thr, double* rv_kms,
                   double* err_kms, int* fallback) {
  hipLaunchKernelGGL(k_gate, blocks(n), dim3(256), 0, st, n, E, calib, thr, rv, rv_kms, err_kms, fallback);
  return hipGetLastError();
}

hipError_t sg_features(hipStream_t st, int64_t n, const double* raw, float* x) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_features, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, raw, x);
  return hipGetLastError();
}

hipError_t sg_pca_project(hipStream_t st, int n, int P, int k, const float* D, int64_t ldd, const float* mean,
                          const int* mean_idx, int n_mean, const float* V, float* coef) {
  const int nb = (k + PCA_N - 1) / PCA_N;
  // 32-row tiles read V half as often, once they still give every CU two blocks
  // (8192 x 128: 482 us against 676; 2048 x 128, 128 blocks of them: 297 against 209)
  const bool wide = (int64_t)((n + 31) / 32) * nb >= 512;
  // a row tile to each wave once the tiles fill the chip, the sooner the fewer the
  // pixels (split and not, us: 8000 rows x 128 components, 1000 tiles, 128 pixels
  // 13.6 and 10.4, 512 pixels 20 and 24; 20000 x 128, 2500 tiles, 256 pixels 32 and
  // 27, 401 pixels 38 and 41; 20000 x 256, 5000 tiles, 512 pixels 87 and 68, 800
  // pixels 108 and 105)
  const bool split = P > std::min((int64_t)1024, (int64_t)((n + 15) / 16) * nb / 7);
  const int tiles = split && wide ? (n + 31) / 32 : (n + 15) / 16;
  const dim3 grid((unsigned)(split ? tiles : (tiles + PCA_W - 1) / PCA_W), nb), block(64 * PCA_W);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, n, P, k, D, ldd, mean, mean_idx, mean_idx ? n_mean : 1, V, coef);
  };
  auto by_rows = [&](auto c4) {
    constexpr bool C4 = decltype(c4)::value;
    if (!split) go(k_pca_project<1, C4, false>);
    else wide ? go(k_pca_project<2, C4, true>) : go(k_pca_project<1, C4, true>);
  };
  k >= 4 ? by_rows(std::true_type()) : by_rows(std::false_type());
  return hipGetLastError();
}

}  // namespace soap
