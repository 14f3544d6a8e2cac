// Final spectra of a chunk of phases over a tile of pixels (section 3.3,
// Algorithm 5 with Eqs. 1-4).
//
// With the quiet integrated spectrum Q resident, Eq. 4 gives each phase's
// spectrum as Q minus the summed per-cell differences of the active cells.
// Grouped by disk column and collapsed onto integer pixel offsets (see
// weights.hip):
//
//   paired tables (one row per active type and mu bin b):
//     F[p][m] = Q[m] + sum_{t,b,j} K[p][t,b][j] * (A_{t,b}(m, j) - S_{q,b}[m - j])
//   with A = C_{t,b}[m] S_{t,b}[m - j]  (Eq. 3, total effect),
//            C_{t,b}[m] S_{q,b}[m - j]  (Eq. 1, flux effect),
//            S_{t,b}[m - j]             (Eq. 2, convective effect);
//   split tables (scalar contrasts other than one): quiet-removal rows with
//   negative taps on S_{q,b} and active rows with contrast-scaled taps on A.
// The contrast multiplies after the shift, at the output pixel m.
//
// Work split: one block of APPLY_WAVES waves per (tile of APPLY_WAVES x 64
// x R pixels, chunk of PC phases); each wave owns 64 x R consecutive pixels
// of the tile (R per lane: 16 bytes of a row) and walks every window of the
// chunk's list over them by itself, with R x PC accumulators per lane in
// registers.  A window's operands (the active row over the wave's pixels and
// APPLY_JW - 1 samples before them, the quiet row likewise for paired tables,
// the contrast at the pixels, and the window's taps) are copied straight from
// memory into one of the wave's DEP LDS slots, the copies of the next DEP - 1
// windows in flight while a window is consumed; the rows are padded with
// their end samples, so no copy needs a bounds check and the end-value hold
// of the interpolation is built in.  Each lane then reads its R + APPLY_JW - 1
// samples per row as 16-byte LDS reads and, offset by offset, forms the
// differences D of its R pixels once and adds k * D for every group of phases
// that has a tap there (a wave-uniform mask test skips the others): in FP32
// four phases per v_mfma_f32_4x4x1_16b, whose lane l takes its own pixel's D
// and the taps of phases 4 g + i from the lanes l % 4 = i of its block of
// four, and which rounds each k * D + acc as one FMA does; in FP64 pairs of
// phases with FMAs.
// The block-to-work mapping keeps the chunks of one tile on one XCD so their
// shared input windows hit the same L2, and either starts the chunks with the
// most windows first or walks the tiles in order.  The final store adds Q in
// double.  Every pixel's sum runs over the offsets in list order, so results
// repeat bit for bit whatever the pipeline depth, item order or chunk size.
//
// What bounds it: for large calls memory and issue together (206k px x 100
// phases, paired with contrast: 82 MB written and 122 MB read in 38.7 us, 5.3
// TB/s; vector and matrix units busy 45% of the time), for small ones the
// chain of a wave's windows (about 0.45 us each).  Before, with operands
// loaded into registers window by window (4 offsets, 8 loads), taps read from
// LDS as broadcasts and one FMA per phase and pixel: 49 us; 500 spots x 8
// phases of 20000 px 162 us, now 107; FP64 100003 px x 60 phases 57.7, now
// 40.2; 60000 px x 100 phases 30 us, now 20.6.  On the way: matrix
// instructions alone 43.9 (16 phases per chunk); operands through LDS in
// windows of 8 offsets 46.2, with the rows' addresses in the record headers,
// reads kept whole and the loop ended by the mask 44.6, with streaming stores
// 39.8.  Headers kept in registers and read back by v_readlane: 42.2 (and
// small calls as now).  Groups of tiles per XCD, heaviest chunk first within
// each: no gain at any group size.
#include <algorithm>
#include <vector>

#include "soap_internal.hpp"

namespace soap {

namespace {

template <typename T>
struct ApplyArgs {
  int64_t P;
  int n_ph, n_chunks, n_tiles, vg_cap, vec_ok, order;
  const double* Q;
  const unsigned char* wins;
  const int* nvg;
  T* out;
  unsigned* started;  // host word that takes seq when the kernel begins (null: none)
  unsigned seq;
};

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

typedef float f32x4 __attribute__((ext_vector_type(4)));

// One LDS slot of a wave: 1 KiB of the wave's pixels per row (the lanes' 16
// bytes in lane order), then the ends of the sample rows (the APPLY_JW
// samples past the 1 KiB: rows start APPLY_JW - 1 samples before the first
// pixel) and the taps.
template <typename T, int PC, int MODE>
struct Slot {
  static constexpr int R = ApplyShape<T, PC>::R;
  static constexpr int ROWS = MODE == MODE_SPLIT ? 1 : 2;              // sample rows
  static constexpr int CON = ROWS * 1024;                               // contrast at the pixels
  static constexpr int TAIL = CON + (MODE == MODE_CONTRAST ? 1024 : 0);
  static constexpr int TB = APPLY_JW * (int)sizeof(T);                  // bytes of a row's end
  static constexpr int TAPS = TAIL + ROWS * TB;
  static constexpr int TAP_BYTES = APPLY_JW * PC * (int)sizeof(T);
  static constexpr int BYTES = TAPS + TAP_BYTES;
  static constexpr int LANES_T = ROWS * TB / 16;                        // lanes that copy the ends
  static constexpr int LANES = LANES_T + TAP_BYTES / 16;                // and the taps
  static constexpr int N16 = (R + APPLY_JW - 1 + R - 1) / R;            // 16-byte reads per row
  static constexpr int COPIES = ROWS + (MODE == MODE_CONTRAST ? 1 : 0) + 1;
  static_assert(LANES <= 64 && BYTES % 16 == 0, "one copy for the ends and the taps");
};

// the compiler keeps nothing in m0 (a reserved register) across statements
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// Copies 16 bytes per lane from memory (any 4-byte alignment) to LDS at lds +
// AT + 16 x lane, without going through registers; counted by vmcnt like a
// load, which the compiler does not see here: every wait is in the loop below.
template <int AT>
__device__ __forceinline__ void copy16(unsigned lds, unsigned long long base, unsigned lane_off) {
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds), "v"(lane_off), "s"(base), "n"(AT)
               : "memory", "m0", "scc");
}
template <int AT>
__device__ __forceinline__ void copy16_lanes(unsigned lds, unsigned long long p) {
  asm volatile("s_add_u32 m0, %0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"(lds), "v"(p), "n"(AT)
               : "memory", "m0", "scc");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_copies() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// A window record's header, through a scalar load.  Scalar loads share their
// counter with LDS reads, and a wait for one waits for all: the header of the
// next copies is loaded right after a window's LDS reads have arrived and is
// used after its arithmetic, so neither is waited for in vain.
struct Head {
  unsigned long long act, quiet, con;
  unsigned gmask;
};
__device__ __forceinline__ Head load_head(unsigned long long rec) {
  typedef unsigned u32x8 __attribute__((ext_vector_type(8)));
  asm volatile("" : "+s"(rec));  // not before this point
  const u32x8 x = *(const __attribute__((address_space(4))) u32x8*)rec;
  auto at = [&](int i) { return (unsigned long long)x[i] | ((unsigned long long)x[i + 1] << 32); };
  return Head{at(0), at(2), at(4), x[6]};
}

// Starts the copies of one window into the slot at LDS address lds.  px_bytes:
// the wave's first pixel in bytes.  Uniform bases in SGPRs, 32-bit lane
// offsets; end_off: the lane's offset in the last copy, from the active row,
// the quiet row or the record (as its lane number says).
template <typename T, int PC, int MODE>
__device__ __forceinline__ void fetch(const Head& h, unsigned long long rec, unsigned long long px_bytes,
                                      unsigned lds, int lane, long long end_off) {
  using S = Slot<T, PC, MODE>;
  const unsigned lo = 16u * lane;
  const unsigned long long act = h.act + px_bytes, quiet = h.quiet + px_bytes;
  copy16<0>(lds, act, lo);
  if constexpr (MODE != MODE_SPLIT) copy16<1024>(lds, quiet, lo);
  if constexpr (MODE == MODE_CONTRAST) copy16<S::CON>(lds, h.con + px_bytes, lo);
  // the ends of the rows and the taps, one copy
  constexpr int LA = S::TB / 16;
  unsigned long long p = rec;
  if constexpr (S::ROWS == 2) p = lane < 2 * LA ? quiet : p;
  p = lane < LA ? act : p;
  if (lane < S::LANES) copy16_lanes<S::TAIL>(lds, p + end_off);
}

// Accumulators of one lane: PC phases x R pixels.  FP32 keeps four phases of a
// pixel together, as the matrix instruction adds them.
template <typename T, int PC>
struct Acc {
  static constexpr int R = ApplyShape<T, PC>::R;
  T v[PC][R];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int p = 0; p < PC; ++p)
#pragma unroll
      for (int r = 0; r < R; ++r) v[p][r] = T(0);
  }
  __device__ __forceinline__ T get(int p, int r) const { return v[p][r]; }
};
template <int PC>
struct Acc<float, PC> {
  static constexpr int R = ApplyShape<float, PC>::R;
  f32x4 v[PC / 4][R];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int g = 0; g < PC / 4; ++g)
#pragma unroll
      for (int r = 0; r < R; ++r) v[g][r] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ float get(int p, int r) const { return v[p / 4][r][p % 4]; }
};

// 16 bytes of LDS
template <typename T>
__device__ __forceinline__ void read16(T* x, const unsigned char* p) {
  if constexpr (sizeof(T) == 4) {
    const float4 f = *reinterpret_cast<const float4*>(p);
    x[0] = f.x;
    x[1] = f.y;
    x[2] = f.z;
    x[3] = f.w;
  } else {
    const double2 f = *reinterpret_cast<const double2*>(p);
    x[0] = f.x;
    x[1] = f.y;
  }
}
// the values are wanted here as they are: the reads before it stay whole and
// together instead of following their uses into the offsets' branches
template <typename T, int N>
__device__ __forceinline__ void settle(T (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}

// Offsets Q0 .. Q0 + NQ - 1 of one window from its slot.  row_at[i]: place of
// the lane's i-th 16 bytes of the active row (past the last lane they are in
// the row's end), row_at[N16 + i] of the quiet row; sample s of the lane is
// m_0 - jlo - (JW - 1) + s, so pixel r at offset jlo + q uses s = r - q + JW -
// 1.  The offsets of a window are mostly its first few, so the loop ends where
// the mask does; within it every group of a pair of groups that has a tap is
// added (a zero tap adds exactly zero).
// then(): called once the reads have arrived.
template <typename T, int PC, int MODE, int Q0, int NQ, typename F>
__device__ __forceinline__ void consume(Acc<T, PC>& acc, unsigned gm, const unsigned char* slot,
                                        const unsigned (&row_at)[2 * Slot<T, PC, MODE>::N16], int lane, F then) {
  using S = Slot<T, PC, MODE>;
  constexpr int R = S::R, JW = APPLY_JW, NG = ApplyShape<T, PC>::NG, N16 = S::N16;
  constexpr int S0 = (JW - Q0 - NQ) / R * R, S1 = R - 1 - Q0 + JW;  // samples S0 .. S1 - 1 are used
  constexpr int I0 = S0 / R, I1 = (S1 + R - 1) / R;
  static_assert(I1 <= N16, "samples of a row");
  T a[(I1 - I0) * R], b[(I1 - I0) * R], c[R];
#pragma unroll
  for (int i = I0; i < I1; ++i) {
    read16(&a[(i - I0) * R], slot + row_at[i]);
    if constexpr (MODE != MODE_SPLIT) read16(&b[(i - I0) * R], slot + row_at[N16 + i]);
  }
  if constexpr (MODE == MODE_CONTRAST) read16(c, slot + S::CON + 16 * lane);
  // FP32: the lane's taps of the offsets; FP64: every phase's taps
  constexpr int NK = sizeof(T) == 4 ? NQ * NG : NQ * PC;
  T k[NK];
  const unsigned char* kp = slot + S::TAPS + (sizeof(T) == 4 ? 4 * NG * (JW * (lane & 3) + Q0) : 8 * PC * Q0);
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int i = 0; i < NK; i += 4) read16(&k[i], kp + 4 * i);
    settle(k);
  }
  settle(a);
  if constexpr (MODE != MODE_SPLIT) settle(b);
  if constexpr (MODE == MODE_CONTRAST) settle(c);
  then();
#pragma unroll
  for (int q = Q0; q < Q0 + NQ; ++q) {
    if (q > Q0 && gm < (1u << (q * NG))) break;  // uniform
    T D[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int s = r - q + JW - 1 - S0;
      D[r] = MODE == MODE_CONTRAST ? fma(c[r], a[s], -b[s]) : (MODE == MODE_PAIRED ? a[s] - b[s] : a[s]);
    }
    const unsigned bits = gm >> (q * NG);
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int g = 0; g < NG; g += 2) {
        if (NG > 2 && !((bits >> g) & 3u)) continue;
#pragma unroll
        for (int u = g; u < g + 2; ++u)
#pragma unroll
          for (int r = 0; r < R; ++r)
            acc.v[u][r] = __builtin_amdgcn_mfma_f32_4x4x1f32(k[(q - Q0) * NG + u], D[r], acc.v[u][r], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int p = 0; p < PC; p += 2) read16(&k[(q - Q0) * PC + p], kp + 8 * ((q - Q0) * PC + p));
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (__builtin_expect((bits >> g) & 1u, 1)) {
#pragma unroll
          for (int p = 2 * g; p < 2 * g + 2; ++p)
#pragma unroll
            for (int r = 0; r < R; ++r) acc.v[p][r] = fma(k[(q - Q0) * PC + p], D[r], acc.v[p][r]);
        }
      }
    }
  }
}

}  // namespace

// final combine of one item: Q (double) plus the accumulated differences,
// written with 16-byte stores where the row allows
template <typename T, int PC>
__device__ __forceinline__ void store_item(const ApplyArgs<T>& A, const Acc<T, PC>& acc, int chunk, int64_t m0) {
  constexpr int R = ApplyShape<T, PC>::R;
  double Qr[R];
#pragma unroll
  for (int r = 0; r < R; ++r) Qr[r] = A.Q[m0 + r];  // Q is padded to whole tiles
  const int p0 = chunk * PC;
  const bool full = A.vec_ok && (m0 + R <= A.P);
#pragma unroll
  for (int p = 0; p < PC; ++p) {
    if (p0 + p >= A.n_ph) break;
    T* row = A.out + (int64_t)(p0 + p) * A.P;
    T vals[R];
#pragma unroll
    for (int r = 0; r < R; ++r) vals[r] = (T)(Qr[r] + (double)acc.get(p, r));
    if (full) {
      typedef T T16 __attribute__((ext_vector_type(16 / sizeof(T))));
      T16 x;
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = vals[r];
      // past the caches' usual order: the output is not read again here, and
      // the input rows stay in L2 (headline 44.8 to 39.8 us at 16 phases)
      __builtin_nontemporal_store(x, reinterpret_cast<T16*>(row + m0));
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (m0 + r < A.P) row[m0 + r] = vals[r];
    }
  }
}

// One (tile, chunk) item: each wave walks all of the chunk's windows over its
// own 64 x R pixels of the tile.  Step v starts the copies of window v + DEP -
// 1 (its slot was consumed in step v - 1: those LDS reads are complete before
// the copies start), waits until only the copies of the later windows are
// outstanding, and consumes window v.  Every copy has arrived before the store.
template <typename T, int PC, int MODE, int DEP>
__device__ __forceinline__ void apply_item(const ApplyArgs<T>& A, int tile, int chunk, unsigned char* lds) {
  using S = Slot<T, PC, MODE>;
  constexpr int R = S::R, WB = ApplyShape<T, PC>::WB, N16 = S::N16, NG = ApplyShape<T, PC>::NG;
  const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
  const int64_t px = (int64_t)tile * ApplyShape<T, PC>::TILE + wave * 64 * R;

  Acc<T, PC> acc;
  acc.clear();
  unsigned row_at[2 * N16];
#pragma unroll
  for (int i = 0; i < N16; ++i) {
    const int u = lane + i;
    row_at[i] = u < 64 ? 16 * u : S::TAIL + 16 * (u - 64);
    row_at[N16 + i] = u < 64 ? 1024 + 16 * u : S::TAIL + S::TB + 16 * (u - 64);
  }
  // the lane's part of the last copy: ends of the rows, then the taps
  constexpr int LA = S::TB / 16;
  const long long end_off = lane < LA ? 1024 + 16 * lane
                            : lane < S::LANES_T ? 1024 + 16 * (lane - LA)
                                                : WIN_HEAD + 16 * (lane - S::LANES_T);

  const int nv = uni(A.nvg[chunk]);
  const unsigned long long gw = (unsigned long long)(uintptr_t)(A.wins + (int64_t)chunk * A.vg_cap * WB);
  unsigned char* ring = lds + wave * (DEP * S::BYTES);
  const unsigned ring_at = uni((unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring);
  const unsigned long long pxb = (unsigned long long)px * sizeof(T);
  if (nv > 0) {
    const unsigned long long last = gw + (unsigned long long)(nv - 1) * WB;
    unsigned long long rf = gw;  // record of the next copies
    Head hf = load_head(rf);     // and its header
    unsigned gm[DEP];            // masks of the windows in flight
#pragma unroll
    for (int i = 0; i + 1 < DEP; ++i) {
      gm[i] = hf.gmask;
      if (i < nv) fetch<T, PC, MODE>(hf, rf, pxb, ring_at + i * S::BYTES, lane, end_off);
      rf = rf < last ? rf + WB : last;
      hf = load_head(rf);
    }
    for (int v0 = 0; v0 < nv; v0 += DEP) {
#pragma unroll
      for (int d = 0; d < DEP; ++d) {
        constexpr int F = DEP - 1, H = APPLY_JW / 2;
        const int v = v0 + d;
        if (v >= nv) break;
        gm[(d + F) % DEP] = hf.gmask;
        if (v + F < nv) {
          fetch<T, PC, MODE>(hf, rf, pxb, ring_at + ((d + F) % DEP) * S::BYTES, lane, end_off);
          wait_copies<F * S::COPIES>();
        } else {
          wait_copies<0>();
        }
        const unsigned m = gm[d];
        const unsigned char* slot = ring + d * S::BYTES;
        consume<T, PC, MODE, 0, H>(acc, m, slot, row_at, lane, [&] {
          rf = rf < last ? rf + WB : last;
          hf = load_head(rf);
        });
        if (m >= (1u << (H * NG))) consume<T, PC, MODE, H, APPLY_JW - H>(acc, m, slot, row_at, lane, [] {});
        // the slot's reads are complete before a later copy may overwrite it
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
      }
    }
  }
  store_item<T, PC>(A, acc, chunk, px + lane * R);
}

// Blocks are dealt to the 8 XCDs in turn (block index mod 8).  Each XCD
// owns a contiguous range of tiles, so the chunks of a tile share its L2,
// and walks its (chunk, tile) items either heaviest chunk first (most
// windows: the long blocks start early and the short ones fill the end) or
// tile by tile (the chunks of a tile run together).  seq8 is
// the block's index within the configuration's 8 * ceil(n_tiles / 8) *
// n_chunks slots; returns false for a slot with no item.
template <typename T>
__device__ __forceinline__ bool map_item(const ApplyArgs<T>& A, int seq8, int* tile, int* chunk) {
  const int xcd = seq8 & 7;
  const int seq = seq8 >> 3;
  const int tpx = (A.n_tiles + 7) / 8;
  const int t0 = xcd * tpx;
  const int nt = min(A.n_tiles, t0 + tpx) - t0;
  if (nt <= 0 || seq >= nt * A.n_chunks) return false;
  if (A.order == 1) {  // tile by tile
    *tile = t0 + seq / A.n_chunks;
    *chunk = seq % A.n_chunks;
    return true;
  }
  const int rank = seq / nt;
  *tile = t0 + (seq - rank * nt);
  *chunk = rank;
  if (A.n_chunks <= APPLY_RANKED) {
    // each wave ranks the chunks by window count (ties in chunk order): one
    // chunk per lane, the counts exchanged across lanes, and takes the chunk
    // of the wanted rank
    const int c = threadIdx.x & 63;
    const int wc = c < A.n_chunks ? A.nvg[c] : 0;
    int r = 0;
    for (int d = 0; d < A.n_chunks; ++d) {
      const int wd = __builtin_amdgcn_readlane(wc, d);
      r += (wd > wc || (wd == wc && d < c)) ? 1 : 0;
    }
    const unsigned long long hit = __ballot(c < A.n_chunks && r == rank);
    *chunk = uni(__ffsll((long long)hit) - 1);
  }
  return true;
}

// waves per SIMD the register budget is sized for
// (as many as its LDS slots allow, at most four)
template <typename T, int PC, int MODE, int DEP>
constexpr int apply_occupancy() {
  constexpr int fit = 160 * 1024 / (APPLY_WAVES * DEP * Slot<T, PC, MODE>::BYTES);
  return fit < 4 ? fit : 4;
}

template <typename T, int PC, int MODE, int DEP>
__global__ void __launch_bounds__(APPLY_WAVES * 64, (apply_occupancy<T, PC, MODE, DEP>())) k_apply(ApplyArgs<T> A) {
  __shared__ __align__(16) unsigned char lds[APPLY_WAVES * DEP * Slot<T, PC, MODE>::BYTES];
  // what was enqueued before this launch is done
  if (A.started && blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(A.started, A.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  int tile, chunk;
  if (!map_item(A, blockIdx.x, &tile, &chunk)) return;
  apply_item<T, PC, MODE, DEP>(A, tile, chunk, lds);
}

// Batched form: one launch over the items of many configurations (each with
// its own arguments, all with PC phases per chunk).  Configuration i owns the
// slots item_off[i] .. item_off[i+1] - 1, a multiple of 8 starting at a
// multiple of 8, mapped as in k_apply.
template <typename T, int PC, int MODE, int DEP>
__global__ void __launch_bounds__(APPLY_WAVES * 64, (apply_occupancy<T, PC, MODE, DEP>()))
    k_apply_batch(const ApplyArgs<T>* __restrict__ args, const int* __restrict__ item_off, int n_cfg) {
  __shared__ __align__(16) unsigned char lds[APPLY_WAVES * DEP * Slot<T, PC, MODE>::BYTES];
  const int b = blockIdx.x;
  int lo = 0, hi = n_cfg;  // last cfg with item_off[cfg] <= b
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (item_off[mid] <= b) lo = mid;
    else hi = mid;
  }
  const ApplyArgs<T> A = args[lo];
  int tile, chunk;
  if (!map_item(A, b - item_off[lo], &tile, &chunk)) return;
  apply_item<T, PC, MODE, DEP>(A, tile, chunk, lds);
}

// contrast rows are read by the total and flux effects of the modes that have
// them; their tables are paired
int apply_table_mode(const soap_ctx* c, const Plan& pl) {
  if (!pl.paired) return MODE_SPLIT;
  return (c->cmode != SOAP_CONTRAST_SCALAR && pl.effect != SOAP_EFFECT_BCONV) ? MODE_CONTRAST : MODE_PAIRED;
}

// as consume() walks a window: the offsets up to the mask's last one, empty ones
// too; per offset a difference unless the table is split, and FP32 phases in
// pairs of groups (of the only pair always), FP64 phases in the groups with a tap
int window_fmas(unsigned gmask, int pc, int esize, int mode) {
  const int gp = win_group(esize), ng = pc / gp, step = esize == 4 ? 2 : 1;
  int n = 0;
  for (int q = 0; q < APPLY_JW && (q == 0 || (gmask >> (q * ng))); ++q) {
    const unsigned bits = gmask >> (q * ng);
    if (mode != MODE_SPLIT) ++n;
    for (int g = 0; g < ng; g += step)
      if ((esize == 4 && ng == 2) || ((bits >> g) & ((1u << step) - 1u))) n += step * gp;
  }
  return n;
}

namespace {

template <typename T, int PC, int MODE>
hipError_t launch_mode(const ApplyArgs<T>& A, int depth, hipStream_t st) {
  const dim3 grid(8 * ((A.n_tiles + 7) / 8) * A.n_chunks), block(APPLY_WAVES * 64);
  if (depth >= 3)
    hipLaunchKernelGGL((k_apply<T, PC, MODE, 3>), grid, block, 0, st, A);
  else
    hipLaunchKernelGGL((k_apply<T, PC, MODE, 2>), grid, block, 0, st, A);
  return hipGetLastError();
}

template <typename T, int PC>
ApplyArgs<T> make_args(soap_ctx* c, const Plan& pl, const void* win, const int* nvg, void* flux, int order) {
  constexpr int R = ApplyShape<T, PC>::R, TILE = ApplyShape<T, PC>::TILE;
  const bool vec_ok = (c->P % R == 0) && (reinterpret_cast<uintptr_t>(flux) % 16 == 0);
  return ApplyArgs<T>{c->P, pl.n_ph, pl.n_chunks, (int)((c->P + TILE - 1) / TILE), pl.vg_cap, vec_ok ? 1 : 0, order,
                      c->d_Q, static_cast<const unsigned char*>(win), nvg, (T*)flux};
}

template <typename T, int PC>
hipError_t launch_apply_pc(soap_ctx* c, const Plan& pl, const void* d_win, const int* d_nvg, void* d_flux, int depth,
                           int order, hipStream_t st, unsigned* started, unsigned seq) {
  ApplyArgs<T> A = make_args<T, PC>(c, pl, d_win, d_nvg, d_flux, order);
  A.started = started;
  A.seq = seq;
  switch (apply_table_mode(c, pl)) {
    case MODE_SPLIT: return launch_mode<T, PC, MODE_SPLIT>(A, depth, st);
    case MODE_PAIRED: return launch_mode<T, PC, MODE_PAIRED>(A, depth, st);
    default: return launch_mode<T, PC, MODE_CONTRAST>(A, depth, st);
  }
}

}  // namespace

namespace {

hipError_t launch_apply_any(soap_ctx* c, const Plan& pl, const void* d_win, const int* d_nvg, void* d_flux, int depth,
                            int order, hipStream_t st, unsigned* started, unsigned seq) {
  const bool fp32 = c->prec == SOAP_PREC_FP32;
  if (!pc_valid(fp32, pl.pc)) return hipErrorInvalidValue;
  auto* f = fp32 ? (pl.pc == PC_F32_WIDE ? launch_apply_pc<float, PC_F32_WIDE> : launch_apply_pc<float, PC_F32>)
                 : (pl.pc == PC_F64_WIDE ? launch_apply_pc<double, PC_F64_WIDE> : launch_apply_pc<double, PC_F64>);
  return f(c, pl, d_win, d_nvg, d_flux, depth, order, st, started, seq);
}

}  // namespace

hipError_t launch_apply(soap_ctx* c, const Plan& pl, const void* d_win, const int* d_nvg, void* d_flux, unsigned seq) {
  return launch_apply_any(c, pl, d_win, d_nvg, d_flux, c->tune_depth, c->tune_order, c->stream, c->started, seq);
}

hipError_t launch_apply_shape(soap_ctx* c, const Plan& pl, const void* d_win, const int* d_nvg, void* d_flux,
                              int depth, int order, hipStream_t st) {
  return launch_apply_any(c, pl, d_win, d_nvg, d_flux, depth, order, st, nullptr, 0);
}

// ---- batched shift-and-sum over many configurations ------------------------

namespace {

template <typename T, int PC>
hipError_t upload_t(const ApplyBatchCfg* cfgs, int n, void* d_buf, ApplyBatchGroup* g) {
  std::vector<ApplyArgs<T>> args(n);
  std::vector<int> off(n + 1, 0);
  for (int i = 0; i < n; ++i) {
    args[i] = make_args<T, PC>(cfgs[i].c, cfgs[i].pl, cfgs[i].win, cfgs[i].nvg, cfgs[i].flux, cfgs[i].c->tune_order);
    off[i + 1] = off[i] + 8 * ((args[i].n_tiles + 7) / 8) * args[i].n_chunks;  // whole XCD rounds
  }
  g->n_cfg = n;
  g->n_items = off[n];
  g->args = d_buf;
  g->off = static_cast<unsigned char*>(d_buf) + 256 * ((sizeof(ApplyArgs<T>) * n + 255) / 256);
  hipError_t e = hipMemcpy(g->args, args.data(), sizeof(ApplyArgs<T>) * n, hipMemcpyHostToDevice);
  if (e != hipSuccess) return e;
  return hipMemcpy(g->off, off.data(), sizeof(int) * (n + 1), hipMemcpyHostToDevice);
}

template <typename T, int PC, int MODE>
void launch_batch_mode(const ApplyBatchGroup& g, hipStream_t st) {
  const dim3 grid((unsigned)g.n_items), block(APPLY_WAVES * 64);
  const auto* a = static_cast<const ApplyArgs<T>*>(g.args);
  const int* off = static_cast<const int*>(g.off);
  if (g.depth >= 3)
    hipLaunchKernelGGL((k_apply_batch<T, PC, MODE, 3>), grid, block, 0, st, a, off, g.n_cfg);
  else
    hipLaunchKernelGGL((k_apply_batch<T, PC, MODE, 2>), grid, block, 0, st, a, off, g.n_cfg);
}

template <typename T, int PC>
void launch_batch_pc(const ApplyBatchGroup& g, hipStream_t st) {
  switch (g.mode) {
    case MODE_SPLIT: launch_batch_mode<T, PC, MODE_SPLIT>(g, st); break;
    case MODE_PAIRED: launch_batch_mode<T, PC, MODE_PAIRED>(g, st); break;
    default: launch_batch_mode<T, PC, MODE_CONTRAST>(g, st); break;
  }
}

}  // namespace

size_t apply_batch_bytes(int n) {
  return 256 * ((sizeof(ApplyArgs<double>) * n + 255) / 256) + sizeof(int) * (n + 1) + 256;
}

hipError_t apply_batch_upload(const ApplyBatchCfg* cfgs, int n, void* d_buf, ApplyBatchGroup* g) {
  g->fp32 = cfgs[0].c->prec == SOAP_PREC_FP32;
  g->mode = apply_table_mode(cfgs[0].c, cfgs[0].pl);
  g->depth = cfgs[0].c->tune_depth;
  g->pc = cfgs[0].pl.pc;
  if (!pc_valid(g->fp32, g->pc)) return hipErrorInvalidValue;
  // one precision, table mode, phases per chunk and depth per group
  for (int i = 1; i < n; ++i)
    if ((cfgs[i].c->prec == SOAP_PREC_FP32) != g->fp32 || apply_table_mode(cfgs[i].c, cfgs[i].pl) != g->mode ||
        cfgs[i].pl.pc != g->pc || cfgs[i].c->tune_depth != g->depth)
      return hipErrorInvalidValue;
  if (g->fp32)
    return g->pc == PC_F32_WIDE ? upload_t<float, PC_F32_WIDE>(cfgs, n, d_buf, g) : upload_t<float, PC_F32>(cfgs, n, d_buf, g);
  return g->pc == PC_F64_WIDE ? upload_t<double, PC_F64_WIDE>(cfgs, n, d_buf, g) : upload_t<double, PC_F64>(cfgs, n, d_buf, g);
}

hipError_t apply_batch_launch(const ApplyBatchGroup& g, hipStream_t st) {
  if (g.n_items <= 0) return hipSuccess;
  if (g.fp32) {
    if (g.pc == PC_F32_WIDE)
      launch_batch_pc<float, PC_F32_WIDE>(g, st);
    else
      launch_batch_pc<float, PC_F32>(g, st);
  } else {
    if (g.pc == PC_F64_WIDE)
      launch_batch_pc<double, PC_F64_WIDE>(g, st);
    else
      launch_batch_pc<double, PC_F64>(g, st);
  }
  return hipGetLastError();
}

}  // namespace soap
