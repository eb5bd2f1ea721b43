// Grouped SwiGLU expert FFN (Table 3 "MoE update": FFN_e on the rows routed
// to expert e).  Two grouped GEMMs over the permuted rows:
//   gate/up : h[rows,F] = silu(A W_g[e]^T) * (A W_u[e]^T)   (SwiGLU fused into
//             the epilogue; both products share the A tile)
//   down    : y[rows,d] = h W_d[e]^T
// Every weight is [out,in] (K-contiguous), so both GEMMs are "NT".  Row r of A
// is either row r of a permuted copy (x_perm) or, with a gather list, row
// gather[r] / kdiv of the unpermuted input: then the permutation is folded
// into the operand loads and x_perm is never written.
//
// bf16, many rows per expert: 8 waves (2 per SIMD) on a 256-row tile,
// v_mfma_f32_16x16x32_bf16 with fp32 accumulation, operands staged through two
// LDS stages.  Loads use buffer resources whose range ends where the valid
// rows / K end, so ragged tiles read zeros without branches.  The MFMA computes
// D = W_tile * A_tile^T: each lane holds 4 consecutive output columns of one
// row.  The expert and row range of a workgroup come from the
// device-side offsets (one wave prefix sum over per-expert tile counts), so no
// host sync is needed.
//
// bf16, few rows per expert (decode, weight-streaming bound): see
// ffn_stream_bf16.  fp32: the same tiles with fp32 MFMAs.
#include <type_traits>

#include "lds_dma.hpp"

// LDS-DMA large-M kernel: (BM, BN, WM, WN, LDS stages, M-tile group of the tile
// order, persistent)
#ifndef FOE_DMA_GU
#define FOE_DMA_GU 256, 128, 2, 4, 2, 4, 1
#endif
#ifndef FOE_DMA_DN
#define FOE_DMA_DN 256, 256, 2, 4, 2, 4, 1
#endif
// plain grouped GEMM over a few wide segments (the q/k/v projection of the
// attention groups): as the down projection, tiles walked XCD by XCD
#ifndef FOE_DMA_SEG
#define FOE_DMA_SEG 256, 256, 2, 4, 2, 4, 2
#endif
// plain GEMM with the residual epilogue (few M rows)
#ifndef FOE_DMA_RES
#define FOE_DMA_RES 128, 256, 2, 4, 3, 4, 1
#endif
// Smaller tiles of both, for products with few large tiles.  Each CU then runs
// at most one tile, a walk down K that waits for its loads, so the tile is the
// largest that still leaves no more tiles than CUs and more stages keep the
// loads in flight: 128 x 128 where the larger tiles would leave CUs idle, and
// 64 x 128 where even those tiles fit the chip at once.  q/k/v product of 8
// groups, 1000 rows, N 288, K 768: 21.6 us with 64 tiles of 256 x 256, 11.4
// with 192 of 128 x 128, 15.2 with 384 of 64 x 128; output projection of 1000
// rows, N 768, K 768: 12.6 with 48 tiles of 128 x 128, 11.3 with 96 of 64 x 128
// (300 rows: 12.8 and 9.8).  At 1500 rows, N 2048, K 2048 the output
// projection has 192 tiles of 128 x 128 (24 us) against 384 of 64 x 128 (31).
#ifndef FOE_DMA_SMALL
#define FOE_DMA_SMALL 128, 128, 2, 4, 3, 4
#endif
#ifndef FOE_DMA_TINY
#define FOE_DMA_TINY 64, 128, 1, 4, 4, 4
#endif
// medium row counts (see ffn_form): 128 rows x (64 gate + 64 up) or 128 columns,
// 4 waves, two workgroups per CU, K walk rotated
#ifndef FOE_MID_GU
#define FOE_MID_GU 128, 64, 2, 2, 2, 4, 3
#endif
#ifndef FOE_MID_DN
#define FOE_MID_DN 128, 128, 2, 2, 2, 4, 3
#endif
// fp32 expert FFN: gate/up and down tiles (two workgroups per CU)
#ifndef FOE_F32_GU
#define FOE_F32_GU 64, 32, 2, 2, 4, 4, 1
#endif
#ifndef FOE_F32_DN
#define FOE_F32_DN 64, 64, 2, 2, 4, 4, 1
#endif
// few rows per expert (decode): LDS-staged weight stream with NS stages, K
// walk rotated per workgroup, and (block decode form) pair lists built in the
// kernel
#ifndef FOE_FFN_SEL
#define FOE_FFN_SEL 1
#endif
#ifndef FOE_STREAM_ROT
#define FOE_STREAM_ROT 1
#endif
#ifndef FOE_STREAM_NS
#define FOE_STREAM_NS 3
#endif

namespace foe {
namespace {

// Most (token, slot) pairs per cluster for which the decode FFN builds each
// expert's pair list itself from the routing decisions.
constexpr int kSelMax = 2048;
constexpr int kScDevice = 16;  // buffer cache policy SC1: device-scope coherence
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Number of M-tiles of BM rows over all experts (segments clamped as in
// find_tile); every lane of the wave gets the total.
// Start of segment e: offsets[e] clamped to [0, rows], or e * (rows / E) when
// offsets is null (E segments of equal length, rows a multiple of E).
__device__ __forceinline__ int seg_start(const int32_t* __restrict__ offsets, int e, int E,
                                         int rows) {
  return offsets == nullptr ? e * (rows / E) : min(max(offsets[e], 0), rows);
}

__device__ int total_mtiles(const int32_t* __restrict__ offsets, int E, int rows, int BM) {
  const int lane = lane_id();
  int mine = 0;
  for (int e = lane; e < E; e += kWave) {
    const int a = seg_start(offsets, e, E, rows);
    const int b = seg_start(offsets, e + 1, E, rows);
    mine += b > a ? (b - a + BM - 1) / BM : 0;
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
  return mine;
}

// Find the (expert, first row, row end) of global M-tile `mt`.  Returns false
// if `mt` is past the last tile.  Offsets are clamped to [0, rows]; a
// decreasing bound gives an empty segment.  Lane l counts the tiles of a
// contiguous range of experts; a wave prefix sum locates the lane holding
// `mt`, which walks its range again to find the expert.
__device__ bool find_tile(const int32_t* __restrict__ offsets_, int E, int rows, int BM, int mt,
                          int& e_out, int& row0, int& row_end) {
  // opaque: in a persistent loop what follows from these is formed anew for
  // every tile (kept across the tile's K loop, which has no register left, it
  // is spilled)
  const int32_t* __restrict__ offsets = opaque_uniform(offsets_);
  const int lane = opaque_int((int)threadIdx.x) & (kWave - 1);
  const int per = (E + kWave - 1) / kWave;
  const int e_begin = min(lane * per, E), e_end = min(e_begin + per, E);
  auto seg = [&](int e, int& a, int& b) {
    a = seg_start(offsets, e, E, rows);
    b = seg_start(offsets, e + 1, E, rows);
    if (b < a) b = a;
  };
  int mine = 0;
  for (int e = e_begin; e < e_end; ++e) {
    int a, b;
    seg(e, a, b);
    mine += (b - a + BM - 1) / BM;
  }
  int incl = mine;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    // (__shfl_up forms its lane addresses from the hardware's lane number)
    const int t = __builtin_amdgcn_ds_bpermute((lane - off) * 4, incl);
    if (lane >= off) incl += t;
  }
  const int excl = incl - mine;
  const uint64_t bal = __ballot(mt >= excl && mt < incl);
  if (bal == 0) return false;
  const int src = __builtin_ctzll(bal);
  int e_sel = 0, r0 = 0, r1 = 0;
  if (lane == src) {
    int t = mt - excl;
    for (int e = e_begin; e < e_end; ++e) {
      int a, b;
      seg(e, a, b);
      const int n = (b - a + BM - 1) / BM;
      if (t < n) {
        e_sel = e;
        r0 = a + t * BM;
        r1 = b;
        break;
      }
      t -= n;
    }
  }
  e_out = __builtin_amdgcn_readlane(e_sel, src);
  row0 = __builtin_amdgcn_readlane(r0, src);
  row_end = __builtin_amdgcn_readlane(r1, src);
  return true;
}

// M-tile table of the fused FFN, held in LDS: entry i (expert, first row,
// row end) is the i-th M-tile of the launch's tile order.  Experts are taken
// in ascending order of their row counts (equal counts: lower id first), each
// expert's tiles in row order.  The least-loaded experts' tiles -- mostly
// partly filled, and reading weight slices that no other M-tile shares, so
// slower than full tiles -- then run first and their down tiles early, and the
// schedule ends on full tiles of the most-loaded experts (in a list-scheduling
// model fitted to measured tile times this is 7% shorter at the Zipf-skewed
// prefill load than id order, and the same for uniform loads).
// kTabMaxE experts at most (their scratch fits the stage buffers), kTileTab
// entries.
constexpr int kTileTab = 2048;
constexpr int kTabMaxE = 1024;

// Builds the table with every thread of the workgroup; `aux` is LDS scratch of
// 4 * kTabMaxE + 1 ints.  Returns the number of M-tiles (the same in every
// thread); the table is complete only if that is at most kTileTab and
// E <= kTabMaxE (otherwise nothing is written and -1 is returned).
template <int NTHR>
__device__ int build_tile_table(const int32_t* __restrict__ offsets, int E, int rows, int BM,
                                int* aux, int* tab) {
  if (E > kTabMaxE) return -1;
  int* cnt = aux;                  // rows of expert e
  int* seg = aux + kTabMaxE;       // first row of expert e
  int* pos = aux + 2 * kTabMaxE;   // expert at position p of the order
  int* first = aux + 3 * kTabMaxE; // first M-tile of position p (E + 1 entries)
  const int tid = threadIdx.x;
  for (int e = tid; e < E; e += NTHR) {
    const int a = seg_start(offsets, e, E, rows);
    const int b = max(seg_start(offsets, e + 1, E, rows), a);
    cnt[e] = b - a;
    seg[e] = a;
  }
  __syncthreads();
  for (int e = tid; e < E; e += NTHR) {
    const int c = cnt[e];
    int r = 0;
    for (int f = 0; f < E; ++f) {
      const int cf = cnt[f];
      r += (cf < c || (cf == c && f < e)) ? 1 : 0;
    }
    pos[r] = e;
  }
  __syncthreads();
  if (tid < kWave) {
    // wave prefix sum of the M-tiles over the positions (contiguous ranges
    // of `per` positions per lane)
    const int per = (E + kWave - 1) / kWave;
    const int p0 = min(tid * per, E), p1 = min(p0 + per, E);
    int mine = 0;
    for (int p = p0; p < p1; ++p) mine += (cnt[pos[p]] + BM - 1) / BM;
    int incl = mine;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int v = __shfl_up(incl, off);
      if (tid >= off) incl += v;
    }
    int run = incl - mine;
    for (int p = p0; p < p1; ++p) {
      first[p] = run;
      run += (cnt[pos[p]] + BM - 1) / BM;
    }
    if (tid == kWave - 1) first[E] = incl;
  }
  __syncthreads();
  const int m_tiles = first[E];
  if (m_tiles > kTileTab) return m_tiles;
  for (int mt = tid; mt < m_tiles; mt += NTHR) {
    // last position p with first[p] <= mt (positions of empty experts share
    // their successor's first tile, so the last such p is the non-empty one)
    int lo = 0, hi = E - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (first[mid] <= mt) lo = mid;
      else hi = mid - 1;
    }
    const int e = pos[lo];
    tab[3 * mt] = e;
    tab[3 * mt + 1] = seg[e] + (mt - first[lo]) * BM;
    tab[3 * mt + 2] = seg[e] + cnt[e];
  }
  __syncthreads();
  return m_tiles;
}

// silu(g) = g * sigmoid(g) with the hardware reciprocal (v_rcp_f32, about one
// ulp) instead of an IEEE division (a ten-instruction sequence); the product
// is rounded to bf16 afterwards, so the two differ far below that rounding.
// g -> -inf: exp overflows to inf and the reciprocal to 0, as the division.
__device__ __forceinline__ float silu_f(float g) {
  return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
}


// Calls f(integral_constant<int, I>) for I = B .. N-1 (compile-time indices).
template <int B, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < N) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, N>(f);
  }
}

// Source row of operand row r: r itself, or gather[r] / kdiv (-1 if that row
// is outside [0, src_rows)).
__device__ __forceinline__ int src_row(const int32_t* __restrict__ gather, int kdiv, int r,
                                       int src_rows) {
  if (gather == nullptr) return r;
  const int g = gather[r];
  const int s = g >= 0 ? g / kdiv : -1;
  return s < src_rows ? s : -1;
}

// ---- LDS-DMA variant of the large-M grouped GEMM ---------------------------
// Operand tiles go from global memory straight into LDS with
// `buffer_load_dwordx4 ... lds`: each lane of a wave deposits 16 bytes at
// M0 + 16 * lane, so one instruction fills 1 KiB of LDS and the tile never
// passes through VGPRs (no ds_write, no staging registers).  The loads are
// issued from inline assembly so that their completion is tracked here with
// explicit vmcnt waits (the compiler does not see them; the kernel issues no
// other global loads inside the main loop and uses M0 nowhere else).
//
// LDS layout of a tile: rows of 128 bytes (64 bf16 or 32 fp32, no padding), the
// 16-byte chunk c of row r stored in slot c ^ swz_tile(r).  A fragment read takes one chunk of 16
// rows, two rows to a 256-byte bank line, so the eight rows of each half need
// eight different slots.  Since a DMA instruction writes 1 KiB contiguously,
// the swizzle is applied on the load side: the lane that lands in slot s of
// row r fetches chunk s ^ swz_tile(r).
__device__ __forceinline__ int swz_tile(int r) { return (r >> 1) & 7; }

template <typename T, int BM, int BN, int WM, int WN, bool GATEUP, int NST>
struct DmaCfg {
  static constexpr int RB = 128;           // bytes per tile row: whole cache lines
  static constexpr int BK = RB / (int)sizeof(T);  // K columns per stage
  static constexpr int NW = WM * WN, NTHR = NW * kWave;
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int SM = WTM / 16, SN = WTN / 16;  // 16-row / 16-column sub-tiles
  static constexpr int NB = GATEUP ? 2 : 1;
  static constexpr int NJ = NB * SN;       // weight fragments of a half stage
  static constexpr int SH = SM / 2;        // A fragments of a row half
  static constexpr int CPR = RB / 16;      // 16-byte chunks per row
  static constexpr int RPI = 1024 / RB;    // rows per DMA instruction
  static constexpr int A_INS = BM / RPI, B_INS = BN / RPI;  // DMA instructions per tile
  // DMA instructions per wave and stage: weights, and each row half of A
  static constexpr int WPW = NB * B_INS / NW, AH = A_INS / 2 / NW;
  static constexpr int NLD = WPW + 2 * AH;
  static constexpr int A_BYTES = BM * RB, B_BYTES = BN * RB;
  static constexpr int STAGE = A_BYTES + NB * B_BYTES;
  static_assert(WTM % 32 == 0 && WTN % 16 == 0, "wave tile");
  static_assert(NB * B_INS % NW == 0 && A_INS % (2 * NW) == 0, "even DMA split");
  static_assert(B_INS % WPW == 0 && (WTM / 16) % AH == 0,
                "a wave's instructions stay inside one weight slice and one run of A rows");
  static_assert(NST >= 2 && NLD * NST <= 63, "vmcnt range");
  static_assert(NST * STAGE <= 160 * 1024, "LDS capacity");
};

// A 16-byte fragment: 8 bf16 or 4 fp32 of one row.
template <typename T> using Frag = T __attribute__((ext_vector_type(16 / sizeof(T))));

// acc[j] += w[j] x^T for the NJ weight fragments of one A fragment, step n of
// NJ (each step the same number of MFMAs), the accumulators fixed in AGPRs.
// bf16: 16 rows x 32 k, v_mfma_f32_16x16x32_bf16, one per weight fragment.
// fp32: 16 rows x 16 k, four v_mfma_f32_16x16x4_f32 per weight fragment (the
// s-th takes element s of every lane's 16 bytes on both operands; fp32
// products and sums), one statement per step so that an accumulator's
// dependent MFMAs stay apart.
// (Through the builtins the register allocator gives each result other
// registers than its addend and spills around 60 of them inside the K loop.)
// The compiler does not see an MFMA here: acc_fence() separates the
// accumulators' first write and last read from the MFMAs by more wait states
// than the instructions need; inside the loop an accumulator returns after at
// least one other MFMA.  Fragments come from LDS reads, which the compiler waits
// for; a vector instruction that wrote one (a register copy) would need two
// wait states before the MFMA.  tests/test_device_code_cpu.py looks for such
// writes, and for results read too early, along every path of the compiled
// kernels (an s_nop 1 in each statement would rule them out too, but costs 4%:
// 16384 tokens x 4 in 32 experts 2116 -> 2196 us a call).
template <int SN, int NJ, typename Acc>
__device__ __forceinline__ void mma_step(Acc& acc, int i, int n, const bf16x8 (&w)[NJ], bf16x8 x) {
  asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
      : "+a"(acc[n / SN][i][n % SN])
      : "v"(w[n]), "v"(x));
}
template <int SN, int NJ, typename Acc>
__device__ __forceinline__ void mma_step(Acc& acc, int i, int n, const f32x4 (&w)[NJ], f32x4 x) {
  static_assert(NJ == 2, "two weight fragments");
  asm("v_mfma_f32_16x16x4_f32 %0, %2, %4, %0\n\t"
      "v_mfma_f32_16x16x4_f32 %1, %3, %4, %1\n\t"
      "v_mfma_f32_16x16x4_f32 %0, %5, %7, %0\n\t"
      "v_mfma_f32_16x16x4_f32 %1, %6, %7, %1"
      : "+a"(acc[0][i][0]), "+a"(acc[1 / SN][i][1 % SN])
      : "v"(w[0][2 * n]), "v"(w[1][2 * n]), "v"(x[2 * n]), "v"(w[0][2 * n + 1]),
        "v"(w[1][2 * n + 1]), "v"(x[2 * n + 1]));
}
template <int N>
__device__ __forceinline__ void acc_fence(f32x4* a) {
  static_assert(N % 4 == 0, "four accumulators per statement");
#pragma unroll
  for (int i = 0; i < N; i += 4)
    asm volatile("s_nop 15\n\ts_nop 15"
                 : "+a"(a[i]), "+a"(a[i + 1]), "+a"(a[i + 2]), "+a"(a[i + 3]));
}

// Residual epilogue of the plain (non gate/up) form: the output becomes
// scale * (acc + x), x an fp32 matrix of the output's shape.
struct GemmResid {
  const float* x = nullptr;
  float scale = 1.f;
};

// Operands of one grouped GEMM: A rows (direct, or gathered as gather[r] /
// kdiv from a_rows source rows), one or two [E, N, K] weight stacks, the
// output [rows, N] (out_bytes = its size, for device-scope stores) and the
// residual epilogue.
template <typename T>
struct GemmArgs {
  const T* A;
  const int32_t* gather;
  int kdiv;
  int a_rows;
  const T* B0;
  const T* B1;
  int N;
  int K;
  T* out;
  uint32_t out_bytes;
  GemmResid res;
  // two-matrix tile shape (GATEUP) used for a plain product: B1 is ignored,
  // and the tile's two BN-row weight slices are rows ntile*2*BN .. +BN and
  // .. +2*BN of B0, stored side by side (no SwiGLU); the tile covers 2*BN
  // output columns
  bool halves;
};

// One BM x BN output tile of expert e (rows row0 .. row_end-1, N-tile ntile)
// over all of K, staged through the workgroup's LDS `smem`.  OUT_CPOL = 0
// stores the output tile through the caches as usual; otherwise the stores
// carry that cache policy (kScDevice: written through past the XCD's L2, so
// that other XCDs can read the tile once the stores have completed).  The
// two-slice form (GemmArgs::halves) always stores as usual, staged through LDS.
//
// Stage kt (64 K columns; 32 in fp32, where the steps below are half as wide)
// lives in LDS buffer kt % NST.  What bounds the loop
// is the delivery of the operands: a 256 x 256 tile needs 64 KiB per stage,
// which takes longer to arrive than the stage's MFMAs take, so the loads must
// be in flight well over one iteration ahead.  With two stage buffers that
// needs each part of a buffer to be free as early as possible.  An iteration
// therefore runs in four quarters, each wave's rows taken as two halves:
//   Q1  A half 0, k 0-31    reads: A half 0 k 32-63, weights k 32-63
//       barrier: A half 1 has landed; nobody reads A half 0 and the weights
//       of this stage any more
//   Q2  A half 0, k 32-63   reads: A half 1 k 0-31
//   Q3  A half 1, k 0-31    reads: A half 1 k 32-63
//       (Q2, Q3 issue the weights and A half 0 of stage kt+NST)
//       barrier: weights and A half 0 of stage kt+1 have landed; nobody reads
//       A half 1 of this stage any more
//   Q4  A half 1, k 32-63   reads: next stage's A half 0 and weights, k 0-31
//       (issues A half 1 of stage kt+NST)
// so every load has between NST-1 and NST-0.5 iterations to arrive (whole
// stages in two buffers left it half to three quarters of one), the waits are
// counted (vmcnt) and never drain the queue, and each row's 64 columns are one
// whole 128-byte line.  Fused expert FFN, against the loop with whole stages
// (us): 2110 -> 1950 at 65536 rows x 32 experts, d 4096, F 1536 (1.17 -> 1.27
// PFLOP/s); 775 -> 735 at 65536 rows x 64 experts, d 2048, F 1024; 207 -> 198
// at 16384 skewed rows x 16 experts.  Without the vmcnt waits (timing only) it
// is no faster; with the loads alone it takes 1490, with the MFMAs and
// fragment reads alone 1630: what is left is the two sharing the clock that
// the power limit allows (1.85 GHz) and the tiles' beginnings and ends.
// 16x16x32 MFMAs: a register-only loop reaches 2.04 PFLOP/s with them and 1.86
// with 32x32x16 ones.
template <typename T, int BM, int BN, int WM, int WN, bool GATEUP, int NST, bool RESID,
          int OUT_CPOL>
__device__ __forceinline__ void gemm_tile(unsigned char* smem, const GemmArgs<T>& g, const int e_,
                                          const int row0_, const int row_end_, const int ntile_,
                                          int32_t* signal = nullptr, const int rot_ = 0) {
  static_assert(!(RESID && GATEUP), "residual epilogue on the plain form only");
  static_assert(sizeof(T) == 2 || OUT_CPOL == 0, "fp32 stores as usual");
  using C = DmaCfg<T, BM, BN, WM, WN, GATEUP, NST>;
  constexpr int BK = C::BK, WPW = C::WPW, AH = C::AH, NLD = C::NLD;
  constexpr uint32_t ES = sizeof(T);
  constexpr bool BF16 = ES == 2;
  // the tile is the same for the whole workgroup: its coordinates (read from
  // LDS) and what follows from them stay in scalar registers
  const int e = __builtin_amdgcn_readfirstlane(e_);
  const int row0 = __builtin_amdgcn_readfirstlane(row0_);
  const int row_end = __builtin_amdgcn_readfirstlane(row_end_);
  const int ntile = __builtin_amdgcn_readfirstlane(ntile_);
  const T* __restrict__ A = g.A;
  // opaque, as the thread index below: conditions and divisors made of them
  // would otherwise be kept from tile to tile in vector registers
  const int32_t* __restrict__ gather = opaque_uniform(g.gather);
  const int kdiv = opaque_uniform(g.kdiv), a_rows = g.a_rows, N = g.N, K = opaque_uniform(g.K);
  const T* __restrict__ B0 = g.B0;
  const T* __restrict__ B1 = g.B1;
  T* __restrict__ out = g.out;
  const GemmResid& res = g.res;

  // opaque: what follows from the lane is formed anew for every tile instead
  // of being kept (spilled) across the persistent loop
  const int tid = opaque_int((int)threadIdx.x);
  const int lane = tid & (kWave - 1);
  const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave_u / WN, wn = wave_u % WN;
  const int n0 = ntile * BN;

  // This wave's DMA: instructions wave*WPW .. of the weight slices and
  // wave*AH .. of each row half of A.  An instruction covers RPI rows (1 KiB);
  // lane l lands in row l / CPR, slot l % CPR and fetches chunk
  // (l % CPR) ^ swz_tile(row).
  const int rl = lane / C::CPR, cl = lane % C::CPR;
  auto kcol = [&](int ii) { return (cl ^ swz_tile(ii * C::RPI + rl)) * (16 / (int)ES); };
  // weights: slice ws, its instruction wi0; a slice past N is empty
  const int wp = wave_u * WPW, ws = wp / C::B_INS, wi0 = wp % C::B_INS;
  int wrow0 = n0;  // first row of the slice
  const T* wmat = B0;
  if constexpr (GATEUP) {
    if (g.halves) wrow0 = ntile * 2 * BN + ws * BN;
    else if (ws == 1) wmat = B1;
  }
  wrow0 = min(wrow0, N);
  const uint64_t w_base = (uint64_t)(uintptr_t)(wmat + ((size_t)e * N + wrow0) * K);
  const uint32_t w_bytes = (uint32_t)min(BN, N - wrow0) * K * ES;
  // A: the tile's rows, or the whole source when gathering
  const uint64_t a_base =
      (uint64_t)(uintptr_t)(gather == nullptr ? A + (size_t)row0 * K : A);
  const uint32_t a_bytes = gather == nullptr ? (uint32_t)min(BM, row_end - row0) * K * ES
                                             : (uint32_t)a_rows * K * ES;
  // instruction q of row half h: rows of one 16-row run after another of the
  // wave rows' halves
  auto a_ins = [&](int h, int q) {
    const int t = wave_u * AH + q;
    constexpr int RUN = C::WTM / 16;  // instructions of half a wave tile's rows
    return (t / RUN) * 2 * RUN + h * RUN + t % RUN;
  };
  uint32_t off_w[WPW], off_a[2][AH];
#pragma unroll
  for (int q = 0; q < WPW; ++q)
    off_w[q] = ((uint32_t)((wi0 + q) * C::RPI + rl) * K + kcol(wi0 + q)) * ES;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < AH; ++q) {
      const int ii = a_ins(h, q), r = ii * C::RPI + rl;
      if (gather == nullptr) {
        off_a[h][q] = ((uint32_t)r * K + kcol(ii)) * ES;
      } else {
        const int rr = opaque_int(row0 + r);
        const int s = rr < row_end ? src_row(gather, kdiv, rr, a_rows) : -1;
        off_a[h][q] = s < 0 ? kOob : ((uint32_t)s * K + kcol(ii)) * ES;
      }
    }
  const uint32_t smem_base = lds_addr(smem);
  const uint32_t lds_w = smem_base + C::A_BYTES + ws * C::B_BYTES + wi0 * 1024;
  const uint32_t lds_a[2] = {smem_base + a_ins(0, 0) * 1024, smem_base + a_ins(1, 0) * 1024};

  // The resource of a stage starts at its first K column (scalar arithmetic),
  // so the per-lane offsets stay fixed; its range shrinks with it and is empty
  // past K.  In a stage that K ends inside, the lanes past K (and in every
  // later stage all lanes) read zeros: their offsets are spoilt once.
  // (signed, below 2^31: the range stays in scalar instructions.  A vector
  // instruction that wrote it would need wait states before the loads, which
  // the compiler cannot see)
  // With `rot` the tile walks its stages from stage rot on and around (only
  // where K is whole stages): tiles that stream weights from memory then read
  // different columns at any moment instead of crowding the channels that one
  // column of the 4 KiB-strided rows lies on.
  const int nkr = (K + BK - 1) / BK;
  const int rot = __builtin_amdgcn_readfirstlane(K % BK == 0 ? rot_ % nkr : 0);
  auto stage_rsrc = [&](uint64_t base, uint32_t bytes, int kt) {
    const int kr = kt < nkr ? (kt + rot >= nkr ? kt + rot - nkr : kt + rot) : kt;
    const int k2 = kr * C::RB;
    return make_rsrc_u(reinterpret_cast<const void*>((uintptr_t)(base + (uint32_t)k2)),
                       (uint32_t)max((int)bytes - k2, 0));
  };
  auto tail_w = [&](int kt) {
    if ((kt + 1) * BK > K) {
#pragma unroll
      for (int q = 0; q < WPW; ++q)
        if (kt * BK + kcol(wi0 + q) >= K) off_w[q] = kOob;
    }
  };
  auto tail_a = [&](int h, int kt) {
    if ((kt + 1) * BK > K) {
#pragma unroll
      for (int q = 0; q < AH; ++q)
        if (kt * BK + kcol(a_ins(h, q)) >= K) off_a[h][q] = kOob;
    }
  };
  auto issue_w = [&](const __amdgpu_buffer_rsrc_t& r, int buf, int q) {
    dma16(r, off_w[q], lds_w, buf * C::STAGE + q * 1024);
  };
  auto issue_a = [&](const __amdgpu_buffer_rsrc_t& r, int buf, int h, int q) {
    dma16(r, off_a[h][q], lds_a[h], buf * C::STAGE + q * 1024);
  };

  constexpr int SM = C::SM, SN = C::SN, NJ = C::NJ, SH = C::SH;
  f32x4 acc[C::NB][SM][SN];
#pragma unroll
  for (int b = 0; b < C::NB; ++b)
#pragma unroll
    for (int i = 0; i < SM; ++i)
#pragma unroll
      for (int j = 0; j < SN; ++j) acc[b][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // LDS offsets of fragment 0 in every buffer and k32 step (fragment rows are
  // congruent to lane % 16 modulo 16, so one swizzle per lane); opaque, so
  // that the fragments are reached by the instructions' offset fields (seen
  // through, each fragment past 64 KiB got an address register of its own)
  const int lrow = lane & 15;
  int oa[NST][2], ob[NST][2];
#pragma unroll
  for (int b = 0; b < NST; ++b)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int x = ((4 * ks + (lane >> 4)) ^ swz_tile(lrow)) * 16 + b * C::STAGE;
      oa[b][ks] = opaque_int((wm * C::WTM + lrow) * C::RB + x);
      ob[b][ks] = opaque_int(C::A_BYTES + (wn * C::WTN + lrow) * C::RB + x);
    }
  Frag<T> xa[2][SH];  // A fragments of this and of the next quarter
  Frag<T> wf[2][NJ];  // weight fragments of the stage's first and second half of K
  auto read_a = [&](int buf, int ks, int h, int i) {
    xa[ks][i] = *reinterpret_cast<const Frag<T>*>(smem + oa[buf][ks] + (h * SH + i) * 16 * C::RB);
  };
  auto read_w = [&](int buf, int ks, int u) {
    wf[ks][u] = *reinterpret_cast<const Frag<T>*>(smem + ob[buf][ks] + (u / SN) * C::B_BYTES +
                                                 (u % SN) * 16 * C::RB);
  };
  // Rows of this wave's tile that exist: with at most half of them the wave
  // leaves out its second half's MFMAs and fragment reads, with none of them
  // all (variants of the loop, which meet the same barriers).  A tile of 256
  // rows with at most 128 then leaves the matrix cores to half of its waves
  // (block calls: 96 rows in each of 40 experts, d = F = 1024: 108 -> 104 us; 24
  // x 2 experts of 160 rows, d = F = 2048: 391 -> 378).
  const int wave_rows = row_end - row0 - wm * C::WTM;

  // K steps rounded up to a multiple of NST: steps past K read zeros.
  const int nk = ((K + BK - 1) / BK + NST - 1) / NST * NST;
  constexpr int QM = SH * NJ;       // MFMAs per quarter
  constexpr int NWA = WPW + AH;     // DMA instructions of Q2 and Q3
  constexpr int VM = (NST - 1) * NLD;  // loads in flight behind the awaited ones
  auto iteration = [&](auto hv, int kt, int b) {
    constexpr bool half = decltype(hv)::value >= 1, none = decltype(hv)::value == 2;
    const int bn = (b + 1) % NST;  // buffer of the next stage
    const int dkt = kt + NST;      // the stage loaded into this buffer
    // quarter q: MFMAs of A half q/2, k32 step q%2, each followed by up to one
    // fragment read (nr of them: rd(n)) and, ahead of it so that it does not
    // queue behind the MFMA, up to one DMA instruction (dma(slot))
    auto quarter = [&](auto qv, auto&& dma, int nr, auto&& rd) {
      constexpr int q = decltype(qv)::value, h = q / 2, ks = q % 2;
      if constexpr (none || (half && h == 1)) {
#pragma unroll
        for (int n = 0; n < QM; ++n) dma(n);
#pragma unroll
        for (int n = 0; n < SH + NJ; ++n)
          if (!none && n < nr) rd(n);
      } else {
#pragma unroll
        for (int n = 0; n < QM; ++n) {
          dma(n);
          const int i = n / NJ, j = n % NJ;
          mma_step<SN, NJ>(acc, h * SH + i, j, wf[ks], xa[ks][i]);
          if (n < nr) rd(n);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = QM; n < SH + NJ; ++n)
          if (n < nr) rd(n);
      }
    };
    using std::integral_constant;
    quarter(integral_constant<int, 0>{}, [&](int) {}, SH + NJ, [&](int n) {
      if (n < SH) read_a(b, 1, 0, n);
      else read_w(b, 1, n - SH);
    });
    vm_barrier<VM>();
    tail_w(dkt);
    tail_a(0, dkt);
    const __amdgpu_buffer_rsrc_t rw = stage_rsrc(w_base, w_bytes, dkt);
    const __amdgpu_buffer_rsrc_t ra = stage_rsrc(a_base, a_bytes, dkt);
    // instruction q of the NWA goes out in slot q * 2 * QM / NWA of Q2 and Q3
    auto dma_wa = [&](int slot) {
#pragma unroll
      for (int q = 0; q < NWA; ++q)
        if (q * 2 * QM / NWA == slot) {
          if (q < AH) issue_a(ra, b, 0, q);
          else issue_w(rw, b, q - AH);
        }
    };
    quarter(integral_constant<int, 1>{}, dma_wa, half ? 0 : SH,
            [&](int n) { read_a(b, 0, 1, n); });
    quarter(integral_constant<int, 2>{}, [&](int slot) { dma_wa(QM + slot); }, half ? 0 : SH,
            [&](int n) { read_a(b, 1, 1, n); });
    vm_barrier<VM>();
    tail_a(1, dkt);
    quarter(integral_constant<int, 3>{},
            [&](int slot) {
#pragma unroll
              for (int q = 0; q < AH; ++q)
                if (q * QM / AH == slot) issue_a(ra, b, 1, q);
            },
            SH + NJ, [&](int n) {
              if (n < SH) read_a(bn, 0, 0, n);
              else read_w(bn, 0, n - SH);
            });
  };
  auto k_loop = [&](auto hv) {
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      tail_w(st);
      tail_a(0, st);
      tail_a(1, st);
      const __amdgpu_buffer_rsrc_t rw = stage_rsrc(w_base, w_bytes, st);
      const __amdgpu_buffer_rsrc_t ra = stage_rsrc(a_base, a_bytes, st);
#pragma unroll
      for (int q = 0; q < AH; ++q) issue_a(ra, st, 0, q);
#pragma unroll
      for (int q = 0; q < WPW; ++q) issue_w(rw, st, q);
#pragma unroll
      for (int q = 0; q < AH; ++q) issue_a(ra, st, 1, q);
    }
    // weights and A half 0 of stage 0 have landed
    if (signal != nullptr) {
      // counted once every wave's earlier stores have completed (the wait
      // drains all of the wave's memory operations, the barrier meets all waves)
      vm_barrier<0>();
      if (threadIdx.x == 0) atomicAdd(signal, 1);
    } else {
      vm_barrier<NST * NLD - NWA>();
    }
#pragma unroll
    for (int i = 0; i < SH; ++i) read_a(0, 0, 0, i);
#pragma unroll
    for (int u = 0; u < NJ; ++u) read_w(0, 0, u);
    acc_fence<C::NB * SM * SN>(&acc[0][0][0]);
    for (int kt = 0; kt < nk; kt += NST) {
#pragma unroll
      for (int u = 0; u < NST; ++u) iteration(hv, kt + u, u);
    }
    acc_fence<C::NB * SM * SN>(&acc[0][0][0]);
    // the last DMAs (zeros past K) land before the buffers are reused
    vm_barrier<0>();
  };
  if (wave_rows > C::WTM / 2) k_loop(std::integral_constant<int, 0>{});
  else if (wave_rows > 0) k_loop(std::integral_constant<int, 1>{});
  else k_loop(std::integral_constant<int, 2>{});

  // Thread indices of the epilogue, taken afresh: address arithmetic on
  // the ones above would be hoisted before the K loop and kept live through
  // it, where the accumulators and fragments leave no registers for it, so
  // the compiler would spill it and reload each value behind a wait for
  // every outstanding store.
  const int tid_e = opaque_int((int)threadIdx.x);
  const int lane_e = tid_e & (kWave - 1);
  const int wm_e = (tid_e >> 6) / WN, wn_e = (tid_e >> 6) % WN;
  const int lrow_e = lane_e & 15;
  // epilogue: lane_e holds row m = .. + lane_e%16, columns n = .. + 4*(lane_e/16) + [0,4)
  const int ncol_e = (lane_e >> 4) * 4;
  [[maybe_unused]] const __amdgpu_buffer_rsrc_t out_rsrc = make_rsrc_u(out, g.out_bytes);
  if constexpr (RESID) {
    // the residual added to the accumulators, the loads of all of the
    // lane_e's outputs in flight together
    f32x4 xv[SM][SN];
#pragma unroll
    for (int i = 0; i < SM; ++i)
#pragma unroll
      for (int j = 0; j < SN; ++j) {
        const int m = row0 + wm_e * C::WTM + i * 16 + lrow_e;
        const int n = n0 + wn_e * C::WTN + j * 16 + ncol_e;
        xv[i][j] = (m < row_end && n < N)
                       ? *reinterpret_cast<const f32x4*>(res.x + (size_t)m * N + n)
                       : f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
    for (int i = 0; i < SM; ++i)
#pragma unroll
      for (int j = 0; j < SN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[0][i][j][v] += xv[i][j][v];
  }
  if constexpr (GATEUP && OUT_CPOL != 0 && BF16) {
    if (!g.halves) {
      // Device-scope stores of whole lines: the SwiGLU tile goes to LDS
      // first (free after the K loop; 16-byte chunk c of tile row r at slot
      // c ^ (r % OCH), so the writes of 16 rows at one chunk spread over the
      // banks), then every lane_e stores 16-byte chunks of whole rows, so the
      // stores that pass the L2 are full 128-byte lines rather than 16-byte
      // pieces of 32.
      constexpr int OCH = BN / 8, ORB = BN * 2;  // chunks and bytes of a staged row
#pragma unroll
      for (int i = 0; i < SM; ++i) {
        const int rr = wm_e * C::WTM + i * 16 + lrow_e;
#pragma unroll
        for (int j = 0; j < SN; ++j) {
          const int ch = (wn_e * C::WTN + j * 16 + ncol_e) / 8;
          bf16x4 o;
#pragma unroll
          for (int v = 0; v < 4; ++v)
            o[v] = (bf16)(silu_f(acc[0][i][j][v]) * acc[1][i][j][v]);
          *reinterpret_cast<bf16x4*>(smem + rr * ORB + ((ch ^ (rr % OCH)) * 16) +
                                     (ncol_e & 4) * 2) = o;
        }
      }
      lds_barrier();
      constexpr int NCH = BM * OCH;
      static_assert(NCH % C::NTHR == 0, "whole store rounds");
#pragma unroll
      for (int k = 0; k < NCH / C::NTHR; ++k) {
        const int c = tid_e + k * C::NTHR;
        const int rr = c / OCH, ch = c % OCH;
        const int m = row0 + rr, n = n0 + ch * 8;
        if (m < row_end && n < N) {
          const bf16x8 o =
              *reinterpret_cast<const bf16x8*>(smem + rr * ORB + ((ch ^ (rr % OCH)) * 16));
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), out_rsrc,
                                                 (uint32_t)(((size_t)m * N + n) * 2), 0,
                                                 OUT_CPOL);
        }
      }
      return;
    }
  }
  if constexpr (GATEUP && OUT_CPOL != 0 && BF16) {
    if (g.halves) {
      // The BM x 2*BN output tile (slice b at columns ntile*2*BN + b*BN + ..)
      // goes to LDS first (the stage buffers are free after the K loop;
      // 16-byte chunk c of tile row r at slot c ^ (r % RCH)), then every lane_e
      // stores 16-byte chunks of whole rows, so a wave instruction writes
      // whole 128-byte lines instead of 16 rows x 32 bytes.
      constexpr int ORB = 2 * BN * 2;                 // bytes per staged row
      constexpr int RCH = 2 * BN / 8;                 // 16-byte chunks per row
      static_assert(BM * ORB <= NST * C::STAGE, "staged tile fits the stage buffers");
#pragma unroll
      for (int i = 0; i < SM; ++i) {
        const int rr = wm_e * C::WTM + i * 16 + lrow_e;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int j = 0; j < SN; ++j) {
            const int ch = b * (BN / 8) + (wn_e * C::WTN + j * 16 + ncol_e) / 8;
            bf16x4 o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = (bf16)acc[b][i][j][v];
            *reinterpret_cast<bf16x4*>(smem + rr * ORB + ((ch ^ (rr % RCH)) * 16) +
                                       (ncol_e & 4) * 2) = o;
          }
      }
      lds_barrier();
      // thread tid_e stores chunk tid_e % RCH of rows tid_e / RCH + k * RPR
      constexpr int RPR = C::NTHR / RCH;  // rows per store round
      static_assert(C::NTHR % RCH == 0 && BM % RPR == 0 && RCH % RPR == 0, "store rounds");
      const int ch = tid_e % RCH, r0 = tid_e / RCH;
      const int n = ntile * 2 * BN + ch * 8;
      if (n < N) {
        // rows r0 + k*RPR take RCH / RPR values modulo RCH, so as many LDS
        // slot offsets serve all rounds
        constexpr int NV = RCH / RPR;
        int slot[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) slot[v] = (ch ^ ((r0 + v * RPR) % RCH)) * 16;
        const unsigned char* src = smem + r0 * ORB;
        bf16* dst = out + (size_t)(row0 + r0) * N + n;
        const int nr = row_end - row0 - r0;  // rows of this thread's column still valid
#pragma unroll
        for (int k = 0; k < BM / RPR; ++k) {
          if (k * RPR < nr)
            *reinterpret_cast<bf16x8*>(dst + (size_t)k * RPR * N) =
                *reinterpret_cast<const bf16x8*>(src + k * RPR * ORB + slot[k % NV]);
        }
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < SM; ++i) {
    const int m = row0 + wm_e * C::WTM + i * 16 + lrow_e;
    if (m >= row_end) continue;
#pragma unroll
    for (int j = 0; j < SN; ++j) {
      const int n = n0 + wn_e * C::WTN + j * 16 + ncol_e;
      if (n >= N) continue;
      typedef T Out4 __attribute__((ext_vector_type(4)));
      Out4 o;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float val = acc[0][i][j][v];
        if constexpr (GATEUP) {
          const float u = acc[C::NB - 1][i][j][v];
          if constexpr (BF16) val = silu_f(val) * u;
          else val = val / (1.0f + expf(-val)) * u;
        }
        if constexpr (RESID) val *= res.scale;
        o[v] = (T)val;
      }
      *reinterpret_cast<Out4*>(out + (size_t)m * N + n) = o;
    }
  }
}

// tile t -> (M-tile, N-tile) of m_tiles x ntn tiles: groups of GM M-tiles are
// walked N-tile by N-tile, so that a run of consecutive tiles shares A rows
// and weight slices
template <int GM>
__device__ __forceinline__ void tile_coords(int t, int ntn, int m_tiles, int& mt, int& nt) {
  if constexpr (GM <= 1) {
    mt = t / ntn;
    nt = t % ntn;
  } else {
    // the last group may hold fewer than GM M-tiles
    const int grp = t / (GM * ntn), i = t % (GM * ntn);
    const int g = min(GM, m_tiles - grp * GM);
    mt = grp * GM + i % g;
    nt = i / g;
  }
}

template <typename T, int BM, int BN, int WM, int WN, bool GATEUP, int NST, int GM, int PERSIST,
          bool RESID = false>
__global__ __launch_bounds__(WM* WN* kWave) __attribute__((amdgpu_waves_per_eu(1, 2)))
void grouped_gemm_dma(const T* __restrict__ A, const int32_t* __restrict__ gather, int kdiv,
                      int a_rows, const int32_t* __restrict__ offsets, int E, int rows,
                      const T* __restrict__ B0, const T* __restrict__ B1, int N, int K,
                      T* __restrict__ out, int n_tiles_n, int n_tiles, GemmResid res) {
  using C = DmaCfg<T, BM, BN, WM, WN, GATEUP, NST>;
  __shared__ __align__(1024) unsigned char smem[NST * C::STAGE];
  const GemmArgs<T> g{A, gather, kdiv, a_rows, B0, B1, N, K, out, 0u, res, false};
  auto run_tile = [&](const int e, const int row0, const int row_end, const int ntile) {
    // rotated K walk (PERSIST == 3): neighbouring tiles start 7 stages apart, a
    // step prime to the usual powers of two.  (K of 7 x 64 n columns leaves n
    // different starts; steps prime to every K gained at most 1% there: d 1792, F
    // 896, 16 experts of 64 rows 56.3 -> 55.7 us a call, F 448 or 1792 nothing.)
    gemm_tile<T, BM, BN, WM, WN, GATEUP, NST, RESID, 0>(
        smem, g, e, row0, row_end, ntile, nullptr,
        PERSIST == 3 ? 7 * (e * n_tiles_n + ntile) : 0);
  };

  // M-tiles that hold rows (persistent form: the tile list is split over
  // the XCDs by this count, not by the launch's upper bound)
  const int m_tiles = PERSIST ? __builtin_amdgcn_readfirstlane(total_mtiles(offsets, E, rows, BM))
                              : n_tiles / n_tiles_n;
  auto tile_coords = [&](int t, int& mt, int& nt) {
    foe::tile_coords<GM>(t, n_tiles_n, m_tiles, mt, nt);
  };
  auto run_t = [&](int t) {
    int mt, nt, e, row0, row_end;
    tile_coords(t, mt, nt);
    if (!find_tile(offsets, E, rows, BM, mt, e, row0, row_end)) return;
    vm_barrier<0>();  // the previous tile's LDS reads are done everywhere
    run_tile(e, row0, row_end, nt);
  };
  if constexpr (PERSIST >= 2) {
    // one workgroup per CU, each XCD walks a contiguous eighth of the tile
    // order (workgroup b runs on XCD b % 8; the grid is a multiple of 8), so
    // the N-tiles of an M-tile and the M-tiles of a segment meet in that
    // XCD's own L2: for a few wide segments (one per XCD) every A row and
    // weight slice is fetched from memory once
    const int n_real = m_tiles * n_tiles_n;
    const int x = blockIdx.x % 8, per = gridDim.x / 8;
    const int chunk = (n_real + 7) / 8;
    const int t_end = min((x + 1) * chunk, n_real);
    for (int t = x * chunk + (int)blockIdx.x / 8; t < t_end; t += per) run_t(t);
  } else if constexpr (PERSIST == 1) {
    // one workgroup per CU, tiles dealt round-robin: the tiles running at any
    // moment are a window of consecutive tiles of the order above, spread
    // over all XCDs, and their shared A rows and weight slices meet in the
    // Infinity Cache that every XCD reads through (measured faster than
    // giving each XCD a contiguous range for its own L2 on the expert GEMMs)
    const int n_real = m_tiles * n_tiles_n;
    for (int t = blockIdx.x; t < n_real; t += gridDim.x) run_t(t);
  } else {
    const int tile = blockIdx.x;
    if (tile >= n_tiles) return;
    int mt, nt, e, row0, row_end;
    tile_coords(tile, mt, nt);
    if (!find_tile(offsets, E, rows, BM, mt, e, row0, row_end)) return;
    run_tile(e, row0, row_end, nt);
  }
}

// Both grouped GEMMs of the expert FFN in one persistent launch.  Work items
// are the gate/up tiles (SwiGLU epilogue, writing h) followed by the down
// tiles (reading h, writing y), numbered in that order; a workgroup's first
// item is its own index and the later ones come one at a time, in order, from
// a device-side counter, so the two GEMMs share one schedule: the
// CUs that finish their last gate/up tile go on to down tiles instead of
// idling through a partly filled last round, and there is no launch between
// the two.
//
// Both tile kinds run the one tile body of the gate/up form (BM rows x two
// BN-row weight slices): a down tile's two slices are consecutive BN-row
// blocks of W_d, stored side by side instead of through SwiGLU.
//
// A down tile of M-tile m needs every gate/up tile of m.  A gate/up tile
// writes its h rows with device-scope stores of whole lines (staged through
// LDS, past its XCD's L2) and is counted in ready[m] once they have completed:
// at the prologue of the workgroup's next gate/up tile, whose wait drains them
// anyway, or before the workgroup's first wait and at its end.  A down tile
// waits until ready[m] holds all of m's gate/up tiles before loading h.  The
// wait always ends: every gate/up tile a down tile waits for is the first
// item of a workgroup of the grid or was taken from the counter, in order,
// before the down tile, by a workgroup that is running it (or holds it as its
// next item behind a gate/up tile); gate/up tiles wait on nothing.  (The
// wait also gives up after a bounded number of polls, so the launch drains
// whatever happens; a give-up is counted in the give-up word of sync.)  No h
// row is read before it is complete, and with rows of whole 128-byte lines (F a
// multiple of 64, checked by the caller) no line is shared by two M-tiles, so
// no XCD's L2 can hold a stale copy of an h line (the L2s hold no h lines from
// earlier launches: each launch starts with them invalidated).
//
// sync: the work counters (one 128-byte line each), give-ups, then ready[m];
// zeroed before the launch (by the index pass).
constexpr int kReadyPollLimit = 1 << 20;  // about a second of polling

// M-tiles per group of the fused FFN's tile order (a group's gate/up tiles
// are walked N-tile by N-tile)
#ifndef FOE_FUSED_GM
#define FOE_FUSED_GM 4
#endif
// per-XCD work lists from this many groups of M-tiles (fewer groups leave the
// lists unbalanced, and the tail goes to taking items from other lists)
#ifndef FOE_FUSED_XCD_MIN_GROUPS
#define FOE_FUSED_XCD_MIN_GROUPS 32
#endif
constexpr int kLineInts = 32;  // one counter per 128-byte line

// Work lists of the fused FFN, one per XCD: list x holds the groups of GM
// M-tiles g = x, x+8, x+16, ... (all their gate/up tiles, then all their down
// tiles, in the tile order), so the 32 workgroups of one XCD work on the tiles
// of a few groups at a time and their A rows and weight slices meet in that
// XCD's L2.  A group's down tiles depend only on the same group's gate/up
// tiles, so every dependency stays inside one list.
struct FusedLists {
  int m_tiles, ntg, ntd, n_groups, gm;
  // groups of list x and M-tiles of its last group
  __device__ int groups(int x) const { return x < n_groups ? (n_groups - 1 - x) / 8 + 1 : 0; }
  __device__ int tiles(int x, int ntn) const {
    const int ng = groups(x);
    if (ng == 0) return 0;
    const int last = x + 8 * (ng - 1);
    return ((ng - 1) * gm + min(gm, m_tiles - last * gm)) * ntn;
  }
  __device__ int size(int x) const { return tiles(x, ntg) + tiles(x, ntd); }
  // global item (tile order: gate/up tiles, then down tiles) of item i of list
  // x, i < size(x)
  __device__ int item(int x, int i) const {
    const int ngu = tiles(x, ntg);
    if (i < ngu) return (x + 8 * (i / (gm * ntg))) * gm * ntg + i % (gm * ntg);
    i -= ngu;
    return m_tiles * ntg + (x + 8 * (i / (gm * ntd))) * gm * ntd + i % (gm * ntd);
  }
};

template <int BM, int BN, int WM, int WN, int NST, int GM>
__global__ __launch_bounds__(WM* WN* kWave) __attribute__((amdgpu_waves_per_eu(1, 2)))
void ffn_fused_dma(const bf16* __restrict__ A, const int32_t* __restrict__ gather, int kdiv,
                   int a_rows, const int32_t* __restrict__ offsets, int E, int rows,
                   const bf16* __restrict__ wg, const bf16* __restrict__ wu,
                   const bf16* __restrict__ wd, int d, int F, bf16* __restrict__ h,
                   bf16* __restrict__ y, int32_t* __restrict__ sync) {
  // one tile shape for both GEMMs: BM rows x (BN gate + BN up) columns, or
  // BM rows x 2*BN down columns read as two BN-row slices of W_d (the same
  // operand loads, LDS layout and MFMA sequence; only the epilogue differs)
  using C = DmaCfg<bf16, BM, BN, WM, WN, true, NST>;
  __shared__ __align__(1024) unsigned char smem[NST * C::STAGE];
  __shared__ int s_item[2];  // alternate slots: a slot is rewritten one barrier after it is read
  // thread 0's own: its current list, and the index it took for the next item
  // (in LDS because a tile's K loop leaves no vector register for them)
  __shared__ int s_list, s_next;
  __shared__ int s_tab[3 * kTileTab];

  // the M-tile order: the table (scratch in the stage buffers, which no DMA
  // uses yet), or experts in id order through find_tile past its capacity
  static_assert(NST * C::STAGE >= (4 * kTabMaxE + 1) * 4, "table scratch fits");
  const int mt_tab = __builtin_amdgcn_readfirstlane(build_tile_table<C::NTHR>(
      offsets, E, rows, BM, reinterpret_cast<int*>(smem), s_tab));
  auto tab_ok = [](int n) { return n >= 0 && n <= kTileTab; };
  const int m_tiles = tab_ok(mt_tab) ? mt_tab
                             : __builtin_amdgcn_readfirstlane(total_mtiles(offsets, E, rows, BM));
  const int ntg = (F + BN - 1) / BN, ntd = (d + 2 * BN - 1) / (2 * BN);
  const int n_gu = m_tiles * ntg, n_all = n_gu + m_tiles * ntd;
  // sync: list counters (one line each), give-ups, then ready[m]
  int32_t* giveups = sync + 8 * kLineInts;
  int32_t* ready = sync + 9 * kLineInts;
  const FusedLists fl{m_tiles, ntg, ntd, (m_tiles + GM - 1) / GM, GM};

  // The first item of a workgroup is fixed (a workgroup that starts early
  // cannot take two first-round items); the next item is taken while the
  // current one runs (its value is needed only at the end), so items come
  // without a wait.  With many groups (xq) workgroup b (on XCD b % 8) works
  // through list b % 8 and then takes the remaining items of the other lists
  // (measured 2.7% faster at 270 and 290 M-tiles, 8% slower at 73);
  // otherwise all items form one list.  Items of a list are taken in order.
  // Deadlock-free: a workgroup blocked on a down tile holds no unstarted
  // gate/up item (its next item was taken after its current, down, item, and
  // a list's gate/up items come before its down items), and first items
  // belong to workgroups of the grid, which run to their end.
  const bool xq = fl.n_groups >= FOE_FUSED_XCD_MIN_GROUPS;
  const int nper = xq ? (int)gridDim.x / 8 : (int)gridDim.x;
  if (threadIdx.x == 0) s_list = xq ? (int)blockIdx.x % 8 : 0;
  auto list_size = [&](int l) { return xq ? fl.size(l) : n_all; };
  auto list_item = [&](int l, int i) { return xq ? fl.item(l, i) : i; };
  // thread 0: the next item after index i of the current list (i from the
  // list's counter), or one taken from the other lists, or -1
  auto next_item = [&](int i) {
    const int list = s_list;
    if (i < list_size(list)) return list_item(list, i);
    for (int k = 1; xq && k < 8; ++k) {
      const int l = (list + k) % 8;
      const int j = nper + atomicAdd(&sync[l * kLineInts], 1);
      if (j < list_size(l)) {
        s_list = l;
        return list_item(l, j);
      }
    }
    return -1;
  };
  if (threadIdx.x == 0) {
    const int i0 = xq ? (int)blockIdx.x / 8 : (int)blockIdx.x, list = s_list;
    s_item[0] = i0 < list_size(list) ? list_item(list, i0)
                                     : next_item(nper + atomicAdd(&sync[list * kLineInts], 1));
  }
  lds_barrier();
  // The item and its tile are the same for the whole workgroup: in scalar
  // registers, since a tile leaves no vector register for what is kept across
  // it (with 24 values spilled, 8192 rows x 2 in 16 experts wrote 128 MB
  // instead of the 101 of h and y and took 199 us instead of 191).
  int t = __builtin_amdgcn_readfirstlane(s_item[0]);
  int slot = 0;
  // M-tile of this workgroup's last gate/up tile, not yet counted in ready[]:
  // it is counted at the next gate/up tile's prologue (whose wait drains the
  // stores anyway) or flushed before a wait and at the end
  int pending = -1;
  auto flush = [&]() {
    if (pending >= 0) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (threadIdx.x == 0) atomicAdd(&ready[pending], 1);
      pending = -1;
    }
  };
  while (t >= 0 && t < n_all) {
    if (threadIdx.x == 0) s_next = nper + atomicAdd(&sync[s_list * kLineInts], 1);
    const bool gu = t < n_gu;
    int mt, nt, e, row0, row_end;
    if (gu)
      tile_coords<GM>(t, ntg, m_tiles, mt, nt);
    else
      tile_coords<GM>(t - n_gu, ntd, m_tiles, mt, nt);
    bool have;
    if (tab_ok(opaque_uniform(mt_tab))) {
      e = __builtin_amdgcn_readfirstlane(s_tab[3 * mt]);
      row0 = __builtin_amdgcn_readfirstlane(s_tab[3 * mt + 1]);
      row_end = __builtin_amdgcn_readfirstlane(s_tab[3 * mt + 2]);
      have = true;
    } else {
      have = find_tile(offsets, E, rows, BM, mt, e, row0, row_end);
    }
    if (have) {
      if (!gu) {
        flush();
        if (threadIdx.x == 0) {
          int polls = 0;
          while (__hip_atomic_load(&ready[mt], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                 ntg) {
            if (++polls >= kReadyPollLimit) {
              atomicAdd(giveups, 1);
              break;
            }
            __builtin_amdgcn_s_sleep(2);
          }
        }
        __syncthreads();
      }
      // h is stored past the XCD's L2 (other XCDs read it in this launch), y
      // as usual (the next kernel reads it)
      const GemmArgs<bf16> g = gu ? GemmArgs<bf16>{A, gather, kdiv, a_rows, wg, wu, F, d, h,
                                       (uint32_t)rows * F * 2u, GemmResid{}, false}
                            : GemmArgs<bf16>{h, nullptr, 1, rows, wd, nullptr, d, F, y,
                                       (uint32_t)rows * d * 2u, GemmResid{}, true};
      gemm_tile<bf16, BM, BN, WM, WN, true, NST, false, kScDevice>(
          smem, g, e, row0, row_end, nt, gu && pending >= 0 ? &ready[pending] : nullptr);
      if (gu) pending = mt;
    }
    // the next item in LDS; this item's LDS use is done everywhere
    slot ^= 1;
    if (threadIdx.x == 0) s_item[slot] = next_item(s_next);
    lds_barrier();
    t = __builtin_amdgcn_readfirstlane(s_item[slot]);
  }
  flush();
}

// Few rows per expert (decode), LDS-staged weight stream.  A workgroup of 4
// waves takes one expert and 4 consecutive weight tiles (each 16 gate + 16 up
// rows, or 32 down rows), one per wave, over all of K, for up to 32 rows of A
// (tokens) at a time.  Operands stream through a ring of NS LDS stages of
// 128 K columns: per stage each wave loads its weight tile with 8 LDS-DMA
// instructions and a quarter of the shared token tile with 2, each
// instruction covering 4 rows x 256 bytes (the access pattern that reads HBM
// fastest).  The 16-byte chunk c of row r of any tile sits in slot
// c ^ (r & 15), so the v_mfma_f32_16x16x32_bf16 fragment reads (16 rows, one
// chunk) are conflict-free.
//
// All loads of the loop are LDS DMA issued from inline assembly with explicit
// vmcnt waits, so NS-2 later stages stay in flight while a stage is used.

// Expert whose workgroups list a pair (selection mode).  A pair without an expert
// (id -1: its token's scores are NaN) goes to the first one, so that its token's
// arrivals become complete and the output row is written; the combine leaves
// it out.
__device__ __forceinline__ int listed_expert(int id, int E) {
  return (unsigned)id < (unsigned)E ? id : 0;
}

// What such a pair adds to its token's arrival count besides one: above any C*k, and
// C*k of them stay below 2^31 (C <= 64, k <= 256).
constexpr int kNoExpert = 1 << 15;

template <bool GATEUP, int NS, bool SEL, bool SLOTS = false, bool PARTS = false>
__global__ __launch_bounds__(256) void ffn_stream_bf16(
    const bf16* __restrict__ A, const int32_t* __restrict__ gather, int kdiv, int a_rows,
    const int32_t* __restrict__ offsets, int E, int rows, const bf16* __restrict__ W0,
    const bf16* __restrict__ W1, int N, int K, bf16* __restrict__ out, int n_groups,
    int e_per_c, int r_sel, int slots, FusedCombine fc) {
  static_assert(NS >= 2 && NS <= 4, "2 to 4 stages");
  constexpr int WPB = 4;
  constexpr int NPW = GATEUP ? 16 : 32;  // output columns per wave
  constexpr int WB = 8192;                // weight bytes per stage and wave
  constexpr int XB = WPB * WB;            // offset of the token rows in a stage
  constexpr int SB = XB + 8192;           // bytes per stage
  constexpr int NI = 10;                  // DMA instructions per stage and wave
  constexpr int SELB = SEL ? kSelMax * 4 : 0;       // staged expert ids of the cluster
  constexpr int LSTB = SEL ? kSelMax * 4 + 64 : 0;  // pair list + wave counts
  static_assert(NS * SB + SELB + LSTB <= 160 * 1024, "LDS capacity");
  __shared__ __align__(1024) unsigned char smem[NS * SB + SELB + LSTB];

  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  const int gpe = (n_groups + WPB - 1) / WPB;                           // workgroups per expert
  const int n0 = ((blockIdx.x % gpe) * WPB + wave) * NPW;
  // expert e of all clusters; selection mode: expert le of cluster hc
  int e = blockIdx.x / gpe, hc = 0, le = 0;
  [[maybe_unused]] uint64_t pairs = 0;  // (SLOTS) the expert's pairs of the cluster, one bit each
  if constexpr (SEL) {
    if constexpr (SLOTS) {
      // Few pairs (at most 64 per cluster): a workgroup takes the s-th
      // distinct expert of its cluster, so none is launched for most of the
      // experts without rows, and none of those loads weights.  Lane j holds
      // pair j's expert; experts are numbered by their first pair.
      hc = e / slots;
      const int s = e - hc * slots;
      const bool ok = lane < r_sel;
      const int id = ok ? listed_expert(gather[(size_t)hc * r_sel + lane], e_per_c) : -1;
      uint64_t same = __ballot(ok);
      for (int b = 0; (1 << b) < e_per_c; ++b) {
        const uint64_t bb = __ballot((id >> b) & 1);
        same &= ((id >> b) & 1) ? bb : ~bb;
      }
      const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
      uint64_t first = __ballot(ok && (same & below) == 0);
      for (int i = 0; i < s; ++i) first &= first - 1;
      if (first == 0) return;  // the same in every wave
      const int at = __builtin_ctzll(first);
      le = __builtin_amdgcn_readlane(id, at);
      pairs = __ballot(ok && id == le);
      e = hc * e_per_c + le;
    } else {
      hc = e / e_per_c;
      le = e - hc * e_per_c;
    }
  }
  if (e >= E) return;
  int off_a = 0, off_b = 0;
  if constexpr (!SEL) {
    off_a = offsets[e];  // scalar loads, waited on below
    off_b = offsets[e + 1];
  }
  const uint32_t lds0 = lds_addr(smem);
  if constexpr (SEL && !SLOTS) {
    // the cluster's r_sel expert ids go to LDS first (256 per wave instruction)
    const __amdgpu_buffer_rsrc_t sr =
        make_rsrc_u(gather + (size_t)hc * r_sel, (uint32_t)r_sel * 4u);
    rsrc_settle(sr);
    for (int c = wave * 256; c < r_sel; c += WPB * 256)
      dma16(sr, (uint32_t)(c + 4 * lane) * 4u, lds0 + NS * SB + c * 4, 0);
  }

  // weight sources: instruction i < 4 reads tile rows 4i.. of W0, i >= 4 rows
  // 4(i-4).. of W1 (gate/up) or rows 4i.. of W0 (down); a wave past N reads
  // zeros (empty range)
  const int nv = max(min(NPW, N - n0), 0);
  const size_t wrow = (size_t)e * N + min(n0, N);
  const __amdgpu_buffer_rsrc_t wr0 = make_rsrc_u(W0 + wrow * K, (uint32_t)nv * K * 2u);
  const __amdgpu_buffer_rsrc_t wr1 =
      GATEUP ? make_rsrc_u(W1 + wrow * K, (uint32_t)nv * K * 2u) : wr0;
  const __amdgpu_buffer_rsrc_t ar = make_rsrc_u(A, (uint32_t)a_rows * K * 2u);
  // output rows of the folded combine (down, selection mode)
  const __amdgpu_buffer_rsrc_t yr = make_rsrc_u(out, (uint32_t)rows * N * 2u);
  rsrc_settle(wr0, wr1);
  const int lr = lane >> 4, lc = lane & 15;
  uint32_t wv[8];  // byte offset of this lane's weight chunk in instruction i (stage 0)
  int wk[8];       // its K column
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int tr = (GATEUP ? (i & 3) : i) * 4 + lr;  // row inside the rsrc range
    const int q = lc ^ (tr & 15);                     // chunk of the 256-byte segment
    wk[i] = q * 8;
    wv[i] = ((uint32_t)tr * K + q * 8) * 2u;
  }
  const int nks = (K + 127) / 128;
  // Workgroups start their K walk at different chunks, so the reads in flight
  // at any moment are spread over all column offsets of the 4 KB-strided
  // weight rows (and so over the HBM channels) instead of one.
  const int rot = FOE_STREAM_ROT ? (int)(blockIdx.x % (unsigned)nks) : 0;
  auto chunk0 = [&](int kt) {
    const int kc = kt + rot;
    return (kc >= nks ? kc - nks : kc) * 128;
  };
  // fragment read offsets inside a stage: row R of a 16-row tile
  const int R = lane & 15, g = lane >> 4;
  const int rbase = (R >> 2) * 1024 + (R & 3) * 256;

  auto issue_w = [&](int kt, int s) {
    const int k0 = chunk0(kt);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t off = k0 + wk[i] < K ? wv[i] + (uint32_t)k0 * 2u : kOob;
      dma16(GATEUP && i >= 4 ? wr1 : wr0, off, lds0 + wave * WB, s * SB + i * 1024);
    }
  };
  // The weights of the first NS-1 stages do not depend on the token rows:
  // they go out before the segment bounds and gather indices are read.
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nks) issue_w(s, s);
  rsrc_settle(ar);
  int a = 0, b = 0;
  const int* lst = reinterpret_cast<const int*>(smem + NS * SB + SELB);
  if constexpr (SEL) {
    // Pair list of this expert in ascending pair order (the stable order of
    // the dispatch): per 256-pair chunk, each wave ballots its matches and
    // the wave counts give the positions.  The weight DMAs stay in flight.
    int* lw = reinterpret_cast<int*>(smem + NS * SB + SELB);
    int* wc = lw + kSelMax;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    int n = 0;
    if constexpr (SLOTS) {  // every wave writes the same list
      if ((pairs >> lane) & 1) lw[__popcll(pairs & below)] = lane;
      n = __popcll(pairs);
      lds_barrier();
    } else {
      if (nks >= NS - 1) vm_wait<8 * (NS - 1)>();
      else vm_wait<0>();
      lds_barrier();
    }
    const int* sel = reinterpret_cast<const int*>(smem + NS * SB);
    for (int c0 = 0; !SLOTS && c0 < r_sel; c0 += WPB * 64) {
      const int f = c0 + (int)threadIdx.x;
      const bool ok = f < r_sel && listed_expert(sel[f], e_per_c) == le;
      const uint64_t m = __ballot(ok);
      if (lane == 0) wc[wave] = __popcll(m);
      lds_barrier();
      int pre = 0, tot = 0;
#pragma unroll
      for (int w = 0; w < WPB; ++w) {
        const int cw = wc[w];
        pre += w < wave ? cw : 0;
        tot += cw;
      }
      if (ok) lw[n + pre + __popcll(m & below)] = f;
      n += tot;
      lds_barrier();
    }
    b = n;
  } else {
    a = min(max(off_a, 0), rows);
    b = max(min(max(off_b, 0), rows), a);
  }
  // (PARTS) the passes of 32 rows are dealt to the parts of the grid
  const int first = a + (PARTS ? (int)blockIdx.y * 32 : 0);
  const int stride = PARTS ? (int)gridDim.y * 32 : 32;
  if (first >= b) {  // uniform over the workgroup; the DMAs land before LDS is released
    vm_wait<0>();
    return;
  }

  for (int t0 = first; t0 < b; t0 += stride) {
    const int tv = min(32, b - t0);
    if (t0 != first) {
#pragma unroll
      for (int s = 0; s < NS - 1; ++s)
        if (s < nks) issue_w(s, s);
    }
    // token instructions 2*wave and 2*wave+1 of this wave (rows 8*wave + 4u +
    // lane/16 of the pass); the wave's 8 gather indices are uniform loads
    uint32_t xv[2];
    int xk[2];
    if constexpr (SEL) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int t = 8 * wave + 4 * u + lr;
        const int q = lc ^ (t & 15);
        int sr = -1;
        if (t < tv) {
          const int f = lst[t0 + t];
          sr = GATEUP ? f / kdiv : hc * r_sel + f;
          if (sr >= a_rows) sr = -1;
        }
        xk[u] = q * 8;
        xv[u] = sr < 0 ? kOob : ((uint32_t)sr * K + q * 8) * 2u;
      }
    } else {
      const int tw = 8 * wave;
      int gi[8];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        gi[j] = (gather != nullptr && tw + j < tv) ? gather[t0 + tw + j] : t0 + tw + j;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int t = tw + 4 * u + lr;
        const int q = lc ^ (t & 15);
        const int gsel = lr == 0 ? gi[4 * u] : lr == 1 ? gi[4 * u + 1] : lr == 2 ? gi[4 * u + 2]
                                                                                 : gi[4 * u + 3];
        int sr = -1;
        if (t < tv) {
          sr = gather == nullptr ? gsel : (gsel >= 0 ? gsel / kdiv : -1);
          if (sr >= a_rows) sr = -1;
        }
        xk[u] = q * 8;
        xv[u] = sr < 0 ? kOob : ((uint32_t)sr * K + q * 8) * 2u;
      }
    }
    auto issue_x = [&](int kt, int s) {
      const int k0 = chunk0(kt);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t off = (k0 + xk[u] < K && xv[u] != kOob) ? xv[u] + (uint32_t)k0 * 2u : kOob;
        dma16(ar, off, lds0 + wave * 2048, s * SB + XB + u * 1024);
      }
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < nks) issue_x(s, s);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // iteration kt: wait for this wave's part of stage kt, meet the other
    // waves (stage kt complete, stage kt-1 no longer read), issue stage
    // kt+NS-1 into the buffer of stage kt-1, use stage kt.  The pass starts
    // with the weights of stages 0..NS-2 and then their token rows, so stage
    // u < NS-1 still has 2*(NS-2-u) token and u*NI loop instructions behind it.
    auto body = [&](int kt, auto U, int s_next) {
      constexpr int u = decltype(U)::value;
      if (kt + NS - 2 >= nks) vm_wait<0>();
      else if (u < NS - 1 && kt == u) vm_wait<2 * (NS - 2 - u) + NI * u>();
      else vm_wait<NI * (NS - 2)>();
      lds_barrier();
      if (kt + NS - 1 < nks) {
        issue_w(kt + NS - 1, s_next);
        issue_x(kt + NS - 1, s_next);
      }
      const unsigned char* src = smem + u * SB + rbase;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int slot = ((c * 4 + g) ^ R) * 16;
        const bf16x8 w0 = *reinterpret_cast<const bf16x8*>(src + wave * WB + slot);
        const bf16x8 w1 = *reinterpret_cast<const bf16x8*>(src + wave * WB + 4096 + slot);
        const bf16x8 x0 = *reinterpret_cast<const bf16x8*>(src + XB + slot);
        const bf16x8 x1 = *reinterpret_cast<const bf16x8*>(src + XB + 4096 + slot);
        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, x0, acc[0][0], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x0, acc[1][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, x1, acc[0][1], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x1, acc[1][1], 0, 0, 0);
      }
    };
    for (int kt0 = 0; kt0 < nks; kt0 += NS) {
      static_for<0, NS>([&](auto U) {
        constexpr int u = decltype(U)::value;
        const int kt = kt0 + u;
        if (kt < nks) body(kt, U, (u + NS - 1) % NS);
      });
    }
    // every wave is done with the ring before the next pass refills it
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // lane holds weight rows 4*(lane/16) + [0,4) of each tile for token lane%16 (+16)
    const int nb = 4 * g;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int t = j * 16 + R;
      if (t >= tv) continue;
      const int orow_i = SEL ? hc * r_sel + lst[t0 + t] : t0 + t;
      bf16* orow = out + (size_t)orow_i * N + n0;
      if constexpr (GATEUP) {
        if (nb < nv) {
          bf16x4 o;
#pragma unroll
          for (int v = 0; v < 4; ++v) o[v] = (bf16)(silu_f(acc[0][j][v]) * acc[1][j][v]);
          *reinterpret_cast<bf16x4*>(orow + nb) = o;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (i * 16 + nb >= nv) continue;
          bf16x4 o;
#pragma unroll
          for (int v = 0; v < 4; ++v) o[v] = (bf16)acc[i][j][v];
          if (SEL && fc.out != nullptr)  // device-scope store: read back by other workgroups
            __builtin_amdgcn_raw_buffer_store_b64(
                __builtin_bit_cast(u32x2, o), yr,
                (uint32_t)(((size_t)orow_i * N + n0 + i * 16 + nb) * 2), 0, kScDevice);
          else
            *reinterpret_cast<bf16x4*>(orow + i * 16 + nb) = o;
        }
      }
    }
  }

  if constexpr (!GATEUP && SEL) {
    if (fc.out != nullptr) {
      // Combine folded in: this workgroup's y columns [cg*128, +128) of its
      // pairs are stored (device-scope stores, past the XCD's own L2, and
      // acknowledged once visible to every XCD); count one arrival per (token,
      // column group).  The workgroup that brings a count to C*k forms that
      // token's output columns from device-scope loads of the y rows, summing
      // the k rows of every cluster in the fixed order (h, j) exactly as the
      // combine kernel does.  Nothing waits on another workgroup.
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int cg = blockIdx.x % gpe;
      int* done = reinterpret_cast<int*>(smem + NS * SB);  // staged ids are dead
      int* ndone = reinterpret_cast<int*>(smem + NS * SB + SELB) + kSelMax;
      if (threadIdx.x == 0) *ndone = 0;
      __syncthreads();
      const int need = fc.C * fc.k;
      // (PARTS: this part's rows, 32 of every `stride` from `first`)
      const int mine = PARTS ? (b - first + stride - 1) / stride * 32 : b;
      for (int j = (int)threadIdx.x; j < mine; j += WPB * 64) {
        const int i = PARTS ? first + j / 32 * stride + j % 32 : j;
        if (PARTS && i >= b) continue;
        const int t = lst[i] / fc.k;
        // a pair without an expert is marked in the count's upper half (the first
        // expert lists it), so that only its token's combine looks at the ids
        int one = 1;
        if (le == 0) {
          const int id = gather[(size_t)hc * r_sel + lst[i]];
          if (id != listed_expert(id, e_per_c)) one += kNoExpert;
        }
        const int sum = atomicAdd(&fc.cnt[(size_t)t * gpe + cg], one) + one;
        if (sum % kNoExpert == need) done[atomicAdd(ndone, 1)] = sum > need ? ~t : t;
      }
      __syncthreads();
      const int nd = *ndone;
      if (nd > 0) {
        const int c0 = cg * 128;
        const int nvec = (min(128, N - c0) + 7) / 8;
        const float cx = (float)fc.C;
        for (int it = (int)threadIdx.x; it < nd * 16; it += WPB * 64) {
          const int v = it & 15;
          if (v >= nvec) continue;
          const int t0 = done[it >> 4], t = t0 < 0 ? ~t0 : t0;
          const int col = c0 + v * 8;
          float acc[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) acc[q] = 0.f;
          const bf16x8 xv = *reinterpret_cast<const bf16x8*>(fc.x + (size_t)t * N + col);
          // the token's rows in the order (h, j), NB of them in flight (one at
          // a time, their latencies added up: 1 token with 16 rows of 8 clusters,
          // 22.5 -> 18.6 us for the kernel)
          constexpr int NB = 8;
          for (int q0 = 0; q0 < need; q0 += NB) {
            bf16x8 yv[NB];
            float wq[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) {
              if (q0 + u < need) {
                const int h = (q0 + u) / fc.k, j = q0 + u - h * fc.k;
                const size_t p = (size_t)h * r_sel + (size_t)t * fc.k + j;
                wq[u] = fc.w[p];
                yv[u] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                yr, (uint32_t)((p * N + col) * 2), 0, kScDevice));
              }
            }
            if (t0 < 0) {  // some of its pairs have no expert: they add nothing
#pragma unroll
              for (int u = 0; u < NB; ++u) {
                const int h = (q0 + u) / fc.k, j = q0 + u - h * fc.k;
                if (q0 + u >= need) break;
                const int id = gather[(size_t)h * r_sel + (size_t)t * fc.k + j];
                if (id != listed_expert(id, e_per_c)) {
                  wq[u] = 0.f;
                  yv[u] = bf16x8{};
                }
              }
            }
#pragma unroll
            for (int u = 0; u < NB; ++u) {
              if (q0 + u < need) {
#pragma unroll
                for (int q = 0; q < 8; ++q) acc[q] = fmaf(wq[u], (float)yv[u][q], acc[q]);
              }
            }
          }
          bf16x8 o;
#pragma unroll
          for (int q = 0; q < 8; ++q) o[q] = (bf16)(fc.scale * fmaf(cx, (float)xv[q], acc[q]));
          *reinterpret_cast<bf16x8*>(fc.out + (size_t)t * N + col) = o;
        }
      }
    }
  }
}


// ---- fp32 with operands past the tiled kernel's 2 GiB offsets: plain FMA ------
__device__ int expert_of_row(const int32_t* __restrict__ offsets, int E, int rows, int row) {
  for (int e = 0; e < E; ++e) {
    int a = min(max(offsets[e], 0), rows);
    int b = min(max(offsets[e + 1], 0), rows);
    if (row >= a && row < b) return e;
  }
  return -1;
}

__global__ __launch_bounds__(256) void gateup_f32(const float* __restrict__ A,
                                                  const int32_t* __restrict__ gather, int kdiv,
                                                  int a_rows, const int32_t* __restrict__ offsets,
                                                  int E, int rows, const float* __restrict__ wg,
                                                  const float* __restrict__ wu, int F, int d,
                                                  float* __restrict__ h) {
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (long long)rows * F) return;
  const int row = (int)(id / F), n = (int)(id % F);
  const int e = expert_of_row(offsets, E, rows, row);
  if (e < 0) return;
  const int s = src_row(gather, kdiv, row, a_rows);
  const float* g = wg + ((size_t)e * F + n) * d;
  const float* u = wu + ((size_t)e * F + n) * d;
  float ag = 0.f, au = 0.f;
  if (s >= 0) {
    const float* xr = A + (size_t)s * d;
    for (int i = 0; i < d; ++i) {
      ag = fmaf(xr[i], g[i], ag);
      au = fmaf(xr[i], u[i], au);
    }
  }
  h[(size_t)row * F + n] = ag / (1.0f + expf(-ag)) * au;
}

__global__ __launch_bounds__(256) void down_f32(const float* __restrict__ h,
                                                const int32_t* __restrict__ offsets, int E,
                                                int rows, const float* __restrict__ wd, int d,
                                                int F, float* __restrict__ y) {
  const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (long long)rows * d) return;
  const int row = (int)(id / d), c = (int)(id % d);
  const int e = expert_of_row(offsets, E, rows, row);
  if (e < 0) return;
  const float* hr = h + (size_t)row * F;
  const float* w = wd + ((size_t)e * d + c) * F;
  float acc = 0.f;
  for (int i = 0; i < F; ++i) acc = fmaf(hr[i], w[i], acc);
  y[(size_t)row * d + c] = acc;
}

// compute units of the current device (one persistent workgroup each)
int device_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8)
    return 256;
  return n / 8 * 8;
}

template <int BM, int BN, int WM, int WN, int NST, int GM, int PERSIST, bool GATEUP,
          bool RESID = false, typename T>
void launch_gemm_dma(const T* A, const int32_t* gather, int kdiv, int a_rows,
                     const int32_t* offsets, int E, int rows, const T* B0, const T* B1,
                     int N, int K, T* out, hipStream_t s, const char* name,
                     GemmResid res = GemmResid{}) {
  const int ntn = ceil_div(N, BN);
  const int max_mt = ceil_div(rows, BM) + E;  // sum_e ceil(M_e/BM) <= rows/BM + E
  const long long n_tiles = (long long)max_mt * ntn;
  long long nb = (n_tiles + 7) / 8 * 8;
  if (PERSIST) {
    // as many workgroups as the CUs hold at once: by LDS, and two waves a SIMD
    using C = DmaCfg<T, BM, BN, WM, WN, GATEUP, NST>;
    constexpr int by_lds = 160 * 1024 / (NST * C::STAGE), by_waves = 8 / C::NW;
    constexpr int per_cu = by_lds < by_waves ? by_lds : by_waves;
    static const int slots = device_cus() * (per_cu > 1 ? per_cu : 1);
    nb = nb < slots ? nb : slots;
  }
  dim3 grid((unsigned)nb);
  ProfileScope ps(name, s);
  FOE_LAUNCH((grouped_gemm_dma<T, BM, BN, WM, WN, GATEUP, NST, GM, PERSIST, RESID>),
             grid, dim3(WM * WN * kWave), 0, s, A, gather, kdiv, a_rows, offsets, E, rows, B0, B1,
             N, K, out, ntn, (int)n_tiles, res);
}

template <int BM, int BN, int WM, int WN, int NST, int GM, int PERSIST>
struct DmaLaunch {
  template <bool GATEUP, bool RESID = false, typename... Args>
  static void run(Args... args) {
    launch_gemm_dma<BM, BN, WM, WN, NST, GM, PERSIST, GATEUP, RESID>(args...);
  }
};

// Calls f with the tile size (0 = 64 x 128, 1 = 128 x 128, 2 = bm x bn) of a
// plain product of E equal segments (see FOE_DMA_SMALL).
template <typename F>
void pick_tile(int E, int rows, int N, int bm, int bn, F&& f) {
  static const int cus = device_cus();
  auto tiles = [&](int m, int n) {
    return (long long)E * ceil_div(rows, (long long)m * E) * ceil_div(N, n);
  };
  if (tiles(64, 128) <= cus) f(std::integral_constant<int, 0>{});
  else if (tiles(bm, bn) < cus) f(std::integral_constant<int, 1>{});
  else f(std::integral_constant<int, 2>{});
}

}  // namespace

FfnForm ffn_form(int E, int d, int F, long long rows) {
  static const int cus = device_cus();
  return ffn_form(E, d, F, rows, cus);
}

size_t ffn_scratch_bytes(foe_dtype dt, int rows, int F) {
  return align_up((size_t)rows * F * (dt == FOE_BF16 ? 2 : 4), 256);
}

hipError_t launch_expert_ffn_ex(foe_dtype dt, int E, int d, int F, int rows, const void* A,
                                const int32_t* gather, int kdiv, int a_rows,
                                const int32_t* offsets, const void* w_gate, const void* w_up,
                                const void* w_down, void* y_perm, void* scratch, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  if (dt == FOE_F32) {
    float* h = reinterpret_cast<float*>(scratch);
    // fp32 products on the matrix cores through the tiled kernel (768 rows, 8
    // experts, d 768, F 512: gate/up 2540 -> 21 us, down 1200 -> 14; 8192 rows,
    // 16 experts, d = F = 1024: 316 + 163 us, 108 TFLOP/s; 64-row tiles, two
    // workgroups per CU: 128-row ones took 31 + 24 and 362 + 200).  A thread
    // per output read a weight row of its own, 64 rows to a wave instruction.
    if (f32_tiled(d, F, gather == nullptr ? 0 : a_rows)) {
      const float* xa = reinterpret_cast<const float*>(A);
      DmaLaunch<FOE_F32_GU>::run<true>(xa, gather, kdiv, a_rows, offsets, E, rows,
                                       reinterpret_cast<const float*>(w_gate),
                                       reinterpret_cast<const float*>(w_up), F, d, h, s,
                                       "ffn_gateup_f32");
      DmaLaunch<FOE_F32_DN>::run<false>(static_cast<const float*>(h), (const int32_t*)nullptr, 1,
                                        rows, offsets, E, rows,
                                        reinterpret_cast<const float*>(w_down),
                                        (const float*)nullptr, d, F,
                                        reinterpret_cast<float*>(y_perm), s, "ffn_down_f32");
      return hipGetLastError();
    }
    {
      ProfileScope ps("ffn_gateup_f32", s);
      FOE_LAUNCH(gateup_f32, dim3(ceil_div((long long)rows * F, 256)), dim3(256), 0, s,
                         reinterpret_cast<const float*>(A), gather, kdiv, a_rows, offsets, E,
                         rows, reinterpret_cast<const float*>(w_gate),
                         reinterpret_cast<const float*>(w_up), F, d, h);
    }
    {
      ProfileScope ps("ffn_down_f32", s);
      FOE_LAUNCH(down_f32, dim3(ceil_div((long long)rows * d, 256)), dim3(256), 0, s, h,
                         offsets, E, rows, reinterpret_cast<const float*>(w_down), d, F,
                         reinterpret_cast<float*>(y_perm));
    }
    return hipGetLastError();
  }
  const bf16* xa = reinterpret_cast<const bf16*>(A);
  const bf16* wg = reinterpret_cast<const bf16*>(w_gate);
  const bf16* wu = reinterpret_cast<const bf16*>(w_up);
  const bf16* wd = reinterpret_cast<const bf16*>(w_down);
  bf16* h = reinterpret_cast<bf16*>(scratch);
  bf16* y = reinterpret_cast<bf16*>(y_perm);
  const FfnForm form = ffn_form(E, d, F, rows);
  if (form == FfnForm::kStream) {
    {
      const int ng = ceil_div(F, 16);
      ProfileScope ps("ffn_gateup", s);
      FOE_LAUNCH((ffn_stream_bf16<true, FOE_STREAM_NS, false>), dim3(E * ceil_div(ng, 4)),
                 dim3(256), 0, s, xa, gather, kdiv, a_rows, offsets, E, rows, wg, wu, F, d, h,
                 ng, 1, 0, 0, FusedCombine{});
    }
    {
      const int ng = ceil_div(d, 32);
      ProfileScope ps("ffn_down", s);
      FOE_LAUNCH((ffn_stream_bf16<false, FOE_STREAM_NS, false>), dim3(E * ceil_div(ng, 4)),
                 dim3(256), 0, s, static_cast<const bf16*>(h), nullptr, 1, rows, offsets, E,
                 rows, wd, nullptr, d, F, y, ng, 1, 0, 0, FusedCombine{});
    }
  } else if (form == FfnForm::kMid) {
    DmaLaunch<FOE_MID_GU>::run<true>(xa, gather, kdiv, a_rows, offsets, E, rows, wg, wu, F, d, h,
                                     s, "ffn_gateup");
    DmaLaunch<FOE_MID_DN>::run<false>(static_cast<const bf16*>(h), (const int32_t*)nullptr, 1,
                                      rows, offsets, E, rows, wd, (const bf16*)nullptr, d, F, y, s,
                                      "ffn_down");
  } else {
    DmaLaunch<FOE_DMA_GU>::run<true>(xa, gather, kdiv, a_rows, offsets, E, rows, wg, wu, F, d, h,
                                     s, "ffn_gateup");
    DmaLaunch<FOE_DMA_DN>::run<false>(static_cast<const bf16*>(h), (const int32_t*)nullptr, 1,
                                      rows, offsets, E, rows, wd, (const bf16*)nullptr, d, F, y, s,
                                      "ffn_down");
  }
  return hipGetLastError();
}

size_t ffn_sync_ints(int E, int rows) { return (size_t)ceil_div(rows, 256) + E + 9 * kLineInts; }

hipError_t launch_expert_ffn_fused(int E, int d, int F, int rows, const void* A,
                                   const int32_t* gather, int kdiv, int a_rows,
                                   const int32_t* offsets, const void* w_gate, const void* w_up,
                                   const void* w_down, void* y, void* h, int32_t* sync,
                                   hipStream_t s) {
  if (rows == 0) return hipSuccess;
  static const int cus = device_cus();
  ProfileScope ps("ffn_fused", s);
  FOE_LAUNCH((ffn_fused_dma<256, 128, 2, 4, 2, FOE_FUSED_GM>), dim3(cus),
             dim3(8 * kWave), 0, s,
             static_cast<const bf16*>(A), gather, kdiv, a_rows, offsets, E, rows,
             static_cast<const bf16*>(w_gate), static_cast<const bf16*>(w_up),
             static_cast<const bf16*>(w_down), d, F, static_cast<bf16*>(h),
             static_cast<bf16*>(y), sync);
  return hipGetLastError();
}

bool ffn_sel_ok(foe_dtype dt, int C, int E, int T, int k, int d, int F) {
  const long long R = (long long)T * k;
  if (!FOE_FFN_SEL || dt != FOE_BF16 || R <= 0 || R > kSelMax) return false;
  static const int cus = device_cus();
  return ffn_form(C * E, d, F, C * R, cus) == FfnForm::kStream ||
         stream_spreads(C, E, (int)R, d, F, cus);
}

hipError_t launch_expert_ffn_sel(int C, int E, int d, int F, int T, int k, const void* x,
                                 const int32_t* topk_idx, const void* w_gate, const void* w_up,
                                 const void* w_down, void* y, void* scratch, hipStream_t s,
                                 const FusedCombine& fc) {
  const int R = T * k;
  const int rows = C * R;
  const bf16* xa = static_cast<const bf16*>(x);
  const bf16* wg = static_cast<const bf16*>(w_gate);
  const bf16* wu = static_cast<const bf16*>(w_up);
  const bf16* wd = static_cast<const bf16*>(w_down);
  bf16* h = static_cast<bf16*>(scratch);
  bf16* yo = static_cast<bf16*>(y);
  // Workgroups by distinct experts of the pairs instead of by expert: reading
  // the ids before the first weights costs every workgroup about 0.7 us, and
  // an expert without rows otherwise takes an eighth of the weight traffic of
  // one with rows (the stages issued before its list is known), so it pays
  // while more than about a fifth of the experts stay empty (e^(-R/E)).  One
  // token, 8 clusters of 16 experts, d 2048, F 1024: gate/up 48 -> 25 us, down
  // 41 -> 21; 4 tokens 89 -> 80 and 60 -> 53; 16 tokens (not taken): 163 + 95.
  const int slots = R <= kWave && 2 * R < 3 * E ? (R < E ? R : E) : 0;
  const int per_c = slots > 0 ? slots : E;
  static const int cus = device_cus();
  auto grid = [&](int ng) {
    const int wgs = C * per_c * ceil_div(ng, 4);
    return dim3(wgs, stream_parts(R, E, wgs, cus));
  };
  auto go = [&](auto by_slot, auto in_parts) {
    constexpr bool SLOTS = decltype(by_slot)::value, PARTS = decltype(in_parts)::value;
    {
      const int ng = ceil_div(F, 16);
      ProfileScope ps("ffn_gateup", s);
      FOE_LAUNCH((ffn_stream_bf16<true, FOE_STREAM_NS, true, SLOTS, PARTS>),
                 grid(ng), dim3(256), 0, s, xa, topk_idx, k, T, nullptr,
                 C * E, rows, wg, wu, F, d, h, ng, E, R, slots, FusedCombine{});
    }
    {
      const int ng = ceil_div(d, 32);
      ProfileScope ps("ffn_down", s);
      FOE_LAUNCH((ffn_stream_bf16<false, FOE_STREAM_NS, true, SLOTS, PARTS>),
                 grid(ng), dim3(256), 0, s, static_cast<const bf16*>(h),
                 topk_idx, 1, rows, nullptr, C * E, rows, wd, nullptr, d, F, yo, ng, E, R, slots,
                 fc);
    }
  };
  // (from 32 rows per expert on; a form of its own, since decode steps lose 2% to
  // the arithmetic: 128 tokens, 16 experts 49.2 -> 50.2 us)
  if (R >= 32 * E) go(std::false_type{}, std::true_type{});
  else if (slots > 0) go(std::true_type{}, std::false_type{});
  else go(std::false_type{}, std::false_type{});
  return hipGetLastError();
}

hipError_t launch_grouped_gemm(const void* A, const int32_t* offsets, int E, int rows,
                               const void* W, int N, int K, void* out, hipStream_t s,
                               const char* name) {
  if (rows == 0) return hipSuccess;
  pick_tile(E, rows, N, 256, 256, [&](auto size) {
    auto go = [&](auto cfg) {
      decltype(cfg)::template run<false>(static_cast<const bf16*>(A), (const int32_t*)nullptr, 1,
                                         rows, offsets, E, rows, static_cast<const bf16*>(W),
                                         (const bf16*)nullptr, N, K, static_cast<bf16*>(out), s,
                                         name);
    };
    if constexpr (size.value == 0) go(DmaLaunch<FOE_DMA_TINY, 2>{});
    else if constexpr (size.value == 1) go(DmaLaunch<FOE_DMA_SMALL, 2>{});
    else go(DmaLaunch<FOE_DMA_SEG>{});
  });
  return hipGetLastError();
}

hipError_t launch_gemm_resid(const void* A, const int32_t* offsets, int rows, const void* W,
                             int N, int K, const float* x, float scale, void* out, hipStream_t s,
                             const char* name) {
  if (rows == 0) return hipSuccess;
  GemmResid res;
  res.x = x;
  res.scale = scale;
  pick_tile(1, rows, N, 128, 256, [&](auto size) {
    auto go = [&](auto cfg) {
      decltype(cfg)::template run<false, true>(
          static_cast<const bf16*>(A), (const int32_t*)nullptr, 1, rows, offsets, 1, rows,
          static_cast<const bf16*>(W), (const bf16*)nullptr, N, K, static_cast<bf16*>(out), s,
          name, res);
    };
    if constexpr (size.value == 0) go(DmaLaunch<FOE_DMA_TINY, 1>{});
    else if constexpr (size.value == 1) go(DmaLaunch<FOE_DMA_SMALL, 1>{});
    else go(DmaLaunch<FOE_DMA_RES>{});
  });
  return hipGetLastError();
}

hipError_t launch_expert_ffn(foe_dtype dt, int E, int d, int F, int rows, const void* x_perm,
                             const int32_t* offsets, const void* w_gate, const void* w_up,
                             const void* w_down, void* y_perm, void* scratch, hipStream_t s) {
  return launch_expert_ffn_ex(dt, E, d, F, rows, x_perm, nullptr, 1, rows, offsets, w_gate, w_up,
                              w_down, y_perm, scratch, s);
}

}  // namespace foe
