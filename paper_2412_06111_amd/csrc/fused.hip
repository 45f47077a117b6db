// Fused one-pass STTNN sketch for trees whose first root child A covers modes
// (1, 2) with two one-mode leaf children (e.g. ((1,2),(3,4)) and ((1,2),(3,(4,5)))).
//
// With M = T^{A} (n_A x n_B, n_A = n_1 n_2, column-major), the nodes A, {1}, {2}
// have S = {}, {}, {{1}} (Sec. 5, Fig. 5), so one pass over M produces
//   R_A = M X_A                                   (Sec. 5: A is sketched on T itself)
//   Z_A = Y_A^T M       -- the contraction T x_A Y_A^T reused by every node right of A
//   R_1 = T^{1} X_1     -- sum over columns of (n_1 x n_2 slab) . X_1 rows
//   R_2 = (T x_1 Y_1^T)^{2} X_2  -- Z1 = Y_1^T slab kept on chip, then Z1 . X_2 rows
// R_B and the right subtree (and the root sketch) follow from Z_A on the generic path.
//
// TTNN mode (template flag TT): R_A, Z_A and R_1 are the same sketches in TTNN (their
// reuse sets are empty), and for a root with two children R_B = T^{(B)} X_B with X_B
// rows over i_A, so R_B^T = X_B^T M is formed like Z_A, by the waves that STTNN spends
// on Z1.  The leaves right of A ({2} and the subtree of B) follow on the other paths.
//
// Each workgroup streams a tile of M (B2 slabs, one i2 and all of i1 each, by a range
// of columns) through LDS once; every product is an MFMA chain on that LDS tile:
//   (a)+(c) share the A fragments of the slab (rows i1, K = columns) against
//           [X_A | X_1] rows;  (b)+(d1) share its B fragments (K = i1) against
//           [Y_A | Y_1] rows;  (d2) contracts the LDS-staged Z1 over (j1, column)
//           (r = 16), or Z1 is written out for a streaming R_2 (r >= 32).
// Partial sums are written per tile in the accumulation precision and summed in a
// fixed order into the FP64 accumulators by sttnn_t4_reduce.
#include "fused.hpp"

#include <type_traits>

#include "engine.hpp"
#include "kernels.hpp"
#include "mfma.hpp"

namespace ttnn {
namespace {

constexpr int N1 = 128;

struct SttnnArgs {
  const void* T;
  int64_t n2, nA, nB;
  int TA, TB, CB;
  const void *XA, *X1, *YA, *Y1, *X2, *XB;
  void *PRA, *PZA, *PR1, *PR2, *PRB;
  void* Z1;            // Z1-out mode: Y_1^T slab for every (i_2, column), [i_2][i_B][j1]
  const uint16_t *YA3, *Y13, *XB3;          // sttnn_t4_x3_kernel: Y_A, Y_1, X_B as three BF16 planes
  uint32_t* redo;      // ... and, per tile and wave, whether sttnn_t4_kernel has to form the tile again
};

// Wide fragment: V = 16 / sizeof(T) consecutive contraction values of one lane (one
// 16-byte load).  A 16 x 16 MFMA step takes KPL of them per lane group (BF16: all 8;
// FP32 / FP64: one), so a wide load feeds SUB = V / KPL MFMAs; sub-step s of every
// operand uses value s, and the SUB steps together cover the 4 V contraction values
// of the lane groups.  Every operand is laid out with the contraction index
// contiguous, in global memory and in LDS.
template <typename P>
struct Wide {
  using T = typename P::T;
  static constexpr int V = 16 / P::ESZ;
  static constexpr int SUB = V / P::KPL;
  static constexpr int KG = 4 * V;            // contraction values per wide step
  typedef T vec __attribute__((ext_vector_type(V)));
  __device__ static inline vec load(const T* p) { return *reinterpret_cast<const vec*>(p); }
  __device__ static inline typename P::Frag frag(const vec& w, int s) {
    if constexpr (P::KPL == 8) {
      (void)s;
      return __builtin_bit_cast(typename P::Frag, w);
    } else {
      return w[s];
    }
  }
};

// LDS plan of the kernel: the slab of T and the DRM rows of one sub-tile are copied
// straight from global memory into one of two LDS stages (global_load_lds, 16 bytes
// per lane, 64 lanes = whole rows per instruction) while the other stage is being
// consumed.  Operands that do not fit the budget are read from global memory (L2)
// instead.  Staged rows are not padded: the 16-byte chunks of row r are stored in
// XOR-swizzled order (chunk c at position c ^ (r mod 16, or mod the chunk count)),
// so reads along a row and gathers down a column spread over the LDS banks.
template <int DT, int R, int KP, int B2, int SC, bool TT, bool YR = false, bool ZO = false>
struct SttnnLayout {
  using P = Pol<DT>;
  using T = typename P::T;
  static constexpr int ESZ = P::ESZ;
  static constexpr int S = N1;                                // slab column stride
  static constexpr int SY = N1;                               // row stride of staged Y_A / Y_1 / X_B rows
  static constexpr int SXB = SY;
  static constexpr int SX = SC;                               // row stride of staged X_A / X_1 rows
  static constexpr size_t MS = size_t(SC) * S * ESZ;
  // Z1 stash rows (one per slab): FP32 rows are padded by 16 elements so that the four
  // rows read together by the 4 x 4 block products of (d2) fall on distinct banks
  static constexpr int ZPAD = DT == TTNN_F32 ? 16 : 0;
  static constexpr int ZS = KP * SC + ZPAD;
  // STTNN keeps Z1 = Y_1^T slab at FP32 accuracy whatever the plan dtype (the chained
  // intermediate of the sequential variant): a BF16 plan stashes FP32 values where Z1
  // is written out (ZF), and a high and a low BF16 half (hi = RNE(z), lo = RNE(z - hi),
  // |z - hi - lo| <= 2^-18 |z|) where it contracts Z1 with X_2 in the tile (ZH), so
  // that the BF16 MFMA takes both halves.
  static constexpr bool ZF = DT == TTNN_BF16 && ZO && !TT;
  static constexpr bool ZH = DT == TTNN_BF16 && !ZO && !TT;
  static constexpr int ZESZ = ZF ? 4 : ESZ;
  static constexpr size_t Z1 = TT ? 0 : size_t(ZH ? 2 : 1) * B2 * ZS * ZESZ;
  static constexpr size_t YAB = size_t(KP) * SY * ESZ;
  static constexpr size_t YB = YAB + (TT ? size_t(R) * SXB * ESZ : 0);
  static constexpr size_t XB = size_t(R) * SX * ESZ;
  static constexpr size_t BUDGET = 156 * 1024;
  // YR: the Y_A rows (TTNN: and the X_B rows) of the tile's B2 slabs stay in LDS for
  // the whole tile (one copy per tile instead of one per sub-tile), after both stages
  static constexpr size_t YRB = YR ? size_t(B2) * YB : 0;
  static constexpr bool STAGE_YA = !YR && 2 * (MS + YB) + Z1 <= BUDGET;
  // X_A / X_1 rows are staged where the Y_A rows are (staged or resident), and in FP64,
  // whose Y_A rows never fit: there every wave would otherwise load the same X fragments
  // from L2 inside its product loop
  static constexpr bool STAGE_X = (STAGE_YA || YR || DT == TTNN_F64) &&
                                  2 * (MS + (STAGE_YA ? YB : 0) + 2 * XB) + Z1 + YRB <= BUDGET;
  static constexpr size_t STAGE = MS + (STAGE_YA ? YB : 0) + (STAGE_X ? 2 * XB : 0);   // one stage
  static constexpr size_t Y1B = size_t(KP) * SY * ESZ;
  static constexpr bool STAGE_Y1 = !TT && 2 * STAGE + Z1 + YRB + Y1B <= BUDGET;
  static constexpr size_t OFF_YA = MS;                         // offsets within a stage
  static constexpr size_t OFF_XB = OFF_YA + YAB;               // TT: X_B rows after Y_A rows
  static constexpr size_t OFF_XA = OFF_YA + (STAGE_YA ? YB : 0);
  static constexpr size_t OFF_X1 = OFF_XA + (STAGE_X ? XB : 0);
  static constexpr size_t OFF_Z1 = 2 * STAGE;                 // after both stages
  static constexpr size_t OFF_YR = OFF_Z1 + Z1;
  static constexpr size_t OFF_Y1 = OFF_YR + YRB;
  static constexpr size_t TOTAL = OFF_Y1 + (STAGE_Y1 ? Y1B : 0);
};

constexpr int kThreadsF = 512;

// One lane's 16 bytes from global memory straight into LDS (global_load_lds_dwordx4);
// the LDS address is the wave's base plus 16 bytes per lane.
__device__ inline void lds_dma16(const void* g, void* l) {
  __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0);
}

// XOR swizzle of the 16-byte chunks of a staged row of RL elements: element k of
// row r lives at r*RL + swz_off<T, RL>(r, k).
template <typename T, int RL>
struct Swz {
  static constexpr int EV = 16 / sizeof(T);
  static constexpr int CPR = RL / EV;                 // chunks per row
  static constexpr int MASK = (CPR < 16 ? CPR : 16) - 1;
  static_assert(CPR >= 1 && CPR <= 64 && (CPR & (CPR - 1)) == 0, "chunks per row");
  __device__ static inline int off(int r, int k) { return r * RL + ((((k / EV) ^ (r & MASK))) * EV) + (k % EV); }
};

// Copy `rows` rows of RL elements (row r from g + r*gs) into LDS at l, swizzled:
// each instruction fills 64 / CPR whole rows (64 lanes x 16 bytes, one contiguous
// kilobyte of LDS); lane L fetches the chunk that belongs at its position.
// Instructions are dealt to the eight waves; the LDS address is wave-uniform.
template <typename T, int RL>
__device__ inline void lds_dma_rows(const T* g, int64_t gs, T* l, int rows, int wave, int lane) {
  using Z = Swz<T, RL>;
  constexpr int RPI = 64 / Z::CPR;                    // rows per instruction
  const int ninstr = rows / RPI;
  const int rl = lane / Z::CPR, p = lane % Z::CPR;
  for (int q = wave; q < ninstr; q += kThreadsF / 64) {
    const int r = q * RPI + rl;
    const int c = p ^ (r & Z::MASK);
    lds_dma16(g + r * gs + static_cast<int64_t>(c) * Z::EV, l + q * RPI * RL);
  }
}

// Issue the copies of the sub-tile (slab i2, columns col0 .. col0+SC-1) into one stage.
template <int DT, int R, int KP, int B2, int SC, bool TT, bool YR, bool ZO>
__device__ inline void sttnn_issue(const SttnnArgs& a, char* sb, int64_t i2, int64_t col0, int wave, int lane) {
  using P = Pol<DT>;
  using Lay = SttnnLayout<DT, R, KP, B2, SC, TT, YR, ZO>;
  using T = typename P::T;
  const int64_t nA = a.nA, nB = a.nB, n2 = a.n2;
  lds_dma_rows<T, N1>(static_cast<const T*>(a.T) + i2 * N1 + nA * col0, nA, reinterpret_cast<T*>(sb), SC, wave,
                      lane);
  if constexpr (Lay::STAGE_YA) {
    lds_dma_rows<T, N1>(static_cast<const T*>(a.YA) + i2 * N1, nA, reinterpret_cast<T*>(sb + Lay::OFF_YA), KP, wave,
                        lane);
    if constexpr (TT)
      lds_dma_rows<T, N1>(static_cast<const T*>(a.XB) + i2 * N1, nA, reinterpret_cast<T*>(sb + Lay::OFF_XB), R, wave,
                          lane);
  }
  if constexpr (Lay::STAGE_X) {
    lds_dma_rows<T, SC>(static_cast<const T*>(a.XA) + col0, nB, reinterpret_cast<T*>(sb + Lay::OFF_XA), R, wave,
                        lane);
    lds_dma_rows<T, SC>(static_cast<const T*>(a.X1) + i2 * nB + col0, n2 * nB, reinterpret_cast<T*>(sb + Lay::OFF_X1),
                        R, wave, lane);
  }
}

// Wait for every outstanding LDS read of the wave (s_waitcnt lgkmcnt(0)).  While a
// global-to-LDS copy is in flight the compiler's own waits before an LDS operand
// cover all reads issued so far, including prefetches; waiting here, before the next
// step's reads are issued, lets those reads run under the current step's products.
__device__ inline void lds_wait_all() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// acc[rb] += A[rb rows, K = i1] . slab[i1, column iBl] over the whole slab (K = N1),
// A rows delivered by loadA(rb, kk) (wide fragment at contraction offset kk).  The
// operands of step kw + 1 are loaded before the MFMAs of step kw are issued, so the
// LDS latency of one step is hidden behind the products of the previous one.
template <typename P, int NB, typename LoadA>
__device__ inline void bd_chain(const typename P::T* Ms, int iBl, int lg, LoadA&& loadA,
                                typename P::CFrag (&acc)[NB]) {
  using W = Wide<P>;
  using vec = typename W::vec;
  using ZN = Swz<typename P::T, N1>;
  constexpr int V = W::V, SUB = W::SUB, KG = W::KG, NK = N1 / KG;
  static_assert(NK % 2 == 0, "steps in pairs");
  auto load = [&](int kw, vec& bw, vec (&ay)[NB]) {
    const int kk = kw * KG + V * lg;
    bw = W::load(&Ms[ZN::off(iBl, kk)]);
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) ay[rb] = loadA(rb, kk);
  };
  auto mma = [&](const vec& bw, const vec (&ay)[NB]) {
#pragma unroll
    for (int sb = 0; sb < SUB; ++sb)
#pragma unroll
      for (int rb = 0; rb < NB; ++rb) acc[rb] = P::mfma(W::frag(ay[rb], sb), W::frag(bw, sb), acc[rb]);
  };
  {
    vec bw0, ay0[NB], bw1, ay1[NB];
    load(0, bw0, ay0);
#pragma unroll
    // each wait, its loads and the products that follow stay in this order
    for (int kw = 0; kw < NK; kw += 2) {
      lds_wait_all();
      load(kw + 1, bw1, ay1);
      __builtin_amdgcn_sched_barrier(0);
      mma(bw0, ay0);
      __builtin_amdgcn_sched_barrier(0);
      lds_wait_all();
      if (kw + 2 < NK) load(kw + 2, bw0, ay0);
      __builtin_amdgcn_sched_barrier(0);
      mma(bw1, ay1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// A barrier without the fence of __syncthreads, which would wait for every copy in flight:
// the waits before it are the caller's, and no access moves across it.
__device__ __forceinline__ void raw_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Tile of this workgroup.  Workgroups are dealt to the eight XCDs round robin; each XCD
// takes a range of slab groups across every column band when TA allows, so the tiles that
// share an L2 run through the same slabs in step and fetch each Y_A row once between them
// (X_A, the smaller operand, is then shared by fewer tiles).
__device__ __forceinline__ void tile_of(const SttnnArgs& a, int& tA, int& tB) {
  const int w = blockIdx.x;
  if (a.TA % 8 == 0) {
    const int x = w % 8, j = w / 8, gpx = a.TA / 8;
    tA = x * gpx + j % gpx;
    tB = j / gpx;
  } else if (a.TB % 8 == 0) {
    const int x = w % 8, j = w / 8, bpx = a.TB / 8;
    tB = x * bpx + j / a.TA;
    tA = j % a.TA;
  } else {
    tB = w / a.TA;
    tA = w % a.TA;
  }
}

// The FP32 forms at r = 32 whose products are split into BF16 ones (sttnn_t4_x3_kernel).  At
// r = 64 the Y_A planes of two slabs (147 KB) leave no room for the stages of T; at r = 16 the
// STTNN form contracts Z1 in the tile, and the TTNN form was left as it was.
constexpr bool split_form(int dt, int R, bool tt, bool zout) { return dt == TTNN_F32 && R == 32 && (tt || zout); }

// ZO (STTNN only): instead of contracting Z1 with X_2 in the tile (which re-reads the
// X_2 rows of the column band in every row tile), write Z1 out; R_2 is then one
// streaming contraction that reads X_2 once (used for r >= 32).
template <int DT, int R, int KP, int B2, int SC, bool TT, bool ZO>
__global__ __launch_bounds__(kThreadsF) void sttnn_t4_kernel(SttnnArgs a) {
  using P = Pol<DT>;
  using W = Wide<P>;
  // FP32 / BF16 Z1-out and TTNN forms at r = 32, and the BF16 Z1-out form at r = 64 (two
  // slabs per tile, 32-column sub-tiles): the tile's Y_A rows (and X_B rows) stay resident
  static constexpr bool YR = ((ZO || TT) && DT != TTNN_F64 && R == 32) || (DT == TTNN_BF16 && ZO && !TT && R == 64);
  using Lay = SttnnLayout<DT, R, KP, B2, SC, TT, YR, ZO>;
  using T = typename P::T;
  using Acc = typename P::Acc;
  using CFrag = typename P::CFrag;
  using vec = typename W::vec;
  constexpr int V = W::V, SUB = W::SUB, KG = W::KG;
  constexpr int CBR = R / 16;               // 16-wide column blocks of an R-wide output
  constexpr int KB = KP / 16;               // 16-row blocks of KP
  constexpr int KBB = R / 16;               // TT: 16-row blocks of R_B^T
  constexpr int NCB = SC / 16;              // 16-wide column blocks of a sub-tile
  static_assert(NCB == 4 || NCB == 2, "sub-tile width");
  constexpr int KT = KP * SC;               // (d2) contraction length per column sub-block
  constexpr int KW = KT / 8;                // per wave
  static_assert(KW % KG == 0 && SC % KG == 0 && N1 % KG == 0, "wide steps");
  // FP32 R_2 stage on 4 x 4 blocks (R <= 32; wider R keeps the 16 x 16 tiles, whose
  // accumulators are 4x smaller)
  constexpr bool D2Q = DT == TTNN_F32 && R <= 32;
  static_assert(!D2Q || KW % 64 == 0, "4 x 4 block steps");
  static_assert(Lay::TOTAL <= 160 * 1024, "LDS budget");
  static_assert(8 * 16 * R * sizeof(Acc) <= Lay::TOTAL, "reduction scratch");
  // With 32-column sub-tiles the (b)/(d1) products occupy waves 0-3 only; then (a)/(c)
  // go to waves 4-7 (two 16-row blocks of i1 each), so that each SIMD runs one wave of
  // either phase side by side instead of one wave alone through (b)/(d1).  Not where
  // the doubled accumulators would crowd the register file: FP64 at r >= 32, r = 64,
  // and, at r = 32, the forms that keep R_2 or R_B accumulators as well.
  constexpr bool SPLIT =
      NCB == 2 && (ZO || YR || R <= 16) && 2 * (B2 + 1) * CBR * int(sizeof(CFrag) / 4) <= 80;
  constexpr int RB1 = SPLIT ? 2 : 1;        // 16-row blocks of i1 per wave in (a)/(c)
  // (b)/(d1) chains software-pipelined where the second register set fits
  constexpr bool PIPE = DT != TTNN_F64 && (R <= 16 || (R == 32 && (ZO || (TT && DT == TTNN_F32))));

  __shared__ __align__(16) char smem[Lay::TOTAL];
  using ZT = typename std::conditional<Lay::ZF, float, T>::type;   // Z1 stash element
  ZT* Z1s = reinterpret_cast<ZT*>(smem + Lay::OFF_Z1);
  T* Z1lo = reinterpret_cast<T*>(smem + Lay::OFF_Z1) + B2 * Lay::ZS;   // ZH: the low halves
  T* Y1s = reinterpret_cast<T*>(smem + Lay::OFF_Y1);

  if constexpr (split_form(DT, R, TT, ZO)) {     // behind sttnn_t4_x3_kernel: the tiles that it marked
    uint32_t again = 0;
#pragma unroll
    for (int w = 0; w < 8; ++w) again |= a.redo[8 * blockIdx.x + w];
    if (!__builtin_amdgcn_readfirstlane(again)) return;
  }
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform

  int tA, tB;
  tile_of(a, tA, tB);
  const int64_t i2_0 = static_cast<int64_t>(tA) * B2;
  const int64_t c_tile = static_cast<int64_t>(tB) * a.CB * SC;
  const T* XA = static_cast<const T*>(a.XA);
  const T* X1 = static_cast<const T*>(a.X1);
  const T* YA = static_cast<const T*>(a.YA);
  const T* Y1 = static_cast<const T*>(a.Y1);
  const T* X2 = static_cast<const T*>(a.X2);
  const T* XB = static_cast<const T*>(a.XB);
  const int64_t nA = a.nA, nB = a.nB, n2 = a.n2;

  auto stage_base = [&](int buf) -> char* { return smem + buf * Lay::STAGE; };
  // issue the copies of sub-tile s into stage buf
  auto issue = [&](int s, int buf) {
    const int cb = s / B2, i2l = s % B2;
    sttnn_issue<DT, R, KP, B2, SC, TT, YR, ZO>(a, stage_base(buf), i2_0 + i2l,
                                               c_tile + static_cast<int64_t>(cb) * SC, wave, lane);
  };
  // Y_1 rows, resident for the whole kernel; YR: the Y_A rows of the tile's slabs
  if constexpr (Lay::STAGE_Y1) lds_dma_rows<T, N1>(Y1, N1, Y1s, KP, wave, lane);
  T* YRs = reinterpret_cast<T*>(smem + Lay::OFF_YR);
  constexpr int YRN = KP + (TT ? R : 0);      // resident rows per slab: Y_A, then X_B
  if constexpr (YR) {
#pragma unroll
    for (int i2l = 0; i2l < B2; ++i2l) {
      lds_dma_rows<T, N1>(YA + (i2_0 + i2l) * N1, nA, YRs + i2l * YRN * N1, KP, wave, lane);
      if constexpr (TT) lds_dma_rows<T, N1>(XB + (i2_0 + i2l) * N1, nA, YRs + (i2l * YRN + KP) * N1, R, wave, lane);
    }
  }
  using ZN = Swz<T, N1>;                    // staged rows of N1 elements (slab columns, Y rows)
  using ZX = Swz<T, SC>;                    // staged rows of SC elements (X_A, X_1 rows)

  CFrag rA[RB1][B2][CBR];
  CFrag r1[RB1][CBR];
  CFrag r2[CBR];
  // FP32 (d2): 16 blocks of 4 x 4 per column group (block = lane / 4, row i2l = register
  // index, column 4 g + lane % 4); summed over blocks and waves at the end of the tile
  f32x4_t r2q[D2Q ? R / 4 : 1];
  CFrag zA[KB];
  CFrag zB[TT ? KBB : 1];
  const CFrag zero = {};
#pragma unroll
  for (int h = 0; h < RB1; ++h)
#pragma unroll
    for (int c = 0; c < CBR; ++c) {
      r1[h][c] = zero;
#pragma unroll
      for (int i = 0; i < B2; ++i) rA[h][i][c] = zero;
    }
#pragma unroll
  for (int c = 0; c < CBR; ++c) r2[c] = zero;
#pragma unroll
  for (int g = 0; g < (D2Q ? R / 4 : 1); ++g) r2q[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // roles in the (b)/(d1) phase: Z_A, or Z1 (STTNN) / R_B^T (TTNN), for one 16-column
  // block of the sub-tile
  const bool bd_active = wave < 2 * NCB;
  const int cblk = wave % NCB;
  const bool bd_zA = (wave / NCB) == 0;
  const int iBl = 16 * cblk + l16;         // column of the sub-tile in the (b)/(d1) phase
  const bool ac_active = !SPLIT || wave >= 2 * NCB;
  const int i1base = SPLIT ? 32 * (wave - 2 * NCB) : 16 * wave;   // first i1 row of (a)/(c)

  const int nsub = a.CB * B2;
  issue(0, 0);
  for (int cb = 0; cb < a.CB; ++cb) {
    const int64_t iBbase = c_tile + static_cast<int64_t>(cb) * SC;
#pragma unroll
    for (int rb = 0; rb < KB; ++rb) zA[rb] = zero;
    if constexpr (TT) {
#pragma unroll
      for (int rb = 0; rb < KBB; ++rb) zB[rb] = zero;
    }

#pragma unroll
    for (int i2l = 0; i2l < B2; ++i2l) {
      const int s = cb * B2 + i2l;
      const int64_t i2 = i2_0 + i2l;
      const int buf = s & 1;
      __builtin_amdgcn_s_waitcnt(0);      // this wave's copies of sub-tile s have landed
      __syncthreads();                    // ... everyone's; and stage buf^1 is free again
      if (s + 1 < nsub) issue(s + 1, buf ^ 1);
      const T* Ms = reinterpret_cast<const T*>(stage_base(buf));
      const T* YAs = YR ? YRs + i2l * YRN * N1 : reinterpret_cast<const T*>(stage_base(buf) + Lay::OFF_YA);
      const T* XBs = YR ? YRs + (i2l * YRN + KP) * N1 : reinterpret_cast<const T*>(stage_base(buf) + Lay::OFF_XB);
      const T* XAs = reinterpret_cast<const T*>(stage_base(buf) + Lay::OFF_XA);
      const T* X1s = reinterpret_cast<const T*>(stage_base(buf) + Lay::OFF_X1);

      // (a) R_A rows of this slab and (c) R_1: A = slab (rows i1, K = columns)
      if constexpr (!SPLIT) {
        const int i1 = 16 * wave + l16;
#pragma unroll
        for (int kw = 0; kw < SC / KG; ++kw) {
          const int kk = kw * KG + V * lg;
          vec aw;
#pragma unroll
          for (int e = 0; e < V; ++e) aw[e] = Ms[ZN::off(kk + e, i1)];
          vec bA[CBR], b1[CBR];
#pragma unroll
          for (int c = 0; c < CBR; ++c) {
            const int j = 16 * c + l16;
            if constexpr (Lay::STAGE_X) {
              bA[c] = W::load(XAs + ZX::off(j, kk));
              b1[c] = W::load(X1s + ZX::off(j, kk));
            } else {
              bA[c] = W::load(XA + static_cast<int64_t>(j) * nB + iBbase + kk);
              b1[c] = W::load(X1 + (static_cast<int64_t>(j) * n2 + i2) * nB + iBbase + kk);
            }
          }
#pragma unroll
          for (int sb = 0; sb < SUB; ++sb) {
            const auto af = W::frag(aw, sb);
#pragma unroll
            for (int c = 0; c < CBR; ++c) {
              rA[0][i2l][c] = P::mfma(af, W::frag(bA[c], sb), rA[0][i2l][c]);
              r1[0][c] = P::mfma(af, W::frag(b1[c], sb), r1[0][c]);
            }
          }
        }
      } else if (ac_active) {
#pragma unroll
      for (int kw = 0; kw < SC / KG; ++kw) {
        const int kk = kw * KG + V * lg;
        vec aw[RB1];
#pragma unroll
        for (int h = 0; h < RB1; ++h)
#pragma unroll
          for (int e = 0; e < V; ++e) aw[h][e] = Ms[ZN::off(kk + e, i1base + 16 * h + l16)];
        vec bA[CBR], b1[CBR];
#pragma unroll
        for (int c = 0; c < CBR; ++c) {
          const int j = 16 * c + l16;
          if constexpr (Lay::STAGE_X) {
            bA[c] = W::load(XAs + ZX::off(j, kk));
            b1[c] = W::load(X1s + ZX::off(j, kk));
          } else {
            bA[c] = W::load(XA + static_cast<int64_t>(j) * nB + iBbase + kk);
            b1[c] = W::load(X1 + (static_cast<int64_t>(j) * n2 + i2) * nB + iBbase + kk);
          }
        }
#pragma unroll
        for (int sb = 0; sb < SUB; ++sb)
#pragma unroll
          for (int h = 0; h < RB1; ++h) {
            const auto af = W::frag(aw[h], sb);
#pragma unroll
            for (int c = 0; c < CBR; ++c) {
              rA[h][i2l][c] = P::mfma(af, W::frag(bA[c], sb), rA[h][i2l][c]);
              r1[h][c] = P::mfma(af, W::frag(b1[c], sb), r1[h][c]);
            }
          }
      }
      }  // ac_active

      // (b) Z_A += Y_A^T slab; (b') TTNN: R_B^T += X_B^T slab; (d1) STTNN: Z1 = Y_1^T slab.
      // B = slab (K = i1, columns)
      // (d1) result: the Z1 rows of this slab go to the LDS stash
      auto stash_z1 = [&](const CFrag (&acc)[KB]) {
#pragma unroll
        for (int rb = 0; rb < KB; ++rb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int j1 = 16 * rb + P::crow(lane, v);
            const int at = i2l * Lay::ZS + iBl * KP + j1;
            if constexpr (Lay::ZF) {
              Z1s[at] = acc[rb][v];
            } else if constexpr (Lay::ZH) {
              const T hi = P::from_acc(acc[rb][v]);
              Z1s[at] = hi;
              Z1lo[at] = P::from_acc(acc[rb][v] - bf16_bits_to_f32(hi));
            } else {
              Z1s[at] = P::from_acc(acc[rb][v]);
            }
          }
      };
      if constexpr (PIPE) {
        if (bd_active && bd_zA) {
          bd_chain<P, KB>(Ms, iBl, lg, [&](int rb, int kk) -> vec {
            const int jr = 16 * rb + l16;
            if constexpr (Lay::STAGE_YA || YR) return W::load(YAs + ZN::off(jr, kk));
            else return W::load(YA + static_cast<int64_t>(jr) * nA + i2 * N1 + kk);
          }, zA);
        } else if (TT && bd_active) {
          bd_chain<P, (TT ? KBB : 1)>(Ms, iBl, lg, [&](int rb, int kk) -> vec {
            const int jr = 16 * rb + l16;
            if constexpr (Lay::STAGE_YA || YR) return W::load(XBs + ZN::off(jr, kk));
            else return W::load(XB + static_cast<int64_t>(jr) * nA + i2 * N1 + kk);
          }, zB);
        } else if (!TT && bd_active) {
          CFrag acc[KB];
#pragma unroll
          for (int rb = 0; rb < KB; ++rb) acc[rb] = zero;
          bd_chain<P, KB>(Ms, iBl, lg, [&](int rb, int kk) -> vec {
            const int jr = 16 * rb + l16;
            if constexpr (Lay::STAGE_Y1) return W::load(Y1s + ZN::off(jr, kk));
            else return W::load(Y1 + static_cast<int64_t>(jr) * N1 + kk);
          }, acc);
          stash_z1(acc);
        }
      } else if (bd_active && bd_zA) {
#pragma unroll 2
        for (int kw = 0; kw < N1 / KG; ++kw) {
          const int kk = kw * KG + V * lg;
          const vec bw = W::load(&Ms[ZN::off(iBl, kk)]);
          vec ay[KB];
#pragma unroll
          for (int rb = 0; rb < KB; ++rb) {
            const int jr = 16 * rb + l16;
            if constexpr (Lay::STAGE_YA || YR) ay[rb] = W::load(YAs + ZN::off(jr, kk));
            else ay[rb] = W::load(YA + static_cast<int64_t>(jr) * nA + i2 * N1 + kk);
          }
#pragma unroll
          for (int sb = 0; sb < SUB; ++sb)
#pragma unroll
            for (int rb = 0; rb < KB; ++rb) zA[rb] = P::mfma(W::frag(ay[rb], sb), W::frag(bw, sb), zA[rb]);
        }
      } else if (TT && bd_active) {
#pragma unroll 2
        for (int kw = 0; kw < N1 / KG; ++kw) {
          const int kk = kw * KG + V * lg;
          const vec bw = W::load(&Ms[ZN::off(iBl, kk)]);
          vec ax[KBB];
#pragma unroll
          for (int rb = 0; rb < KBB; ++rb) {
            const int jr = 16 * rb + l16;
            if constexpr (Lay::STAGE_YA || YR) ax[rb] = W::load(XBs + ZN::off(jr, kk));
            else ax[rb] = W::load(XB + static_cast<int64_t>(jr) * nA + i2 * N1 + kk);
          }
#pragma unroll
          for (int sb = 0; sb < SUB; ++sb)
#pragma unroll
            for (int rb = 0; rb < KBB; ++rb) zB[rb] = P::mfma(W::frag(ax[rb], sb), W::frag(bw, sb), zB[rb]);
        }
      } else if (!TT && bd_active) {
        CFrag acc[KB];
#pragma unroll
        for (int rb = 0; rb < KB; ++rb) acc[rb] = zero;
#pragma unroll 2
        for (int kw = 0; kw < N1 / KG; ++kw) {
          const int kk = kw * KG + V * lg;
          const vec bw = W::load(&Ms[ZN::off(iBl, kk)]);
          vec ay[KB];
#pragma unroll
          for (int rb = 0; rb < KB; ++rb) {
            const int jr = 16 * rb + l16;
            if constexpr (Lay::STAGE_Y1) ay[rb] = W::load(Y1s + ZN::off(jr, kk));
            else ay[rb] = W::load(Y1 + static_cast<int64_t>(jr) * N1 + kk);
          }
#pragma unroll
          for (int sb = 0; sb < SUB; ++sb)
#pragma unroll
            for (int rb = 0; rb < KB; ++rb) acc[rb] = P::mfma(W::frag(ay[rb], sb), W::frag(bw, sb), acc[rb]);
        }
        stash_z1(acc);
      }
    }  // i2l
    // Z_A partials of this tile's row range for the sub-block's columns (before (d2),
    // so that the stores overlap it and zA's registers are free)
    if (bd_active && bd_zA) {
      Acc* PZA = static_cast<Acc*>(a.PZA);
      const int64_t iB = iBbase + iBl;
#pragma unroll
      for (int rb = 0; rb < KB; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int jA = 16 * rb + P::crow(lane, v);
          PZA[(static_cast<int64_t>(tA) * KP + jA) * nB + iB] = zA[rb][v];
        }
    }
    if constexpr (ZO) {
      // the tile's Z1 rows for this column block: B2 runs of SC * KP contiguous values
      __syncthreads();
      typedef ZT zvec __attribute__((ext_vector_type(16 / sizeof(ZT))));
      constexpr int ZV = 16 / sizeof(ZT);
      constexpr int NZ = SC * KP / ZV;
      ZT* Z1g = static_cast<ZT*>(a.Z1);
      for (int e = tid; e < B2 * NZ; e += kThreadsF) {
        const int i2l = e / NZ, q = e % NZ;
        const zvec v = *reinterpret_cast<const zvec*>(&Z1s[i2l * Lay::ZS + q * ZV]);
        *reinterpret_cast<zvec*>(&Z1g[((i2_0 + i2l) * nB + iBbase) * KP + q * ZV]) = v;
      }
    } else if constexpr (!TT && D2Q) {
      __syncthreads();
      // (d2) R_2[i2 rows] += Z1 (rows i2l, K = (column, j1)) . X_2 rows (column, j1) on
      // the 16-block 4 x 4 x 1 MFMA: only B2 <= 4 rows are live, so 16 x 16 tiles would
      // idle three quarters of the unit.  Block q = lane / 4 takes its own contraction
      // values (4 consecutive per wide load), lane % 4 is the row i2l for A and the
      // column within a group of 4 for B; group g covers columns 4 g .. 4 g + 3.
      const int q = lane >> 2, iq = lane & 3;
#pragma unroll
      for (int kw = 0; kw < KW / 64; ++kw) {
        const int K = wave * KW + kw * 64 + 4 * q;
        f32x4_t az;
        if (iq < B2) az = *reinterpret_cast<const f32x4_t*>(&Z1s[iq * Lay::ZS + K]);
        else az = f32x4_t{0.f, 0.f, 0.f, 0.f};
        f32x4_t bx[R / 4];
#pragma unroll
        for (int g = 0; g < R / 4; ++g)
          bx[g] = *reinterpret_cast<const f32x4_t*>(X2 + (static_cast<int64_t>(4 * g + iq) * nB + iBbase) * KP + K);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int g = 0; g < R / 4; ++g) r2q[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(az[s], bx[g][s], r2q[g], 0, 0, 0);
      }
    } else if constexpr (!TT) {
      __syncthreads();
      // (d2) R_2[i2 rows] += Z1 (rows i2l, K = (column, j1)) . X_2 rows (column, j1);
      // fully unrolled so that every X_2 load of the wave is in flight at once
#pragma unroll
      for (int kw = 0; kw < KW / KG; ++kw) {
        const int K = wave * KW + kw * KG + V * lg;
        vec azw, azl;
        if (l16 < B2) azw = W::load(reinterpret_cast<const T*>(&Z1s[l16 * Lay::ZS + K]));
        else azw = vec{};
        if constexpr (Lay::ZH) {
          if (l16 < B2) azl = W::load(&Z1lo[l16 * Lay::ZS + K]);
          else azl = vec{};
        }
        vec bx[CBR];
#pragma unroll
        for (int c = 0; c < CBR; ++c) {
          const int j = 16 * c + l16;
          bx[c] = W::load(X2 + (static_cast<int64_t>(j) * nB + iBbase) * KP + K);
        }
#pragma unroll
        for (int sb = 0; sb < SUB; ++sb)
#pragma unroll
          for (int c = 0; c < CBR; ++c) {
            r2[c] = P::mfma(W::frag(azw, sb), W::frag(bx[c], sb), r2[c]);
            if constexpr (Lay::ZH) r2[c] = P::mfma(W::frag(azl, sb), W::frag(bx[c], sb), r2[c]);
          }
      }
    }

    // TTNN R_B^T partials of this tile's row range for the sub-block's columns
    if constexpr (TT) {
      if (bd_active && !bd_zA) {
        Acc* PRB = static_cast<Acc*>(a.PRB);
        const int64_t iB = iBbase + iBl;
#pragma unroll
        for (int rb = 0; rb < KBB; ++rb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int j = 16 * rb + P::crow(lane, v);
            PRB[(static_cast<int64_t>(tA) * R + j) * nB + iB] = zB[rb][v];
          }
      }
    }
  }  // cb

  // ---- partial results of the tile
  if (ac_active) {
    Acc* PRA = static_cast<Acc*>(a.PRA);
    Acc* PR1 = static_cast<Acc*>(a.PR1);
#pragma unroll
    for (int h = 0; h < RB1; ++h)
#pragma unroll
      for (int c = 0; c < CBR; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i1 = i1base + 16 * h + P::crow(lane, v);
          const int j = 16 * c + l16;
#pragma unroll
          for (int i2l = 0; i2l < B2; ++i2l) {
            const int64_t iA = (i2_0 + i2l) * N1 + i1;
            PRA[(static_cast<int64_t>(tB) * nA + iA) * R + j] = rA[h][i2l][c][v];
          }
          PR1[((static_cast<int64_t>(tA) * a.TB + tB) * N1 + i1) * R + j] = r1[h][c][v];
        }
  }
  if constexpr (TT || ZO) return;
  __syncthreads();
  Acc* red = reinterpret_cast<Acc*>(smem);          // 8 waves x 16 rows x R
  if constexpr (D2Q) {
    // sum the 16 blocks (lanes 4 q + jj, q = 0..15) by a fixed butterfly; lanes 0..3 of
    // each wave then hold rows i2l = v, columns 4 g + lane
#pragma unroll
    for (int g = 0; g < R / 4; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float x = r2q[g][v];
        x += __shfl_xor(x, 4);
        x += __shfl_xor(x, 8);
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        if (lane < 4) red[(wave * 16 + v) * R + 4 * g + lane] = x;
      }
  } else {
#pragma unroll
    for (int c = 0; c < CBR; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[(wave * 16 + P::crow(lane, v)) * R + 16 * c + l16] = r2[c][v];
  }
  __syncthreads();
  {
    Acc* PR2 = static_cast<Acc*>(a.PR2);
    for (int e = tid; e < B2 * R; e += kThreadsF) {
      const int row = e / R, j = e % R;
      Acc s = 0;
#pragma unroll
      for (int w = 0; w < 8; ++w) s += red[(w * 16 + row) * R + j];
      PR2[(static_cast<int64_t>(tB) * n2 + i2_0 + row) * R + j] = s;
    }
  }
}

// ---------------------------------------------------------------- FP32 at r = 32 on BF16 products
// An FP32 value is the exact sum of three BF16 ones, x = h + m + l (h = RNE(x), m = RNE(x -
// h), l the rest: 8 + 8 + 8 bits), so an FP32 product is a sum of BF16 products, of which
// h h', h m', m h', h l', l h', m m' are formed (the rest is below 2^-24 |x x'|), each
// exact, accumulated in FP32 like the FP32 products they stand for.  Six 16x16x32 BF16
// MFMAs take 0.375 of the time of the eight 16x16x4 FP32 ones: the 85.9 GFLOP of a 128^4
// sweep, 546 us on the FP32 MFMA, 205 us, which leaves the sweep to its bytes (1.95 GB:
// T, X_1, Z_1 and the partials).
//
// The tile and the results are those of sttnn_t4_kernel with two slabs a tile and 32-column
// sub-tiles.  Waves 4-7 take (a) R_A and (c) R_1, 32 rows of i1 each; waves 0, 1 (b) Z_A and
// waves 2, 3 (d1) Z_1 (TT: (b') R_B^T), 16 columns each.  The slab's values are split in
// registers as they are read (5.5 vector instructions a value); the Y_A, Y_1 and X_B rows,
// read by every sub-tile, are split once in a plan ([3][row][i1] planes): Y_A stays in LDS
// for the tile, Y_1 or X_B in the registers of waves 2, 3.  X_A and X_1 come from global
// memory a column block ahead into the registers of waves 4-7 and are split there (a split
// copy of X_1 would add 134 MB to the sweep's bytes).  That leaves room for four stages of T:
// waves 0, 1, which load nothing else, issue the slab's copies three sub-tiles ahead.
//
// 128^4, r = 32, whole update, in turns with the FP32 MFMA form: STTNN 1021 -> 814 us, TTNN
// 1660 -> 1459 us (with two stages, Y_1 in LDS and the copies issued by all waves a quarter
// more for STTNN).  Over twelve shapes and five kinds of data the sketches' errors against
// FP64 are 0.2 to 0.75 of those of the FP32 MFMA form (R_1 of a 128^4 tensor 3e-7, there
// 1.6e-6), R_2's, whose second pass is the same in both, 0.8 to 1.07.
//
// A tile with results outside the range where the split is exact (SplitRange) is marked, and
// sttnn_t4_kernel, launched behind this kernel, forms it again; with no mark that launch
// takes 4 us.  A tensor scaled so that its sketches lie below 2^-80, or whose values decay so
// far inside every tile, pays for both kernels on every tile.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

struct Bf3 {
  bf16x8_t p[3];      // h, m, l
};
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ Bf3 split3(const float (&x)[8]) {
  u32x4_t h, m, l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = bf16_pair(x[2 * i], x[2 * i + 1]);
    const float r0 = x[2 * i] - __uint_as_float(h[i] << 16), r1 = x[2 * i + 1] - __uint_as_float(h[i] & 0xFFFF0000u);
    m[i] = bf16_pair(r0, r1);
    l[i] = bf16_pair(r0 - __uint_as_float(m[i] << 16), r1 - __uint_as_float(m[i] & 0xFFFF0000u));
  }
  return Bf3{{__builtin_bit_cast(bf16x8_t, h), __builtin_bit_cast(bf16x8_t, m), __builtin_bit_cast(bf16x8_t, l)}};
}
// The six products, smallest first, onto NB accumulators in turn (neighbouring products
// then do not wait for one another).
template <int NB>
__device__ __forceinline__ void mfma3(const Bf3 (&a)[NB], const Bf3& b, f32x4_t (&acc)[NB]) {
  constexpr int A[6] = {1, 2, 0, 1, 0, 0}, B[6] = {1, 0, 2, 0, 1, 0};
#pragma unroll
  for (int q = 0; q < 6; ++q)
#pragma unroll
    for (int i = 0; i < NB; ++i)
      acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i].p[A[q]], b.p[B[q]], acc[i], 0, 0, 0);
}

struct X3Layout {
  static constexpr int R = 32, KP = 48, B2 = 2, SC = 32, NST = 4;
  static constexpr size_t MS = size_t(SC) * N1 * 4;           // one stage of T
  static constexpr int YROWS = 3 * KP;                        // resident rows a slab: Y_A planes
  static constexpr size_t OFF_YR = NST * MS;
  static constexpr size_t TOTAL = OFF_YR + size_t(B2) * YROWS * N1 * 2;
  static_assert(TOTAL <= 160 * 1024, "LDS");
};

// Whether results leave the range of the split: infinite or NaN (an infinity, or an FP32
// value above the largest BF16 one, splits into NaN), so small that a part of the split may
// have fallen below the smallest BF16 number, or all zero where a value that is not zero
// entered their sums (every part of every product fell below it; where only some have, a
// neighbouring result is not zero and too small).  One zero says nothing: sums of ordinary
// values cancel to it, too, a few among the 100M of a Z_1.
struct SplitRange {
  uint32_t least = 0xFFFFFFFFu;             // twice the bits of the smallest magnitude, less one: zero is greatest
  uint32_t lost = 0;                        // whether the sums of values not all zero came out zero
  float nan = 0.f;                          // NaN from the first infinity or NaN on
  // any: the bits of the values that entered the sums x
  __device__ __forceinline__ void zeros(const f32x4_t& x, uint32_t any) {
    uint32_t b = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) b |= __float_as_uint(x[v]);
    lost |= b << 1 == 0 && any << 1 != 0 ? 1u : 0u;
  }
  __device__ __forceinline__ void add(const f32x4_t& x) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      least = min(least, (__float_as_uint(x[v]) << 1) - 1);
      nan = __builtin_fmaf(x[v], 0.f, nan);
    }
  }
  __device__ __forceinline__ bool left() const {
    constexpr uint32_t kLeast = uint32_t(127 - 80) << 24;      // 2^-80, twice its bits
    return __any(nan != nan || least < kLeast || lost);
  }
};

template <bool TT>
__global__ __launch_bounds__(kThreadsF) void sttnn_t4_x3_kernel(SttnnArgs a) {
  using Lay = X3Layout;
  constexpr int R = Lay::R, KP = Lay::KP, B2 = Lay::B2, SC = Lay::SC, NST = Lay::NST;
  constexpr int CBR = R / 16, KB = KP / 16, NCB = SC / 16, NK = N1 / 32;
  using ZN = Swz<float, N1>;
  using ZY = Swz<uint16_t, N1>;
  __shared__ __align__(16) char smem[Lay::TOTAL];
  uint16_t* YRs = reinterpret_cast<uint16_t*>(smem + Lay::OFF_YR);

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tA, tB;
  tile_of(a, tA, tB);
  const int64_t i2_0 = static_cast<int64_t>(tA) * B2;
  const int64_t c_tile = static_cast<int64_t>(tB) * a.CB * SC;
  const int64_t nA = a.nA, nB = a.nB, n2 = a.n2;
  const float* T = static_cast<const float*>(a.T);
  const float* XA = static_cast<const float*>(a.XA);
  const float* X1 = static_cast<const float*>(a.X1);
  const bool bd = wave < 4;                 // (b)/(d1) waves; the others (a)/(c)
  const int nsub = a.CB * B2;

  auto stage = [&](int s) { return reinterpret_cast<float*>(smem + (s % NST) * Lay::MS); };
  // Waves 0, 1: the slab's copy of sub-tile s (or, past the last, of the last one into a
  // stage that nobody reads: the copies in flight are then the same in every sub-tile, and
  // a wait can count them), eight loads a wave.
  auto issue = [&](int s) {
    constexpr int RPI = 64 / ZN::CPR;       // rows a load
    static_assert(SC == 16 * RPI, "eight loads a wave");
    const int e = s < nsub ? s : nsub - 1;
    const float* g = T + (i2_0 + e % B2) * N1 + nA * (c_tile + static_cast<int64_t>(e / B2) * SC);
    float* l = stage(s);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = 2 * u + wave, r = q * RPI + lane / ZN::CPR;
      lds_dma16(g + r * nA + ((lane % ZN::CPR) ^ (r & ZN::MASK)) * ZN::EV, l + q * RPI * N1);
    }
  };
#pragma unroll
  for (int i = 0; i < B2; ++i)
    lds_dma_rows<uint16_t, N1>(a.YA3 + (i2_0 + i) * N1, nA, YRs + i * Lay::YROWS * N1,
                               3 * KP, wave, lane);
  __syncthreads();                          // the resident rows are there

  static_assert(B2 == 2, "the loops' slabs");
  auto next_stage = [&]() {
    lds_wait_all();                         // this wave's reads of the last stage are done
    raw_barrier();
  };
  // The roles run loops of their own, so that neither's registers are held through the
  // other's code; both pass one barrier a sub-tile.
  const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
  SplitRange range;
  auto mark = [&]() {
    const bool left = range.left();
    if (lane == 0) a.redo[8 * blockIdx.x + wave] = left;
  };

  if (bd) {
    // (b) Z_A += Y_A^T slab; (b') R_B^T += X_B^T slab; (d1) Z1 = Y_1^T slab: B = slab (K =
    // i1, columns).  Waves 0, 1 take Z_A, its A rows from LDS; waves 2, 3 the other, whose A
    // fragments (the same for every sub-tile of a slab) stay in registers, which leaves the
    // LDS to two more stages of T.
    // The BF16 MFMA rounds its sums down, which adds up over the tiles: every second step's
    // products go, negated (the planes hold those values of Y_A, Y_1 and X_B so), to sums of
    // their own, where down is the other way.  R_B of a 128 x 1024 x 8 x 4 tensor is 1.6e-7 off
    // its FP64 value (4.2e-7 in one chain, 2.8e-7 on the FP32 MFMA).
    const int iBl = 16 * (wave % NCB) + l16;
    const bool zA_role = wave < NCB;
    constexpr int NB = TT ? CBR : KB, NS = TT ? B2 : 1;      // row blocks, slabs with rows of their own
    auto slab8 = [&](const float* Ms, int t, f32x4_t (&b)[2]) {
      b[0] = *reinterpret_cast<const f32x4_t*>(&Ms[ZN::off(iBl, 32 * t + 8 * lg)]);
      b[1] = *reinterpret_cast<const f32x4_t*>(&Ms[ZN::off(iBl, 32 * t + 8 * lg + 4)]);
    };
    // any: bits of the column's values (the lane's quarter of them).  R_B^T leaves the look at
    // zeros to the waves of Z_A, whose sums are of the same values.
    uint32_t any = 0;
    auto split8 = [&](const f32x4_t (&b)[2], bool look) {
      const float x[8] = {b[0][0], b[0][1], b[0][2], b[0][3], b[1][0], b[1][1], b[1][2], b[1][3]};
      if (look) {
#pragma unroll
        for (int e = 0; e < 8; ++e) any |= __float_as_uint(x[e]);
      }
      return split3(x);
    };
    if (zA_role) {
      f32x4_t zA[2][KB];
      float* PZ = static_cast<float*>(a.PZA) + static_cast<int64_t>(tA) * KP * nB + c_tile + iBl;
#pragma unroll
      for (int s = 0; s < NST - 1; ++s) issue(s);
      // Before the barrier of sub-tile s this wave's copies of it have to have landed.
      // Loads and stores complete in order, and after those copies the wave issued the
      // sixteen of s + 1 and s + 2 and the twelve stores of each column block that ended
      // after them (a barrier keeps either from moving to another sub-tile).
      auto copy_stage = [&](int s) {
        if (s < 2) __builtin_amdgcn_s_waitcnt(0x4070);          // vmcnt(16) lgkmcnt(0)
        else if (s == 2 || s % 2) __builtin_amdgcn_s_waitcnt(0x407c);   // vmcnt(28) lgkmcnt(0)
        else __builtin_amdgcn_s_waitcnt(0x8078);                // vmcnt(40) lgkmcnt(0)
        raw_barrier();                      // everyone's reads of s - 1's stage are done too
        issue(s + NST - 1);
        __builtin_amdgcn_sched_barrier(0);
      };
      static_assert(KB == 3 && NST == 4 && B2 == 2, "the counts of copy_stage");
      for (int cb = 0; cb < a.CB; ++cb) {
#pragma unroll
        for (int rb = 0; rb < KB; ++rb) zA[0][rb] = zA[1][rb] = zero;
#pragma unroll
        for (int i2l = 0; i2l < B2; ++i2l) {
          copy_stage(cb * B2 + i2l);
          const float* Ms = stage(cb * B2 + i2l);
          const uint16_t* Ys = YRs + i2l * Lay::YROWS * N1;
          // a step's reads go out before the previous step's products
          f32x4_t b[2][2];
          Bf3 y[2][KB];
          auto load = [&](int t, int q) {
            slab8(Ms, t, b[q]);
#pragma unroll
            for (int rb = 0; rb < KB; ++rb)
#pragma unroll
              for (int p = 0; p < 3; ++p)
                y[q][rb].p[p] = __builtin_bit_cast(
                    bf16x8_t, *reinterpret_cast<const u16x8_t*>(Ys + ZY::off(p * KP + 16 * rb + l16, 32 * t + 8 * lg)));
          };
          load(0, 0);
#pragma unroll
          for (int t = 0; t < NK; ++t) {
            lds_wait_all();
            if (t + 1 < NK) load(t + 1, (t + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma3(y[t & 1], split8(b[t & 1], true), zA[t & 1]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        // the tile's row range of Z_A for these columns
#pragma unroll
        for (int rb = 0; rb < KB; ++rb) {
          const f32x4_t z = zA[0][rb] - zA[1][rb];
          if (rb == 0) range.zeros(z, any);
          range.add(z);
#pragma unroll
          for (int v = 0; v < 4; ++v) PZ[(16 * rb + 4 * lg + v) * nB + cb * SC] = z[v];
        }
        any = 0;
      }
      __builtin_amdgcn_s_waitcnt(0);        // no copy outlives the workgroup
      mark();
      return;
    }
    Bf3 y[NS][NK][NB];
    {
      const uint16_t* Y = TT ? a.XB3 : a.Y13;
      const int64_t ld = TT ? nA : N1, rows = TT ? R : KP;
#pragma unroll
      for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int t = 0; t < NK; ++t)
#pragma unroll
          for (int rb = 0; rb < NB; ++rb)
#pragma unroll
            for (int p = 0; p < 3; ++p)
              y[i][t][rb].p[p] = __builtin_bit_cast(
                  bf16x8_t, *reinterpret_cast<const u16x8_t*>(Y + (p * rows + 16 * rb + l16) * ld +
                                                              (TT ? (i2_0 + i) * N1 : 0) + 32 * t + 8 * lg));
    }
    f32x4_t zB[2][NB];
    float* PZ = TT ? static_cast<float*>(a.PRB) + static_cast<int64_t>(tA) * R * nB + c_tile + iBl
                   : static_cast<float*>(a.Z1) + (i2_0 * nB + c_tile + iBl) * KP + 4 * lg;
    for (int cb = 0; cb < a.CB; ++cb) {
#pragma unroll
      for (int i2l = 0; i2l < B2; ++i2l) {
        if (!TT || i2l == 0) {
#pragma unroll
          for (int rb = 0; rb < NB; ++rb) zB[0][rb] = zB[1][rb] = zero;
        }
        next_stage();
        const float* Ms = stage(cb * B2 + i2l);
        f32x4_t b[TT ? 1 : 2][2];           // TT: the registers hold X_B rows instead
        if (!TT) slab8(Ms, 0, b[0]);
#pragma unroll
        for (int t = 0; t < NK; ++t) {
          if (TT) slab8(Ms, t, b[0]);
          lds_wait_all();
          if (!TT && t + 1 < NK) slab8(Ms, t + 1, b[TT ? 0 : (t + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          mfma3(y[TT ? i2l : 0][t], split8(b[TT ? 0 : t & 1], !TT), zB[t & 1]);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!TT) {                // Z1 rows [i_2][i_B][j1], 64-byte pieces a lane group
#pragma unroll
          for (int rb = 0; rb < NB; ++rb) {
            const f32x4_t z = zB[0][rb] - zB[1][rb];
            if (rb == 0) range.zeros(z, any);
            range.add(z);
            *reinterpret_cast<f32x4_t*>(PZ + (i2l * nB + cb * SC) * KP + 16 * rb) = z;
          }
          any = 0;
        }
      }
      if constexpr (TT) {                   // the tile's row range of R_B^T for these columns
#pragma unroll
        for (int rb = 0; rb < NB; ++rb) {
          const f32x4_t z = zB[0][rb] - zB[1][rb];
          range.add(z);
          int64_t ld = nB;                  // the rows' addresses formed here, not held through the loop
          asm volatile("" : "+s"(ld));
#pragma unroll
          for (int v = 0; v < 4; ++v) PZ[(16 * rb + 4 * lg + v) * ld + cb * SC] = z[v];
        }
      }
    }
    mark();
    return;
  }

  // (a) R_A and (c) R_1: A = slab (rows i1, K = the sub-tile's 32 columns)
  f32x4_t rA[2][B2][CBR], r1[2][CBR];       // [i1 block][slab][column block]
  uint32_t any[2][B2] = {};                 // bits of the values of row i1base + 16 h + l16 (the lane's quarter)
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < CBR; ++c) {
      r1[h][c] = zero;
#pragma unroll
      for (int i = 0; i < B2; ++i) rA[h][i][c] = zero;
    }
  const int i1base = 32 * (wave - 4);
  const float *xrow[CBR], *x1row[CBR];      // X_A row j, X_1 row (j, i2_0) at the lane's first column
#pragma unroll
  for (int c = 0; c < CBR; ++c) {
    const int64_t j = 16 * c + l16;
    xrow[c] = XA + j * nB + c_tile + 8 * lg;
    x1row[c] = X1 + (j * n2 + i2_0) * nB + c_tile + 8 * lg;
  }
  float xa[CBR][8], x1[B2][CBR][8];         // the next column block's X values of the lane
  auto load_x = [&](const float* const (&row)[CBR], int64_t off, float (&x)[CBR][8]) {
#pragma unroll
    for (int c = 0; c < CBR; ++c) {
      const f32x4_t u = *reinterpret_cast<const f32x4_t*>(row[c] + off);
      const f32x4_t v = *reinterpret_cast<const f32x4_t*>(row[c] + off + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[c][e] = u[e];
        x[c][e + 4] = v[e];
      }
    }
  };
  load_x(xrow, 0, xa);
#pragma unroll
  for (int i = 0; i < B2; ++i) load_x(x1row, i * nB, x1[i]);
  Bf3 xas[CBR];
  for (int cb = 0; cb < a.CB; ++cb) {
    const int64_t next = static_cast<int64_t>(cb + 1 < a.CB ? cb + 1 : cb) * SC;
#pragma unroll
    for (int i2l = 0; i2l < B2; ++i2l) {
      next_stage();
      const float* Ms = stage(cb * B2 + i2l);
      // The BF16 MFMA rounds its sums down, not to nearest, which adds up over thousands of
      // columns.  So a sub-tile's sums start from zero and are added to the tile's with
      // rounding to nearest, and every second sub-tile of a sum is formed negated, where down
      // is the other way: R_1 of a 128^4 tensor is 3e-7 off its FP64 value (6.7e-6 in one
      // chain, 1.6e-6 without the negation and on the FP32 MFMA).
      const float sign = (cb + i2l) % 2 ? -1.f : 1.f;
      float v[2][8];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[h][e] = sign * Ms[ZN::off(8 * lg + e, i1base + 16 * h + l16)];
          any[h][i2l] |= __float_as_uint(v[h][e]);
        }
      Bf3 x1s[CBR];
#pragma unroll
      for (int c = 0; c < CBR; ++c) {
        if (i2l == 0) xas[c] = split3(xa[c]);
        x1s[c] = split3(x1[i2l][c]);
      }
      if (i2l == 0) load_x(xrow, next, xa);
      load_x(x1row, i2l * nB + next, x1[i2l]);
      const Bf3 as[2] = {split3(v[0]), split3(v[1])};
#pragma unroll
      for (int c = 0; c < CBR; ++c) {
        f32x4_t t[2] = {zero, zero}, u[2] = {zero, zero};
        mfma3(as, xas[c], t);
        mfma3(as, x1s[c], u);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            rA[h][i2l][c][e] = __builtin_fmaf(sign, t[h][e], rA[h][i2l][c][e]);
            r1[h][c][e] = __builtin_fmaf(sign, u[h][e], r1[h][c][e]);
          }
      }
    }
  }
  float* PRA = static_cast<float*>(a.PRA);
  float* PR1 = static_cast<float*>(a.PR1);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < CBR; ++c) {
      range.add(r1[h][c]);
#pragma unroll
      for (int i = 0; i < B2; ++i) range.add(rA[h][i][c]);
    }
  // the lane's results are of rows 4 lg + v: their values are in four other lanes
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < B2; ++i) {
      const uint64_t b = __ballot(any[h][i] << 1 != 0);
      const uint32_t rows = static_cast<uint32_t>(b | b >> 16 | b >> 32 | b >> 48);
#pragma unroll
      for (int v = 0; v < 4; ++v)
        range.zeros(f32x4_t{rA[h][i][0][v], rA[h][i][1][v], 0.f, 0.f}, rows >> (4 * lg + v) & 1 ? 2u : 0u);
    }
  mark();
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < CBR; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i1 = i1base + 16 * h + 4 * lg + v, j = 16 * c + l16;
#pragma unroll
        for (int i = 0; i < B2; ++i)
          PRA[(static_cast<int64_t>(tB) * nA + (i2_0 + i) * N1 + i1) * R + j] = rA[h][i][c][v];
        PR1[((static_cast<int64_t>(tA) * a.TB + tB) * N1 + i1) * R + j] = r1[h][c][v];
      }
}

// ---------------------------------------------------------------- FP64 Z1-out at r = 32
// Bound by the FP64 MFMA: 85.9 GFLOP for a 128^4 tensor, 1193 us at the 72 TFLOP/s that a
// large product reaches.  A sub-tile (one slab, 32 columns) is 640 MFMAs, 160 a SIMD: waves
// 0, 1 take Z_A and waves 2, 3 Z1 for 16 columns each (96), waves 4-7 R_A and R_1 for 32
// rows of i1 each (64), so that the two waves of a SIMD have the same work on every SIMD
// and one barrier a sub-tile is all that holds them together.  For that the operands that
// every sub-tile reads stay where they are used: the Y_A rows of the tile's two slabs in LDS
// (96 KB, beside two 32 KB stages of T), Y_1 in the registers of waves 2, 3 (192 a lane).
// X_A and X_1 go from global memory to the registers of waves 4-7, each value right after its
// last product for its next use, a sub-tile on.  (At r = 64 the Y_A rows of two slabs are 192
// KB.)  Waves 0, 1, which load nothing else, copy
// the slab a sub-tile ahead.
// 128^4, r = 32: the sweep 2450 -> 1495 us in sttnn_t4_kernel's place (one phase for (b)/(d1)
// and one for (a)/(c), the matrix cores 47% busy; now 85%, at the 2.07 GHz that the card
// holds there), the whole step with the FP64 tail 2902 -> 1910 us.  Two slabs a tile in place
// of four double the partials of Z_A: their reduction takes 116 us where it took 63.
typedef double f64x2_t __attribute__((ext_vector_type(2)));

struct F64Layout {
  static constexpr int R = 32, KP = 48, B2 = 2, SC = 32, NST = 2;
  static constexpr size_t MS = size_t(SC) * N1 * 8;           // one stage of T
  static constexpr size_t OFF_YR = NST * MS;
  static constexpr size_t TOTAL = OFF_YR + size_t(B2) * KP * N1 * 8;
  static_assert(TOTAL <= 160 * 1024, "LDS");
};

__global__ __launch_bounds__(kThreadsF) void sttnn_t4_f64_kernel(SttnnArgs a) {
  using Lay = F64Layout;
  using P = Pol<TTNN_F64>;
  constexpr int R = Lay::R, KP = Lay::KP, B2 = Lay::B2, SC = Lay::SC;
  constexpr int CBR = R / 16, KB = KP / 16, NCB = SC / 16, NT = N1 / 8;
  using Z = Swz<double, N1>;
  __shared__ __align__(16) char smem[Lay::TOTAL];
  double* YRs = reinterpret_cast<double*>(smem + Lay::OFF_YR);

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tA, tB;
  tile_of(a, tA, tB);
  const int64_t i2_0 = static_cast<int64_t>(tA) * B2;
  const int64_t c_tile = static_cast<int64_t>(tB) * a.CB * SC;
  const int64_t nA = a.nA, nB = a.nB, n2 = a.n2;
  const int nsub = a.CB * B2;
  static_assert(B2 == 2 && NCB == 2 && CBR == 2 && Lay::NST == 2 && Z::CPR == 64, "the loops' slabs and roles");
  const f64x4_t zero = {0.0, 0.0, 0.0, 0.0};

  auto stage = [&](int s) { return reinterpret_cast<double*>(smem + (s % 2) * Lay::MS); };
#pragma unroll
  for (int i = 0; i < B2; ++i)
    lds_dma_rows<double, N1>(static_cast<const double*>(a.YA) + (i2_0 + i) * N1, nA, YRs + i * KP * N1, KP, wave, lane);
  __syncthreads();                          // the resident rows are there
  auto next_stage = [&]() {
    lds_wait_all();                         // this wave's reads of the last stage are done
    raw_barrier();
  };

  if (wave < 4) {
    const int iBl = 16 * (wave % NCB) + l16;
    // a step is eight values of i1: 2 lg, 2 lg + 1 of the lane, in two products
    auto pair = [&](const double* row0, int r, int t) {
      return *reinterpret_cast<const f64x2_t*>(&row0[Z::off(r, 8 * t + 2 * lg)]);
    };
    if (wave < NCB) {
      const double* T = static_cast<const double*>(a.T);
      // sixteen rows a wave of the slab's copy of sub-tile s (none past the last)
      auto issue = [&](int s) {
        if (s >= nsub) return;
        const double* g = T + (i2_0 + s % B2) * N1 + nA * (c_tile + static_cast<int64_t>(s / B2) * SC);
        double* l = stage(s);
#pragma unroll
        for (int u = 0; u < SC / 2; ++u) {
          const int r = 2 * u + wave;
          lds_dma16(g + r * nA + (lane ^ (r & Z::MASK)) * Z::EV, l + r * N1);
        }
      };
      f64x4_t zA[KB];
      double* PZ = static_cast<double*>(a.PZA) + static_cast<int64_t>(tA) * KP * nB + c_tile + iBl;
      issue(0);
      for (int cb = 0; cb < a.CB; ++cb) {
#pragma unroll
        for (int rb = 0; rb < KB; ++rb) zA[rb] = zero;
#pragma unroll
        for (int i2l = 0; i2l < B2; ++i2l) {
          // The copies of this sub-tile have to have landed.  Loads and stores complete in
          // order, and after those copies, issued a sub-tile ago, come the twelve stores of
          // the last column block if one has just ended.
          if (i2l == 0 && cb > 0) __builtin_amdgcn_s_waitcnt(0x007c);   // vmcnt(12) lgkmcnt(0)
          else __builtin_amdgcn_s_waitcnt(0x0070);                      // vmcnt(0) lgkmcnt(0)
          raw_barrier();
          issue(cb * B2 + i2l + 1);         // everyone's reads of that stage are done
          __builtin_amdgcn_sched_barrier(0);
          const double* Ms = stage(cb * B2 + i2l);
          const double* Ys = YRs + i2l * KP * N1;
          f64x2_t b[2], y[2][KB];
          auto load = [&](int t, int q) {
            b[q] = pair(Ms, iBl, t);
#pragma unroll
            for (int rb = 0; rb < KB; ++rb) y[q][rb] = pair(Ys, 16 * rb + l16, t);
          };
          load(0, 0);
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            lds_wait_all();
            if (t + 1 < NT) load(t + 1, (t + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
              for (int rb = 0; rb < KB; ++rb) zA[rb] = P::mfma(y[t & 1][rb][v], b[t & 1][v], zA[rb]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
        for (int rb = 0; rb < KB; ++rb)     // the tile's row range of Z_A for these columns
#pragma unroll
          for (int v = 0; v < 4; ++v) PZ[(16 * rb + P::crow(lane, v)) * nB + cb * SC] = zA[rb][v];
      }
      return;
    }
    // Z1: Y_1's rows dealt so that a lane's four results of a block are neighbours
    f64x2_t y[NT][KB];
    const double* Y1 = static_cast<const double*>(a.Y1) + (4 * (l16 % 4) + l16 / 4) * N1 + 2 * lg;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int rb = 0; rb < KB; ++rb) y[t][rb] = *reinterpret_cast<const f64x2_t*>(Y1 + 16 * rb * N1 + 8 * t);
    double* PZ = static_cast<double*>(a.Z1) + (i2_0 * nB + c_tile + iBl) * KP + 4 * lg;
    for (int s = 0; s < nsub; ++s) {
      f64x4_t z1[KB];
#pragma unroll
      for (int rb = 0; rb < KB; ++rb) z1[rb] = zero;
      next_stage();
      const double* Ms = stage(s);
      f64x2_t b[2];
      b[0] = pair(Ms, iBl, 0);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        lds_wait_all();
        if (t + 1 < NT) b[(t + 1) & 1] = pair(Ms, iBl, t + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
          for (int rb = 0; rb < KB; ++rb) z1[rb] = P::mfma(y[t][rb][v], b[t & 1][v], z1[rb]);
        __builtin_amdgcn_sched_barrier(0);
      }
      double* o = PZ + ((s % B2) * nB + (s / B2) * SC) * KP;
#pragma unroll
      for (int rb = 0; rb < KB; ++rb) *reinterpret_cast<f64x4_t*>(o + 16 * rb) = z1[rb];
    }
    return;
  }

  // R_A and R_1: A = slab (rows i1, K = the sub-tile's columns, 8 lg + e of the lane)
  f64x4_t rA[2][B2][CBR], r1[2][CBR];       // [i1 block][slab][column block]
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < CBR; ++c) {
      r1[h][c] = zero;
#pragma unroll
      for (int i = 0; i < B2; ++i) rA[h][i][c] = zero;
    }
  const int i1base = 32 * (wave - 4);
  // X_A row j = l16, X_1 row (j, i2_0), at the lane's first column; 16 rows on the next block
  const double* XA = static_cast<const double*>(a.XA) + l16 * nB + c_tile + 8 * lg;
  const double* X1 = static_cast<const double*>(a.X1) + (l16 * n2 + i2_0) * nB + c_tile + 8 * lg;
  const int64_t ca = 16 * nB, c1 = 16 * n2 * nB;
  f64x2_t xa[4][CBR], x1[4][CBR];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int c = 0; c < CBR; ++c) {
      xa[q][c] = *reinterpret_cast<const f64x2_t*>(XA + c * ca + 2 * q);
      x1[q][c] = *reinterpret_cast<const f64x2_t*>(X1 + c * c1 + 2 * q);
    }
  for (int cb = 0; cb < a.CB; ++cb) {
    const int64_t next = static_cast<int64_t>(cb + 1 < a.CB ? cb + 1 : cb) * SC;
#pragma unroll
    for (int i2l = 0; i2l < B2; ++i2l) {
      next_stage();
      const double* Ms = stage(cb * B2 + i2l);
      double v[2][8];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[h][e] = Ms[Z::off(8 * lg + e, i1base + 16 * h + l16)];
      const double* x1n = X1 + (i2l == 0 ? nB + static_cast<int64_t>(cb) * SC : next);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int c = 0; c < CBR; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h) rA[h][i2l][c] = P::mfma(v[h][2 * q + u], xa[q][c][u], rA[h][i2l][c]);
        if (i2l == B2 - 1) {
#pragma unroll
          for (int c = 0; c < CBR; ++c) xa[q][c] = *reinterpret_cast<const f64x2_t*>(XA + c * ca + next + 2 * q);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int c = 0; c < CBR; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h) r1[h][c] = P::mfma(v[h][2 * q + u], x1[q][c][u], r1[h][c]);
#pragma unroll
        for (int c = 0; c < CBR; ++c) x1[q][c] = *reinterpret_cast<const f64x2_t*>(x1n + c * c1 + 2 * q);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  double* PRA = static_cast<double*>(a.PRA);
  double* PR1 = static_cast<double*>(a.PR1);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < CBR; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i1 = i1base + 16 * h + P::crow(lane, v), j = 16 * c + l16;
#pragma unroll
        for (int i = 0; i < B2; ++i)
          PRA[(static_cast<int64_t>(tB) * nA + (i2_0 + i) * N1 + i1) * R + j] = rA[h][i][c][v];
        PR1[((static_cast<int64_t>(tA) * a.TB + tB) * N1 + i1) * R + j] = r1[h][c][v];
      }
}

// ---------------------------------------------------------------- BF16 Z1-out at r = 64, four slabs
// Bound by its bytes: for a 128^4 tensor 0.8 GB read (T, X_1) and 1.0 GB written (Z1 in FP32,
// the partials of Z_A, which halve with four slabs a tile in place of two).  The roles are
// those of sttnn_t4_f64_kernel: waves 0, 1 Z_A and the copies of T and X_1, three sub-tiles
// ahead into four stages, and of X_A, a column block ahead; waves 2, 3 Z1, Y_1 in registers,
// written straight from the products; waves 4-7 R_A and R_1.  The Y_A rows of the four slabs
// (96 KB) stay in LDS.  Z_A's FP32 sums start anew for every slab and are then added: in one
// chain over the four slabs Z_A was 1.4 times as far from its FP64 value as with two slabs a
// tile, now 0.85 times.
// 128^4, r = 64: the sweep 540 -> 440 us and the reduction of its partials 103 -> 63, the
// whole update 1083 -> 944 (sttnn_t4_kernel: two slabs, Z1 through an LDS stash, every wave
// waiting for its copies; with the X values fetched by waves 4-7 a sub-tile ahead: 583).
struct Bf64Layout {
  static constexpr int R = 64, KP = 96, B2 = 4, SC = 32, NST = 4;
  static constexpr size_t MT = size_t(SC) * N1 * 2, MX = size_t(R) * SC * 2;
  static constexpr size_t MS = MT + MX;                       // one stage: T, then X_1
  static constexpr size_t OFF_XA = NST * MS;                  // X_A of two column blocks
  static constexpr size_t OFF_YR = OFF_XA + 2 * MX;
  static constexpr size_t TOTAL = OFF_YR + size_t(B2) * KP * N1 * 2;
  static_assert(TOTAL <= 160 * 1024, "LDS");
};

__global__ __launch_bounds__(kThreadsF) void sttnn_t4_bf64_kernel(SttnnArgs a) {
  using Lay = Bf64Layout;
  using P = Pol<TTNN_BF16>;
  constexpr int R = Lay::R, KP = Lay::KP, B2 = Lay::B2, SC = Lay::SC, NST = Lay::NST;
  constexpr int CBR = R / 16, KB = KP / 16, NCB = SC / 16, NK = N1 / 32;
  using Z = Swz<uint16_t, N1>;
  using ZX = Swz<uint16_t, SC>;
  __shared__ __align__(16) char smem[Lay::TOTAL];
  uint16_t* YRs = reinterpret_cast<uint16_t*>(smem + Lay::OFF_YR);

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tA, tB;
  tile_of(a, tA, tB);
  const int64_t i2_0 = static_cast<int64_t>(tA) * B2;
  const int64_t c_tile = static_cast<int64_t>(tB) * a.CB * SC;
  const int64_t nA = a.nA, nB = a.nB, n2 = a.n2;
  const int nsub = a.CB * B2;
  static_assert(B2 == 4 && NCB == 2 && NST == 4 && Z::CPR == 16 && KB == 6, "the loops' slabs, roles and counts");
  const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};

  auto stage = [&](int s) { return reinterpret_cast<uint16_t*>(smem + (s % NST) * Lay::MS); };
  auto stage_x1 = [&](int s) { return stage(s) + SC * N1; };
  auto stage_xa = [&](int cb) { return reinterpret_cast<uint16_t*>(smem + Lay::OFF_XA + (cb % 2) * Lay::MX); };
  auto frag = [&](const uint16_t* rows, int r, int k) { return P::load8(&rows[Z::off(r, k)]); };
#pragma unroll
  for (int i = 0; i < B2; ++i)
    lds_dma_rows<uint16_t, N1>(static_cast<const uint16_t*>(a.YA) + (i2_0 + i) * N1, nA, YRs + i * KP * N1, KP, wave,
                               lane);
  __syncthreads();                          // the resident rows are there
  auto next_stage = [&]() {
    lds_wait_all();                         // this wave's reads of the last stage are done
    raw_barrier();
  };

  if (wave < 4) {
    const int iBl = 16 * (wave % NCB) + l16;
    if (wave < NCB) {
      const uint16_t* T = static_cast<const uint16_t*>(a.T);
      const uint16_t* XA = static_cast<const uint16_t*>(a.XA);
      const uint16_t* X1 = static_cast<const uint16_t*>(a.X1);
      // A wave's loads of sub-tile s, four of T and two of X_1 (past the last sub-tile, of the
      // last one into a stage that nobody reads, so that the loads in flight are the same in
      // every sub-tile), and its two of a column block's X_A.
      auto issue = [&](int s) {
        constexpr int RPI = 64 / Z::CPR, RPX = 64 / ZX::CPR;
        const int e = s < nsub ? s : nsub - 1;
        const int64_t i2 = i2_0 + e % B2, col = c_tile + static_cast<int64_t>(e / B2) * SC;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = 2 * u + wave, r = q * RPI + lane / Z::CPR;
          lds_dma16(T + i2 * N1 + nA * (col + r) + ((lane % Z::CPR) ^ (r & Z::MASK)) * Z::EV, stage(s) + q * RPI * N1);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int q = 2 * u + wave, r = q * RPX + lane / ZX::CPR;
          lds_dma16(X1 + (r * n2 + i2) * nB + col + ((lane % ZX::CPR) ^ (r & ZX::MASK)) * ZX::EV,
                    stage_x1(s) + q * RPX * SC);
        }
      };
      auto issue_xa = [&](int cb) {
        constexpr int RPX = 64 / ZX::CPR;
        const int64_t col = c_tile + static_cast<int64_t>(cb < a.CB ? cb : a.CB - 1) * SC;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int q = 2 * u + wave, r = q * RPX + lane / ZX::CPR;
          lds_dma16(XA + r * nB + col + ((lane % ZX::CPR) ^ (r & ZX::MASK)) * ZX::EV, stage_xa(cb) + q * RPX * SC);
        }
      };
      f32x4_t zA[KB];
      float* PZ = static_cast<float*>(a.PZA) + static_cast<int64_t>(tA) * KP * nB + c_tile + iBl;
      issue_xa(0);
#pragma unroll
      for (int s = 0; s < NST - 1; ++s) issue(s);
      for (int cb = 0; cb < a.CB; ++cb) {
#pragma unroll
        for (int rb = 0; rb < KB; ++rb) zA[rb] = zero;
#pragma unroll
        for (int i2l = 0; i2l < B2; ++i2l) {
          // The copies of this sub-tile have to have landed.  Loads and stores complete in
          // order, and after those copies, issued three sub-tiles ago, come the twelve of the
          // next two, the two of X_A if a column block began in between, and the 24 stores of
          // a column block that ended since.
          if (i2l == 0) {
            if (cb > 0) __builtin_amdgcn_s_waitcnt(0x8074);             // vmcnt(36) lgkmcnt(0)
            else __builtin_amdgcn_s_waitcnt(0x007c);                    // vmcnt(12) lgkmcnt(0)
          } else if (i2l < 3) {
            if (cb > 0) __builtin_amdgcn_s_waitcnt(0x8076);             // vmcnt(38) lgkmcnt(0)
            else __builtin_amdgcn_s_waitcnt(0x007e);                    // vmcnt(14) lgkmcnt(0)
          } else {
            __builtin_amdgcn_s_waitcnt(0x007c);                         // vmcnt(12) lgkmcnt(0)
          }
          raw_barrier();                    // everyone's reads of the stages filled now are done
          if (i2l == 0) issue_xa(cb + 1);
          issue(cb * B2 + i2l + NST - 1);
          __builtin_amdgcn_sched_barrier(0);
          const uint16_t* Ms = stage(cb * B2 + i2l);
          const uint16_t* Ys = YRs + i2l * KP * N1;
          f32x4_t z[KB];                    // this slab's sums (see above)
#pragma unroll
          for (int rb = 0; rb < KB; ++rb) z[rb] = zero;
          bf16x8_t b[2], y[2][KB];
          auto load = [&](int t, int q) {
            b[q] = frag(Ms, iBl, 32 * t + 8 * lg);
#pragma unroll
            for (int rb = 0; rb < KB; ++rb) y[q][rb] = frag(Ys, 16 * rb + l16, 32 * t + 8 * lg);
          };
          load(0, 0);
#pragma unroll
          for (int t = 0; t < NK; ++t) {
            lds_wait_all();
            if (t + 1 < NK) load(t + 1, (t + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rb = 0; rb < KB; ++rb) z[rb] = P::mfma(y[t & 1][rb], b[t & 1], z[rb]);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int rb = 0; rb < KB; ++rb) zA[rb] += z[rb];
        }
#pragma unroll
        for (int rb = 0; rb < KB; ++rb)     // the tile's row range of Z_A for these columns
#pragma unroll
          for (int v = 0; v < 4; ++v) PZ[(16 * rb + P::crow(lane, v)) * nB + cb * SC] = zA[rb][v];
      }
      __builtin_amdgcn_s_waitcnt(0);        // no copy outlives the workgroup
      return;
    }
    bf16x8_t y[NK][KB];
    const uint16_t* Y1 = static_cast<const uint16_t*>(a.Y1) + l16 * N1 + 8 * lg;
#pragma unroll
    for (int t = 0; t < NK; ++t)
#pragma unroll
      for (int rb = 0; rb < KB; ++rb) y[t][rb] = P::load8(Y1 + 16 * rb * N1 + 32 * t);
    float* PZ = static_cast<float*>(a.Z1) + (i2_0 * nB + c_tile + iBl) * KP + 4 * lg;
    for (int s = 0; s < nsub; ++s) {
      f32x4_t z1[KB];
#pragma unroll
      for (int rb = 0; rb < KB; ++rb) z1[rb] = zero;
      next_stage();
      const uint16_t* Ms = stage(s);
      bf16x8_t b[NK];
#pragma unroll
      for (int t = 0; t < NK; ++t) b[t] = frag(Ms, iBl, 32 * t + 8 * lg);
#pragma unroll
      for (int t = 0; t < NK; ++t)
#pragma unroll
        for (int rb = 0; rb < KB; ++rb) z1[rb] = P::mfma(y[t][rb], b[t], z1[rb]);
      float* o = PZ + ((s % B2) * nB + (s / B2) * SC) * KP;
#pragma unroll
      for (int rb = 0; rb < KB; ++rb) *reinterpret_cast<f32x4_t*>(o + 16 * rb) = z1[rb];
    }
    return;
  }

  // R_A and R_1: A = slab (rows i1, K = the sub-tile's 32 columns, 8 lg + e of the lane)
  f32x4_t rA[2][B2][CBR], r1[2][CBR];       // [i1 block][slab][column block]
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < CBR; ++c) {
      r1[h][c] = zero;
#pragma unroll
      for (int i = 0; i < B2; ++i) rA[h][i][c] = zero;
    }
  const int i1base = 32 * (wave - 4);
  bf16x8_t xa[CBR];
  for (int cb = 0; cb < a.CB; ++cb) {
#pragma unroll
    for (int i2l = 0; i2l < B2; ++i2l) {
      next_stage();
      const uint16_t* Ms = stage(cb * B2 + i2l);
      bf16x8_t v[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        u16x8_t w;
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = Ms[Z::off(8 * lg + e, i1base + 16 * h + l16)];
        v[h] = __builtin_bit_cast(bf16x8_t, w);
      }
      bf16x8_t x1[CBR];
#pragma unroll
      for (int c = 0; c < CBR; ++c) {
        const int o = ZX::off(16 * c + l16, 8 * lg);
        x1[c] = P::load8(stage_x1(cb * B2 + i2l) + o);
        if (i2l == 0) xa[c] = P::load8(stage_xa(cb) + o);
      }
#pragma unroll
      for (int c = 0; c < CBR; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          r1[h][c] = P::mfma(v[h], x1[c], r1[h][c]);
          rA[h][i2l][c] = P::mfma(v[h], xa[c], rA[h][i2l][c]);
        }
    }
  }
  float* PRA = static_cast<float*>(a.PRA);
  float* PR1 = static_cast<float*>(a.PR1);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int c = 0; c < CBR; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i1 = i1base + 16 * h + P::crow(lane, v), j = 16 * c + l16;
#pragma unroll
        for (int i = 0; i < B2; ++i)
          PRA[(static_cast<int64_t>(tB) * nA + (i2_0 + i) * N1 + i1) * R + j] = rA[h][i][c][v];
        PR1[((static_cast<int64_t>(tA) * a.TB + tB) * N1 + i1) * R + j] = r1[h][c][v];
      }
}

// sum_{t < n} p[t * stride] in FP64 with eight interleaved partial sums (t mod 8),
// combined in a fixed order: eight loads in flight per thread.
template <typename Acc>
__device__ inline double sum_strided(const Acc* p, int n, int64_t stride) {
  double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  int t = 0;
  for (; t + 8 <= n; t += 8) {
    Acc v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(t + u) * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] += static_cast<double>(v[u]);
  }
  for (int q = 0; t < n; ++t, ++q) s[q] += static_cast<double>(p[t * stride]);
  return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// Tile of the transposing reductions: 16 output-fast x 32 input-fast entries per
// 256-thread block, two per thread.
constexpr int kRTX = 16, kRTY = 32;

// O[x + ldo y] (+)= alpha * sum_t P[t * tstride + x * ldx + y] for the tile (x0, y0):
// the partials are read along y (their contiguous index) and, through an LDS
// transpose, the output is written along x (its contiguous index).
template <typename Acc>
__device__ inline void reduce_transpose_tile(const Acc* P, int nt, int64_t tstride, int64_t ldx, int64_t X, int64_t Y,
                                             int64_t x0, int64_t y0, double* O, int64_t ldo, double alpha, bool acc,
                                             double (*tile)[kRTX + 1]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int u = 0; u < kRTX * kRTY / 256; ++u) {
    const int e = tid + 256 * u;
    const int xl = e / kRTY, yl = e % kRTY;
    const int64_t x = x0 + xl, y = y0 + yl;
    double v = 0.0;
    if (x < X && y < Y) v = sum_strided(P + x * ldx + y, nt, tstride);
    tile[yl][xl] = v;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kRTX * kRTY / 256; ++u) {
    const int e = tid + 256 * u;
    const int xl = e % kRTX, yl = e / kRTX;
    const int64_t x = x0 + xl, y = y0 + yl;
    if (x < X && y < Y) {
      double* o = O + x + ldo * y;
      *o = acc ? *o + alpha * tile[yl][xl] : tile[yl][xl];
    }
  }
}

// Few entries, many partials: O[x + ldo y] = sum_t P[t * tstride + x * ldx + y] for 32 values
// of y at one x, eight threads an entry (thread g sums t = g mod 8), their sums added in a
// fixed tree.
constexpr int kSplitY = 32, kSplitT = 256 / kSplitY;
template <typename Acc>
__device__ inline void reduce_split_row(const Acc* P, int nt, int64_t tstride, int64_t ldx, int64_t Y, int64_t x,
                                        int64_t y0, double* O, int64_t ldo, double* red) {
  const int yl = threadIdx.x % kSplitY, g = threadIdx.x / kSplitY;
  const int64_t y = y0 + yl;
  double v = 0.0;
  if (y < Y && g < nt) v = sum_strided(P + g * tstride + x * ldx + y, (nt - g + kSplitT - 1) / kSplitT, kSplitT * tstride);
  red[g * kSplitY + yl] = v;
  __syncthreads();
#pragma unroll
  for (int w = kSplitT / 2; w > 0; w /= 2) {
    if (g < w) red[g * kSplitY + yl] += red[(g + w) * kSplitY + yl];
    __syncthreads();
  }
  if (g == 0 && y < Y) O[x + ldo * y] = red[yl];
}

// Sum the tile partials in a fixed order into the FP64 state.  Blocks [0, nbA) do R_A
// (PRA [tB][iA][R] -> RA[iA + nA j]) and [nbA, nbA + nbZ) Z_A (PZA [tA][jA][iB] ->
// ZA[jA + k iB]) tile by tile (zsplit: 32 entries a block), [nbA + nbZ, + nb1) R_1 (16 lanes per entry), and the
// remaining blocks the last segment, entry by entry: R_2 (mode 0, STTNN; PR2
// [tB][n2][R]), R_B (mode 1, TTNN; PRB [tA][R][nB]) or nothing (mode 2, STTNN with Z1
// written out).
template <typename Acc>
__global__ __launch_bounds__(256) void sttnn_t4_reduce(const Acc* PRA, const Acc* PZA, const Acc* PR1, const Acc* PR2,
                                                       int TA, int TB, int64_t n2, int64_t nA, int64_t nB, int R,
                                                       int KP, int k, double alpha, double* RA, double* ZA, double* R1,
                                                       double* R2, int tt, int nbA, int nbZ, int zsplit, int nb1) {
  __shared__ double tile[kRTY][kRTX + 1];
  const int64_t b = blockIdx.x;
  if (b < nbA) {
    const int64_t ty = (R + kRTY - 1) / kRTY;
    reduce_transpose_tile(PRA, TB, nA * R, R, nA, R, (b / ty) * kRTX, (b % ty) * kRTY, RA, nA, alpha, true, tile);
    return;
  }
  if (b < nbA + nbZ) {
    const int64_t bz = b - nbA;
    if (zsplit) {
      reduce_split_row(PZA, TA, static_cast<int64_t>(KP) * nB, nB, nB, bz % k, (bz / k) * kSplitY, ZA, k, &tile[0][0]);
      return;
    }
    const int64_t tx = (k + kRTX - 1) / kRTX;
    reduce_transpose_tile(PZA, TA, static_cast<int64_t>(KP) * nB, nB, k, nB, (bz % tx) * kRTX, (bz / tx) * kRTY, ZA,
                          k, 1.0, false, tile);
    return;
  }
  const int64_t nR1 = static_cast<int64_t>(N1) * R;
  if (b < nbA + nbZ + nb1) {
    // R_1: TA * TB partials per entry, 16 lanes per entry (lane g sums partials
    // t = g mod 16), the 16 sums combined by a fixed butterfly
    const int g = threadIdx.x & 15;
    const int64_t f = ((b - nbA - nbZ) * blockDim.x + threadIdx.x) >> 4;
    if (f >= nR1) return;                       // whole 16-lane groups leave together
    const int64_t i1 = f / R, j = f % R;
    const int nt = TA * TB;
    const int64_t st = static_cast<int64_t>(N1) * R;
    double x = g < nt ? sum_strided(PR1 + i1 * R + j + g * st, (nt - g + 15) / 16, 16 * st) : 0.0;
    x += __shfl_xor(x, 8);
    x += __shfl_xor(x, 4);
    x += __shfl_xor(x, 2);
    x += __shfl_xor(x, 1);
    if (g == 0) R1[i1 + N1 * j] += alpha * x;
    return;
  }
  const int64_t nR2 = tt == 1 ? nB * R : tt == 0 ? n2 * R : 0;
  const int64_t nb = gridDim.x - nbA - nbZ - nb1;
  for (int64_t f = (b - nbA - nbZ - nb1) * blockDim.x + threadIdx.x; f < nR2; f += nb * blockDim.x) {
    if (tt == 0) {
      const int64_t i2 = f / R, j = f % R;
      R2[i2 + n2 * j] += alpha * sum_strided(PR2 + i2 * R + j, TB, n2 * R);
    } else {
      const int64_t j = f / nB, c = f % nB;
      R2[c + nB * j] += alpha * sum_strided(PR2 + j * nB + c, TA, static_cast<int64_t>(R) * nB);
    }
  }
}

// out[i0 + d0 (i1 + d1 i2)] = (valid) ? round(src[i0 s0 + i1 s1 + i2 s2]) : 0,
// valid: the coordinate `cdim` is below `lim`.
template <typename TO>
__global__ void gather_copy(const double* src, TO* out, int64_t d0, int64_t d1, int64_t d2, int64_t s0, int64_t s1,
                            int64_t s2, int cdim, int64_t lim) {
  const int64_t total = d0 * d1 * d2;
  for (int64_t o = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; o < total;
       o += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t i0 = o % d0, t = o / d0, i1 = t % d1, i2 = t / d1;
    const int64_t c = cdim == 0 ? i0 : cdim == 1 ? i1 : i2;
    double v = 0.0;
    if (c < lim) v = src[i0 * s0 + i1 * s1 + i2 * s2];
    if constexpr (sizeof(TO) == 2) {
      const uint32_t b = __float_as_uint(static_cast<float>(v));
      out[o] = static_cast<uint16_t>((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
    } else {
      out[o] = static_cast<TO>(v);
    }
  }
}

// The same copy split into the BF16 planes of split3: out[p][o], p = h, m, l, every second
// 32 values of i_0 negated (sttnn_t4_x3_kernel's second sums).
__global__ void gather_split(const double* src, uint16_t* out, int64_t d0, int64_t d1, int64_t s0, int64_t s1,
                             int64_t lim) {
  const int64_t total = d0 * d1;
  for (int64_t o = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; o < total;
       o += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t i0 = o % d0, i1 = o / d0;
    float v = i1 < lim ? static_cast<float>(src[i0 * s0 + i1 * s1]) : 0.0f;
    if (i0 & 32) v = -v;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const uint32_t b = __float_as_uint(v);
      const uint16_t q = static_cast<uint16_t>((b + 0x7FFFu + ((b >> 16) & 1u)) >> 16);
      out[p * total + o] = q;
      v -= bf16_bits_to_f32(q);
    }
  }
}

}  // namespace

void copy_layout(const double* src, void* out, int dt, int64_t d0, int64_t d1, int64_t d2, int64_t s0, int64_t s1,
                 int64_t s2, int cdim, int64_t lim, hipStream_t st) {
  const int64_t total = d0 * d1 * d2;
  const int blocks = static_cast<int>(std::min<int64_t>((total + 255) / 256, 16384));
  if (dt == TTNN_BF16)
    hipLaunchKernelGGL(gather_copy<uint16_t>, dim3(blocks), dim3(256), 0, st, src, static_cast<uint16_t*>(out), d0,
                       d1, d2, s0, s1, s2, cdim, lim);
  else if (dt == TTNN_F32)
    hipLaunchKernelGGL(gather_copy<float>, dim3(blocks), dim3(256), 0, st, src, static_cast<float*>(out), d0, d1, d2,
                       s0, s1, s2, cdim, lim);
  else
    hipLaunchKernelGGL(gather_copy<double>, dim3(blocks), dim3(256), 0, st, src, static_cast<double*>(out), d0, d1,
                       d2, s0, s1, s2, cdim, lim);
}

namespace {

struct Shape {
  int B2, SC;
};

// Tile shape per dtype: B2 slabs of i_2 per tile, SC columns per sub-tile (sized so
// that the slab, the DRM rows of a sub-tile and the Z1 stash fit the LDS budget).
// The FP32 Z1-out and TTNN forms and the FP64 Z1-out form at r = 32 take two slabs, so that
// their Y_A (and X_B) rows stay in LDS.
template <int DT, int R, bool TT, bool ZO = false>
constexpr int b2_of() {
  return DT == TTNN_BF16 ? (R >= 64 ? 2 : (ZO || TT) && R == 32 ? 4 : 8)
         : DT == TTNN_F32 ? (R >= 64 || ((ZO || TT) && R == 32) ? 2 : 4)
                          : (R >= 64 || TT || (ZO && R == 32) ? 2 : 4);
}
// BF16 Z1-out at r = 64 takes 32-column sub-tiles: with them the FP32 Z1 stash, the
// resident Y_A rows of both slabs and staged X_A / X_1 rows fit the LDS (at 64 columns
// the Y_A rows were re-copied every sub-tile and X_A / X_1 read from L2).
template <int DT, int R = 32, bool ZO = false>
constexpr int sc_of() {
  return DT == TTNN_BF16 ? (ZO && R >= 64 ? 32 : 64) : 32;
}

Shape shape_for(int dt, int R, bool tt, bool zout) {
  if (dt == TTNN_BF16) return {R >= 64 ? 2 : (zout || tt) && R == 32 ? 4 : 8, zout && !tt && R >= 64 ? 32 : 64};
  if (dt == TTNN_F32) return {R >= 64 || ((zout || tt) && R == 32) ? 2 : 4, 32};
  return {R >= 64 || tt || (zout && R == 32) ? 2 : 4, 32};
}

template <int DT, int R, int KP>
void launch_sttnn(bool tt, bool zout, const SttnnArgs& a, hipStream_t st) {
  constexpr int SC = sc_of<DT>(), SCZ = sc_of<DT, R, true>();
  constexpr int B2T = b2_of<DT, R, true>(), B2S = b2_of<DT, R, false>(), B2Z = b2_of<DT, R, false, true>();
  const dim3 grid(a.TA * a.TB);
  if constexpr (split_form(DT, R, true, false)) {
    static_assert(B2T == X3Layout::B2 && B2Z == X3Layout::B2 && SC == X3Layout::SC && KP == X3Layout::KP,
                  "one tile shape");
    if (tt) hipLaunchKernelGGL(sttnn_t4_x3_kernel<true>, grid, dim3(kThreadsF), 0, st, a);
    else if (zout) hipLaunchKernelGGL(sttnn_t4_x3_kernel<false>, grid, dim3(kThreadsF), 0, st, a);
  }
  if (tt) hipLaunchKernelGGL((sttnn_t4_kernel<DT, R, KP, B2T, SC, true, false>), grid, dim3(kThreadsF), 0, st, a);
  else if (zout && DT == TTNN_F64 && R == 32) hipLaunchKernelGGL(sttnn_t4_f64_kernel, grid, dim3(kThreadsF), 0, st, a);
  else if (zout) {
    if (DT == TTNN_BF16 && R == 64 && a.n2 == int64_t(a.TA) * Bf64Layout::B2) {
      hipLaunchKernelGGL(sttnn_t4_bf64_kernel, grid, dim3(kThreadsF), 0, st, a);
      return;
    }
    if constexpr (DT != TTNN_F64 || R != 32)
      hipLaunchKernelGGL((sttnn_t4_kernel<DT, R, KP, B2Z, SCZ, false, true>), grid, dim3(kThreadsF), 0, st, a);
  }
  else hipLaunchKernelGGL((sttnn_t4_kernel<DT, R, KP, B2S, SC, false, false>), grid, dim3(kThreadsF), 0, st, a);
}

template <int DT>
void launch_sttnn_dt(int R, bool tt, bool zout, const SttnnArgs& a, hipStream_t st) {
  if (R == 16) launch_sttnn<DT, 16, 32>(tt, zout, a, st);
  else if (R == 32) launch_sttnn<DT, 32, 48>(tt, zout, a, st);
  else launch_sttnn<DT, 64, 96>(tt, zout, a, st);
}

int64_t elem_size(int dt) { return dt == TTNN_F64 ? 8 : dt == TTNN_F32 ? 4 : 2; }

}  // namespace

// ---------------------------------------------------------------- plan-time setup
void fused_prepare(Plan& P, hipStream_t st) {
  FusedT4& F = P.fused;
  F.enabled = false;
  const bool tt = P.variant == TTNN_TTNN;
  if (P.d < 3) return;
  const Node& root = P.nodes[0];
  if (root.children.size() < 2) return;
  if (tt && root.children.size() != 2) return;            // X_B rows must be exactly i_A
  const int A = root.children[0];
  const Node& nA_ = P.nodes[A];
  if (nA_.first != 0 || nA_.last != 1 || nA_.children.size() != 2) return;
  const int c1 = nA_.children[0], c2 = nA_.children[1];
  const Node &L1 = P.nodes[c1], &L2 = P.nodes[c2];
  if (!L1.leaf() || !L2.leaf()) return;
  const int R = nA_.r;
  if (L1.r != R || L2.r != R || L1.k != nA_.k || L2.k != nA_.k) return;
  int KP = 0;
  if (R == 16 && nA_.k <= 32) KP = 32;
  else if (R == 32 && nA_.k <= 48) KP = 48;
  else if (R == 64 && nA_.k <= 96) KP = 96;
  if (KP == 0) return;
  if (P.dims[0] != N1) return;
  const int64_t n2 = P.dims[1], nAs = N1 * n2, nB = P.N / nAs;
  // Z1-out form (STTNN, r >= 32): Z1 is written out and R_2 formed by one streaming
  // contraction that reads X_2 once, instead of re-reading X_2 in every row tile
  // (a BF16 plan writes Z1 in FP32 and contracts it with an FP32 copy of X_2)
  const int zdt = P.dtype == TTNN_BF16 ? TTNN_F32 : P.dtype;
  const bool zout = !tt && R >= 32 && right_mfma_eligible(static_cast<int64_t>(KP) * nB, n2, 1, R, zdt);
  Shape sh = shape_for(P.dtype, R, tt, zout);
  if (n2 % sh.B2 != 0 || nB % sh.SC != 0) return;
  int TA = static_cast<int>(n2 / sh.B2);
  // column tiles: the fewest that give every compute unit a tile (else as many as divide)
  int TB = 0;
  for (int cand = 1; cand <= 256; cand *= 2) {
    if (nB % (static_cast<int64_t>(sh.SC) * cand) != 0) continue;
    TB = cand;
    if (static_cast<int64_t>(TA) * cand >= 256) break;
  }
  if (TB == 0) return;
  // sttnn_t4_bf64_kernel, tiles of twice the slabs by half the columns, where both divide: R_1's
  // sums run over as many products as in the two-slab form's tiles
  if (P.dtype == TTNN_BF16 && R == 64 && zout && n2 % Bf64Layout::B2 == 0 && TB <= 128 &&
      nB % (static_cast<int64_t>(sh.SC) * 2 * TB) == 0) {
    sh.B2 = Bf64Layout::B2;
    TA /= 2;
    TB *= 2;
  }
  F.R = R;
  F.KP = KP;
  F.k = nA_.k;
  F.B2 = sh.B2;
  F.SC = sh.SC;
  F.TA = TA;
  F.TB = TB;
  F.CB = static_cast<int>(nB / (static_cast<int64_t>(sh.SC) * TB));
  F.n2 = n2;
  F.nA = nAs;
  F.nB = nB;
  F.node_A = A;
  F.node_1 = c1;
  F.node_2 = c2;
  F.tt = tt;
  F.node_B = root.children[1];
  if (tt && (P.nodes[F.node_B].r != R || P.nodes[F.node_B].m != nAs)) return;

  const int dt = P.dtype;
  const int64_t es = elem_size(dt);
  const bool x3 = split_form(dt, R, tt, zout);            // Y_A, Y_1, X_B as three BF16 planes as well
  // DRM copies in the fragment layouts of the kernel (the FP64 arrays of a lower-precision
  // plan hold the rounded values already, so these copies are exact)
  F.XA = P.alloc(es * nB * R);
  F.X1 = P.alloc(es * nAs / N1 * nB * R);
  F.YA = P.alloc(es * nAs * KP);
  if (x3) {
    F.YA3 = P.alloc(6 * nAs * KP);
    if (tt) F.XB3 = P.alloc(6 * nAs * R);
    else F.Y13 = P.alloc(6 * static_cast<int64_t>(N1) * KP);
    F.redo = P.alloc(4 * int64_t(8) * TA * TB);
  }
  const int x2dt = zout ? zdt : dt;
  if (tt) {
    F.XB = P.alloc(es * nAs * R);
  } else {
    F.Y1 = P.alloc(es * N1 * KP);
    F.X2 = P.alloc(elem_size(x2dt) * nB * KP * R);
  }
  const Node& NA = P.nodes[A];
  const double* XB64 = P.nodes[F.node_B].X64;
  const int k = nA_.k;
  // contraction index contiguous for every dtype
  if (!P.dry) {
    copy_layout(NA.X64, F.XA, dt, nB, R, 1, R, 1, 0, 0, nB, st);                     // [j][iB]
    copy_layout(L1.X64, F.X1, dt, nB, n2, R, n2 * R, R, 1, 0, nB, st);               // [j][i2][iB]
    auto rows = [&](const double* src, void* out, void* out3, int64_t d0, int64_t d1, int64_t s0) {   // [j][i]
      copy_layout(src, out, dt, d0, d1, 1, s0, 1, 0, 1, s0, st);
      if (!x3) return;
      const int blocks = static_cast<int>(std::min<int64_t>((d0 * d1 + 255) / 256, 16384));
      hipLaunchKernelGGL(gather_split, dim3(blocks), dim3(256), 0, st, src, static_cast<uint16_t*>(out3), d0, d1, s0,
                         int64_t(1), s0);
    };
    rows(NA.Y64, F.YA, F.YA3, nAs, KP, k);                                           // [jA][iA]
    if (tt) {
      rows(XB64, F.XB, F.XB3, nAs, R, R);                                            // [j][iA]
    } else {
      rows(L1.Y64, F.Y1, F.Y13, N1, KP, k);                                          // [j1][i1]
      copy_layout(L2.X64, F.X2, x2dt, KP, nB, R, R, static_cast<int64_t>(k) * R, 1, 0, k, st);  // [j][iB][j1]
    }
  }
  const int64_t as = dt == TTNN_F64 ? 8 : 4;
  F.PRA = P.alloc(as * TB * nAs * R);
  F.PZA = P.alloc(as * TA * KP * nB);
  F.PR1 = P.alloc(as * static_cast<int64_t>(TA) * TB * N1 * R);
  F.zout = zout;
  if (tt) F.PRB = P.alloc(as * TA * R * nB);
  else if (F.zout) F.Z1 = P.alloc(elem_size(zdt) * KP * n2 * nB);
  else F.PR2 = P.alloc(as * TB * n2 * R);
  F.enabled = true;
}

bool try_fused_update(Plan& P, const void* block, const int64_t* off, const int64_t* ext, double alpha,
                      hipStream_t st, std::vector<int>* done_nodes, std::vector<std::vector<int>>* done_prefixes) {
  const FusedT4& F = P.fused;
  if (!F.enabled) return false;
  for (int mu = 0; mu < P.d; ++mu)
    if (off[mu] != 0 || ext[mu] != P.dims[mu]) return false;
  SttnnArgs a;
  a.T = block;
  a.n2 = F.n2;
  a.nA = F.nA;
  a.nB = F.nB;
  a.TA = F.TA;
  a.TB = F.TB;
  a.CB = F.CB;
  a.XA = F.XA;
  a.X1 = F.X1;
  a.YA = F.YA;
  a.Y1 = F.Y1;
  a.X2 = F.X2;
  a.XB = F.XB;
  a.PRA = F.PRA;
  a.PZA = F.PZA;
  a.PR1 = F.PR1;
  a.PR2 = F.PR2;
  a.PRB = F.PRB;
  a.Z1 = F.Z1;
  a.YA3 = static_cast<const uint16_t*>(F.YA3);
  a.Y13 = static_cast<const uint16_t*>(F.Y13);
  a.XB3 = static_cast<const uint16_t*>(F.XB3);
  a.redo = static_cast<uint32_t*>(F.redo);
  if (P.dtype == TTNN_BF16) launch_sttnn_dt<TTNN_BF16>(F.R, F.tt, F.zout, a, st);
  else if (P.dtype == TTNN_F32) launch_sttnn_dt<TTNN_F32>(F.R, F.tt, F.zout, a, st);
  else launch_sttnn_dt<TTNN_F64>(F.R, F.tt, F.zout, a, st);
  if (P.timing) {
    TTNN_HIP(hipEventRecord(P.sweep_ev[1], st));
    P.sweep_recorded = true;
  }

  if (F.zout) {
    // R_2 += alpha Z1 X_2: Z1 [i_2][(i_B, j1)] against X_2 [j][(i_B, j1)], one pass over both
    // on the caller's stream.  Beside the reduction and the FP64 jobs that follow, on a stream
    // of its own, every one of them took longer than alone (R_2 of a 128^4 tensor at FP32, r =
    // 32, 220 us for 134, the reduction 83 for 48, the FP64 jobs 120 for 32), and the update
    // 797 us for 774 (BF16 at r = 64: 1120 for 1112, FP64: 1895 for 1809).
    const int64_t K = static_cast<int64_t>(F.KP) * F.nB;
    const int zdt = P.dtype == TTNN_BF16 ? TTNN_F32 : P.dtype;      // Z1 and this X_2 copy
    const int nch = launch_right_mfma(F.Z1, zdt, K, F.n2, 1, F.X2, K, F.R, P.partial, P.partial_elems, st);
    const Node& n2d = P.nodes[F.node_2];
    launch_reduce(P.partial, nch, F.n2, F.R, 0, alpha, box_rows(P, n2d.first, n2d.last, off, ext), n2d.n, n2d.R, 1, 1,
                  st);
  }

  const std::vector<int> pre{F.node_A};
  double* ZA = P.chain + P.prefix_offset.at(pre);
  const int node_last = F.tt ? F.node_B : F.node_2;
  const void* plast = F.tt ? F.PRB : F.PR2;
  const int64_t nbA = ((F.nA + kRTX - 1) / kRTX) * ((F.R + kRTY - 1) / kRTY);
  // Z_A: a tile's threads sum an entry's TA partials by themselves, which leaves the chip idle
  // where there are fewer tiles than compute units; then eight threads share an entry.  r = 32,
  // whole update, one thread and eight: 128 x 1024 x 32 FP64 (512 partials, 3 tiles) 210 -> 170
  // us, 128 x 1024 x 1024 FP32 (96 tiles) 538 -> 492, 128 x 256 x 1024 FP64 327 -> 312, 128 x 32 x
  // 4096 (16 partials, 384 tiles) as before.
  const int64_t zt = ((F.k + kRTX - 1) / kRTX) * ((F.nB + kRTY - 1) / kRTY);
  const bool zsplit = zt < 256 && F.TA >= 2 * kSplitT;
  const int64_t nbZ = zsplit ? F.k * ((F.nB + kSplitY - 1) / kSplitY) : zt;
  const int mode = F.tt ? 1 : F.zout ? 2 : 0;
  const int64_t nb1 = (static_cast<int64_t>(N1) * F.R * 16 + 255) / 256;
  const int64_t rest = (F.tt ? F.nB : F.zout ? 0 : F.n2) * F.R;
  const int64_t nbE = std::min<int64_t>((rest + 255) / 256, 2048);
  const dim3 grid(static_cast<unsigned>(nbA + nbZ + nb1 + nbE));
  if (P.dtype == TTNN_F64)
    hipLaunchKernelGGL(sttnn_t4_reduce<double>, grid, dim3(256), 0, st, static_cast<const double*>(F.PRA),
                       static_cast<const double*>(F.PZA), static_cast<const double*>(F.PR1),
                       static_cast<const double*>(plast), F.TA, F.TB, F.n2, F.nA, F.nB, F.R, F.KP, F.k, alpha,
                       P.nodes[F.node_A].R, ZA, P.nodes[F.node_1].R, P.nodes[node_last].R, mode,
                       static_cast<int>(nbA), static_cast<int>(nbZ), zsplit ? 1 : 0, static_cast<int>(nb1));
  else
    hipLaunchKernelGGL(sttnn_t4_reduce<float>, grid, dim3(256), 0, st, static_cast<const float*>(F.PRA),
                       static_cast<const float*>(F.PZA), static_cast<const float*>(F.PR1),
                       static_cast<const float*>(plast), F.TA, F.TB, F.n2, F.nA, F.nB, F.R, F.KP, F.k, alpha,
                       P.nodes[F.node_A].R, ZA, P.nodes[F.node_1].R, P.nodes[node_last].R, mode,
                       static_cast<int>(nbA), static_cast<int>(nbZ), zsplit ? 1 : 0, static_cast<int>(nb1));
  done_nodes->assign({F.node_A, F.node_1, node_last});
  done_prefixes->assign({pre});
  return true;
}

}  // namespace ttnn
