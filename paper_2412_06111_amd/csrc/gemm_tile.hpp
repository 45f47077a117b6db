// Device code of the generic contraction (see gemm.hip), shared by the translation units
// that instantiate it, one per storage type so that they compile side by side: the tile,
// the fixed-order sums of chunk partials and the persistent ingest kernel.
#pragma once

#include <cstring>
#include <type_traits>

#include "kernels.hpp"
#include "mfma.hpp"

namespace ttnn {

// ---------------------------------------------------------------- the contraction tile
// A workgroup of four waves owns TR output rows (16, 32 or 64), one block of 16 NCB
// columns and one chunk of the contraction, taken in steps of BKX values staged in LDS
// (two buffers, one barrier a step, the next step's loads in flight while a step is
// multiplied).  TR < 64: the waves that the rows leave over take slices of every step,
// and their sums are added in wave order at the end.
//
// The addresses separate: operand entry (m, i) sits at koff(contraction index) +
// roff(row), and the contraction index alone gives the DRM row.  A thread keeps the
// pointers of its few rows in registers; the offsets of the next kTab contraction values
// (mixed-radix digits of the box, in 32-bit divisions while the indices fit) are worked
// out one a thread and kept in LDS.  A form that divided in 64 bits for every entry and
// worked out a step's DRM rows on 16 threads took 2.5 us for a step of 16 values; now a
// wave issues ~60 vector instructions beside the 16 MFMAs of a 64 x 32 x 32 step, and the
// tile is bound by those two and the barrier between steps (MFMA busy 40% and 37% in the two
// workloads below).  Measured
// with it before and now: a whole 97 x 113 x 61 x 75 FP32 tensor (r = 21, TTNN) 1250 ->
// 500 us (a pass over the 200 MB 140-220 -> 55-90 us); a 33.9M-entry box of a 64^5 FP32
// tensor (r = 24) 1764 -> 686 us, the faster packing included; two steps of loads in flight
// at three workgroups a compute unit 519 and 685, at four (spilling) 525 and 718.
//
// Products run on the 16x16x4 MFMA of the compute type CT: FP64 when an operand is FP64,
// else FP32 with the running sums moved to FP64 registers every kFlush steps, so a
// chunk's length does not change its accuracy and chunks can be as long as the machine's
// parallelism allows (fewer partials to write and add).  A lane reads V = 16 / sizeof(CT)
// consecutive contraction values of a row with one 16-byte LDS read and feeds them to V
// MFMAs; row pitches of BKX + V put the 16 rows of a read on distinct banks.
constexpr int kTab = 256;        // contraction values per offset table (one a thread)
constexpr int kFlush = 4;        // steps between moves of the FP32 sums to FP64

template <typename CT, int TR> struct TileDims {
  static constexpr int V = 16 / static_cast<int>(sizeof(CT));
  static constexpr int BKX = (TR == 64 ? 8 : 16) * V;   // contraction values per step
  static constexpr int PITCH = BKX + V;
  static constexpr int KW = 64 / TR;                    // waves along the contraction
};

struct TileOff {
  int64_t h;      // operand offset of the contraction value, in bytes
  int64_t d;      // DRM offset of its row, in bytes (both 0 past the end of the chunk)
};

constexpr size_t kTabBytes = 2 * kTab * sizeof(TileOff);
// Dynamic LDS of a form: both buffers of both operands, then the offset tables.
constexpr size_t tile_lds(int tr, int ncb) {
  return 2 * static_cast<size_t>(tr + 16 * ncb) * ((tr == 64 ? 8 : 16) + 1) * 16 + kTabBytes + 8 * static_cast<size_t>(tr);
}

__device__ inline int64_t map_at(const IndexMap& m, int64_t idx) {
  if (idx >> 32) return m(idx);
  uint32_t x = static_cast<uint32_t>(idx);
  int64_t row = 0;
  for (int p = 0; p < m.n; ++p) {
    const uint32_t e = static_cast<uint32_t>(m.ext[p]);      // a wider extent leaves x as it is
    const uint32_t q = m.ext[p] >> 32 ? 0u : x / e;
    const uint32_t i = x - q * e;
    x = q;
    row += (m.off[p] + i) * m.stride[p];
  }
  return row;
}
// a = idx mod L, b = idx / L
__device__ inline void split_at(int64_t idx, int64_t L, int64_t& a, int64_t& b) {
  if ((idx | L) >> 32) {
    b = idx / L;
    a = idx - b * L;
  } else {
    const uint32_t q = static_cast<uint32_t>(idx) / static_cast<uint32_t>(L);
    b = q;
    a = static_cast<uint32_t>(idx) - q * static_cast<uint32_t>(L);
  }
}

// A task's pointers come out of LDS, where the compiler cannot see that they are global: its
// flat loads count as LDS reads too, and every wait for an LDS operand would wait for them.
#define TTNN_GLOBAL __attribute__((address_space(1)))
typedef const char TTNN_GLOBAL* GlobalPtr;
template <typename T> __device__ __forceinline__ T load_global(GlobalPtr p) {
  return *reinterpret_cast<const T TTNN_GLOBAL*>(p);
}

template <typename CT> __device__ inline CT to_ct(float v) { return static_cast<CT>(v); }
template <typename CT> __device__ inline CT to_ct(double v) { return static_cast<CT>(v); }
template <typename CT> __device__ inline CT to_ct(uint16_t v) { return static_cast<CT>(bf16_bits_to_f32(v)); }

template <bool RIGHT, typename TH, typename TD, int TR, int NCB>
__device__ __forceinline__ void gemm_tile(const GemmTask& t, int64_t row0, int64_t c, int j0, char* lds) {
  using CT = std::conditional_t<std::is_same_v<TH, double> || std::is_same_v<TD, double>, double, float>;
  using P = Pol<std::is_same_v<CT, double> ? TTNN_F64 : TTNN_F32>;
  using Dm = TileDims<CT, TR>;
  constexpr bool F32 = std::is_same_v<CT, float>;
  constexpr int V = Dm::V, BKX = Dm::BKX, PITCH = Dm::PITCH, KW = Dm::KW, NJ = 16 * NCB;
  constexpr int KG = 4 * V;                       // contraction values per fragment read
  constexpr int NA = TR * BKX / 256;              // operand entries a thread stages per step
  constexpr int GK = BKX / V;                     // groups of V contraction values of a step
  constexpr int RS = 256 / GK;                    // contraction along memory: rows apart of a thread's groups
  constexpr int RW = TR < 32 ? TR : 32;           // rows along memory: rows per pass ...
  constexpr int KS = V * 256 / RW, NK = BKX / KS; // ... and values apart of its groups, groups of a row
  constexpr int NBK = BKX / 16;                   // DRM rows a thread stages per step
  static_assert(NA == V * NK * (TR / RW) && NA == V * (TR / RS) && BKX <= kTab && kTab % BKX == 0 && 256 % BKX == 0, "tile shape");
  typedef CT vec_t __attribute__((ext_vector_type(V)));

  CT* As = reinterpret_cast<CT*>(lds);            // [2][TR][PITCH]
  CT* Bs = As + 2 * TR * PITCH;                   // [2][NJ][PITCH]
  TileOff* tab = reinterpret_cast<TileOff*>(Bs + 2 * NJ * PITCH);   // [2][kTab]
  int64_t* rows = reinterpret_cast<int64_t*>(tab + 2 * kTab);       // [TR]: row offsets, -1 past the end

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave & (TR / 16 - 1), kw = wave / (TR / 16);
  const int64_t L = t.L, n = t.n, Q = t.Q;
  const int64_t rows_total = RIGHT ? n : L * Q;
  const int64_t K = RIGHT ? L * Q : n;
  const int64_t k_begin = c * t.kchunk;
  const int64_t k_end = (k_begin + t.kchunk < K) ? k_begin + t.kchunk : K;
  const bool kfast = RIGHT ? (L > 1) : (L == 1);  // the contraction runs along memory
  const int ncols = t.ncols;
  auto fill = [&](int tb, int64_t k0) {           // the table of [k0, k0 + kTab)
    const int64_t kg = k0 + tid;
    TileOff o{0, 0};
    if (kg < k_end) {
      if constexpr (RIGHT) {
        int64_t l, q;
        split_at(kg, L, l, q);
        o.h = t.hm.strided ? map_at(t.hm.ml, l) + map_at(t.hm.mq, q) : l + L * n * q;
        o.d = (map_at(t.amap, l) + map_at(t.bmap, q)) * t.sDr;
      } else {
        o.h = t.hm.strided ? map_at(t.hm.mi, kg) : L * kg;
        o.d = map_at(t.amap, kg) * t.sDr;
      }
    }
    o.h *= static_cast<int64_t>(sizeof(TH));
    o.d *= static_cast<int64_t>(sizeof(TD));
    tab[tb * kTab + tid] = o;
  };
  if (tid < TR) {
    const int64_t row = row0 + tid;
    int64_t o = -1;
    if (row < rows_total) {
      if constexpr (RIGHT) {
        o = t.hm.strided ? map_at(t.hm.mi, row) : L * row;
      } else {
        int64_t l, q;
        split_at(row, L, l, q);
        o = t.hm.strided ? map_at(t.hm.ml, l) + map_at(t.hm.mq, q) : l + L * n * q;
      }
    }
    rows[tid] = o;
  }
  fill(0, k_begin);
  __syncthreads();

  // Staging map of a thread, which takes groups of V consecutive contraction values of a row
  // (one 16-byte LDS store each): contraction along memory, group kk0 of rows rr0 + RS s;
  // rows along memory, groups kk0 + KS u of rows rr0 + RW b.  Along memory a group inside one
  // run of it is one load (of any alignment).  With single values, a load and a 4-byte store
  // each, and flat loads the whole 97 x 113 x 61 x 75 FP32 tensor took 549 us, with single
  // values and global loads 517, now 500 (the 33.9M-entry box 727, 686, 686).
  const int kk0 = V * (kfast ? tid % GK : tid / RW);
  const int rr0 = kfast ? tid / GK : tid % RW;
  const bool runs = !t.hm.strided;
  // Rows past the end read row 0 of the operand and columns past the end column j0 of the
  // DRM: what they form lands in rows and columns that are not written.
  constexpr int NR = TR / RS > TR / RW ? TR / RS : TR / RW;    // rows of a thread
  GlobalPtr hp[NR];
#pragma unroll
  for (int s = 0; s < NR; ++s) {
    const int64_t o = rows[(kfast ? rr0 + RS * s : rr0 + RW * s) % TR];
    hp[s] = (GlobalPtr)t.H + (o < 0 ? 0 : o) * static_cast<int64_t>(sizeof(TH));
  }
  const int jl = tid & 15, kb0 = tid >> 4;
  GlobalPtr dp[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const int col = j0 + 16 * cb + jl < ncols ? j0 + 16 * cb + jl : j0;
    dp[cb] = (GlobalPtr)t.D + col * t.sDc * static_cast<int64_t>(sizeof(TD));
  }

  // A step's loads, and its stores to LDS.  Values past the end of the chunk read value 0
  // and are zeroed when they are stored (both operands: 0 x inf): only a chunk's last step
  // can hold any, and nothing in fetch looks at a loaded value, so no wait stands between
  // these loads and the products of the step before (with the zeroing in fetch every step
  // waited for its operand loads, then for its DRM loads, before its first product:
  // 1.9 times the time).
  struct Stage {
    TH a[NA];
    TD b[NBK * NCB];
  };
  auto fetch = [&](int64_t k0, Stage& g) {
    const TileOff* tp = tab + static_cast<int>((k0 - k_begin) & (2 * kTab - 1));
    if (kfast) {
      const int64_t h = tp[kk0].h;
      if (runs && tp[kk0 + V - 1].h - h == static_cast<int64_t>((V - 1) * sizeof(TH))) {
        typedef TH group_t __attribute__((ext_vector_type(V), aligned(sizeof(TH))));
#pragma unroll
        for (int s = 0; s < TR / RS; ++s) {
          const group_t q = load_global<group_t>(hp[s] + h);
#pragma unroll
          for (int v = 0; v < V; ++v) g.a[s * V + v] = q[v];
        }
      } else {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const int64_t hv = tp[kk0 + v].h;
#pragma unroll
          for (int s = 0; s < TR / RS; ++s) g.a[s * V + v] = load_global<TH>(hp[s] + hv);
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < NK; ++u)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const int64_t h = tp[kk0 + KS * u + v].h;
#pragma unroll
          for (int b = 0; b < TR / RW; ++b) g.a[(b * NK + u) * V + v] = load_global<TH>(hp[b] + h);
        }
    }
#pragma unroll
    for (int u = 0; u < NBK; ++u) {
      const int64_t d = tp[kb0 + 16 * u].d;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) g.b[u * NCB + cb] = load_global<TD>(dp[cb] + d);
    }
  };
  // LAST: only the first klen values of the step exist
  auto store = [&](int buf, const Stage& g, auto last, int klen) {
    constexpr bool LAST = decltype(last)::value;
    CT* A = As + buf * TR * PITCH + rr0 * PITCH + kk0;
    CT* B = Bs + buf * NJ * PITCH + jl * PITCH + kb0;
    auto put = [&](CT* to, const TH* x, int k) {
      vec_t w;
#pragma unroll
      for (int v = 0; v < V; ++v) w[v] = !LAST || k + v < klen ? to_ct<CT>(x[v]) : CT(0);
      *reinterpret_cast<vec_t*>(to) = w;
    };
    if (kfast) {
#pragma unroll
      for (int s = 0; s < TR / RS; ++s) put(A + RS * s * PITCH, &g.a[s * V], kk0);
    } else {
#pragma unroll
      for (int b = 0; b < TR / RW; ++b)
#pragma unroll
        for (int u = 0; u < NK; ++u) put(A + RW * b * PITCH + KS * u, &g.a[(b * NK + u) * V], kk0 + KS * u);
    }
#pragma unroll
    for (int u = 0; u < NBK; ++u)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        B[16 * cb * PITCH + 16 * u] = !LAST || kb0 + 16 * u < klen ? to_ct<CT>(g.b[u * NCB + cb]) : CT(0);
  };

  typename P::CFrag acc[NCB];
  f64x4_t sum[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    acc[cb] = typename P::CFrag{};
    sum[cb] = f64x4_t{};
  }

  Stage g;
  if (k_begin < k_end) fetch(k_begin, g);
  int step = 0;
  for (int64_t k = k_begin; k < k_end; k += BKX, ++step) {
    const int buf = step & 1;
    if (k + BKX > k_end) store(buf, g, std::true_type{}, static_cast<int>(k_end - k));
    else store(buf, g, std::false_type{}, BKX);
    // the first step of a table fills the next one: its buffer was last read by loads
    // issued before the previous step's barrier, and is first read after this one
    const int in_tab = static_cast<int>((k - k_begin) & (2 * kTab - 1));
    if (in_tab % kTab == 0 && k + kTab < k_end) fill(in_tab == 0 ? 1 : 0, k + kTab);
    __syncthreads();
    if (k + BKX < k_end) fetch(k + BKX, g);
    const CT* A = As + buf * TR * PITCH + (16 * wr + l16) * PITCH + kw * (BKX / KW) + V * lg;
    const CT* B = Bs + buf * NJ * PITCH + l16 * PITCH + kw * (BKX / KW) + V * lg;
#pragma unroll
    for (int h = 0; h < BKX / KW / KG; ++h) {
      const vec_t a = *reinterpret_cast<const vec_t*>(A + h * KG);
      vec_t b[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) b[cb] = *reinterpret_cast<const vec_t*>(B + 16 * cb * PITCH + h * KG);
#pragma unroll
      for (int s = 0; s < V; ++s)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[cb] = P::mfma(a[s], b[cb][s], acc[cb]);
    }
    if constexpr (F32) {
      if (step % kFlush == kFlush - 1) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
          for (int v = 0; v < 4; ++v) sum[cb][v] += static_cast<double>(acc[cb][v]);
          acc[cb] = typename P::CFrag{};
        }
      }
    }
  }
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int v = 0; v < 4; ++v) sum[cb][v] += static_cast<double>(acc[cb][v]);

  if constexpr (KW > 1) {                         // the slices' sums, in wave order
    static_assert(sizeof(double) * 1024 * NCB <= 2 * (TR + NJ) * PITCH * sizeof(CT), "sums fit the buffers");
    double* red = reinterpret_cast<double*>(lds);
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[((wave * NCB + cb) * 4 + v) * 64 + lane] = sum[cb][v];
    __syncthreads();
    if (kw != 0) return;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int w = 1; w < KW; ++w) sum[cb][v] += red[(((wave + w * (TR / 16)) * NCB + cb) * 4 + v) * 64 + lane];
  }

  // lane holds C[16 wr + crow(lane, v)][16 cb + l16]
  double TTNN_GLOBAL* out = (double TTNN_GLOBAL*)t.out + c * t.ol.cs;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t row = row0 + 16 * wr + P::crow(lane, v);
    if (row >= rows_total) continue;
    int64_t lo = row, hi = 0;
    if (t.ol.Lo <= row) split_at(row, t.ol.Lo, lo, hi);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int j = j0 + 16 * cb + l16;
      if (j < ncols) out[lo * t.ol.s0 + static_cast<int64_t>(j) * t.ol.s1 + hi * t.ol.s2] = sum[cb][v];
    }
  }
}

// Tile rel of a task, in the task's form (rows per tile and column blocks).
template <bool RIGHT, typename TH, typename TD, int TR>
__device__ __forceinline__ void gemm_form(const GemmTask& t, int64_t rb, int64_t c, int cb, char* lds) {
  const int ncb = t.ncb, j0 = cb * 16 * ncb;
  if (ncb == 1) gemm_tile<RIGHT, TH, TD, TR, 1>(t, rb * TR, c, j0, lds);
  else if (ncb == 2) gemm_tile<RIGHT, TH, TD, TR, 2>(t, rb * TR, c, j0, lds);
  else if constexpr (TR == 64) gemm_tile<RIGHT, TH, TD, TR, 3>(t, rb * TR, c, j0, lds);
}
template <typename TH, typename TD>
__device__ __forceinline__ void gemm_any(const GemmTask& t, int64_t rel, char* lds) {
  int64_t rb, c, cb;
  split_at(rel, t.row_blocks, rb, rel);
  split_at(rel, t.nch, c, cb);
  const int jb = static_cast<int>(cb);
  if (!t.right) gemm_form<false, TH, TD, 64>(t, rb, c, jb, lds);
  else if (t.tr == 16) gemm_form<true, TH, TD, 16>(t, rb, c, jb, lds);
  else if (t.tr == 32) gemm_form<true, TH, TD, 32>(t, rb, c, jb, lds);
  else gemm_form<true, TH, TD, 64>(t, rb, c, jb, lds);
}

// Copy a descriptor from global memory into LDS (8-byte words) after finding the task
// that owns this workgroup, the last one whose first_block is not past it: a wave looks
// at 64 tasks with one load (a binary search by one thread was a chain of up to six
// dependent loads, 3-4 us before a tile's first load).
template <typename Task>
__device__ inline int64_t load_task(const Task* __restrict__ tasks, int ntasks, Task* t, int64_t b) {
  __shared__ int idx;
  if (threadIdx.x < 64) {
    int found = 0;
    for (int base = 0; base < ntasks; base += 64) {
      const int i = base + static_cast<int>(threadIdx.x);
      const bool ge = i < ntasks && tasks[i].first_block <= b;
      const uint64_t m = __ballot(ge);
      if (m) found = base + 63 - __builtin_clzll(m);
      if (m != ~0ull) break;
    }
    if (threadIdx.x == 0) idx = found;
  }
  __syncthreads();
  static_assert(sizeof(Task) % 8 == 0, "task size");
  const uint64_t* src = reinterpret_cast<const uint64_t*>(tasks + idx);
  uint64_t* dst = reinterpret_cast<uint64_t*>(t);
  for (int w = threadIdx.x; w < static_cast<int>(sizeof(Task) / 8); w += blockDim.x) dst[w] = src[w];
  __syncthreads();
  return b - t->first_block;
}

// Every workgroup serves one tile of one task; tasks of one launch may belong to
// different updates (of different plans) and have different sizes.
// Tile b of a batched contraction launch.
template <typename TH, typename TD>
__device__ __forceinline__ void gemm_task_tile(const GemmTask* __restrict__ tasks, int ntasks, int64_t b, char* lds) {
  __shared__ __align__(16) char tbuf[sizeof(GemmTask)];      // raw storage: IndexMap has initialisers
  GemmTask& t = *reinterpret_cast<GemmTask*>(tbuf);
  const int64_t rel = load_task(tasks, ntasks, &t, b);
  gemm_any<TH, TD>(t, rel, lds);
}

// The tasks of a launch: a table in device memory (ntasks > 0), one task passed by value
// (0), or -ntasks linear ones passed by value; right and left ones side by side.  A task's maps are indexed at run time,
// which the compiler would serve from a private copy in scratch, so the workgroup copies
// the task from the argument segment to LDS.
struct GemmByValue {
  union {
    char one[sizeof(GemmTask)];
    GemmLin lin[kLinTasks];
  };
};
template <typename TH, typename TD>
__global__ __launch_bounds__(256, 4) void hm_gemm(const GemmTask* __restrict__ tasks, int64_t ntasks, GemmByValue) {
  extern __shared__ __align__(16) char tile_mem[];
  __shared__ __align__(16) char tbuf[sizeof(GemmTask)];      // raw storage: IndexMap has initialisers
  GemmTask& t = *reinterpret_cast<GemmTask*>(tbuf);
  int64_t rel = static_cast<int64_t>(blockIdx.x);
  const char* args = (const char*)__builtin_amdgcn_kernarg_segment_ptr() + 16;   // past the two scalars
  if (ntasks > 0) {
    rel = load_task(tasks, static_cast<int>(ntasks), &t, rel);
  } else if (ntasks == 0) {
    for (int w = threadIdx.x; w < static_cast<int>(sizeof(GemmTask) / 8); w += 256)
      reinterpret_cast<uint64_t*>(tbuf)[w] = reinterpret_cast<const uint64_t*>(args)[w];
    __syncthreads();
  } else {
    __shared__ GemmLin lin;
    rel = load_task(reinterpret_cast<const GemmLin*>(args), static_cast<int>(-ntasks), &lin, rel);
    if (threadIdx.x == 0) {
      t.H = lin.H;
      t.D = lin.D;
      t.out = lin.out;
      t.L = lin.L;
      t.n = lin.n;
      t.Q = lin.Q;
      t.sDr = lin.sDr;
      t.sDc = 1;
      t.kchunk = lin.kchunk;
      t.row_blocks = lin.row_blocks;
      t.nch = lin.nch;
      t.ncols = lin.ncols;
      t.tr = lin.tr;
      t.ncb = lin.ncb;
      t.right = lin.right;
      // the DRM row of (l, q) is l + L q, of a left value the value itself
      t.amap.n = t.bmap.n = 1;
      t.amap.ext[0] = t.bmap.ext[0] = INT64_MAX;
      t.amap.off[0] = t.bmap.off[0] = 0;
      t.amap.stride[0] = 1;
      t.bmap.stride[0] = lin.L;
      t.hm.strided = 0;
      t.ol = lin.store ? OutLayout{lin.L, 1, lin.L, lin.L * lin.ncols, 0}
                       : OutLayout{INT64_MAX, lin.ncols, 1, 0, (lin.right ? lin.n : lin.L * lin.Q) * lin.ncols};
    }
    __syncthreads();
  }
  gemm_any<TH, TD>(t, rel, tile_mem);
}

// part[c * stride + e] summed over c in [c0, c1) in the order of c: the loads go out
// eight at a time with no dependence between them, the additions stay in order, so the
// sum is bitwise that of the plain loop.
__device__ __forceinline__ double sum_chunks(const double* __restrict__ part, int c0, int c1, int64_t stride,
                                             int64_t e) {
  double s = 0.0;
  int c = c0;
  for (; c + 8 <= c1; c += 8) {
    double v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = part[(c + i) * stride + e];
#pragma unroll
    for (int i = 0; i < 8; ++i) s += v[i];
  }
  for (; c < c1; ++c) s += part[c * stride + e];
  return s;
}

__device__ inline void reduce_range(const double* __restrict__ part, int nchunks, int64_t rows, int ncols, int mode,
                                    double alpha, const IndexMap& rmap, int64_t ldr, double* __restrict__ dst,
                                    int64_t L, int64_t kdim, int64_t start, int64_t step, int64_t stride) {
  const int64_t total = rows * ncols;
  for (int64_t e = start; e < total; e += step) {
    int64_t row, j;
    split_at(e, ncols, j, row);
    const double s = sum_chunks(part, 0, nchunks, stride, e);
    if (mode == 0) {
      dst[map_at(rmap, row) + ldr * j] += alpha * s;
    } else {
      int64_t l, q;
      split_at(row, L, l, q);
      const int64_t o = l + L * (j + kdim * q);
      if (mode == 1) dst[o] += alpha * s;
      else dst[o] = s;
    }
  }
}

__device__ __forceinline__ void reduce_task_tile(const ReduceTask* __restrict__ tasks, int ntasks, int64_t b) {
  __shared__ __align__(16) char tbuf[sizeof(ReduceTask)];
  ReduceTask& t = *reinterpret_cast<ReduceTask*>(tbuf);
  const int64_t rel = load_task(tasks, ntasks, &t, b);
  reduce_range(t.part, t.nchunks, t.rows, t.ncols, t.mode, t.alpha, t.rmap, t.ldr, t.dst, t.L, t.kdim,
               rel * 256 + threadIdx.x, t.nblocks * 256, t.cstride ? t.cstride : t.rows * t.ncols);
}

constexpr int kFold = 32;

// Fold groups of kFold consecutive chunks into each group's first slot (see
// fold_chunks_kernel); workgroup -> (task, element block, group).
__device__ __forceinline__ void fold_task_tile(const ReduceTask* __restrict__ tasks, int ntasks, int64_t b) {
  __shared__ __align__(16) char tbuf[sizeof(ReduceTask)];
  ReduceTask& t = *reinterpret_cast<ReduceTask*>(tbuf);
  const int64_t rel = load_task(tasks, ntasks, &t, b);
  const int64_t E = t.rows * t.ncols;
  const int64_t eblocks = (E + 255) / 256;
  const int64_t e = (rel % eblocks) * 256 + threadIdx.x;
  const int g = static_cast<int>(rel / eblocks);
  if (e >= E) return;
  const int c0 = g * kFold, c1 = c0 + kFold < t.nchunks ? c0 + kFold : t.nchunks;
  t.part[c0 * E + e] = sum_chunks(t.part, c0, c1, E, e);
}

// ---------------------------------------------------------------- persistent ingest
// One launch for a whole batched round of box updates: the workgroups sweep, phase by
// phase, every tile of every task list of the round (a level's contractions of all
// kinds, then its chunk folds, then its reductions, level after level) and meet at a
// grid-wide barrier between phases.  The tiles are those of the per-level launches, so
// results are bitwise the same.  Launched cooperatively (every workgroup resident), so
// each barrier ends; the wait is still bounded, and a wait that ran out marks the
// round's plans (their sticky numerical status).
struct IngestSeg {
  int64_t tasks;        // byte offset of the task table from the program
  int64_t blocks;
  int32_t kind, ntasks;
};
struct IngestPhase {
  IngestSeg seg[kIngestSegs];
  int32_t nseg, pad_;
};
struct IngestProgram {
  uint32_t counter;     // barrier arrivals (zero as staged)
  int32_t nphases, nsticky, pad_;
  int* sticky[kIngestPlans];
  IngestPhase ph[kIngestPhases];
};

__device__ inline bool grid_barrier(uint32_t* counter, uint32_t target) {
  __shared__ int ok;
  __syncthreads();                                     // the workgroup's writes are done
  if (threadIdx.x == 0) {
    __threadfence();                                   // ... and visible device-wide
    __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t spins = 0;
    ok = 1;
    while (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      __builtin_amdgcn_s_sleep(2);
      if (++spins > (1u << 24)) {                      // ~1 s: cannot happen with resident workgroups
        ok = 0;
        break;
      }
    }
    __threadfence();                                   // later reads see the other workgroups' writes
  }
  __syncthreads();
  return ok != 0;
}

template <typename TC>
__global__ __launch_bounds__(256) void ingest_kernel(char* base) {
  extern __shared__ __align__(16) char tile_mem[];
  IngestProgram* prog = reinterpret_cast<IngestProgram*>(base);
  uint32_t* counter = &prog->counter;
  const int nph = prog->nphases;
  for (int p = 0; p < nph; ++p) {
    const IngestPhase& P = prog->ph[p];
    int64_t total = 0;
    for (int s = 0; s < P.nseg; ++s) total += P.seg[s].blocks;
    for (int64_t b = blockIdx.x; b < total; b += gridDim.x) {
      int s = 0;
      int64_t rel = b;
      while (rel >= P.seg[s].blocks) rel -= P.seg[s++].blocks;
      const IngestSeg& g = P.seg[s];
      const void* tasks = base + g.tasks;
      switch (g.kind) {
        case kSegRaw:
          gemm_task_tile<TC, TC>(static_cast<const GemmTask*>(tasks), g.ntasks, rel, tile_mem);
          break;
        case kSegF64:
          gemm_task_tile<double, double>(static_cast<const GemmTask*>(tasks), g.ntasks, rel, tile_mem);
          break;
        case kSegFold:
          fold_task_tile(static_cast<const ReduceTask*>(tasks), g.ntasks, rel);
          break;
        default:
          reduce_task_tile(static_cast<const ReduceTask*>(tasks), g.ntasks, rel);
          break;
      }
    }
    if (p + 1 < nph && !grid_barrier(counter, static_cast<uint32_t>(p + 1) * gridDim.x)) {
      if (threadIdx.x == 0)
        for (int i = 0; i < prog->nsticky; ++i) atomicOr(prog->sticky[i], 1);
      return;
    }
  }
}

// What a translation unit provides for its storage type T: the contraction launches with
// raw operands of type T, and its ingest kernel.
template <typename T>
void launch_tiles(const GemmTask* tasks, int nt, const GemmTask& one, int64_t blocks, size_t lds, hipStream_t st) {
  GemmByValue v{};
  if (!tasks) std::memcpy(v.one, &one, sizeof(one));
  hipLaunchKernelGGL((hm_gemm<T, T>), dim3(static_cast<unsigned>(blocks)), dim3(256), lds, st, tasks,
                     static_cast<int64_t>(tasks ? nt : 0), v);
}
template <typename T>
void launch_tiles_lin(const GemmLin* tasks, int nt, int64_t blocks, size_t lds, hipStream_t st) {
  GemmByValue v{};
  std::memcpy(v.lin, tasks, static_cast<size_t>(nt) * sizeof(GemmLin));
  hipLaunchKernelGGL((hm_gemm<T, T>), dim3(static_cast<unsigned>(blocks)), dim3(256), lds, st, nullptr,
                     static_cast<int64_t>(-nt), v);
}
using LaunchTiles = void (*)(const GemmTask*, int, const GemmTask&, int64_t, size_t, hipStream_t);
using LaunchLin = void (*)(const GemmLin*, int, int64_t, size_t, hipStream_t);
struct TileKernels {
  LaunchTiles table;
  LaunchLin lin;
  const void* ingest;
};
TileKernels tile_kernels_f64();
TileKernels tile_kernels_f32();
TileKernels tile_kernels_bf16();

}  // namespace ttnn
