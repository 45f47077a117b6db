// Generic contraction kernels of the engine (any tree, any box, any dtype).
//
// One LDS-tiled kernel (gemm_tile.hpp) covers both contractions the method needs on a
// 3-index view H[L][n][Q] of a (partially contracted) tensor:
//   RIGHT  R(i, j)    = sum_{l,q} H[l, i, q] X[row(l, q), j]   (right sketch T^{t} X_t,
//                                                           Sec. 4; STTNN on T_{S_t}, Sec. 5)
//   LEFT   Z(l, j, q) = sum_i     H[l, i, q] Y[row(i), j]      (mode product with Y_s^T,
//                                                           Def. 1 / Sec. 5 contractions)
// The contraction is split in chunks; each chunk writes an FP64 partial that a
// second kernel sums in a fixed order, so the result does not depend on timing.
// This path is the reference engine for arbitrary shapes; the fused kernels for
// the large dense trees live in separate files.
#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>

#include "gemm_tile.hpp"

namespace ttnn {
namespace {

constexpr int kTargetBlocks = 768;    // workgroups a contraction is split for: one round of three a compute unit
constexpr int kMinSteps = 8;          // and the least steps a chunk is worth (below, a tile's
                                      // descriptor, tables and first loads outweigh its steps)

// The kernels of a contraction's operand types: the raw block with the compute-type maps,
// or an FP64 intermediate with the FP64 maps.
TileKernels kernels_for(int th, int td) {
  TTNN_REQUIRE(th == td, TTNN_E_INVALID, "contraction operands of different types");
  return th == TTNN_F64 ? tile_kernels_f64() : th == TTNN_F32 ? tile_kernels_f32() : tile_kernels_bf16();
}

__global__ __launch_bounds__(256) void reduce_batched_kernel(const ReduceTask* __restrict__ tasks, int ntasks) {
  reduce_task_tile(tasks, ntasks, static_cast<int64_t>(blockIdx.x));
}

// The same two passes over tables passed with the launch (identity row maps).
struct ReduceLinList {
  ReduceLin t[kLinTasks];
};
__global__ __launch_bounds__(256) void reduce_lin_kernel(int64_t ntasks, ReduceLinList) {
  __shared__ ReduceLin t;
  const ReduceLin* tasks = (const ReduceLin*)((const char*)__builtin_amdgcn_kernarg_segment_ptr() + 8);
  const int64_t rel = load_task(tasks, static_cast<int>(ntasks), &t, static_cast<int64_t>(blockIdx.x));
  const int64_t total = t.rows * t.ncols;
  for (int64_t e = rel * 256 + threadIdx.x; e < total; e += static_cast<int64_t>(t.nblocks) * 256) {
    int64_t row, j;
    split_at(e, t.ncols, j, row);
    const double s = sum_chunks(t.part, 0, t.nchunks, t.cstride, e);
    int64_t o;
    if (t.mode == 0) {
      o = row + t.ldr * j;
    } else {
      int64_t l, q;
      split_at(row, t.L, l, q);
      o = l + t.L * (j + t.kdim * q);
    }
    if (t.mode == 2) t.dst[o] = s;
    else t.dst[o] += t.alpha * s;
  }
}
// Groups of kFold chunks summed into each group's first slot; nblocks: element blocks.
__global__ __launch_bounds__(256) void fold_lin_kernel(int64_t ntasks, ReduceLinList) {
  __shared__ ReduceLin t;
  const ReduceLin* tasks = (const ReduceLin*)((const char*)__builtin_amdgcn_kernarg_segment_ptr() + 8);
  const int64_t rel = load_task(tasks, static_cast<int>(ntasks), &t, static_cast<int64_t>(blockIdx.x));
  const int64_t E = t.rows * t.ncols;
  const int64_t e = (rel % t.nblocks) * 256 + threadIdx.x;
  const int c0 = static_cast<int>(rel / t.nblocks) * kFold, c1 = c0 + kFold < t.nchunks ? c0 + kFold : t.nchunks;
  if (e < E) t.part[c0 * E + e] = sum_chunks(t.part, c0, c1, E, e);
}

__global__ __launch_bounds__(256) void fold_batched_kernel(const ReduceTask* __restrict__ tasks, int ntasks) {
  fold_task_tile(tasks, ntasks, static_cast<int64_t>(blockIdx.x));
}

__global__ void reduce_kernel(const double* __restrict__ part, int nchunks, int64_t rows, int ncols, int mode,
                              double alpha, IndexMap rmap, int64_t ldr, double* __restrict__ dst, int64_t L,
                              int64_t kdim, int64_t stride) {
  reduce_range(part, nchunks, rows, ncols, mode, alpha, rmap, ldr, dst, L, kdim,
               static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x,
               static_cast<int64_t>(gridDim.x) * blockDim.x, stride);
}

// Many chunks, few elements: fold each group of kFold consecutive chunks into the
// group's first chunk slot (in place, fixed order), so that the final pass sums
// ceil(nchunks / kFold) values per element.  Element e of group g is read and
// written by one thread only.
__global__ void fold_chunks_kernel(double* __restrict__ part, int nchunks, int64_t E) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int g = blockIdx.y;
  if (e >= E) return;
  const int c0 = g * kFold, c1 = c0 + kFold < nchunks ? c0 + kFold : nchunks;
  part[c0 * E + e] = sum_chunks(part, c0, c1, E, e);
}

__global__ void copy_kernel(double* y, const double* x, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    y[i] = x[i];
}
__global__ void zero_int_kernel(int* p, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = 0;
}
// Block b of a list launch serves segment `seg` (blocks are dealt to segments in
// proportion to their length, at most kSegBlocks each).
__device__ inline int seg_of(const SegList& s, int b, int* first) {
  int acc = 0;
  for (int i = 0; i < s.count; ++i) {
    int64_t nb = (s.n[i] + 255) / 256;
    if (nb > kSegBlocks) nb = kSegBlocks;
    if (nb < 1) nb = 1;
    if (b < acc + nb) {
      *first = acc;
      return i;
    }
    acc += static_cast<int>(nb);
  }
  *first = acc;
  return -1;
}
__global__ void zero_list_kernel(SegList s) {
  int first = 0;
  const int i = seg_of(s, blockIdx.x, &first);
  if (i < 0) return;
  int64_t nb = (s.n[i] + 255) / 256;
  nb = nb > kSegBlocks ? kSegBlocks : (nb < 1 ? 1 : nb);
  for (int64_t e = static_cast<int64_t>(blockIdx.x - first) * 256 + threadIdx.x; e < s.n[i]; e += nb * 256)
    s.p[i][e] = 0.0;
}
// flag[b] = whether block b met an entry that is not finite (every block's word is written,
// so that nothing has to clear them first: a launch of its own, 4 us of a 79 us step)
__global__ void finite_list_kernel(SegList s, int* flag) {
  int first = 0;
  const int i = seg_of(s, blockIdx.x, &first);
  if (i < 0) return;
  int bad = 0;
  int64_t nb = (s.n[i] + 255) / 256;
  nb = nb > kSegBlocks ? kSegBlocks : (nb < 1 ? 1 : nb);
  for (int64_t e = static_cast<int64_t>(blockIdx.x - first) * 256 + threadIdx.x; e < s.n[i]; e += nb * 256)
    if (!isfinite(s.p[i][e])) bad = 1;
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) flag[blockIdx.x] = bad;
}

inline bool fold_pays(int nchunks, int64_t E) { return nchunks > 2 * kFold && E < (int64_t(1) << 20); }

inline int grid_for(int64_t n) {
  const int64_t b = (n + 255) / 256;
  return static_cast<int>(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

}  // namespace

// Rows per tile: a right contraction of few rows takes smaller row tiles (the spare waves
// split each step) so that its products are not mostly padding.
static int tile_rows(bool right, int64_t rows) { return !right || rows > 32 ? 64 : rows > 16 ? 32 : 16; }
// Columns: at most 48 a tile (32 in the small row tiles, by registers), spread evenly over
// the column blocks.
static int col_blocks_of(int tr, int ncols) { return tr == 64 ? (ncols + 47) / 48 : (ncols + 31) / 32; }
static int ncb_of(int tr, int ncols) { return ((ncols + 15) / 16 + col_blocks_of(tr, ncols) - 1) / col_blocks_of(tr, ncols); }
static int step_of(const GemmArgs& a) {
  const bool f64 = a.th == TTNN_F64 || a.td == TTNN_F64;
  return (tile_rows(a.right, a.right ? a.n : a.L * a.Q) == 64 ? 8 : 16) * (f64 ? 2 : 4);
}

int pick_chunks(const GemmArgs& a, size_t partial_cap) {
  const int64_t rows = a.right ? a.n : a.L * a.Q, K = a.right ? a.L * a.Q : a.n;
  if (rows <= 0 || a.ncols <= 0) return 1;
  const int tr = tile_rows(a.right, rows);
  const int64_t blocks = (rows + tr - 1) / tr * col_blocks_of(tr, a.ncols);
  int64_t want = kTargetBlocks / blocks;
  const int64_t by_len = (K + kMinSteps * step_of(a) - 1) / (kMinSteps * step_of(a));
  if (want > by_len) want = by_len;
  const int64_t cap = static_cast<int64_t>(partial_cap / static_cast<size_t>(rows * a.ncols));
  if (want > cap) want = cap;
  if (want > 65535) want = 65535;
  return static_cast<int>(want < 1 ? 1 : want);
}

int gemm_chunks(const GemmArgs& a, int64_t* kchunk_out) {
  const int64_t rows = a.right ? a.n : a.L * a.Q;
  const int64_t K = a.right ? a.L * a.Q : a.n;
  if (rows <= 0 || a.ncols <= 0) return 0;
  const int64_t bk = step_of(a);
  int64_t kchunk = (K + a.nchunks - 1) / a.nchunks;
  kchunk = ((kchunk + bk - 1) / bk) * bk;
  if (kchunk < bk) kchunk = bk;
  const int nch = static_cast<int>((K + kchunk - 1) / kchunk);
  if (kchunk_out) *kchunk_out = kchunk;
  return nch > 0 ? nch : 1;
}

static bool fill_task(const GemmArgs& a, GemmTask& t, size_t& lds) {
  const int nch = gemm_chunks(a, &t.kchunk);
  if (nch == 0) return false;
  const int64_t rows = a.right ? a.n : a.L * a.Q;
  t.H = a.H;
  t.D = a.D;
  t.out = a.out;
  t.L = a.L;
  t.n = a.n;
  t.Q = a.Q;
  t.sDr = a.sDr;
  t.sDc = a.sDc;
  t.ncols = a.ncols;
  t.amap = a.amap;
  t.bmap = a.bmap;
  t.hm = a.hm;
  t.ol = a.ol;
  t.tr = tile_rows(a.right, rows);
  t.ncb = ncb_of(t.tr, a.ncols);
  t.right = a.right ? 1 : 0;
  t.row_blocks = (rows + t.tr - 1) / t.tr;
  t.nch = nch;
  t.col_blocks = col_blocks_of(t.tr, a.ncols);
  lds = std::max(lds, tile_lds(t.tr, t.ncb));
  return true;
}

int launch_gemm(const GemmArgs& a, hipStream_t st) {
  GemmTask t{};
  size_t lds = 0;
  if (!fill_task(a, t, lds)) return 0;
  const int64_t blocks = t.row_blocks * t.nch * t.col_blocks;
  TTNN_REQUIRE(blocks < (int64_t(1) << 31), TTNN_E_INVALID, "contraction launch too large");
  kernels_for(a.th, a.td).table(nullptr, 0, t, blocks, lds, st);
  return static_cast<int>(t.nch);
}

BatchedGemm plan_gemm_batched(const std::vector<GemmArgs>& args) {
  BatchedGemm b;
  if (args.empty()) return b;
  b.th = args[0].th;
  b.td = args[0].td;
  b.tasks.reserve(args.size());
  for (const GemmArgs& a : args) {
    TTNN_REQUIRE(a.th == b.th && a.td == b.td, TTNN_E_INVALID,
                 "batched contraction with mixed kinds");
    GemmTask t{};
    if (!fill_task(a, t, b.lds)) continue;
    t.first_block = b.blocks;
    b.blocks += t.row_blocks * t.nch * t.col_blocks;
    b.tasks.push_back(t);
  }
  TTNN_REQUIRE(b.blocks < (int64_t(1) << 31), TTNN_E_INVALID, "batched launch too large");
  return b;
}

void launch_gemm_staged(const BatchedGemm& b, const GemmTask* d, hipStream_t st) {
  if (b.tasks.empty()) return;
  const int nt = static_cast<int>(b.tasks.size());
  kernels_for(b.th, b.td).table(d, nt, GemmTask{}, b.blocks, b.lds, st);
}

void launch_level_lin(const std::vector<GemmArgs>& args, const std::vector<ReduceTask>& reds, hipStream_t st) {
  std::vector<bool> taken(args.size(), false);
  for (size_t a = 0; a < args.size(); ++a) {              // one launch per operand type
    if (taken[a]) continue;
    std::vector<GemmLin> v;
    size_t lds = 0;
    int64_t blocks = 0;
    auto flush = [&]() {
      if (!v.empty()) kernels_for(args[a].th, args[a].td).lin(v.data(), static_cast<int>(v.size()), blocks, lds, st);
      v.clear();
      lds = 0;
      blocks = 0;
    };
    for (size_t b = a; b < args.size(); ++b) {
      if (taken[b] || args[b].th != args[a].th || args[b].td != args[a].td) continue;
      taken[b] = true;
      GemmTask t{};
      size_t mem = 0;
      if (!fill_task(args[b], t, mem)) continue;
      const int64_t mine = t.row_blocks * t.nch * t.col_blocks;
      TTNN_REQUIRE(!args[b].hm.strided && t.sDc == 1 && mine < (int64_t(1) << 31), TTNN_E_INVALID,
                   "contraction launch too large");
      if (v.size() == static_cast<size_t>(kLinTasks) || blocks + mine >= (int64_t(1) << 31)) flush();
      v.push_back(GemmLin{t.H, t.D, t.out, t.L, t.n, t.Q, t.sDr, t.kchunk, t.ncols, t.tr, t.ncb, t.right,
                          static_cast<int32_t>(blocks), static_cast<int32_t>(t.row_blocks), static_cast<int32_t>(t.nch),
                          t.ol.cs == 0 ? 1 : 0});
      blocks += mine;
      lds = std::max(lds, mem);
    }
    flush();
  }
  for (size_t i0 = 0; i0 < reds.size(); i0 += kLinTasks) {
    ReduceLinList folds{}, tasks{};
    int nf = 0, nt = 0;
    int64_t fblocks = 0, blocks = 0;
    for (size_t i = i0; i < std::min(reds.size(), i0 + kLinTasks); ++i) {
      const ReduceTask& t = reds[i];
      if (t.rows <= 0 || t.ncols <= 0 || t.nchunks <= 0) continue;
      const int64_t E = t.rows * t.ncols;
      ReduceLin r{t.part, t.dst, t.rows, t.ldr, t.L, t.kdim, E, t.alpha, t.nchunks, t.ncols, t.mode, 0, 0, 0};
      if (fold_pays(t.nchunks, E)) {
        ReduceLin f = r;
        const int groups = (t.nchunks + kFold - 1) / kFold;
        f.first_block = static_cast<int32_t>(fblocks);
        f.nblocks = static_cast<int32_t>((E + 255) / 256);
        fblocks += static_cast<int64_t>(f.nblocks) * groups;
        folds.t[nf++] = f;
        r.nchunks = groups;
        r.cstride = E * kFold;
      }
      r.first_block = static_cast<int32_t>(blocks);
      r.nblocks = grid_for(E);
      blocks += r.nblocks;
      tasks.t[nt++] = r;
    }
    if (nf) hipLaunchKernelGGL(fold_lin_kernel, dim3(static_cast<unsigned>(fblocks)), dim3(256), 0, st,
                               static_cast<int64_t>(nf), folds);
    if (nt) hipLaunchKernelGGL(reduce_lin_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st,
                               static_cast<int64_t>(nt), tasks);
  }
}

BatchedReduce plan_reduce_batched(const std::vector<ReduceTask>& in) {
  // the same two passes as launch_reduce, so batched and single results are bitwise equal
  BatchedReduce b;
  for (ReduceTask t : in) {
    if (t.rows <= 0 || t.ncols <= 0 || t.nchunks <= 0) continue;
    const int64_t E = t.rows * t.ncols;
    if (fold_pays(t.nchunks, E)) {
      ReduceTask f = t;
      f.groups = (t.nchunks + kFold - 1) / kFold;
      f.first_block = b.fblocks;
      b.fblocks += (E + 255) / 256 * f.groups;
      b.folds.push_back(f);
      t.nchunks = f.groups;
      t.cstride = E * kFold;
    }
    t.nblocks = grid_for(E);
    t.first_block = b.blocks;
    b.blocks += t.nblocks;
    b.tasks.push_back(t);
  }
  TTNN_REQUIRE(b.fblocks < (int64_t(1) << 31) && b.blocks < (int64_t(1) << 31), TTNN_E_INVALID,
               "batched launch too large");
  return b;
}

void launch_reduce_staged(const BatchedReduce& b, const ReduceTask* dfolds, const ReduceTask* dtasks,
                          hipStream_t st) {
  if (b.tasks.empty()) return;
  if (!b.folds.empty())
    hipLaunchKernelGGL(fold_batched_kernel, dim3(static_cast<unsigned>(b.fblocks)), dim3(256), 0, st, dfolds,
                       static_cast<int>(b.folds.size()));
  hipLaunchKernelGGL(reduce_batched_kernel, dim3(static_cast<unsigned>(b.blocks)), dim3(256), 0, st, dtasks,
                     static_cast<int>(b.tasks.size()));
}

void launch_reduce(double* part, int nchunks, int64_t rows, int ncols, int mode, double alpha,
                   const IndexMap& rmap, int64_t ldr, double* dst, int64_t L, int64_t kdim, hipStream_t st) {
  if (rows <= 0 || ncols <= 0) return;
  const int64_t E = rows * ncols;
  int64_t stride = E;
  if (fold_pays(nchunks, E)) {
    const int groups = (nchunks + kFold - 1) / kFold;
    hipLaunchKernelGGL(fold_chunks_kernel, dim3(static_cast<unsigned>((E + 255) / 256), groups), dim3(256), 0, st,
                       part, nchunks, E);
    nchunks = groups;
    stride = E * kFold;
  }
  hipLaunchKernelGGL(reduce_kernel, dim3(grid_for(E)), dim3(256), 0, st, part, nchunks, rows, ncols, mode, alpha,
                     rmap, ldr, dst, L, kdim, stride);
}

void launch_copy_f64(double* y, const double* x, int64_t n, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(copy_kernel, dim3(grid_for(n)), dim3(256), 0, st, y, x, n);
}
void launch_zero_int(int* p, int64_t n, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(zero_int_kernel, dim3(grid_for(n)), dim3(256), 0, st, p, n);
}
int list_blocks(const SegList& s) {
  int64_t b = 0;
  for (int i = 0; i < s.count; ++i) {
    int64_t nb = (s.n[i] + 255) / 256;
    b += nb > kSegBlocks ? kSegBlocks : (nb < 1 ? 1 : nb);
  }
  return static_cast<int>(b);
}
void launch_zero_list(const SegList& s, hipStream_t st) {
  if (s.count > 0) hipLaunchKernelGGL(zero_list_kernel, dim3(list_blocks(s)), dim3(256), 0, st, s);
}
void launch_finite_list(const SegList& s, int* flag, hipStream_t st) {
  if (s.count > 0) hipLaunchKernelGGL(finite_list_kernel, dim3(list_blocks(s)), dim3(256), 0, st, s, flag);
}

// ---------------------------------------------------------------- persistent ingest (host)
namespace {
int ingest_grid(const void* kernel, int64_t want, size_t lds) {
  static std::mutex mu;
  static std::map<std::tuple<int, const void*, size_t>, int> slots;   // resident workgroups by device, kernel and LDS
  int dev = 0;
  TTNN_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(mu);
  auto it = slots.find({dev, kernel, lds});
  if (it == slots.end()) {
    int coop = 0, cus = 0, per = 0;
    TTNN_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    TTNN_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    TTNN_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, 256, lds));
    it = slots.emplace(std::make_tuple(dev, kernel, lds), coop ? per * cus : 0).first;
  }
  if (it->second <= 0) return 0;
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(want, it->second)));
}
}  // namespace

bool launch_ingest(int cd, const std::vector<BatchedGemm>& gl, const std::vector<size_t>& level_end,
                   const std::vector<BatchedReduce>& rl, const std::vector<int*>& sticky, hipStream_t st) {
  if (sticky.size() > static_cast<size_t>(kIngestPlans)) return false;
  std::vector<IngestPhase> phases;
  // task tables follow the program, each 64-byte aligned
  const size_t head = (sizeof(IngestProgram) + 63) / 64 * 64;
  std::vector<std::pair<const void*, size_t>> tables;     // (host data, bytes)
  size_t off = head;
  auto add_table = [&](const void* data, size_t bytes) {
    const size_t at = off;
    tables.emplace_back(data, bytes);
    off = (off + bytes + 63) / 64 * 64;
    return static_cast<int64_t>(at);
  };
  int64_t most = 0;
  size_t g0 = 0, lds = 0;
  for (size_t lv = 0; lv < rl.size(); ++lv) {
    IngestPhase ph{};
    for (size_t k = g0; k < level_end[lv]; ++k) {
      const BatchedGemm& b = gl[k];
      if (b.tasks.empty()) continue;
      lds = std::max(lds, b.lds);
      if (ph.nseg == kIngestSegs) return false;
      int kind;
      if (b.th == cd && b.td == cd) kind = kSegRaw;
      else if (b.th == TTNN_F64 && b.td == TTNN_F64) kind = kSegF64;
      else return false;
      IngestSeg& g = ph.seg[ph.nseg++];
      g.kind = kind;
      g.ntasks = static_cast<int32_t>(b.tasks.size());
      g.blocks = b.blocks;
      g.tasks = add_table(b.tasks.data(), b.tasks.size() * sizeof(GemmTask));
    }
    g0 = level_end[lv];
    auto push = [&](IngestPhase& q) {
      if (q.nseg == 0) return;
      int64_t t = 0;
      for (int i = 0; i < q.nseg; ++i) t += q.seg[i].blocks;
      most = std::max(most, t);
      phases.push_back(q);
    };
    push(ph);
    const BatchedReduce& r = rl[lv];
    if (!r.folds.empty()) {
      IngestPhase f{};
      f.nseg = 1;
      f.seg[0] = IngestSeg{add_table(r.folds.data(), r.folds.size() * sizeof(ReduceTask)), r.fblocks, kSegFold,
                           static_cast<int32_t>(r.folds.size())};
      push(f);
    }
    if (!r.tasks.empty()) {
      IngestPhase q{};
      q.nseg = 1;
      q.seg[0] = IngestSeg{add_table(r.tasks.data(), r.tasks.size() * sizeof(ReduceTask)), r.blocks, kSegReduce,
                           static_cast<int32_t>(r.tasks.size())};
      push(q);
    }
  }
  if (phases.empty()) return true;
  if (phases.size() > static_cast<size_t>(kIngestPhases)) return false;
  const void* kernel = (cd == TTNN_BF16 ? tile_kernels_bf16() : cd == TTNN_F32 ? tile_kernels_f32() : tile_kernels_f64()).ingest;
  const int grid = ingest_grid(kernel, most, lds);
  if (grid <= 0) return false;
  std::vector<char> host(off, 0);
  IngestProgram* prog = reinterpret_cast<IngestProgram*>(host.data());
  prog->counter = 0;
  prog->nphases = static_cast<int32_t>(phases.size());
  prog->nsticky = static_cast<int32_t>(sticky.size());
  for (size_t i = 0; i < sticky.size(); ++i) prog->sticky[i] = sticky[i];
  for (size_t i = 0; i < phases.size(); ++i) prog->ph[i] = phases[i];
  size_t at = head;
  for (auto& t : tables) {
    std::memcpy(host.data() + at, t.first, t.second);
    at = (at + t.second + 63) / 64 * 64;
  }
  StagingLock lock;
  char* d = static_cast<char*>(stage_descriptors(host.data(), host.size(), st));
  void* args[] = {&d};
  const hipError_t e = hipLaunchCooperativeKernel(kernel, dim3(grid), dim3(256), args, lds, st);
  TTNN_HIP(e);
  fence_descriptors(st);
  return true;
}

}  // namespace ttnn
