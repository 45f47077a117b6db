// Batched strided FP64 GEMM on MFMA (v_mfma_f64_16x16x4f64) for the dense FP64
// work of the engine: the epilogue (Omega_t = Y_t^T R_t, Psi_t), the cores of the
// recovery phase, the reconstruction, and contractions of FP64 intermediates.
//
// A job computes, for every output batch cb < nbC,
//   C[cb](m, n) = (accumulate ? C[cb](m, n) : 0)
//                 + alpha * sum_{kb < nbK} sum_{k < K} A(m, k; cb, kb) B(k, n; cb, kb)
// with A(m, k; cb, kb) = A[m sAm + k sAk + cb sAc + kb sAkb] (B, C likewise).
// Long contractions are split over several workgroups whose partial tiles a second
// launch adds in split order, so results do not depend on scheduling.  (A last-block
// combine would need a device-scope fence, which on this chip writes back and
// invalidates the whole L2 of the XCD for every workgroup.)  Several jobs share one
// launch.
#include <type_traits>

#include "kernels.hpp"
#include "mfma.hpp"

namespace ttnn {
namespace {

// A K-step of 64 keeps 16 loads a thread in flight: these products are short, so
// their time is the number of dependent memory round trips, not arithmetic.
constexpr int TM = 32, TN = 32, TK = 64;
constexpr int LPT = TM * TK / 256;          // elements of each operand tile per thread (8)

__global__ __launch_bounds__(256) void bgemm64_kernel(GJobList L) {
  __shared__ double As[TK][TM + 1];
  __shared__ double Bs[TK][TN + 1];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int64_t b = blockIdx.x;
  int ji = 0;
  while (ji + 1 < L.n && L.jobs[ji + 1].first_block <= b) ++ji;
  const GJob& J = L.jobs[ji];
  int64_t rel = b - J.first_block;
  const int split = static_cast<int>(rel % J.splits);
  rel /= J.splits;
  const int64_t tn = rel % J.tiles_n;
  rel /= J.tiles_n;
  const int64_t tm = rel % J.tiles_m;
  const int64_t cb = rel / J.tiles_m;
  const int64_t m0 = tm * TM, n0 = tn * TN;

  // contraction range of this split over the flattened (kb, k) space
  const int64_t KK = static_cast<int64_t>(J.nbK) * J.K;
  const int64_t k_begin = (KK * split) / J.splits;
  const int64_t k_end = (KK * (split + 1)) / J.splits;

  const int wm = wave >> 1, wn = wave & 1;    // 16 x 16 block of the wave
  f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
  const double* Ab = J.A + cb * J.sAc;
  const double* Bb = J.B + cb * J.sBc;
  // thread -> (row, k) map of the tile loads: contiguous index fastest
  const bool a_k_fast = J.sAk == 1 && J.sAm != 1;
  const bool b_k_fast = J.sBk == 1 && J.sBn != 1;

  // A thread's entries of a step sit at one pointer plus multiples of one stride (forming
  // the index products for every entry cost some 250 vector instructions a step: a TTN
  // rounding of order 6, n = 500, r = 32 took 306 us, now 298; a 16^4 FP64 step 93, now
  // 90).  Entries past M, N or the split are zeros.
  const int am = a_k_fast ? tid / TK : tid % TM, ak = a_k_fast ? tid % TK : tid / TM;
  const int bn = b_k_fast ? tid / TK : tid % TN, bk = b_k_fast ? tid % TK : tid / TN;
  constexpr int MU = 256 / TK, KU = 256 / TM;   // rows, or contraction values, apart of its entries
  static_assert(TM == TN, "one map for both operands");
  const int64_t ast = a_k_fast ? MU * J.sAm : KU * J.sAk, bst = b_k_fast ? MU * J.sBn : KU * J.sBk;
  unsigned aok = 0, bok = 0;                     // entries inside M, N
#pragma unroll
  for (int u = 0; u < LPT; ++u) {
    aok |= (m0 + am + (a_k_fast ? MU * u : 0) < J.M ? 1u : 0u) << u;
    bok |= (n0 + bn + (b_k_fast ? MU * u : 0) < J.N ? 1u : 0u) << u;
  }
  double ra[LPT], rb[LPT];
  unsigned la = 0, lb = 0;                       // entries of the staged step that exist
  int64_t kk = k_begin;
  int64_t kcur = 0;   // length of the staged step
  auto fetch = [&](int64_t kpos, int64_t& klen) {
    const int64_t kb = J.nbK == 1 ? 0 : kpos / J.K;
    const int64_t k0 = kpos - kb * J.K;
    int64_t kstop = J.K - k0;                  // stay inside one kb
    if (kstop > k_end - kpos) kstop = k_end - kpos;
    if (kstop > TK) kstop = TK;
    klen = kstop;
    const double* pa = Ab + kb * J.sAkb + (m0 + am) * J.sAm + (k0 + ak) * J.sAk;
    const double* pb = Bb + kb * J.sBkb + (n0 + bn) * J.sBn + (k0 + bk) * J.sBk;
    la = aok;
    lb = bok;
    const int ks = static_cast<int>(kstop);
    if (a_k_fast) la = ak < ks ? la : 0u;
    if (b_k_fast) lb = bk < ks ? lb : 0u;
    if (ks < TK) {                             // (a full step has every value)
#pragma unroll
      for (int u = 0; u < LPT; ++u) {
        if (!a_k_fast && ak + KU * u >= ks) la &= ~(1u << u);
        if (!b_k_fast && bk + KU * u >= ks) lb &= ~(1u << u);
      }
    }
    const bool whole = la == (1u << LPT) - 1 && lb == (1u << LPT) - 1;
    if (__all(whole)) {
#pragma unroll
      for (int u = 0; u < LPT; ++u) {
        ra[u] = pa[u * ast];
        rb[u] = pb[u * bst];
      }
    } else {
#pragma unroll
      for (int u = 0; u < LPT; ++u) {
        ra[u] = (la >> u) & 1u ? pa[u * ast] : 0.0;
        rb[u] = (lb >> u) & 1u ? pb[u * bst] : 0.0;
      }
    }
  };
  if (kk < k_end) fetch(kk, kcur);
  while (kk < k_end) {
#pragma unroll
    for (int u = 0; u < LPT; ++u) {
      As[ak + (a_k_fast ? 0 : KU * u)][am + (a_k_fast ? MU * u : 0)] = ra[u];
      Bs[bk + (b_k_fast ? 0 : KU * u)][bn + (b_k_fast ? MU * u : 0)] = rb[u];
    }
    __syncthreads();
    const int64_t knext = kk + kcur;
    int64_t klen_next = 0;
    if (knext < k_end) fetch(knext, klen_next);   // next step's loads overlap the MFMAs
    // rows past the staged length are zero; skip whole groups of 4 beyond it
    const int nmf = static_cast<int>((kcur + 3) / 4);
    if (nmf == TK / 4) {
#pragma unroll
      for (int s = 0; s < TK / 4; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(As[4 * s + lg][16 * wm + l16], Bs[4 * s + lg][16 * wn + l16], acc, 0,
                                                   0, 0);
    } else {
      for (int s = 0; s < nmf; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(As[4 * s + lg][16 * wm + l16], Bs[4 * s + lg][16 * wn + l16], acc, 0,
                                                   0, 0);
    }
    __syncthreads();
    kk = knext;
    kcur = klen_next;
  }

  // C fragment: lane holds C[16 wm + 4 v + lg][16 wn + l16]
  if (J.splits == 1) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t m = m0 + 16 * wm + 4 * v + lg, n = n0 + 16 * wn + l16;
      if (m < J.M && n < J.N) {
        double* c = J.C + cb * J.sCc + m * J.sCm + n * J.sCn;
        *c = (J.accumulate ? *c : 0.0) + J.alpha * acc[v];
      }
    }
    return;
  }
  // split contraction: store the partial tile; bgemm64_combine_kernel adds them
  const int64_t tile_id = (cb * J.tiles_m + tm) * J.tiles_n + tn;
  double* part = J.part + (tile_id * J.splits + split) * (TM * TN);
#pragma unroll
  for (int v = 0; v < 4; ++v) part[(16 * wm + 4 * v + lg) * TN + 16 * wn + l16] = acc[v];
}

// Four workgroups per tile of a split job, one element a thread: C = (accumulate ? C :
// 0) + alpha * sum of the partial tiles in split order (32 interleaved sums, combined
// pairwise in a fixed tree), so results do not depend on scheduling and a thread keeps
// 32 loads in flight.  A launch of its own: the kernel boundary makes the partials
// visible without a device-wide fence.
constexpr int kCombineParts = 4;          // workgroups per 32 x 32 tile
static_assert(kCombineParts * 256 == TM * TN, "one tile element per thread");
__global__ __launch_bounds__(256) void bgemm64_combine_kernel(GJobList L) {
  const int tid = threadIdx.x;
  const int64_t b = blockIdx.x / kCombineParts;
  const int part_of = static_cast<int>(blockIdx.x % kCombineParts);
  int ji = 0;
  while (ji + 1 < L.n && L.jobs[ji + 1].first_tile <= b) ++ji;
  const GJob& J = L.jobs[ji];
  const int64_t tile_id = b - J.first_tile;
  int64_t rel = tile_id;
  const int64_t tn = rel % J.tiles_n;
  rel /= J.tiles_n;
  const int64_t tm = rel % J.tiles_m;
  const int64_t cb = rel / J.tiles_m;
  const int64_t m0 = tm * TM, n0 = tn * TN;
  const double* parts = J.part + tile_id * J.splits * (TM * TN);
  const int e = part_of * 256 + tid;        // element of the tile
  constexpr int NS = 32;
  double s[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) s[q] = 0.0;
  // split sp + q goes to sum q; splits past the end add nothing (static indices only)
  for (int sp = 0; sp < J.splits; sp += NS) {
    double v[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) v[q] = sp + q < J.splits ? parts[(sp + q) * (TM * TN) + e] : 0.0;
#pragma unroll
    for (int q = 0; q < NS; ++q) s[q] += v[q];
  }
#pragma unroll
  for (int w = NS / 2; w > 0; w /= 2)
#pragma unroll
    for (int q = 0; q < w; ++q) s[q] += s[q + w];
  const int mm = e / TN, nn = e % TN;
  const int64_t m = m0 + mm, n = n0 + nn;
  if (m >= J.M || n >= J.N) return;
  double* c = J.C + cb * J.sCc + m * J.sCm + n * J.sCn;
  *c = (J.accumulate ? *c : 0.0) + J.alpha * s[0];
}

// out[l + M j] = sum_i A[l + M i] B[j + N i], i < K: the reconstruction's last step, a dense
// tensor from its halves (M and N in the ten thousands, K a rank).  Bound by the FP64 MFMA
// (2 M N K) and the M N results written.  A wave owns 64 x 32 results (eight accumulators);
// six 8-byte loads a lane feed eight MFMAs of 64 cycles, so the operands, a few megabytes
// in the second-level cache, go straight to registers, one step of four values ahead.
// Vector instructions beside an FP64 MFMA cost their issue time whole, so there are few:
// edge tiles are moved back inside (their results are formed twice, the same) instead of
// masked, the pointers advance by one addition, and B is the MFMA's row operand, results
// going through LDS so that a store writes 64 of them along l (not kept in the cache, which
// the operands need).  128^4 FP32 from rank-32 halves: the generic tile took 960 us, this
// with masked edges and 64-byte stores 420, now 315 (MFMA busy 78%; 17.2 GFLOP take 239 us
// at the rate of a large FP64 product).
// SMALL (M < 64 or N < 32): rows past the end read the last one and are not written.
//
// A workgroup's waves are wl along l by 4 / wl along j, XCDs xl along l by 8 / xl along j
// (OuterSplit): with the one fixed split, 2 x 2 waves and all XCDs along l, M <= 128 left
// seven of the eight XCDs idle.
struct OuterSplit {
  int wl, xl;
  uint32_t lx, jx;               // tiles of an XCD along l and j
};
template <typename TO, bool SMALL>
__global__ __launch_bounds__(256, 4) void outer64_kernel(const double* __restrict__ A, const double* __restrict__ B,
                                                         int64_t M, int64_t N, int K, OuterSplit sp,
                                                         TO* __restrict__ out) {
  // results of 16 rows of B by 64 of A; the pitch puts the lane groups' rows 16 banks apart
  __shared__ TO tile[4][16][80];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // workgroups go to the XCDs in turn: XCD x takes part x % xl of the l tiles (its part of A
  // stays in its cache) and part x / xl of the j tiles, and walks them l first
  const int x = blockIdx.x % 8;
  const uint32_t rel = blockIdx.x / 8;
  const int64_t lt = static_cast<int64_t>(x % sp.xl) * sp.lx + rel % sp.lx;
  const int64_t jt = static_cast<int64_t>(x / sp.xl) * sp.jx + rel / sp.lx;
  int64_t l0 = (lt * sp.wl + wave % sp.wl) * 64;
  int64_t j0 = (jt * (4 / sp.wl) + wave / sp.wl) * 32;
  if (l0 >= M || j0 >= N) return;                 // no barrier follows
  if (!SMALL) {
    if (l0 > M - 64) l0 = M - 64;
    if (j0 > N - 32) j0 = N - 32;
  }
  int al[4], bl[2];                               // offsets of the lane's rows
#pragma unroll
  for (int q = 0; q < 4; ++q) al[q] = !SMALL || l0 + 16 * q + l16 < M ? 16 * q : static_cast<int>(M - 1 - l0) - l16;
#pragma unroll
  for (int q = 0; q < 2; ++q) bl[q] = !SMALL || j0 + 16 * q + l16 < N ? 16 * q : static_cast<int>(N - 1 - j0) - l16;
  const double* pa = A + l0 + l16 + M * lg;
  const double* pb = B + j0 + l16 + N * lg;
  auto fetch = [&](double* a, double* b) {
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = pa[al[q]];
#pragma unroll
    for (int q = 0; q < 2; ++q) b[q] = pb[bl[q]];
    pa += 4 * M;
    pb += 4 * N;
  };
  f64x4_t acc[2][4];                              // [j block][l block]
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) acc[x][y] = f64x4_t{};
  auto multiply = [&](const double* ca, const double* cb) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(cb[x], ca[y], acc[x][y], 0, 0, 0);
  };
  double a0[4], b0[2], a1[4], b1[2];              // two steps in turn (no copies between them)
  const int whole = K / 4;
  if (whole > 0) fetch(a0, b0);
  for (int k = 0; k < whole; k += 2) {
    if (k + 1 < whole) fetch(a1, b1);
    multiply(a0, b0);
    if (k + 1 >= whole) break;
    if (k + 2 < whole) fetch(a0, b0);
    multiply(a1, b1);
  }
  if (K % 4) {                                    // the last, partial step
    const bool live = 4 * whole + lg < K;
#pragma unroll
    for (int q = 0; q < 4; ++q) a0[q] = live ? pa[al[q]] : 0.0;
#pragma unroll
    for (int q = 0; q < 2; ++q) b0[q] = live ? pb[bl[q]] : 0.0;
    multiply(a0, b0);
  }
  TO* row = out + M * j0 + l0;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int y = 0; y < 4; ++y) tile[wave][4 * v + lg][16 * y + l16] = static_cast<TO>(acc[x][y][v]);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");   // a wave's LDS accesses are in order
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (!SMALL || (j0 + 16 * x + r < N && l0 + lane < M)) __builtin_nontemporal_store(tile[wave][r][lane], row + lane);
      row += M;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }
}

}  // namespace

void launch_bgemm64(std::vector<GJob>& jobs, double* part, size_t part_elems, hipStream_t st) {
  for (size_t j0 = 0; j0 < jobs.size(); j0 += kMaxGJobs) {
    GJobList L{};
    GJobList LC{};                              // split jobs, for the combine launch
    L.n = static_cast<int>(std::min<size_t>(kMaxGJobs, jobs.size() - j0));
    int64_t blocks = 0, ctiles = 0;
    size_t part_used = 0;
    for (int i = 0; i < L.n; ++i) {
      GJob j = jobs[j0 + i];
      j.tiles_m = (j.M + TM - 1) / TM;
      j.tiles_n = (j.N + TN - 1) / TN;
      const int64_t tiles = j.tiles_m * j.tiles_n * j.nbC;
      // split long contractions so that the launch has enough workgroups
      const int64_t KK = static_cast<int64_t>(j.nbK) * j.K;
      int64_t sp = 1;
      if (tiles < 512 && KK > 256) {
        sp = std::min<int64_t>((KK + 255) / 256, std::max<int64_t>(1, 1024 / tiles));
        sp = std::min<int64_t>(sp, 256);
      }
      const size_t need = static_cast<size_t>(tiles * sp * TM * TN);
      if (sp > 1 && part_used + need > part_elems) sp = 1;
      j.splits = static_cast<int>(sp);
      if (sp > 1) {
        j.part = part + part_used;
        part_used += need;
        j.first_tile = ctiles;
        ctiles += tiles;
      }
      j.first_block = blocks;
      blocks += tiles * sp;
      L.jobs[i] = j;
      if (sp > 1) LC.jobs[LC.n++] = j;
    }
    if (blocks > 0)
      hipLaunchKernelGGL(bgemm64_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, L);
    if (ctiles > 0)
      hipLaunchKernelGGL(bgemm64_combine_kernel, dim3(static_cast<unsigned>(ctiles * kCombineParts)), dim3(256), 0,
                         st, LC);
  }
}

void launch_outer64(const double* A, const double* B, int64_t M, int64_t N, int K, void* out, bool f32,
                    hipStream_t st) {
  if (M <= 0 || N <= 0) return;
  // Waves: 2 x 2 of 64 x 32 results, or all four along the other side where one side is no
  // more than a wave's.  XCDs: all along l while that leaves none with more than an eighth
  // over the evenest split's share of tiles (M = 16,384: 16 l tiles each), else fewer.
  // FP32 results, the whole reconstruction, with 2 x 2 waves and all XCDs along l and now: M =
  // 97, N = 2^20 (K = 32) 1386 -> 414 us, 128, 2^20 1352 -> 398, 500, 2^18 352 -> 290, 33,
  // 810,000 (K = 16) 500 -> 136, 8, 9e6 (K = 8) 3817 -> 761; 16,384 x 16,384 350 both.
  OuterSplit sp{};
  sp.wl = M <= 64 ? 1 : N <= 32 ? 4 : 2;
  const int64_t lts = (M + 64 * sp.wl - 1) / (64 * sp.wl), jts = (N + 128 / sp.wl - 1) / (128 / sp.wl);
  auto share = [&](int xl) { return (lts + xl - 1) / xl * ((jts * xl + 7) / 8); };
  int64_t least = share(8);
  for (int xl = 4; xl > 0; xl /= 2) least = std::min(least, share(xl));
  for (sp.xl = 8; 8 * share(sp.xl) > 9 * least; sp.xl /= 2) {}
  const int64_t lx = (lts + sp.xl - 1) / sp.xl, jx = (jts * sp.xl + 7) / 8, tiles = 8 * lx * jx;
  TTNN_REQUIRE(tiles < (int64_t(1) << 31), TTNN_E_INVALID, "reconstruction too large for one launch");
  sp.lx = static_cast<uint32_t>(lx);
  sp.jx = static_cast<uint32_t>(jx);
  const dim3 grid(static_cast<unsigned>(tiles));
  auto go = [&](auto o, auto small) {
    using TO = decltype(o);
    hipLaunchKernelGGL((outer64_kernel<TO, decltype(small)::value>), grid, dim3(256), 0, st, A, B, M, N, K, sp,
                       static_cast<TO*>(out));
  };
  const bool small = M < 64 || N < 32;
  if (f32) small ? go(float{}, std::true_type{}) : go(float{}, std::false_type{});
  else small ? go(double{}, std::true_type{}) : go(double{}, std::false_type{});
}

}  // namespace ttnn
