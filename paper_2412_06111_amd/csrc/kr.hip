// Tree contractions of a TTN-format tensor with Khatri-Rao maps (Sec. 7).
//
// Every contraction of the structured sketch that shares one column index j over all
// of its operands has the form
//   out[o, j] = sum over every core index except axis `oax` of
//               core[idx] * prod_{q != oax} F_q[idx_q, j]
// (core column-major, first axis fastest; F_q row-major size_q x cols, j fastest; out
// row-major size_o x cols).  With F_q the per-mode factors or the children's vectors it
// gives the down vectors of a node; with the siblings' and the parent's vectors, the up
// vectors of a child.  Split the reduction index into the first non-output axis a
// (size n0) and the rest e (the outer combinations):
//   out[o, j] = sum_e w_e[j] sum_a C_e[o, a] F_0[a, j],  w_e[j] = prod_{q>=1} F_q[e_q, j].
//
// The order of the sums is part of what the kernel promises: the cores of a rounding are
// R Omega^+ with an Omega that the ranks' decay leaves ill conditioned, and summing in
// another order moves them by up to 2e-9 (a two-child root, ranks decaying as 1 / i^2, r =
// 28).  A unit is one outer combination e and one chunk of at most 32 values of a (the chunks
// of equal length); its t = sum_a C F_0 is a chain of fused multiply-adds in the order of a,
// and out the chain out = fma(w_e, t, out) in the order of the units.  The units are cut into
// G contiguous slices, one workgroup each, whose results a second kernel adds in order.
//
// The chains over a run on the FP64 MFMA, which adds its four products one after the other by
// fused multiply-adds in the order of the contraction index, operands straight from global
// memory (a core is read once, the factors stay in the caches): a wave takes one unit of 32
// values of o (two row blocks) by up to 64 columns, the eight waves of a workgroup
// neighbouring units (a slice of 70^3 cores has seven), and after each round its threads, a
// share of the results each, add the t in order.
//
// Bound by latency: the six 70^3 cores of a 500^6 tensor's tree are 1 to 4 us of MFMA work a
// level.  A level's launch takes 7 to 25 us, 14 on average; with FP64 VALU products of LDS
// tiles, seven serial units of a load, a barrier and 24 steps, it took 24-30 (the rounding
// 303 us, now 242).
#include "kr.hpp"

#include <algorithm>

#include "mfma.hpp"

namespace ttnn {

namespace {

constexpr int kTO = 32, kTJ = 64, kKC = 32;   // values of o, columns (at most), of a (at most) of a unit
constexpr int kAhead = 4;                     // steps of four values of a loaded together
constexpr int kUnits = 8;                     // units of a round: waves of a workgroup

// Chunks of the inner axis: as few as hold n0 in chunks of at most kKC, of equal length.
__host__ __device__ inline int64_t kr_nchunks(int64_t n0) { return (n0 + kKC - 1) / kKC; }
__host__ __device__ inline int kr_chunk(int64_t n0) {
  const int64_t nch = kr_nchunks(n0);
  return static_cast<int>((n0 + nch - 1) / nch);
}

template <int NCB>
__global__ __launch_bounds__(64 * kUnits) void kr_contract_kernel(KJobList) {
  using P = Pol<TTNN_F64>;
  // the job's fields by scalar loads (indexing a by-value argument would copy it to scratch)
  typedef const KJobList __attribute__((address_space(4))) ConstList;
  ConstList& L = *(ConstList*)__builtin_amdgcn_kernarg_segment_ptr();
  const int64_t b = blockIdx.x;
  int jid = 0;
  while (jid + 1 < L.n && b >= L.jobs[jid + 1].first_block) ++jid;
  const auto& J = L.jobs[jid];
  int64_t local = b - J.first_block;
  const int j0 = static_cast<int>(local % J.colchunks) * 16 * NCB;
  local /= J.colchunks;
  const int64_t o0 = (local % J.otiles) * kTO;
  const int64_t g = local / J.otiles;
  const int oax = J.oax, naxes = J.naxes, cols = J.cols;
  const int64_t so = J.size[oax];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int in = oax == 0 ? 1 : 0;          // the inner axis; none when there is only the output axis
  const bool one = in >= naxes;
  const int64_t n0 = one ? 1 : J.size[in];
  const double* F0 = one ? nullptr : J.fac[in];
  int64_t so_stride = 1;
  for (int q = 0; q < oax; ++q) so_stride *= J.size[q];
  const int64_t st0 = in == 0 ? 1 : so;
  const int64_t nch = kr_nchunks(n0);
  const int kc = kr_chunk(n0);
  const int64_t units = J.kred / n0 * nch;
  const int64_t ulo = units * g / J.G, uhi = units * (g + 1) / J.G;

  // Rows past the end read the last row and columns past the end the last column: what they
  // form is not delivered.
  const double* row[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t o = o0 + 16 * i + l16;
    row[i] = J.core + (o < so ? o : so - 1) * so_stride;
  }
  int jc[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) jc[cb] = j0 + 16 * cb + l16 < cols ? j0 + 16 * cb + l16 : cols - 1;

  // The unit being loaded: its values of a, core offset and column weights
  int run = 0;
  int64_t a0 = 0, off = 0;
  double w[NCB];
  auto open = [&](int64_t u) {
    run = 0;
    if (u >= uhi) return;
    const int64_t e = u / nch;
    a0 = (u - e * nch) * kc;
    run = static_cast<int>(n0 - a0 < kc ? n0 - a0 : kc);
    off = 0;
    int64_t rest = e, stride = 1;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) w[cb] = 1.0;
    for (int q = 0; q < naxes; ++q) {
      const int64_t sz = J.size[q];
      if (q != oax && q != in) {
        const int64_t up = rest / sz, d = rest - up * sz;
        rest = up;
        off += d * stride;
        const double* F = J.fac[q] + d * cols;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) w[cb] *= F[jc[cb]];
      }
      stride *= sz;
    }
  };
  // Half of a unit: kAhead steps of four values of a from 4 kAhead H on
  struct Half {
    double a[2][kAhead], f[NCB][kAhead];
  };
  static_assert(kKC == 8 * kAhead, "two halves a unit");
  auto fetch = [&](Half& k, int h) {
    if (4 * kAhead * h >= run) return;
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {
      // past the unit's values: its first one, zeroed before its product
      const int v = 4 * (kAhead * h + s) + lg;
      const int64_t a = a0 + (v < run ? v : 0);
#pragma unroll
      for (int i = 0; i < 2; ++i) k.a[i][s] = row[i][off + a * st0];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) k.f[cb][s] = F0 ? F0[a * cols + jc[cb]] : 1.0;
    }
  };
  f64x4_t t[2][NCB];
  auto products = [&](const Half& k, int h, int n) {
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {
      const int at = 4 * (kAhead * h + s);
      if (at >= n) break;
      const bool live = at + lg < n;
      double x[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = live ? k.a[i][s] : 0.0;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        if (j0 + 16 * cb >= cols) continue;
        const double y = live ? k.f[cb][s] : 0.0;
#pragma unroll
        for (int i = 0; i < 2; ++i) t[i][cb] = P::mfma(x[i], y, t[i][cb]);
      }
    }
  };

  // [wave][result register][lane] and [wave][column]: the units of a round and their weights.
  // A thread adds up register `wave` of the eight of its lane's row blocks.
  __shared__ double red[kUnits][8 * NCB][64];
  __shared__ double wl[kUnits][16 * NCB];
  static_assert(kUnits == 8, "a register of each column block a wave");
  double acc[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) acc[cb] = 0.0;
  Half k0, k1;
  open(ulo + wave);
  fetch(k0, 0);
  fetch(k1, 1);
  for (int64_t u0 = ulo; u0 < uhi; u0 += kUnits) {
    const int n = run;                       // of this round's unit; 0: none
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) t[i][cb] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    if (lg == 0) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) wl[wave][16 * cb + l16] = w[cb];
    }
    open(u0 + kUnits + wave);                // the next round's loads go out behind the products
    products(k0, 0, n);
    fetch(k0, 0);
    products(k1, 1, n);
    fetch(k1, 1);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][(2 * cb + i) * 4 + v][lane] = t[i][cb][v];
    __syncthreads();
    const int nu = static_cast<int>(uhi - u0 < kUnits ? uhi - u0 : kUnits);
    for (int u = 0; u < nu; ++u)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        acc[cb] = fma(wl[u][16 * cb + l16], red[u][8 * cb + wave][lane], acc[cb]);
    __syncthreads();
  }
  const int64_t o = o0 + 16 * (wave / 4) + P::crow(lane, wave % 4);
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const int64_t j = j0 + 16 * cb + l16;
    if (o < so && j < cols) {
      if (J.G == 1) J.out[o * cols + j] = acc[cb];
      else J.part[(g * so + o) * cols + j] = acc[cb];
    }
  }
}

// out[e] = sum_{g < G} part[g * size + e] in order, for the jobs split over G > 1.
__global__ __launch_bounds__(256) void kr_fold_kernel(KJobList L) {
  const int64_t b = blockIdx.x;
  int jid = -1;
  for (int i = 0; i < L.n; ++i)
    if (L.jobs[i].G > 1 && b >= L.jobs[i].fold_first) jid = i;
  if (jid < 0) return;
  const KJob& J = L.jobs[jid];
  const int64_t size = J.size[J.oax] * static_cast<int64_t>(J.cols);
  const int64_t e = (b - J.fold_first) * 256 + threadIdx.x;
  if (e >= size) return;
  // loads issued eight at a time, added in the fixed order g = 0, 1, ..
  double v = 0.0;
  int g = 0;
  for (; g + 8 <= J.G; g += 8) {
    double x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = J.part[(g + i) * size + e];
#pragma unroll
    for (int i = 0; i < 8; ++i) v += x[i];
  }
  for (; g < J.G; ++g) v += J.part[g * size + e];
  J.out[e] = v;
}

}  // namespace

int kr_split(int64_t so, int cols, int64_t n0, int64_t nouter) {
  const int64_t tiles = ((so + kTO - 1) / kTO) * ((cols + kTJ - 1) / kTJ);
  const int64_t units = nouter * kr_nchunks(n0);
  int64_t G = tiles >= 512 ? 1 : 512 / tiles;
  if (G > units / 2) G = units / 2;                    // at least two units per slice
  if (G > 32) G = 32;                                  // the fold reads G partials per output
  return G < 1 ? 1 : static_cast<int>(G);
}

size_t kr_part_elems(const KJob& j) {
  return j.G > 1 ? static_cast<size_t>(j.G) * j.size[j.oax] * j.cols : 0;
}

void launch_kr_contract(std::vector<KJob> jobs, hipStream_t stream) {
  for (size_t at = 0; at < jobs.size(); at += kMaxKJobs) {
    KJobList L{};
    int64_t blocks = 0, fblocks = 0;
    int width = 1;                                     // 16-column blocks of a workgroup
    for (size_t i = at; i < jobs.size() && i < at + kMaxKJobs; ++i)
      width = std::max(width, std::min((jobs[i].cols + 15) / 16, kTJ / 16));
    for (size_t i = at; i < jobs.size() && L.n < kMaxKJobs; ++i) {
      KJob j = jobs[i];
      TTNN_REQUIRE(j.naxes >= 1 && j.naxes <= kMaxAxes && j.oax >= 0 && j.oax < j.naxes && j.cols >= 1,
                   TTNN_E_INVALID, "bad tree contraction");
      TTNN_REQUIRE(j.G == 1 || j.part != nullptr, TTNN_E_INVALID, "split tree contraction without scratch");
      j.colchunks = (j.cols + 16 * width - 1) / (16 * width);
      j.otiles = (j.size[j.oax] + kTO - 1) / kTO;
      j.kred = 1;
      for (int q = 0; q < j.naxes; ++q)
        if (q != j.oax) j.kred *= j.size[q];
      j.first_block = blocks;
      blocks += j.otiles * j.colchunks * j.G;
      if (j.G > 1) {
        j.fold_first = fblocks;
        fblocks += (j.size[j.oax] * j.cols + 255) / 256;
      }
      L.jobs[L.n++] = j;
    }
    const dim3 grid(static_cast<unsigned>(blocks));
    if (blocks > 0) {
      if (width == 1) kr_contract_kernel<1><<<grid, dim3(64 * kUnits), 0, stream>>>(L);
      else if (width == 2) kr_contract_kernel<2><<<grid, dim3(64 * kUnits), 0, stream>>>(L);
      else if (width == 3) kr_contract_kernel<3><<<grid, dim3(64 * kUnits), 0, stream>>>(L);
      else kr_contract_kernel<4><<<grid, dim3(64 * kUnits), 0, stream>>>(L);
    }
    if (fblocks > 0) kr_fold_kernel<<<dim3(static_cast<unsigned>(fblocks)), dim3(256), 0, stream>>>(L);
  }
}

}  // namespace ttnn
