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
//   out[o, j] = sum_e w_e[j] sum_a C_e[o, a] F_0[a, j],  w_e[j] = prod_{q>=1} F_q[e_q, j],
// one contraction over (a, e) whose right operand F_0[a, j] w_e[j] is formed in registers.
// It runs on the FP64 MFMA, operands straight from global memory (a core is read once, the
// factors stay in the caches): a wave takes 32 values of o (two row blocks) by up to 64
// columns and a contiguous slice of the steps, four values of a of one combination each,
// loading four steps ahead.  The four waves of a workgroup take neighbouring slices and add
// their sums in wave order through LDS; the steps are cut into 4 G slices, and for G > 1 a
// second kernel adds the G partials in a fixed order, so the result depends only on the
// shapes.
//
// Bound by latency: the six 70^3 cores of a 500^6 tensor's tree are 1 to 4 us of MFMA work a
// level.  A level took 24-30 us on FP64 VALU products of LDS tiles (seven serial units of a
// load, a barrier and 24 steps); now 10-17.
#include "kr.hpp"

#include <algorithm>

#include "mfma.hpp"

namespace ttnn {

namespace {

constexpr int kTO = 32, kTJ = 64;          // values of o and columns (at most) of a workgroup
constexpr int kAhead = 4;                  // steps of loads in flight

template <int NCB>
__global__ __launch_bounds__(256) void kr_contract_kernel(KJobList) {
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
  const int64_t nst = (n0 + 3) / 4, steps = J.kred / n0 * nst;
  const int64_t slice = 4 * g + wave;
  const int64_t hi = steps * (slice + 1) / (4 * J.G);
  int64_t at = steps * slice / (4 * J.G);    // the next step to load: values 4 t.. of combination e
  int64_t e = at / nst, t = at - e * nst;

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

  // Up to kAhead steps of one combination: operands and, per column, the other axes' product
  struct Block {
    double a[2][kAhead], f[NCB][kAhead], w[NCB];
    int n;                                   // steps in it
    int64_t last;                            // values of a from its first on
  };
  auto fetch = [&](Block& k) {
    k.n = 0;
    if (at >= hi) return;
    int64_t n = nst - t < hi - at ? nst - t : hi - at;
    k.n = static_cast<int>(n < kAhead ? n : kAhead);
    k.last = n0 - 4 * t;
    int64_t off = 0, rest = e, stride = 1;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) k.w[cb] = 1.0;
    for (int q = 0; q < naxes; ++q) {
      const int64_t sz = J.size[q];
      if (q != oax && q != in) {
        const int64_t up = rest / sz, d = rest - up * sz;
        rest = up;
        off += d * stride;
        const double* F = J.fac[q] + d * cols;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) k.w[cb] *= F[jc[cb]];
      }
      stride *= sz;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      // past the block or past n0: the first value, zeroed before its product
      const int64_t v = 4 * (t + u) + lg, a = u < k.n && v < n0 ? v : 0;
#pragma unroll
      for (int i = 0; i < 2; ++i) k.a[i][u] = row[i][off + a * st0];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) k.f[cb][u] = F0 ? F0[a * cols + jc[cb]] : 1.0;
    }
    at += k.n;
    t += k.n;
    if (t == nst) {
      t = 0;
      ++e;
    }
  };
  f64x4_t acc[2][NCB];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[i][cb] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  auto products = [&](const Block& k) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (u >= k.n) break;
      const bool live = 4 * u + lg < k.last;
      double x[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) x[i] = live ? k.a[i][u] : 0.0;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        if (j0 + 16 * cb >= cols) continue;
        const double y = live ? k.f[cb][u] * k.w[cb] : 0.0;
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][cb] = P::mfma(x[i], y, acc[i][cb]);
      }
    }
  };
  Block k0, k1;
  fetch(k0);
  while (k0.n) {
    fetch(k1);
    products(k0);
    if (!k1.n) break;
    fetch(k0);
    products(k1);
  }

  // the four waves' sums, added in wave order
  __shared__ double red[4][8][64];
  for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][4 * i + v][lane] = acc[i][cb][v];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int x = wave + 4 * h;            // row block x / 4, result x % 4 of this lane
      const double sum = red[0][x][lane] + red[1][x][lane] + red[2][x][lane] + red[3][x][lane];
      const int64_t o = o0 + 16 * (x / 4) + P::crow(lane, x % 4);
      const int64_t j = j0 + 16 * cb + l16;
      if (o < so && j < cols) {
        if (J.G == 1) J.out[o * cols + j] = sum;
        else J.part[(g * so + o) * cols + j] = sum;
      }
    }
    __syncthreads();
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
  const int64_t steps = nouter * ((n0 + 3) / 4);
  int64_t G = tiles >= 512 ? 1 : 512 / tiles;
  if (G > steps / 32) G = steps / 32;                  // at least eight steps a wave
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
      if (width == 1) kr_contract_kernel<1><<<grid, dim3(256), 0, stream>>>(L);
      else if (width == 2) kr_contract_kernel<2><<<grid, dim3(256), 0, stream>>>(L);
      else if (width == 3) kr_contract_kernel<3><<<grid, dim3(256), 0, stream>>>(L);
      else kr_contract_kernel<4><<<grid, dim3(256), 0, stream>>>(L);
    }
    if (fblocks > 0) kr_fold_kernel<<<dim3(static_cast<unsigned>(fblocks)), dim3(256), 0, stream>>>(L);
  }
}

}  // namespace ttnn
