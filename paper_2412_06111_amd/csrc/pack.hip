// Packing of a strided block: dst (column-major over the box extents, first mode
// fastest) = the block read through its element strides.  A large box read in place
// takes the generic contractions with per-position address maps for every node; packed
// once (one read and one write of the box at streaming speed) it takes the same
// kernels on contiguous data, with the same chunks and sums (so the same bits).
#include "kernels.hpp"

namespace ttnn {
namespace {

constexpr int kPer = 8;                     // entries a thread carries side by side
constexpr int64_t kPackMax = int64_t(1) << 30;   // entries of one launch: places fit 31 bits

// n / d for 0 <= n < 2^31 as one multiplication: with s = ceil(log2 d), mul = floor(2^(31 + s)
// / d) + 1 is at most 2^32 - 1 for d > 1 and 2^31 + 1 for d = 1, and mul d - 2^(31 + s) <= d
// <= 2^s, so the error n (mul / 2^(31 + s) - 1 / d) stays below 1 / d.
struct PackDiv {
  uint32_t mul, shift;
};
PackDiv pack_div(int64_t d) {
  uint32_t s = 0;
  while ((int64_t(1) << s) < d) ++s;
  return PackDiv{static_cast<uint32_t>((uint64_t(1) << (31 + s)) / static_cast<uint64_t>(d) + 1), 31 + s};
}
__device__ __forceinline__ uint32_t pack_quot(uint32_t n, PackDiv v) {
  return static_cast<uint32_t>((static_cast<uint64_t>(n) * v.mul) >> v.shift);
}

struct PackArgs {
  int d;
  uint32_t ext[TTNN_MAX_ORDER];
  PackDiv div[TTNN_MAX_ORDER];
  int64_t stride[TTNN_MAX_ORDER];
};

// Bound by its bytes: the box written once and read in runs of the first extent.  A unit is
// 256 kPer consecutive entries of dst.  Mode by mode, its first entry's digit (the same for
// all threads) plus what the mode before carried gives every entry's digit; each thread
// takes kPer entries 256 apart, so that their loads are in flight together.
// 33 x 21 x 47 x 40 x 26 FP32 entries (136 MB) of a 64^5 tensor: 153 -> 72 us (five 64-bit divisions an entry before)
template <typename W>
__global__ __launch_bounds__(256) void pack_box_kernel(const W* __restrict__ src, PackArgs a, W* __restrict__ dst,
                                                       uint32_t total) {
  constexpr uint32_t UNIT = 256 * kPer;
  for (uint32_t e0 = blockIdx.x * UNIT; e0 < total; e0 += gridDim.x * UNIT) {
    uint32_t first = e0, carry[kPer];
    int64_t off[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      carry[u] = threadIdx.x + 256 * u;
      off[u] = 0;
    }
    for (int m = 0; m < a.d; ++m) {
      const uint32_t up = pack_quot(first, a.div[m]), digit = first - up * a.ext[m];
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const uint32_t n = digit + carry[u];
        carry[u] = pack_quot(n, a.div[m]);
        off[u] += static_cast<int64_t>(n - carry[u] * a.ext[m]) * a.stride[m];
      }
      first = up;
    }
    W v[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u)          // places past the end: the digits wrap, the loads stay in the box
      v[u] = src[off[u]];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const uint32_t e = e0 + threadIdx.x + 256 * u;
      if (e < total) dst[e] = v[u];
    }
  }
}

template <typename W>
void pack_as(const void* src, int d, const int64_t* ext, const int64_t* strides, void* dst, hipStream_t st) {
  int64_t total = 1;
  for (int m = 0; m < d; ++m) total *= ext[m];
  if (total <= 0) return;
  const W* s = static_cast<const W*>(src);
  W* o = static_cast<W*>(dst);
  if (total >= kPackMax) {                  // halves along the last mode
    int last = d - 1;
    while (ext[last] == 1) --last;
    int64_t part[TTNN_MAX_ORDER];
    for (int m = 0; m < d; ++m) part[m] = ext[m];
    const int64_t half = ext[last] / 2, row = total / ext[last];
    part[last] = half;
    pack_as<W>(s, d, part, strides, o, st);
    part[last] = ext[last] - half;
    pack_as<W>(s + half * strides[last], d, part, strides, o + half * row, st);
    return;
  }
  // modes of extent 1 have no digit; a mode that continues the one before it in memory is
  // one mode with it
  PackArgs a{};
  int64_t len = 1;
  for (int m = 0; m < d; ++m) {
    if (ext[m] == 1) continue;
    if (a.d > 0 && strides[m] == a.stride[a.d - 1] * len) {
      len *= ext[m];
    } else {
      a.stride[a.d++] = strides[m];
      len = ext[m];
    }
    a.ext[a.d - 1] = static_cast<uint32_t>(len);
    a.div[a.d - 1] = pack_div(len);
  }
  const int64_t units = (total + 256 * kPer - 1) / (256 * kPer);
  const dim3 grid(static_cast<unsigned>(units < 65536 ? units : 65536));
  hipLaunchKernelGGL(pack_box_kernel<W>, grid, dim3(256), 0, st, s, a, o, static_cast<uint32_t>(total));
}

}  // namespace

void launch_pack_box(const void* src, int dt, int d, const int64_t* ext, const int64_t* strides, void* dst,
                     hipStream_t st) {
  if (dt == TTNN_F64) pack_as<uint64_t>(src, d, ext, strides, dst, st);
  else if (dt == TTNN_F32) pack_as<uint32_t>(src, d, ext, strides, dst, st);
  else pack_as<uint16_t>(src, d, ext, strides, dst, st);
  TTNN_HIP(hipGetLastError());
}

}  // namespace ttnn
