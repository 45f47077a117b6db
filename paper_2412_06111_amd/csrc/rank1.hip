// Rank-1 updates H = a_1 o a_2 o ... o a_d (streaming by linearity, Sec. 4).
//
// Every sketch of a rank-1 tensor factorises.  With u_I = kron of the factors of a
// mode group I (first mode fastest):
//   T^{(t)} = u_{I_t} u_{D\I_t}^T,  so  R_t = u_{I_t} (X_t^T u_{rows of X_t})^T;
// for STTNN the rows of X_t run over contracted groups s, whose factor becomes
// g_s = Y_s^T u_{I_s}; the root sketch is kron_c g_c.  Each product X^T u is a
// GEMV whose vector is never formed: the weight of a row is the product of one
// factor entry per position, read from the row's mixed-radix digits.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"
#include "mfma.hpp"

namespace ttnn {
namespace {

constexpr int kThreadsR = 256;
constexpr int kFacCache = 2048;   // factor entries of a term group kept in LDS by the GEMV (16 KB)

// partial[(y nb + b) ncols + j] = sum over the rows of block b of D[row * ncols + j] *
// weight_y(row), for the terms y of the batch.  The block's rows are contiguous in D:
// each step copies RB of them into LDS with 16-byte loads (rows padded by one element
// against bank conflicts); two lanes take a row, each half of its columns (NCH), two rows
// RH apart a step, and accumulate the products with the weights of up to MT terms in
// FP64, so one staged row serves every term of the block's group; a fixed-order reduction (shuffles over the
// lanes of a half, then the waves in order) ends the block.  A term's sums depend only
// on its own weights and on the row partition, which the batch does not change, so its
// result is bitwise the same in any batch.  A lane's row advances by RH at a time, so
// its mixed-radix digits (one per factor) advance by the digits of RH with one carry
// test each.  Blocks: the chunks of rows, padded to a multiple of 8, times the groups of MT
// terms, the groups of one chunk 8 blocks apart (the same XCD, dispatched together):
// block b takes chunk x = 8 (b / 8G) + b % 8 and group (b % 8G) / 8.  rows_per_block is
// a multiple of RB, so every step but the block's last is whole.
template <typename TD, int NCH, int MT, typename DI>
__global__ __launch_bounds__(kThreadsR) void kron_gemv_kernel(const TD* __restrict__ D, int64_t rows, int ncols,
                                                              KronBatch kb, int64_t rows_per_block, int64_t nb,
                                                              double* __restrict__ partial) {
  constexpr int NC = 2 * NCH;
  constexpr int RH = kThreadsR / 2;                                   // rows at once: two lanes a row
  constexpr int RB = 2 * RH;                                          // rows a step: two rows a lane pair
  constexpr int V = 16 / static_cast<int>(sizeof(TD));                // elements a 16-byte load
  constexpr int PER = (NC * RB + kThreadsR * V - 1) / (kThreadsR * V);  // loads a thread a step
  typedef TD vec_t __attribute__((ext_vector_type(V)));
  __shared__ __align__(16) TD tile[RB * (NC + 1)];
  __shared__ double red[kThreadsR / 64][MT][NC];
  __shared__ double fac[kFacCache];
  const int G = (kb.m + MT - 1) / MT;
  const int64_t bx = blockIdx.x, g8 = 8 * static_cast<int64_t>(G);
  const int64_t chunk = 8 * (bx / g8) + bx % 8;
  const int t0 = MT * static_cast<int>((bx % g8) / 8);                 // first term of the group
  if (chunk >= nb) return;                 // padding chunks (whole block, before any barrier)
  const int mg = kb.m - t0 < MT ? kb.m - t0 : MT;                     // terms of the group
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = tid >> 1, half = tid & 1;
  const int64_t r0 = chunk * rows_per_block;
  const int64_t r1 = r0 + rows_per_block < rows ? r0 + rows_per_block : rows;
  const int ld = ncols + 1;
  const KronVec& k0 = kb.kv[0];            // every term has the same factor lengths
  const int np = k0.n;
  // the group's factors in LDS when they fit (the usual case: a few hundred entries a
  // term), so that the weights never wait on global memory: a wait for a global gather
  // issued after the next step's loads would also wait for those loads (the counter is
  // in order).  Every loop over the factor positions runs to the compile-time maximum
  // with a guard, so that these small arrays stay in registers.
  int foff[kMaxPos];
  int64_t flen = 0;
#pragma unroll
  for (int p = 0; p < kMaxPos; ++p) {
    foff[p] = static_cast<int>(flen < kFacCache ? flen : 0);
    if (p < np) flen += k0.len[p];
  }
  const bool cached = flen * mg <= kFacCache;
  if (cached)
    for (int y = 0; y < mg; ++y)
#pragma unroll
      for (int p = 0; p < kMaxPos; ++p)
        if (p < np)
          for (int64_t i = tid; i < k0.len[p]; i += kThreadsR) fac[y * flen + foff[p] + i] = kb.kv[t0 + y].v[p][i];
  // (row, column) of this thread's first element of each load, and the stride between
  // its loads (kThreadsR * V elements)
  const int x0 = tid * V;
  const int row0 = x0 / ncols, col0 = x0 - row0 * ncols;
  const int dr = (kThreadsR * V) / ncols, dc = (kThreadsR * V) % ncols;
  // digits of this lane's first row and of RH (a lane pair takes rows RH apart)
  DI dig[kMaxPos], stp[kMaxPos], len[kMaxPos];
  {
    int64_t a = r0 + row, b = RH;
#pragma unroll
    for (int p = 0; p < kMaxPos; ++p) {
      const int64_t e = p < np ? k0.len[p] : 1;
      len[p] = static_cast<DI>(e);
      dig[p] = static_cast<DI>(a % e);
      a /= e;
      stp[p] = static_cast<DI>(b % e);
      b /= e;
    }
  }
  double acc[MT][NCH];
#pragma unroll
  for (int y = 0; y < MT; ++y)
#pragma unroll
    for (int j = 0; j < NCH; ++j) acc[y][j] = 0.0;
  vec_t v[PER];
  auto fetch = [&](int64_t b) {            // the step's loads, all in flight together
    const int64_t nr = r1 - b < RB ? r1 - b : RB;
    const TD* src = D + b * ncols;
    if (nr == RB) {
      // a whole step: RB * ncols elements, a multiple of V, 16-byte aligned (RB rows);
      // one predicated vector load each, no dependence between them
      const int total = RB * ncols;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int e = (tid + k * kThreadsR) * V;
        v[k] = e < total ? *reinterpret_cast<const vec_t*>(src + e) : vec_t{};
      }
    } else {
      // the block's last, partial step: element by element
      const int total = static_cast<int>(nr) * ncols;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int e = (tid + k * kThreadsR) * V;
        vec_t t{};
#pragma unroll
        for (int i = 0; i < V; ++i)
          if (e + i < total) t[i] = src[e + i];
        v[k] = t;
      }
    }
  };
  __syncthreads();                              // the factor cache is written
  if (r0 < r1) fetch(r0);
  for (int64_t base = r0; base < r1; base += RB) {
    const int nr = static_cast<int>(r1 - base < RB ? r1 - base : RB);
    const int total = nr * ncols;
    int rr = row0, cc = col0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = (tid + k * kThreadsR) * V;
      int r = rr, c = cc;
#pragma unroll
      for (int i = 0; i < V; ++i) {
        if (e + i < total) tile[r * ld + c] = v[k][i];
        if (++c == ncols) {
          c = 0;
          ++r;
        }
      }
      rr += dr;
      cc += dc;
      if (cc >= ncols) {
        cc -= ncols;
        ++rr;
      }
    }
    __syncthreads();
    if (base + RB < r1) fetch(base + RB);  // next step's loads overlap this step's products
#pragma unroll
    for (int h = 0; h < 2; ++h) {
    const int rl = row + h * RH;               // this pair's row within the step
    if (rl < nr) {
      double w[MT];
#pragma unroll
      for (int y = 0; y < MT; ++y) {
        w[y] = 1.0;
        if (y < mg) {
          if (cached) {
            const int fb = y * static_cast<int>(flen);
#pragma unroll
            for (int p = 0; p < kMaxPos; ++p)
              if (p < np) w[y] *= fac[fb + foff[p] + static_cast<int>(dig[p])];
          } else {
#pragma unroll
            for (int p = 0; p < kMaxPos; ++p)
              if (p < np) w[y] *= kb.kv[t0 + y].v[p][dig[p]];
          }
        }
      }
      const TD* q = tile + rl * ld + half * NCH;
#pragma unroll
      for (int j = 0; j < NCH; ++j)
        if (half * NCH + j < ncols) {
          const double x = to_f64(q[j]);
#pragma unroll
          for (int y = 0; y < MT; ++y)
            if (y < mg) acc[y][j] += x * w[y];
        }
    }
    DI carry = 0;                            // row += RH in mixed radix
#pragma unroll
    for (int p = 0; p < kMaxPos; ++p) {
      const DI x = dig[p] + stp[p] + carry;
      carry = x >= len[p];
      dig[p] = carry ? x - len[p] : x;
    }
    }
    __syncthreads();
  }
  // the lanes of one half hold the same columns: add them (lane bits 1..5), then the
  // waves in order
#pragma unroll
  for (int y = 0; y < MT; ++y)
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      double x = acc[y][j];
#pragma unroll
      for (int o = 2; o < 64; o <<= 1) x += __shfl_xor(x, o);
      if (lane < 2) red[wave][y][lane * NCH + j] = x;
    }
  __syncthreads();
  for (int e = tid; e < mg * ncols; e += kThreadsR) {
    const int y = e / ncols, j = e - y * ncols;
    double sum = red[0][y][j];
#pragma unroll
    for (int q = 1; q < kThreadsR / 64; ++q) sum += red[q][y][j];
    partial[(static_cast<int64_t>(t0 + y) * nb + chunk) * ncols + j] = sum;
  }
}

template <typename TD, int NCH, typename DI>
void launch_gemv_nch(const TD* D, int64_t rows, int ncols, const KronBatch& kb, int64_t per, int64_t nb,
                     double* partial, hipStream_t st) {
  // term slots a block: one for a single term (the fewest registers), else two, or four
  // where the accumulators fit (up to 24 columns).  A term's arithmetic is the same in
  // every instance: its slot only repeats the same operations for it.
  const int mt = kb.m == 1 ? 1 : (kb.m == 2 || NCH > 12) ? 2 : 4;
  const dim3 grid(static_cast<unsigned>((nb + 7) / 8 * 8 * ((kb.m + mt - 1) / mt)));
  if (mt == 1)
    hipLaunchKernelGGL((kron_gemv_kernel<TD, NCH, 1, DI>), grid, dim3(kThreadsR), 0, st, D, rows, ncols, kb, per, nb,
                       partial);
  else if (mt == 2)
    hipLaunchKernelGGL((kron_gemv_kernel<TD, NCH, 2, DI>), grid, dim3(kThreadsR), 0, st, D, rows, ncols, kb, per, nb,
                       partial);
  else
    hipLaunchKernelGGL((kron_gemv_kernel<TD, NCH, (NCH > 12 ? 2 : 4), DI>), grid, dim3(kThreadsR), 0, st, D, rows,
                       ncols, kb, per, nb, partial);
}

template <typename TD, typename DI>
void launch_gemv_di(const TD* D, int64_t rows, int ncols, const KronBatch& kb, int64_t per, int64_t nb,
                    double* partial, hipStream_t st) {
  if (ncols <= 8) launch_gemv_nch<TD, 4, DI>(D, rows, ncols, kb, per, nb, partial, st);
  else if (ncols <= 16) launch_gemv_nch<TD, 8, DI>(D, rows, ncols, kb, per, nb, partial, st);
  else if (ncols <= 24) launch_gemv_nch<TD, 12, DI>(D, rows, ncols, kb, per, nb, partial, st);
  else if (ncols <= 32) launch_gemv_nch<TD, 16, DI>(D, rows, ncols, kb, per, nb, partial, st);
  else if (ncols <= 48) launch_gemv_nch<TD, 24, DI>(D, rows, ncols, kb, per, nb, partial, st);
  else launch_gemv_nch<TD, 32, DI>(D, rows, ncols, kb, per, nb, partial, st);
}

template <typename TD>
void launch_gemv_dt(const TD* D, int64_t rows, int ncols, const KronBatch& kb, int64_t per, int64_t nb,
                    double* partial, hipStream_t st) {
  bool short_factors = true;
  for (int y = 0; y < kb.m; ++y)
    for (int p = 0; p < kb.kv[y].n; ++p) short_factors = short_factors && kb.kv[y].len[p] < (int64_t(1) << 30);
  if (short_factors) launch_gemv_di<TD, int>(D, rows, ncols, kb, per, nb, partial, st);
  else launch_gemv_di<TD, int64_t>(D, rows, ncols, kb, per, nb, partial, st);
}

// Kronecker GEMV with the two fastest factor positions (lengths e0, e1) contracted on
// the FP64 MFMA.  Block b holds the e0 e1 consecutive map rows of its outer index b (the
// digits of positions 2, 3, ..); for every term y
//   C_y[j] = sum_{i1 < e1} v1_y[i1] sum_{i0 < e0} v0_y[i0] D[i0 + e0 (i1 + e1 b)][j],
// the inner sum as a 16 x 16 x 4 MFMA product with the terms as rows (A[y][i0] =
// v0_y[i0]) and a 16-column block of the map as columns (B[i0][j], K = e0 in steps of
// 4), each scaled by v1_y[i1] times the remaining factors at b's digits.
//
// A wave takes one i1 at a time, or (PAIR) two neighbouring ones whose columns share the
// MFMA's 16-column blocks: 24 columns fill one and a half, so two i1 of 24 take three
// instead of four.  The A operand never changes and stays in registers; the map entries
// go from memory straight into the registers that the MFMA reads (a lane's entry of a
// step is one load; a row's 96 bytes are read by the loads of neighbouring column blocks
// while in the first-level cache), and the register of a step just multiplied takes the
// same step of the wave's next i1, so a wave keeps a whole i1's entries in flight and no
// LDS copy, guard or barrier stands in the loop.  Columns past the end
// are read from clamped places: what they form is not written.
//
// NBW consecutive blocks share a workgroup (fewer partials to add); a block's i1 range may
// be split over S workgroups instead.  A term's row of the product does not depend on the
// other rows, so its partials are the same in any batch.
//
// Bound by the map's bytes: a 64^5 leaf map (64^4 x 24 FP32, 1.61 GB, 16 terms) takes 365 us,
// 4.4 TB/s (the products alone 165 us at the FP64 MFMA's rate); through LDS tiles with a
// guard an entry and no pairing it took 530 us.  A group of 16 terms on 64^5: 3390 -> 1976
// us, with the wide maps (36 columns) here too (417 -> 24 us) and the outer products in
// one launch.
constexpr int kKmE0 = 64;         // largest e0
constexpr int kKmE1 = 64;         // largest e1
constexpr int kKmBlocks = 16;     // most blocks a workgroup

template <typename TD, int NCB, bool PAIR, int KSTEPS>
__global__ __launch_bounds__(256, sizeof(TD) == 8 || NCB == 4 ? 2 : 3) void kron_mfma_kernel(const TD* __restrict__ D, int ncols,
                                                                                 KronBatch kb, int64_t nb, int S,
                                                                                 int NBW, int64_t np,
                                                                                 double* __restrict__ partial) {
  using P = Pol<TTNN_F64>;
  // KSTEPS steps of 4 values cover e0; US of them are in flight (FP64 entries: half an i1)
  constexpr int US = sizeof(TD) == 8 || KSTEPS == 8 ? 8 : 16;
  constexpr int NH = KSTEPS / US;
  // [wave][term][column] sums at the end; the A operand's table at the start
  __shared__ double red[4 * 16 * 16 * NCB];
  // factor tables [position value][term]: the 16 lanes of a group read 16 consecutive
  // doubles (with [term][value] rows of 512 bytes they hit one bank)
  __shared__ double W1[kKmE1][16];
  __shared__ double Wr[kKmBlocks][16];
  static_assert(4 * 16 * 16 * NCB >= kKmE0 * 16, "the A table fits the sums");

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t g = blockIdx.x;             // partial row: block group g / S, i1 split g % S
  const int64_t b0 = g / S * NBW, b1 = b0 + NBW < nb ? b0 + NBW : nb;
  const int sp = static_cast<int>(g % S);
  const int m = kb.m;
  const KronVec& k0 = kb.kv[0];             // every term has the same factor lengths
  const int e0 = static_cast<int>(k0.len[0]), e1 = static_cast<int>(k0.len[1]);
  const int blk = e0 * ncols;               // entries of one i1

  for (int e = tid; e < 16 * kKmE0; e += 256) {
    const int y = e / kKmE0, i = e % kKmE0;
    red[i * 16 + y] = (y < m && i < e0) ? kb.kv[y].v[0][i] : 0.0;
    W1[i][y] = (y < m && i < e1) ? kb.kv[y].v[1][i] : 0.0;
  }
  static_assert(kKmE0 == kKmE1, "one loop fills both tables");
  for (int e = tid; e < 16 * static_cast<int>(b1 - b0); e += 256) {
    const int y = e % 16;
    double w = 0.0;
    if (y < m) {                            // the remaining factors at the block's digits
      w = 1.0;
      int64_t rem = b0 + e / 16;
      for (int p = 2; p < k0.n; ++p) {
        const int64_t len = k0.len[p], q = rem / len;
        w *= kb.kv[y].v[p][rem - q * len];
        rem = q;
      }
    }
    Wr[e / 16][y] = w;
  }
  __syncthreads();
  double w0[KSTEPS];
#pragma unroll
  for (int s = 0; s < KSTEPS; ++s) {
    const int i0 = (4 * s < e0 - 4 ? 4 * s : e0 - 4) + lg;
    w0[s] = i0 >= 4 * s ? red[i0 * 16 + l16] : 0.0;
  }
  __syncthreads();                          // red is free for the sums

  // byte offsets of the lane's entries: row lg of a step, column 16 cb + l16 of the i1 (pair)
  uint32_t lo[NCB];
  uint32_t sec = 0;                         // column blocks whose entry is of the pair's second i1
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    int c = 16 * cb + l16;
    const int nc = PAIR ? 2 * ncols : ncols;
    if (c >= nc) c = nc - 1;
    const bool two = PAIR && c >= ncols;
    sec |= (two ? 1u : 0u) << cb;
    lo[cb] = static_cast<uint32_t>(sizeof(TD)) * static_cast<uint32_t>(lg * ncols + (two ? blk + c - ncols : c));
  }

  TD buf[US][NCB];
  // step gs of the i1 (pair) at ub into buf[s]; steps that reach past e0 take its last four
  // values (those they repeat meet zeros of A).  No step is skipped: a branch around a
  // step's loads made the compiler wait for all loads in flight (466 us a leaf map)
  auto load = [&](const TD* ub, const uint32_t* at, int gs, int s) {
    const int r0 = 4 * gs < e0 - 4 ? 4 * gs : e0 - 4;
    const char* row = reinterpret_cast<const char*>(ub + r0 * ncols);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) buf[s][cb] = *reinterpret_cast<const TD*>(row + at[cb]);
  };
  // lane offsets of an i1: an odd e1's last i1 stands in for its missing pair
  auto offsets = [&](bool odd, uint32_t* at) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
      at[cb] = PAIR && odd && ((sec >> cb) & 1u) ? lo[cb] - static_cast<uint32_t>(sizeof(TD)) * blk : lo[cb];
  };
  typename P::CFrag acc[NCB], c[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) acc[cb] = typename P::CFrag{};
  // multiply half h of an i1 out of buf, taking half hn of the i1 at nub in its place
  auto turn = [&](auto hc, auto hn, const TD* nub, bool nodd) {
    constexpr int HC = decltype(hc)::value, HN = decltype(hn)::value;
    uint32_t at[NCB];
    offsets(nodd, at);
#pragma unroll
    for (int s = 0; s < US; ++s) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) c[cb] = P::mfma(w0[HC * US + s], to_f64(buf[s][cb]), c[cb]);
      load(nub, at, HN * US + s, s);
    }
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, NH - 1>;

  constexpr int PW = PAIR ? 2 : 1;
  const int nu = (e1 + PW - 1) / PW, u0 = 4 * sp + wave, ust = 4 * S;
  auto at = [&](int64_t b, int u) { return D + (b * e1 + u * PW) * static_cast<int64_t>(blk); };
  auto alone = [&](int u) { return PAIR && 2 * u + 1 == e1; };
  if (u0 < nu && b0 < b1) {
    int64_t b = b0;
    int u = u0;
    const TD* ub = at(b, u);
    uint32_t first[NCB];
    offsets(alone(u), first);
#pragma unroll
    for (int s = 0; s < US; ++s) load(ub, first, s, s);
    for (;;) {
      int64_t bn = b;
      int un = u + ust;
      if (un >= nu) {
        un = u0;
        ++bn;
      }
      const bool more = bn < b1;
      const TD* nub = more ? at(bn, un) : ub;        // past the last i1: its own entries again
      const bool nodd = alone(more ? un : u);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) c[cb] = typename P::CFrag{};
      if constexpr (NH == 1) {
        turn(H0{}, H0{}, nub, nodd);
      } else {
        turn(H0{}, H1{}, ub, alone(u));
        turn(H1{}, H0{}, nub, nodd);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int y = P::crow(lane, v);
        const double wr = Wr[b - b0][y];
        const double s1 = W1[u * PW][y] * wr;
        const double s2 = PAIR ? W1[(u * PW + 1) & (kKmE1 - 1)][y] * wr : s1;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[cb][v] += ((sec >> cb) & 1u ? s2 : s1) * c[cb][v];
      }
      if (!more) break;
      b = bn;
      u = un;
      ub = nub;
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) red[(wave * 16 + P::crow(lane, v)) * (16 * NCB) + 16 * cb + l16] = acc[cb][v];
  __syncthreads();
  for (int e = tid; e < 16 * ncols; e += 256) {
    const int y = e / ncols, j = e % ncols;
    if (y >= m) continue;
    const int o = y * (16 * NCB) + j, ws = 16 * 16 * NCB;
    double sum = ((red[o] + red[o + ws]) + red[o + 2 * ws]) + red[o + 3 * ws];
    if (PAIR) sum += ((red[o + ncols] + red[o + ncols + ws]) + red[o + ncols + 2 * ws]) + red[o + ncols + 3 * ws];
    partial[(static_cast<int64_t>(y) * np + g) * ncols + j] = sum;
  }
}

// How a map of nb blocks goes over workgroups: NBW blocks each (about 2,048 workgroups, a
// partial row each), or for few blocks each block's i1 range over S workgroups (up to
// 1,024 partial rows, a wave at least one i1 or pair).  A function of the map's shape only,
// never of the batch.
struct KronSplit {
  int S, NBW;
  int64_t np;
  bool pair;
};
KronSplit kron_mfma_split(int64_t nb, int64_t e1, int ncols) {
  const int one = (ncols + 15) / 16, two = (2 * ncols + 15) / 16;
  KronSplit k{1, 1, 0, two < 2 * one && two <= 3};
  if (nb >= 1024) {
    k.NBW = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(nb / 2048, kKmBlocks)));
  } else {
    const int64_t units = k.pair ? (e1 + 1) / 2 : e1;
    k.S = static_cast<int>(std::min<int64_t>((1024 + nb - 1) / nb, std::max<int64_t>(1, units / 4)));
  }
  k.np = (nb + k.NBW - 1) / k.NBW * k.S;
  return k;
}

// Whether the MFMA form covers this map and batch shape (never depends on the number
// of terms, so a term takes the same form alone and in any batch).
bool kron_mfma_eligible(int64_t rows, int ncols, const KronVec& k0, size_t partial_elems) {
  if (k0.n < 2) return false;
  const int64_t e0 = k0.len[0], e1 = k0.len[1];
  if (e0 < 16 || e0 > kKmE0 || e1 < 4 || e1 > kKmE1) return false;
  const int64_t nb = rows / (e0 * e1);
  if (nb < 1 || nb * e0 * e1 != rows) return false;
  const KronSplit k = kron_mfma_split(nb, e1, ncols);
  return static_cast<size_t>(k.np) * static_cast<size_t>(ncols) * kRank1Batch <= partial_elems;
}

template <typename TD, int NCB, bool PAIR>
void launch_kron_form(const TD* D, int ncols, const KronBatch& kb, int64_t nb, const KronSplit& k, double* partial,
                      hipStream_t st) {
  const dim3 grid(static_cast<unsigned>(k.np));
  if (kb.kv[0].len[0] <= 32)
    hipLaunchKernelGGL((kron_mfma_kernel<TD, NCB, PAIR, 8>), grid, dim3(256), 0, st, D, ncols, kb, nb, k.S, k.NBW,
                       k.np, partial);
  else
    hipLaunchKernelGGL((kron_mfma_kernel<TD, NCB, PAIR, 16>), grid, dim3(256), 0, st, D, ncols, kb, nb, k.S, k.NBW,
                       k.np, partial);
}
template <typename TD>
void launch_kron_mfma(const TD* D, int ncols, const KronBatch& kb, int64_t nb, const KronSplit& k, double* partial,
                      hipStream_t st) {
  if (k.pair) {
    if (2 * ncols <= 16) launch_kron_form<TD, 1, true>(D, ncols, kb, nb, k, partial, st);
    else launch_kron_form<TD, 3, true>(D, ncols, kb, nb, k, partial, st);
    return;
  }
  switch ((ncols + 15) / 16) {
    case 1: launch_kron_form<TD, 1, false>(D, ncols, kb, nb, k, partial, st); break;
    case 2: launch_kron_form<TD, 2, false>(D, ncols, kb, nb, k, partial, st); break;
    case 3: launch_kron_form<TD, 3, false>(D, ncols, kb, nb, k, partial, st); break;
    default: launch_kron_form<TD, 4, false>(D, ncols, kb, nb, k, partial, st); break;
  }
}

// w[y wstride + j] = sum_b partial[y nb + b][j]: a workgroup takes eight columns of a term,
// 128 rows at a time (64-byte pieces of a row; one wave per column read 8 bytes of each
// row, 17 us for 4,096 rows of 24 columns and 16 terms), 16 loads of a thread in flight;
// the 128 row sums of a column are added in a fixed tree.
__global__ __launch_bounds__(1024) void sum_blocks_kernel(const double* __restrict__ partial, int nb, int ncols,
                                                          double* __restrict__ w, int64_t wstride) {
  __shared__ double red[128][9];
  const int j = 8 * blockIdx.x + (threadIdx.x & 7), y = blockIdx.y, r = threadIdx.x >> 3;
  const double* p = partial + static_cast<int64_t>(y) * nb * ncols + (j < ncols ? j : ncols - 1);
  double s = 0.0;
  int b = r;
  for (; b + 15 * 128 < nb; b += 16 * 128) {
    double v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = p[static_cast<int64_t>(b + 128 * i) * ncols];
#pragma unroll
    for (int i = 0; i < 16; ++i) s += v[i];
  }
  for (; b < nb; b += 128) s += p[static_cast<int64_t>(b) * ncols];
  red[r][threadIdx.x & 7] = s;
  __syncthreads();
  for (int h = 64; h > 0; h >>= 1) {
    if (r < h) red[r][threadIdx.x & 7] += red[r + h][threadIdx.x & 7];
    __syncthreads();
  }
  if (r == 0 && j < ncols) w[y * wstride + j] = red[0][threadIdx.x & 7];
}

// R_t[i + n_t j] += alpha_y u_y(i) w_y[j], the terms in order, for the nodes of a list in
// one launch (a launch a node left most of them a few workgroups, 17-20 us each for a
// 64 x 24 sketch; 223 us of a 64^5 group of 16, now 45).  A thread takes a row: it splits
// the row into factor digits once, forms alpha_y u_y for every term (each weight
// multiplied out in factor order) and sweeps its share of the columns; neighbouring lanes
// take neighbouring rows, so every column access coalesces.
constexpr int kOuterNodes = 24;
struct OuterTask {
  double* R;
  const double* w;                 // [term][ncols]; null: 1
  int64_t n;
  int32_t ncols, first, cnt;       // factors first .. first + cnt - 1; first < 0: the root's
  int32_t row_blocks, groups, first_block;
};
struct OuterLaunch {
  OuterTask t[kOuterNodes];
  const double* f[kRank1Batch][TTNN_MAX_ORDER];
  int64_t len[TTNN_MAX_ORDER];
  const double* g[TTNN_MAX_ORDER];           // the root's factors: term y's at g[c] + y gstride
  int64_t glen[TTNN_MAX_ORDER];
  int64_t gstride;
  double alpha[kRank1Batch];
  int32_t m, count;
};
__device__ inline double lane_value(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(b), l);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(b >> 32), l);
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}
__global__ __launch_bounds__(256) void outer_acc_kernel(OuterLaunch L) {
  int ti = 0;
  while (ti + 1 < L.count && L.t[ti + 1].first_block <= static_cast<int>(blockIdx.x)) ++ti;
  const OuterTask& t = L.t[ti];
  const int rel = static_cast<int>(blockIdx.x) - t.first_block;
  int64_t i = static_cast<int64_t>(rel % t.row_blocks) * 256 + threadIdx.x;
  const bool live = i < t.n;                 // every lane stays: the wave reads lanes 0 .. 15
  if (!live) i = 0;
  double a[kRank1Batch];
#pragma unroll
  for (int y = 0; y < kRank1Batch; ++y) a[y] = 1.0;
  int64_t row = i;
  for (int p = 0; p < t.cnt; ++p) {
    const bool root = t.first < 0;
    const int64_t e = root ? L.glen[p] : L.len[t.first + p];
    int64_t dgt;
    if ((row | e) >> 32) {
      const int64_t q = row / e;
      dgt = row - q * e;
      row = q;
    } else {
      const uint32_t q = static_cast<uint32_t>(row) / static_cast<uint32_t>(e);
      dgt = static_cast<uint32_t>(row) - q * static_cast<uint32_t>(e);
      row = q;
    }
    // (terms past the last read term 0's factors, with a scale of 0)
    double x[kRank1Batch];
#pragma unroll
    for (int y = 0; y < kRank1Batch; ++y) x[y] = (root ? L.g[p] + (y < L.m ? y : 0) * L.gstride : L.f[y][t.first + p])[dgt];
#pragma unroll
    for (int y = 0; y < kRank1Batch; ++y) a[y] *= x[y];
  }
#pragma unroll
  for (int y = 0; y < kRank1Batch; ++y) a[y] = y < L.m ? a[y] * L.alpha[y] : 0.0;
  // four columns at a time, all their loads before any use; lane y of 16 holds term y's
  // w of the column and is read by the whole wave
  const int ly = threadIdx.x & 15;
  const bool lw = t.w && ly < L.m;
  for (int j0 = rel / t.row_blocks; j0 < t.ncols; j0 += 4 * t.groups) {
    double r[4], w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = j0 + q * t.groups < t.ncols ? j0 + q * t.groups : j0;
      r[q] = live ? t.R[i + t.n * j] : 0.0;
      w[q] = lw ? t.w[ly * t.ncols + j] : (t.w ? 0.0 : 1.0);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (j0 + q * t.groups >= t.ncols) break;
#pragma unroll
      for (int y = 0; y < kRank1Batch; ++y) r[q] += a[y] * lane_value(w[q], y);
      if (live) t.R[i + t.n * (j0 + q * t.groups)] = r[q];
    }
  }
}

}  // namespace

void launch_kron_gemv(const void* D, int dt, int64_t rows, int ncols, const KronBatch& kb, double* partial,
                      size_t partial_elems, double* w, int64_t wstride, bool grouped, hipStream_t st) {
  if (ncols <= 0 || kb.m <= 0) return;
  TTNN_REQUIRE(ncols <= 64, TTNN_E_INVALID, "rank-1 update with more than 64 map columns");
  TTNN_REQUIRE(kb.m <= kRank1Batch, TTNN_E_INVALID, "too many rank-1 terms in one launch");
  const dim3 sum_grid(static_cast<unsigned>((ncols + 7) / 8), static_cast<unsigned>(kb.m));
  if (grouped && kron_mfma_eligible(rows, ncols, kb.kv[0], partial_elems)) {
    const int64_t nbm = rows / (kb.kv[0].len[0] * kb.kv[0].len[1]);
    const KronSplit k = kron_mfma_split(nbm, kb.kv[0].len[1], ncols);
    if (dt == TTNN_F64) launch_kron_mfma(static_cast<const double*>(D), ncols, kb, nbm, k, partial, st);
    else if (dt == TTNN_F32) launch_kron_mfma(static_cast<const float*>(D), ncols, kb, nbm, k, partial, st);
    else launch_kron_mfma(static_cast<const uint16_t*>(D), ncols, kb, nbm, k, partial, st);
    hipLaunchKernelGGL(sum_blocks_kernel, sum_grid, dim3(1024), 0, st, partial, static_cast<int>(k.np), ncols, w,
                       wstride);
    return;
  }
  // >= 512 rows a block, at most 2048 blocks a term; the chunking depends on rows and
  // ncols only, never on the batch, so a term's sums are the same in any batch
  int64_t nb = (rows + 511) / 512;
  if (nb < 1) nb = 1;
  if (nb > 2048) nb = 2048;
  const int64_t cap = static_cast<int64_t>(partial_elems / (static_cast<size_t>(ncols) * kRank1Batch));
  if (nb > cap) nb = cap;
  TTNN_REQUIRE(nb >= 1, TTNN_E_INVALID, "rank-1 scratch too small");
  // rows a block: a multiple of the kernel's step (256 rows)
  const int64_t rb = kThreadsR;
  int64_t per = (rows + nb - 1) / nb;
  per = (per + rb - 1) / rb * rb;
  if (per < rb) per = rb;
  nb = rows > 0 ? (rows + per - 1) / per : 1;
  if (dt == TTNN_F64)
    launch_gemv_dt(static_cast<const double*>(D), rows, ncols, kb, per, nb, partial, st);
  else if (dt == TTNN_F32)
    launch_gemv_dt(static_cast<const float*>(D), rows, ncols, kb, per, nb, partial, st);
  else
    launch_gemv_dt(static_cast<const uint16_t*>(D), rows, ncols, kb, per, nb, partial, st);
  hipLaunchKernelGGL(sum_blocks_kernel, sum_grid, dim3(1024), 0, st, partial, static_cast<int>(nb), ncols, w, wstride);
}

void launch_outer_list(const OuterList& o, hipStream_t st) {
  TTNN_REQUIRE(o.m <= kRank1Batch, TTNN_E_INVALID, "too many rank-1 terms in one launch");
  for (size_t i0 = 0; i0 < o.nodes.size(); i0 += kOuterNodes) {
    OuterLaunch L{};
    L.m = o.m;
    L.count = static_cast<int32_t>(std::min<size_t>(kOuterNodes, o.nodes.size() - i0));
    for (int y = 0; y < kRank1Batch; ++y) {
      L.alpha[y] = y < o.m ? o.alpha[y] : 0.0;
      for (int mu = 0; mu < o.d; ++mu) L.f[y][mu] = o.f[(y < o.m ? y : 0) * o.d + mu];
    }
    for (int mu = 0; mu < o.d; ++mu) L.len[mu] = o.len[mu];
    for (int c = 0; c < o.root.n; ++c) {
      L.g[c] = o.root.v[c];
      L.glen[c] = o.root.len[c];
    }
    L.gstride = o.gstride;
    int64_t blocks = 0;
    for (int i = 0; i < L.count; ++i) {
      const OuterNode& x = o.nodes[i0 + i];
      OuterTask& t = L.t[i];
      const int64_t rb = (x.n + 255) / 256;
      // column groups enough for about 2,048 workgroups (the weights are formed once a group)
      const int64_t cg = std::min<int64_t>(x.ncols, std::max<int64_t>(1, 2048 / rb));
      t = OuterTask{x.R, x.w, x.n, x.ncols, x.first, x.cnt, static_cast<int32_t>(rb), static_cast<int32_t>(cg),
                    static_cast<int32_t>(blocks)};
      blocks += rb * cg;
      TTNN_REQUIRE(blocks < (int64_t(1) << 31), TTNN_E_INVALID, "rank-1 outer products: launch too large");
    }
    if (blocks > 0) hipLaunchKernelGGL(outer_acc_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, L);
  }
}

}  // namespace ttnn
