// The tile contraction of stride-1 rulebooks, on the bf16 matrix cores in
// three-way split fp32 (split.h):
//   dst[row] = act(add + sum over offsets k of (src[row_k] - sub) W_k)
// where row_k is the row that offset k gives the accumulator row, if any.
//
// One wave owns 64 accumulator rows and 64 columns, its 64 x 64 accumulators
// in registers: no scatter, one write per row.  It walks items (offset,
// channel chunk); an item's 64 rows are gathered while the item before is
// multiplied, turned through LDS into the layout of the MFMA operand, split
// and multiplied by the split W_k.  A row without the item's offset reads
// `sub` itself, so its difference is exactly zero.
//
// What bounds it: per 16 channels a wave issues 24 MFMAs of 32 clocks (768)
// against about 110 vector instructions (440) and, per CU, 10 KB of LDS reads
// and 6 KB of L1 traffic per wave.  With everything in LDS the loop runs at
// 1570 TFLOP/s of bf16 (the MFMAs alone at 2190); on the 1M-site 64 -> 64
// layer the input gradient, whose tiles are full, runs at 905 (1.46 ms; 2.11
// on the fp32 instruction with LDS accumulators), the clock at 1.95 GHz.
// Gathering 1024 fixed rows takes 0.09 ms off it, no gather at all 0.2.
// Measured and not kept there: LDS reads and splits of the next step
// interleaved with a step's MFMAs (1.33 ms against 1.23 left in blocks, before
// the sums went in two levels: the two waves of a SIMD then contend instead of
// alternating), eight waves sharing weights (1.32), every wave loading its
// weights from L2 (1.6), four steps per item (1.31), raised priority around
// the MFMAs (1.37).
#include <hip/hip_runtime.h>

#include "split.h"
#include "tile.h"

namespace scn {
namespace {

constexpr int NT = 256;  // threads per work-group (4 waves)

// Fewer (tile, column block) items than this, one per SIMD: four waves share
// each.  (35 -> 50 channels on 1.8k tiles: 66 us shared, 54 not; the networks and
// the stack are within 1% from 512 to 4096.)
constexpr int64_t TILE_SPLIT = 1024;

// Channels go in chunks of one or two 16-channel steps, few of them padded.
// (Longer chunks take registers that a third or second work-group per CU
// needs: four steps per item, two work-groups, 2.71 ms for the forward of the
// benchmark's layer against 2.60.  An odd number of steps rounded up for
// chunks of two: 48 and 80 channels 4 to 14% slower but for single cases.)
int chunk_steps(int Rk) { return Rk >= 32 && ceil_div(Rk, 16) % 2 == 0 ? 2 : 1; }

constexpr int PRE_COLS = 4;

// The channel that entry j of the reduction holds, of a row of Rk >= 4 read in
// chunks of C = 16 TC entries.  A last chunk that the row does not fill starts
// earlier and overlaps the one before (in a row shorter than one chunk, its
// last piece of four does, and pieces past the row repeat it), so that every
// piece of four entries is four channels in a row, of any alignment, and none
// leaves it.  Entries that repeat a channel (one below their unit's start) carry
// zero weights.
struct Entries {
  int mask, last;  // start of entry j's unit: j & mask; where the last unit starts
  __host__ __device__ Entries(int Rk, int C)  // C = 1: entry j is channel j
      : mask(-(Rk >= C ? C : 4)), last(Rk - (Rk >= C ? C : 4)) {}
  __device__ int channel(int j) const { return min(j & mask, last) + (j & ~mask); }
  __device__ bool repeats(int j) const { return channel(j) < (j & mask); }
};
// Where piece `piece` of the first step of chunk ch starts is
// min(C ch + 4 piece, piece_limit); the second step's is 16 channels on.
__device__ inline int piece_limit(int piece, int Rk, int C) {
  return Rk >= C ? Rk - C + 4 * piece : Rk - 4;
}

// Wp[k][cb][step][ct][part][lane][4 words]: the eight reduction entries
// j = 16 step + 8 (lane >> 5) + 0..7 of column n = 64 cb + 32 ct + (lane & 31).
__global__ void __launch_bounds__(NT) tile_pack_kernel(const float* __restrict__ W, int64_t wk,
                                                       int64_t wj, int64_t wn, int K, int Rk,
                                                       int Nc, int nst, int ncb, Entries E,
                                                       const float* __restrict__ g, int gm,
                                                       const float* __restrict__ bias, int relu,
                                                       v4u* __restrict__ Wp,
                                                       uint32_t* __restrict__ wtiny,
                                                       float* __restrict__ sub, int np,
                                                       float* __restrict__ g_pre,
                                                       float* __restrict__ g_out) {
  if ((int)blockIdx.x >= np) {
    // Per column n whether it is tiny (split.h), the largest sum that a tiny row
    // can have there (sum |W| 2^-95, rounded up), and, if asked for, g_pre[n] = B[n] +
    // sum_k g W_k(., n) and g_out = act(g_pre): PRE_COLS columns per block, NT /
    // PRE_COLS threads each, in 64 bits (few products, and every output starts
    // from them)
    __shared__ double part[2][NT / 64][PRE_COLS];
    __shared__ uint32_t obits[NT / 64][PRE_COLS];
    const int c = threadIdx.x % PRE_COLS, t = threadIdx.x / PRE_COLS;
    const int n = ((int)blockIdx.x - np) * PRE_COLS + c;
    const float* const gs = g ? g : W;  // without g (gm = 1) some sum, not used
    double s = 0., l = 0.;
    uint32_t o = 0;
    if (n < Nc) {
      const int tot = K * Rk;
#pragma unroll 8
      for (int q = t; q < tot; q += NT / PRE_COLS) {
        const int k = q / Rk, j = q - k * Rk;
        const float v = W[k * wk + j * wj + n * wn];
        o |= __float_as_uint(v);
        l += (double)fabsf(v);
        s = fma((double)gs[j % gm], (double)v, s);
      }
    }
    // over a wave's threads of a column, then the waves in order
#pragma unroll
    for (int d = PRE_COLS; d < 64; d <<= 1) {
      o |= (uint32_t)__shfl_xor((int)o, d, 64);
      l += __shfl_xor(l, d, 64);
      s += __shfl_xor(s, d, 64);
    }
    if ((threadIdx.x & 63) < PRE_COLS) {
      const int w = threadIdx.x >> 6;
      obits[w][c] = o;
      part[0][w][c] = s;
      part[1][w][c] = l;
    }
    __syncthreads();
    if (t == 0 && n < Nc) {
#pragma unroll
      for (int w = 1; w < NT / 64; ++w) {
        o |= obits[w][c];
        s += part[0][w][c];
        l += part[1][w][c];
      }
      wtiny[n] = tiny_floats(o);
      wtiny[Nc + n] = __float_as_uint((float)(l * 0x1.01p-95));
    }
    if (g_pre && t == 0 && n < Nc) {
      const float v = (float)(s + (bias ? (double)bias[n] : 0.));
      g_pre[n] = v;
      g_out[n] = relu && !(v > 0.f) ? 0.f : v;
    }
    return;
  }
  const int i = blockIdx.x * NT + threadIdx.x;
  if (i < TILE_PAD) sub[i] = g && i < Rk ? g[i % gm] : 0.f;
  const int lane = i & 63, ct = (i >> 6) & 1;
  const int f = i >> 7;  // (k*ncb + cb)*nst + step
  if (f >= K * ncb * nst) return;
  const int step = f % nst, kc = f / nst, cb = kc % ncb, k = kc / ncb;
  const int n = 64 * cb + 32 * ct + (lane & 31), j0 = 16 * step + 8 * (lane >> 5);
  const float* const Wn = W + k * wk + min(n, Nc - 1) * wn;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = Wn[E.channel(j0 + e) * wj];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (n < Nc) & !E.repeats(j0 + e) ? v[e] : 0.f;
  if (k & 1) {  // odd offsets negated (add_item)
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = -v[e];
  }
  const Frag3 s = split8(v);
#pragma unroll
  for (int p = 0; p < 3; ++p) Wp[(((int64_t)f * 2 + ct) * 3 + p) * 64 + lane] = s.s[p];
}

// Orders the wave's LDS accesses: a lane reads what other lanes wrote, which
// the compiler, seeing one lane's addresses, cannot know.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// An offset's index words of a lane's row, loaded ahead of their use.
struct Idx {
  int g, s;
};

// Where the 64 rows of a wave's tile come from: lane l knows accumulator row
// row0 + l.  U: the offsets that any of the rows has.
template <bool SORTED>
struct Rows {
  int64_t row0;
  uint32_t U;
  int64_t P;        // lists: lane k holds the tile's range of list k
  int N;
  uint32_t m, off;  // sorted: the lane's mask and list
  const int32_t *gidx, *aidx;
  int64_t last;     // lists: the last pair

  __device__ inline void init(const TileArgs& a, int64_t tile, int lane) {
    row0 = tile * TILE;
    if (SORTED) {
      const int64_t pos = row0 + lane;
      gidx = a.nb;
      m = pos < a.nrows ? a.fmask[pos] : 0u;
      off = a.nb_off[pos < a.nrows ? a.fperm[pos] : 0];
      uint32_t o = m;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) o |= (uint32_t)__shfl_xor((int)o, d, 64);
      U = (uint32_t)__builtin_amdgcn_readfirstlane((int)o);
    } else {
      const int k = lane < a.K ? lane : 0;
      gidx = a.gidx;
      aidx = a.aidx;
      P = a.tpos[(int64_t)k * a.ntile + tile];
      N = lane < a.K ? (int)(a.tpos[(int64_t)k * a.ntile + tile + 1] - P) : 0;
      U = (uint32_t)__ballot(N > 0);
      last = a.npairs - 1;
    }
  }
  __device__ inline Idx load(int k, int lane) const {
    Idx x;
    if (SORTED) {
      // read unconditionally (the list has a spare entry)
      x.g = gidx[off + __popc(m & ((1u << k) - 1u))];
      x.s = 0;
    } else {
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)P, k);
      const uint32_t hi =
          (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)P >> 32), k);
      const int n = __builtin_amdgcn_readlane(N, k);
      // lanes past the pairs repeat the last one; an offset without pairs
      // here reads some pair
      const int64_t p = min((int64_t)(((uint64_t)hi << 32) | lo) + max(min(lane, n - 1), 0), last);
      x.g = gidx[p];
      x.s = aidx[p];
    }
    return x;
  }
  // row of src for the lane's accumulator row at offset k, or -1
  __device__ inline int row(const Idx& x, int k) const {
    if (SORTED) return (m >> k) & 1u ? x.g : -1;
    // the pair's row takes it; a row that no pair names receives 0
    const int r = __builtin_amdgcn_ds_permute((int)(x.s - row0) * 4, x.g + 1) - 1;
    return (U >> k) & 1u ? r : -1;
  }
};

// Items in (offset, chunk) order; past the last one an item stays where it is
// (its loads are in bounds and unused).
struct Item {
  int k, ch;
  uint32_t rest;  // offsets after k
  __device__ inline void advance(int nchunk) {
    if (ch + 1 < nchunk) {
      ++ch;
    } else if (rest) {
      k = __builtin_ctz(rest);
      rest &= rest - 1;
      ch = 0;
    }
  }
};

typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

// Gather of an item's 64 rows.  Load layout: lane 4 rl + cq takes 16 bytes of
// row 16 g + rl, so four adjacent lanes read 64 contiguous bytes (in the MFMA
// layout adjacent lanes hold different rows, and the L1 would serve each
// 16-byte piece on its own).
template <int TC, bool VEC>
__device__ inline void gather_rows(v4f (&nx)[4][TC], const float* src, int Rk, int64_t absent,
                                   int row, int ch, int rl, int piece) {
  const int c0 = min(16 * TC * ch + 4 * piece, piece_limit(piece, Rk, 16 * TC));
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int r = __builtin_amdgcn_ds_bpermute((16 * g + rl) * 4, row);
    const float* const p = src + (r >= 0 ? (int64_t)r * Rk : absent) + c0;
#pragma unroll
    for (int s = 0; s < TC; ++s)
      nx[g][s] = VEC ? *reinterpret_cast<const v4f*>(p + 16 * s)
                     : *reinterpret_cast<const v4f_any*>(p + 16 * s);
  }
}

// A step's 64 rows pass through 4 KB of LDS into the MFMA layout: lane
// (n32, h) of row tile rt holds row 32 rt + n32, channels 16 s + 8 h + 0..7.
// Piece p of row 16 g + rl sits at g*1024 + rl*64 + 16*(p ^ ((rl >> 1) & 3)):
// the exchange of pieces (made on the addresses loaded from) puts the eight
// rows that a read serves at once on different banks.
struct Turn {
  int wr, rd0, rd1;  // byte offsets: lane's write; reads of the two halves
  __device__ inline explicit Turn(int lane) {
    const int n32 = lane & 31, h = lane >> 5, rr = n32 & 15, sw = (rr >> 1) & 3;
    wr = lane * 16;
    rd0 = (n32 >> 4) * 1024 + rr * 64 + 16 * ((2 * h) ^ sw);
    rd1 = (n32 >> 4) * 1024 + rr * 64 + 16 * ((2 * h + 1) ^ sw);
  }
};

// Reads one row tile of a step, shifts and splits it; NEG: times sgn (1 or
// -1), with g0 and g1 already so.
template <bool SUB, bool NEG>
__device__ inline Frag3 turn_read(const char* b, const Turn& t, int rt, v4f g0, v4f g1,
                                  float sgn) {
  const v4f x0 = *reinterpret_cast<const v4f*>(b + rt * 2048 + t.rd0);
  const v4f x1 = *reinterpret_cast<const v4f*>(b + rt * 2048 + t.rd1);
  float v[8];
#pragma unroll
  for (int z = 0; z < 4; ++z) {
    v[z] = NEG ? fmaf(x0[z], sgn, -g0[z]) : SUB ? x0[z] - g0[z] : x0[z];
    v[4 + z] = NEG ? fmaf(x1[z], sgn, -g1[z]) : SUB ? x1[z] - g1[z] : x1[z];
  }
  return split8(v);
}

// One step: 2 x 2 tiles of 32 rows x 32 columns, products q0 .. q1 - 1 of the
// six, added to acc (FIRST: acc starts from zero).
template <bool FIRST, int q0 = 0, int q1 = SPLIT_PROD>
__device__ inline void step_products(v16f (&acc)[2][2], const v4u (&W)[2][3], const Frag3 (&X)[2]) {
  v16f zero;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero[r] = 0.f;
#pragma unroll
  for (int q = q0; q < q1; ++q)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
        acc[rt][ct] = mfma_bf16(W[ct][split_a(q)], X[rt].s[split_b(q)],
                                FIRST && q == q0 ? zero : acc[rt][ct]);
}

// Sums in two levels, of 64 channels of an offset (tile_wg_kernel; 32 in
// tile_split_kernel) and over these: a chain over all of a row's products
// would round with every one of their MFMAs.  An item's ten small products
// come before its two large ones, so that a sum's first ones round while it is
// still small.  Error of the benchmark's input gradient against 64-bit sums:
// 3.1e-7 in one chain, 1.45e-7 in two levels without that order, 1.52e-7 in
// levels of 32 channels, 1.33e-7 as it is, 1.42e-7 on the fp32 instruction.
// The matrix core drops the bits of small addends below its adder, always
// downwards; odd offsets' weights are packed negated and their sums
// subtracted, so that these drifts cancel as well.
__device__ inline void add_item(v16f (&acc)[2][2], const v16f (&part)[2][2], int k) {
  const float sgn = k & 1 ? -1.f : 1.f;
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        acc[rt][ct][r] = fmaf(part[rt][ct][r], sgn, acc[rt][ct][r]);
}

// STREAM: written past the caches (a large layer's output is read only by
// later calls: 2.70 -> 2.60 ms for the forward of the benchmark's layer).
template <bool SORTED, bool STREAM>
__device__ inline void put4(const TileArgs& a, int64_t pos, int col, v4f v) {
  if (pos >= a.nrows || col >= a.Nc) return;
  const bool dvec = (a.Nc & 3) == 0 && (reinterpret_cast<uintptr_t>(a.dst) & 15) == 0;
  const int64_t drow = SORTED ? (int64_t)a.fperm[pos] : a.wmap ? (int64_t)a.wmap[pos] : pos;
  float* const dp = a.dst + drow * a.Nc + col;
#pragma unroll
  for (int z = 0; z < 4; ++z) {
    if (a.add && col + z < a.Nc) v[z] += a.add[col + z];
    if (a.relu) v[z] = v[z] > 0.f ? v[z] : 0.f;
  }
  if (dvec) {
    if (STREAM)
      __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(dp));
    else
      *reinterpret_cast<v4f*>(dp) = v;
  } else {
#pragma unroll
    for (int z = 0; z < 4; ++z)
      if (col + z < a.Nc) dp[z] = v[z];
  }
}

// 0 if a quarter's sums are finite, else NaN
__device__ inline float not_finite(const v16f& e) {
  float t = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) t = fmaf(e[r], 0.f, t);
  return t;
}
// Whether column `lane` of a column block is tiny.
__device__ inline bool column_tiny(const TileArgs& a, int cb, int lane) {
  return a.wtiny[min(64 * cb + lane, a.Nc - 1)] != 0;
}

// The registers of a quarter whose row (the lane's) or column is tiny; cols:
// bit c of column 32 ct + c.
__device__ inline uint32_t tiny_sums(bool row, uint32_t cols, int lane) {
  uint32_t m = cols >> 4 * (lane >> 5) & 0x0f0f0f0fu;  // columns 8 j + 4 h + z
  m = (m | m >> 4) & 0x00ff00ffu;
  return row ? 0xffffu : (m | m >> 8) & 0xffffu;
}
// The largest sum that a tiny row can have at a column.
__device__ inline float row_limit(const TileArgs& a, int col) {
  return __uint_as_float(a.wtiny[a.Nc + min(col, a.Nc - 1)]);
}
// The rows of a quarter (bit n32) that have a sum but zero, and one too large for
// a tiny row; limit(c): of the quarter's column c.
struct RowSums {
  uint32_t any, big;
};
template <class Limit>
__device__ inline RowSums row_sums(const v16f& e, int lane, Limit limit) {
  bool any = false, big = false;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    any |= e[r] != 0.f;
    const float l = limit(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3));  // all lanes take part
    big |= fabsf(e[r]) > l;
    __builtin_amdgcn_sched_barrier(0);  // seldom run: one limit in registers at a time
  }
  const uint64_t m = __ballot(any), b = __ballot(big);
  return {(uint32_t)(m | m >> 32), (uint32_t)(b | b >> 32)};
}

// the registers of a quarter that are not finite
__device__ inline uint32_t bad_sums(const v16f& e) {
  uint32_t m = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) m |= e[r] * 0.f == 0.f ? 0u : 1u << r;
  return m;
}

// Computes sums of a 32 x 32 quarter of a tile again on the fp32 matrix
// instruction and writes those that `bad` names: where a sum is not finite, the
// operands held an infinity, a NaN or a value past bf16's range (or the sum
// itself overflows); where a row or a column is tiny, its low parts are lost
// (split.h).  A lane holds row 32 rt + n32 and, in register 4 j + z,
// column 64 cb + 32 ct + 8 j + 4 h + z; each offset's products are summed by
// themselves and added for the rows that have it, so that a weight that is not
// finite reaches those rows only.  Runs after the tile's own stores, when its
// accumulators need no registers any more (kept beside them, this seldom run
// code cost the kernels a third of their waves).  An input gradient (64 ->
// 64, 90k sites) whose every sum is NaN takes 590 us, a finite one 97, one with
// a NaN weight 350; a first layer's forward (1M outputs) 1.26 ms, 0.15, 0.75.
template <bool SUB, bool SORTED>
__device__ inline void redo_quarter(const TileArgs& a, const Rows<SORTED>& R, int rt, int ct,
                                    int cb, int lane, uint32_t bad) {
  const int n32 = lane & 31, h = lane >> 5, col0 = 64 * cb + 32 * ct;
  const float* const Wc = a.W + min(col0 + n32, a.Nc - 1) * a.wn;
  v16f e;
#pragma unroll
  for (int r = 0; r < 16; ++r) e[r] = 0.f;
  uint32_t rest = R.U;
  while (rest) {
    const int k = __builtin_ctz(rest);
    rest &= rest - 1;
    const int row = __builtin_amdgcn_ds_bpermute((32 * rt + n32) * 4, R.row(R.load(k, lane), k));
    const float* const xp = a.src + (int64_t)max(row, 0) * a.Rk;
    const float* const wp = Wc + k * a.wk;
    v16f part;
#pragma unroll
    for (int r = 0; r < 16; ++r) part[r] = 0.f;
#pragma unroll 1
    for (int j0 = 0; j0 < a.Rk; j0 += 8) {
      float x[4], w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + 2 * u + h, jj = min(j, a.Rk - 1);
        x[u] = SUB ? xp[jj] - a.sub[jj] : xp[jj];
        w[u] = wp[jj * a.wj];
        x[u] = j < a.Rk ? x[u] : 0.f;
        w[u] = j < a.Rk ? w[u] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        part = __builtin_amdgcn_mfma_f32_32x32x2f32(w[u], x[u], part, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) e[r] = row >= 0 ? e[r] + part[r] : e[r];
  }
  const int64_t pos = R.row0 + 32 * rt + n32;
  if (pos >= a.nrows) return;
  float* const dp = a.dst + (SORTED ? (int64_t)a.fperm[pos] : a.wmap ? (int64_t)a.wmap[pos] : pos) *
                                a.Nc;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int col = col0 + 8 * (r >> 2) + 4 * h + (r & 3);
    if (col < a.Nc && (bad >> r & 1)) {
      float v = e[r];
      if (a.add) v += a.add[col];
      dp[col] = a.relu && !(v > 0.f) ? 0.f : v;
    }
  }
}

// Work items are contiguous per XCD (work-groups are dispatched round-robin
// over the eight), so that neighbouring tiles share its L2.
__device__ inline int64_t xcd_item(int64_t b, int64_t n) {
  const int64_t x = b & 7, j = b >> 3, base = n >> 3, rem = n & 7;
  return x * base + min(x, rem) + j;
}

// The accumulators leave through LDS (ob, the wave's own), 32 rows at a time,
// so that a store instruction writes whole rows, 16 lanes each: 16-byte pieces
// of 32 rows at a time cost the 1.1 GB output of the benchmark's layer 0.56 ms.
constexpr int OUT_LD = 68;                 // floats per row
constexpr int OUT_B = 32 * OUT_LD * 4;     // bytes of ob
template <bool SUB, bool SORTED>
__device__ inline void store_tile(const TileArgs& a, const Rows<SORTED>& R,
                                  const v16f (&acc)[2][2], uint64_t tiny_cols, float* ob,
                                  int cb, int lane) {
  // A row is not tiny if one of its sums is too large for that; the first column's
  // mostly are.
  const float limit = row_limit(a, 64 * cb + lane);
  const float first = __shfl(limit, 4 * (lane >> 5), 64);
  const uint64_t big0 = __ballot(fabsf(acc[0][0][0]) > first);
  const uint64_t big1 = __ballot(fabsf(acc[1][0][0]) > first);
  uint64_t tiny_rows = 0;
  if (__builtin_expect(~((uint32_t)(big0 | big0 >> 32) & (uint32_t)(big1 | big1 >> 32)), 0)) {
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const RowSums l = row_sums(acc[rt][0], lane, [&](int c) { return __shfl(limit, c, 64); });
      const RowSums r =
          row_sums(acc[rt][1], lane, [&](int c) { return __shfl(limit, 32 + c, 64); });
      tiny_rows |= (uint64_t)((l.any | r.any) & ~(l.big | r.big)) << 32 * rt;
    }
  }
  const bool redo = tiny_rows || tiny_cols ||
                    __ballot(!(not_finite(acc[0][0]) + not_finite(acc[0][1]) +
                                   not_finite(acc[1][0]) + not_finite(acc[1][1]) == 0.f)) != 0;
  uint32_t bad0 = 0, bad1 = 0;  // 16 bits per quarter
  if (__builtin_expect(redo, 0)) {
    const bool row0 = tiny_rows >> (lane & 31) & 1, row1 = tiny_rows >> (32 + (lane & 31)) & 1;
    const uint32_t col0 = (uint32_t)tiny_cols, col1 = (uint32_t)(tiny_cols >> 32);
    bad0 = bad_sums(acc[0][0]) | tiny_sums(row0, col0, lane) |
           (bad_sums(acc[0][1]) | tiny_sums(row0, col1, lane)) << 16;
    bad1 = bad_sums(acc[1][0]) | tiny_sums(row1, col0, lane) |
           (bad_sums(acc[1][1]) | tiny_sums(row1, col1, lane)) << 16;
  }
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    wave_sync();
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *reinterpret_cast<v4f*>(ob + (lane & 31) * OUT_LD + 32 * ct + 8 * j + 4 * (lane >> 5)) =
            v4f{acc[rt][ct][4 * j], acc[rt][ct][4 * j + 1], acc[rt][ct][4 * j + 2],
                acc[rt][ct][4 * j + 3]};
    wave_sync();
    const int col = 64 * cb + 4 * (lane & 15);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = 4 * i + (lane >> 4);
      put4<SORTED, SORTED>(a, R.row0 + 32 * rt + r, col,
                           *reinterpret_cast<const v4f*>(ob + r * OUT_LD + 4 * (lane & 15)));
    }
  }
  if (__builtin_expect(redo, 0)) {
    __threadfence();  // the stores that are replaced come from other lanes
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      const uint32_t bad = ((q >> 1 ? bad1 : bad0) >> 16 * (q & 1)) & 0xffffu;
      if (__ballot(bad != 0)) redo_quarter<SUB, SORTED>(a, R, q >> 1, q & 1, cb, lane, bad);
    }
  }
}

// Large layers: four waves, a tile of 64 rows each, walk the same items; the
// item's weights are loaded into LDS once for all of them, an item ahead, and
// so are each step's rows into registers.  Two or three work-groups per CU:
// one's splits, waits, prologue and stores run under the others' products.
// TC: 16-channel steps per item.  VEC: pieces of rows are 16-byte
// aligned.  SUB: rows are shifted by a.sub.  SORTED: rows from the dense
// forward view, else from pair lists; its sums run in one chain (3.1e-7 off
// 64-bit sums on the benchmark's layer, as before it 3.7e-7), the lists' in
// two levels.
constexpr int WGW = 4;              // waves per work-group
constexpr size_t wg_lds(int tc) {
  return std::max<size_t>((size_t)tc * 12288 + WGW * 4096, (size_t)WGW * OUT_B);
}
template <int TC, bool VEC, bool SUB, bool SORTED>
__global__ void __launch_bounds__(64 * WGW, SORTED ? 3 : 2) tile_wg_kernel(TileArgs a, int nchunk, int ncb) {
  extern __shared__ char smem[];
  constexpr int WB = TC * 6144;                    // bytes of an item's weights
  constexpr int NR = TC * 384 / (64 * WGW);        // ... 16-byte pieces per thread
  constexpr int NX = TC * 384 % (64 * WGW);        // ... and threads with one more
  char* const wbuf = smem;                         // [2][WB]
  uint32_t* const ush = reinterpret_cast<uint32_t*>(smem + wg_lds(TC));
  float* const gsh = reinterpret_cast<float*>(smem + wg_lds(TC) + 64);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  char* const buf = smem + 2 * WB + w * 4096;      // one step of the wave's rows
  const int rl = lane >> 2, piece = (lane & 3) ^ ((rl >> 1) & 3);
  const int nst = nchunk * TC;
  if (SUB)
    for (int c = tid; c < 16 * nst; c += 64 * WGW)
      gsh[c] = a.sub[Entries(a.Rk, 16 * TC).channel(c)];
  const int64_t u = xcd_item(blockIdx.x, gridDim.x);
  const int64_t grp = u / ncb;
  const int cb = (int)(u - grp * ncb);
  const int64_t tile = min(grp * WGW + w, a.ntile - 1);
  const bool live = grp * WGW + w < a.ntile;
  const bool wtiny = column_tiny(a, cb, lane);
  Rows<SORTED> R;
  R.init(a, tile, lane);
  const uint64_t tiny_cols = __ballot(wtiny);
  if (lane == 0) ush[w] = R.U;
  __syncthreads();
  uint32_t U = 0;
#pragma unroll
  for (int i = 0; i < WGW; ++i) U |= ush[i];
  U = (uint32_t)__builtin_amdgcn_readfirstlane((int)U);

  const float* const src = a.src;
  const int Rk = a.Rk;
  const Turn turn(lane);
  const v4u* const Wb = reinterpret_cast<const v4u*>(a.Wp);
  v4u wr[NR + (NX > 0)];  // weights on their way to LDS
  auto wload = [&](const Item& t) {
    const v4u* p = Wb + (((int64_t)t.k * ncb + cb) * nst + t.ch * TC) * 384;
#pragma unroll
    for (int i = 0; i < NR; ++i) wr[i] = p[tid + 64 * WGW * i];
    if (NX) wr[NR] = p[64 * WGW * NR + min(tid, NX - 1)];
  };
  auto wstore = [&](char* b) {
#pragma unroll
    for (int i = 0; i < NR; ++i)
      *reinterpret_cast<v4u*>(b + (tid + 64 * WGW * i) * 16) = wr[i];
    if (NX && tid < NX) *reinterpret_cast<v4u*>(b + (tid + 64 * WGW * NR) * 16) = wr[NR];
  };
  // Where the lane gathers from, in the load layout: the row's piece, or that of
  // `sub` for a row without the offset.  The product is taken where a lane knows one
  // row, not after the spread, where it knows four (VEC: in 16-byte units).
  struct From {
    const float* p[4];
  };
  const int limit = piece_limit(piece, Rk, 16 * TC);
  auto spread = [&](int row, int ch) -> From {
    From q;
    const int c0 = min(16 * TC * ch + 4 * piece, limit);
    const int at = VEC ? (row < 0 ? -1 : (int)((uint32_t)row * (uint32_t)(Rk >> 2))) : row;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int v = __builtin_amdgcn_ds_bpermute((16 * g + rl) * 4, at);
      const float* const f = VEC ? src + ((int64_t)(uint32_t)v << 2) : src + (int64_t)v * Rk;
      q.p[g] = (v == -1 ? a.sub : f) + c0;
    }
    return q;
  };
  v4f nx[4][TC];  // rows on their way to LDS
  auto gather = [&](const From& q, int s) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      nx[g][s] = VEC ? *reinterpret_cast<const v4f*>(q.p[g] + 16 * s)
                     : *reinterpret_cast<const v4f_any*>(q.p[g] + 16 * s);
  };
  auto commit = [&](int s) {
    wave_sync();
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<v4f*>(buf + g * 1024 + turn.wr) = nx[g][s];
    wave_sync();
  };
  v16f acc[2][2], part[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nit = __builtin_popcount(U) * nchunk;
  if (nit > 0) {
    Item c{__builtin_ctz(U), 0, U & (U - 1)};
    Item n = c;
    n.advance(nchunk);
    Item n2 = n;
    n2.advance(nchunk);
    const Idx xc = R.load(c.k, lane);
    Idx xn = R.load(n.k, lane);
    wload(c);
    {
      const From q = spread(R.row(xc, c.k), c.ch);
#pragma unroll
      for (int s = 0; s < TC; ++s) gather(q, s);
    }
    wstore(wbuf);
    wload(n);
    __syncthreads();
    // drained once, so that the waits in the loop follow from its own loads
    __builtin_amdgcn_s_waitcnt(0);
    for (int it = 0; it < nit; ++it) {
      const char* const wl = wbuf + (it & 1) * WB + lane * 16;
      // the other half held the item before, which every wave has left
      wstore(wbuf + ((it & 1) ^ 1) * WB);
      wload(n2);
      const From qn = spread(R.row(xn, n.k), n.ch);
      xn = R.load(n2.k, lane);
      // lists: sums of two items of an offset
      const bool first = SORTED || TC == 1 || !(c.ch & 1);
      Frag3 X[TC][2];
      v4u Wf[TC][2][3];
#pragma unroll
      for (int s = 0; s < TC; ++s) {
        commit(s);
        gather(qn, s);
        v4f g0 = {}, g1 = {};
        if (SUB) {
          const float* gp = gsh + 16 * (TC * c.ch + s) + 8 * (lane >> 5);
          g0 = *reinterpret_cast<const v4f*>(gp);
          g1 = *reinterpret_cast<const v4f*>(gp + 4);
        }
        // one chain (SORTED) needs odd offsets' rows negated like their weights
        const float sgn = SORTED && (c.k & 1) ? -1.f : 1.f;
        if (SORTED) {
          g0 *= sgn;
          g1 *= sgn;
        }
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
          X[s][rt] = turn_read<SUB, SORTED>(buf, turn, rt, g0, g1, sgn);
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
          for (int q = 0; q < 3; ++q)
            Wf[s][ct][q] = *reinterpret_cast<const v4u*>(wl + ((s * 2 + ct) * 3 + q) * 1024);
        if (SORTED)
          step_products<false>(acc, Wf[s], X[s]);
        else if (s == 0 && first)
          step_products<true, 0, SPLIT_PROD - 1>(part, Wf[s], X[s]);
        else
          step_products<false, 0, SPLIT_PROD - 1>(part, Wf[s], X[s]);
      }
      if (!SORTED) {
#pragma unroll
        for (int s = 0; s < TC; ++s)
          step_products<false, SPLIT_PROD - 1, SPLIT_PROD>(part, Wf[s], X[s]);
        if (TC == 1 || (c.ch & 1) || c.ch == nchunk - 1) add_item(acc, part, c.k);
      }
      c = n;
      n = n2;
      n2.advance(nchunk);
      __syncthreads();
    }
  }
  if (!live) return;
  store_tile<SUB, SORTED>(a, R, acc, tiny_cols, reinterpret_cast<float*>(smem + w * OUT_B), cb,
                          lane);
}

// Small layers: the four waves of a work-group share one tile and take every
// fourth item, with their own weights from L2; their sums are added in wave
// order.
template <int TC, bool VEC, bool SUB, bool SORTED>
__global__ void __launch_bounds__(NT, 2) tile_split_kernel(TileArgs a, int nchunk,
                                                                     int ncb) {
  extern __shared__ char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rl = lane >> 2, piece = (lane & 3) ^ ((rl >> 1) & 3);
  constexpr int GOFF = 65536;
  char* const buf = smem + w * 16384;
  const int nst = nchunk * TC;
  float* const gsh = reinterpret_cast<float*>(smem + GOFF);
  if (SUB) {
    for (int c = tid; c < 16 * nst; c += NT) gsh[c] = a.sub[Entries(a.Rk, 16 * TC).channel(c)];
    __syncthreads();
  }
  const int64_t u = xcd_item(blockIdx.x, gridDim.x);
  const int64_t tile = u / ncb;
  const int cb = (int)(u - tile * ncb);
  Rows<SORTED> R;
  R.init(a, tile, lane);
  // the columns' limits and whether they are tiny, for the end
  uint32_t* const limits = reinterpret_cast<uint32_t*>(smem + GOFF + 1024);
  if (tid < 128) {
    const int n = min(64 * cb + (tid & 63), a.Nc - 1);
    limits[tid] = a.wtiny[tid < 64 ? a.Nc + n : n];
  }
  const uint32_t U = R.U;
  const float* const src = a.src;
  const int Rk = a.Rk;
  const int64_t absent = a.sub - a.src;  // where rows without the offset read
  const Turn turn(lane);

  struct WSet {
    v4u f[2][3];
  };
  const v4u* const Wb = reinterpret_cast<const v4u*>(a.Wp) + lane;
  auto wload = [&](const Item& t, int s, WSet& A) {
    const v4u* p = Wb + (((int64_t)t.k * ncb + cb) * nst + (t.ch * TC + s)) * 384;
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int q = 0; q < 3; ++q) A.f[ct][q] = p[(ct * 3 + q) * 64];
  };
  v16f acc[2][2], part[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto mult = [&](int s, int ch, const WSet& A) {
    Frag3 X[2];
    v4f g0 = {0.f, 0.f, 0.f, 0.f}, g1 = g0;
    if (SUB) {
      const float* gp = gsh + 16 * (TC * ch + s) + 8 * (lane >> 5);
      g0 = *reinterpret_cast<const v4f*>(gp);
      g1 = *reinterpret_cast<const v4f*>(gp + 4);
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) X[rt] = turn_read<SUB, false>(buf + s * 4096, turn, rt, g0, g1, 1.f);
    if (s == 0)
      step_products<true>(part, A.f, X);
    else
      step_products<false>(part, A.f, X);
  };

  auto step_item = [&](Item t) -> Item {
#pragma unroll
    for (int i = 0; i < 4; ++i) t.advance(nchunk);
    return t;
  };
  const int cnt = (__builtin_popcount(U) * nchunk - w + 3) >> 2;
  if (cnt > 0) {
    Item c{__builtin_ctz(U), 0, U & (U - 1)};
    for (int i = 0; i < w; ++i) c.advance(nchunk);
    Item n = step_item(c), nn = step_item(n);
    WSet A[TC];
    v4f nx[4][TC];
    const Idx xc = R.load(c.k, lane);
    Idx xn = R.load(n.k, lane);
    gather_rows<TC, VEC>(nx, src, Rk, absent, R.row(xc, c.k), c.ch, rl, piece);
#pragma unroll
    for (int s = 0; s < TC; ++s) wload(c, s, A[s]);
    __builtin_amdgcn_sched_barrier(0);
    for (int it = 0; it < cnt; ++it) {
      wave_sync();
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int s = 0; s < TC; ++s)
          *reinterpret_cast<v4f*>(buf + s * 4096 + g * 1024 + turn.wr) = nx[g][s];
      wave_sync();
      // Loads return in order, so a wait for one waits for all before it: the
      // next item's rows and the indices after them are issued ahead of its
      // weights, so that no wait for weights drains them early.
      __builtin_amdgcn_sched_barrier(0);
      gather_rows<TC, VEC>(nx, src, Rk, absent, R.row(xn, n.k), n.ch, rl, piece);
      xn = R.load(nn.k, lane);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < TC; ++s) {
        mult(s, c.ch, A[s]);
        __builtin_amdgcn_sched_barrier(0);
        wload(n, s, A[s]);
        __builtin_amdgcn_sched_barrier(0);
      }
      add_item(acc, part, c.k);
      c = n;
      n = nn;
      nn = step_item(nn);
    }
  }

  // quarter j = 2 rt + ct of the tile goes to wave j, which adds the four
  // waves' sums in wave order
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const v16f& q = acc[j >> 1][j & 1];
      *reinterpret_cast<v4f*>(smem + ((j * 4 + w) * 4 + r) * 1024 + lane * 16) =
          v4f{q[4 * r], q[4 * r + 1], q[4 * r + 2], q[4 * r + 3]};
    }
  __syncthreads();
  v16f e;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    v4f s = *reinterpret_cast<const v4f*>(smem + ((w * 4 + 0) * 4 + r) * 1024 + lane * 16);
#pragma unroll
    for (int v = 1; v < 4; ++v)
      s += *reinterpret_cast<const v4f*>(smem + ((w * 4 + v) * 4 + r) * 1024 + lane * 16);
#pragma unroll
    for (int z = 0; z < 4; ++z) e[4 * r + z] = s[z];
  }
  // as in store_tile
  const float* const lim = reinterpret_cast<const float*>(limits) + 32 * (w & 1);
  const uint64_t tiny_cols = __ballot(limits[64 + lane] != 0);
  const uint64_t big = __ballot(fabsf(e[0]) > lim[4 * (lane >> 5)]);
  uint32_t tiny_rows = 0;
  if (__builtin_expect(~(uint32_t)(big | big >> 32), 0)) {
    const RowSums sums = row_sums(e, lane, [&](int c) { return lim[c]; });
    tiny_rows = sums.any & ~sums.big;
  }
  const uint32_t bad = bad_sums(e) | tiny_sums(tiny_rows >> (lane & 31) & 1,
                                               (uint32_t)(tiny_cols >> 32 * (w & 1)), lane);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    put4<SORTED, false>(a, R.row0 + 32 * (w >> 1) + (lane & 31),
                 64 * cb + 32 * (w & 1) + 8 * j + 4 * (lane >> 5),
                 v4f{e[4 * j], e[4 * j + 1], e[4 * j + 2], e[4 * j + 3]});
  if (__builtin_expect(__ballot(bad != 0) != 0, 0)) {
    __threadfence();  // as in store_tile
    redo_quarter<SUB, SORTED>(a, R, w >> 1, w & 1, cb, lane, bad);
  }
}

// ---------------------------------------------------------------------------
// Few input channels (a network's first layer): the offsets join the
// reduction.  A row's window values, x - g_in at j = k Cin + c and zero where
// the offset is absent, make one reduction of J = K Cin entries (27 for a
// 3x3x3 filter on one channel) against W as the J x Cout matrix it is; with
// 16-channel steps per offset, 15 of 16 products were padding.  The forward is
// then bound by its output (1.8M rows x 64: 0.46 GB), the weight gradient by
// reading dy (and y), each once.
// ---------------------------------------------------------------------------
constexpr int FEW_C = 4, FEW_J = 96;

// V(row, j) of the wave's tile: v[row * ldr + j * ldj], times sgn; zeroed first.
// All channels of eight offsets' rows are on their way together: with a round
// of loads for each channel, a layer of three channels waited three times
// (3 -> 32 channels on 1.4M tetrahedral outputs, ten offsets: 350 -> 247 us).
// REDO: a NaN is stored as any but ABSENT, which few_values fills in first.
constexpr uint32_t ABSENT = 0xffffffffu;
template <bool SORTED, int C, bool REDO>
__device__ inline void few_rows(const TileArgs& a, const Rows<SORTED>& R, float* v, int ldr,
                                int ldj, float sgn, int lane) {
  float g[C];
#pragma unroll
  for (int c = 0; c < C; ++c) g[c] = a.sub[c];
  uint32_t rest = R.U;
  while (rest) {
    // eight offsets at a time, so that their loads overlap (past the last one
    // it is repeated: the same value again)
    int k[8], r[8];
    Idx x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      k[i] = rest ? __builtin_ctz(rest) : k[i ? i - 1 : 0];
      rest &= rest - 1;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = R.load(k[i], lane);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = R.row(x[i], k[i]);
    float t[8][C];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int c = 0; c < C; ++c) t[i][c] = a.src[(int64_t)max(r[i], 0) * C + c];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (r[i] >= 0) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const float d = sgn * (t[i][c] - g[c]);
          v[lane * ldr + (k[i] * C + c) * ldj] = REDO && d != d ? __uint_as_float(0x7fc00000u) : d;
        }
      }
  }
}

template <bool SORTED, bool REDO = false>
__device__ inline void few_values(const TileArgs& a, const Rows<SORTED>& R, float* v, int ldr,
                                  int ldj, int words, float sgn, int lane) {
  for (int i = lane; i < words / 4; i += 64)
    reinterpret_cast<v4u*>(v)[i] = REDO ? v4u{ABSENT, ABSENT, ABSENT, ABSENT} : v4u{0, 0, 0, 0};
  wave_sync();
  switch (a.Rk) {
    case 1: few_rows<SORTED, 1, REDO>(a, R, v, ldr, ldj, sgn, lane); break;
    case 2: few_rows<SORTED, 2, REDO>(a, R, v, ldr, ldj, sgn, lane); break;
    case 3: few_rows<SORTED, 3, REDO>(a, R, v, ldr, ldj, sgn, lane); break;
    default: few_rows<SORTED, 4, REDO>(a, R, v, ldr, ldj, sgn, lane); break;
  }
  wave_sync();
}

__host__ __device__ constexpr int few_lds(int nst, int ncb) {
  const int v = 256 * (16 * nst + 4);
  return ncb > 1 ? v + OUT_B : v > OUT_B ? v : OUT_B;
}

template <bool SORTED>
__global__ void __launch_bounds__(64 * WGW, 3) few_fwd_kernel(TileArgs a, int nst, int ncb) {
  extern __shared__ char smem[];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ldr = 16 * nst + 4;
  const int64_t tile = xcd_item(blockIdx.x, gridDim.x) * WGW + w;
  if (tile >= a.ntile) return;
  float* const v = reinterpret_cast<float*>(smem + w * few_lds(nst, ncb));
  // one column block: the values' room is free when the tile leaves
  float* const ob = ncb == 1 ? v : v + 64 * ldr;
  Rows<SORTED> R;
  R.init(a, tile, lane);
  few_values<SORTED>(a, R, v, ldr, 1, 64 * ldr, 1.f, lane);
  const int n32 = lane & 31, h = lane >> 5;
  for (int cb = 0; cb < ncb; ++cb) {
    const v4u* wp = reinterpret_cast<const v4u*>(a.Wp) + (int64_t)cb * nst * 384 + lane;
    v16f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    // The small products of all steps first, in one chain.  Then each step's
    // large products, summed from zero and added in the vector unit, which
    // rounds to nearest where the matrix core truncates; every second step's
    // are negated and subtracted, so that what is left of its drift cancels.
    // (In one chain over all products the error of a 3x3x3 layer of three
    // channels was 9.1e-8 against 64-bit sums, 6.0e-8 to 7.7e-8 on the fp32
    // instruction; 3.6e-8 as it is.)
#pragma unroll 1
    for (int s = 0; s < nst; ++s) {
      v4u Wf[2][3];
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int q = 0; q < 3; ++q) Wf[ct][q] = wp[(s * 6 + ct * 3 + q) * 64];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const float* p = v + (32 * rt + n32) * ldr + 16 * s + 8 * h;
        const v4f p0 = *reinterpret_cast<const v4f*>(p), p1 = *reinterpret_cast<const v4f*>(p + 4);
        const float e[8] = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
        const Frag3 X = split8(e);
#pragma unroll
        for (int q = 0; q < SPLIT_PROD - 1; ++q)
#pragma unroll
          for (int ct = 0; ct < 2; ++ct)
            acc[rt][ct] = mfma_bf16(Wf[ct][split_a(q)], X.s[split_b(q)], acc[rt][ct]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll 1
    for (int s = 0; s < nst; ++s) {
      const uint32_t neg = s & 1 ? 0x80008000u : 0u;
      const float sgn = s & 1 ? -1.f : 1.f;
      v4u Wh[2];
#pragma unroll
      for (int ct = 0; ct < 2; ++ct) Wh[ct] = wp[(s * 6 + ct * 3) * 64];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const float* p = v + (32 * rt + n32) * ldr + 16 * s + 8 * h;
        const v4f p0 = *reinterpret_cast<const v4f*>(p), p1 = *reinterpret_cast<const v4f*>(p + 4);
        const v4u X = {cvt2_bf16(p0[0], p0[1]) ^ neg, cvt2_bf16(p0[2], p0[3]) ^ neg,
                       cvt2_bf16(p1[0], p1[1]) ^ neg, cvt2_bf16(p1[2], p1[3]) ^ neg};
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          v16f zero;
#pragma unroll
          for (int r = 0; r < 16; ++r) zero[r] = 0.f;
          const v16f t = mfma_bf16(Wh[ct], X, zero);
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[rt][ct][r] = fmaf(t[r], sgn, acc[rt][ct][r]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    store_tile<true, SORTED>(a, R, acc, __ballot(column_tiny(a, cb, lane)), ob, cb, lane);
  }
}

// dW partials and column sums of dy (masked by y > 0 under ReLU) of one 64
// column block: every wave takes tiles in turn, JT tiles of 32 reduction
// entries by 64 columns in registers; a work-group adds its four waves' sums.
// Odd waves sum the negated products (see dw_partial_kernel).
struct FewArgs {
  TileArgs t;          // rows of x; nrows, ntile of the outputs
  const float *dy, *y; // [nrows][Cout]; y null without ReLU
  int Cout, J;
  float* part;         // [work-groups][J][Cout]
  float* partS;        // [work-groups][Cout]
};

template <int JT, bool SORTED, bool V4>
__global__ void __launch_bounds__(64 * WGW, JT == 1 ? 3 : 2) few_dw_kernel(FewArgs f) {
  extern __shared__ char smem[];
  const TileArgs& a = f.t;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pg = lane >> 4, cq = lane & 15, n32 = lane & 31, h = lane >> 5;
  constexpr int LDJ = 68;  // floats per reduction entry: 64 rows and padding
  float* const v = reinterpret_cast<float*>(smem) + w * (32 * JT * LDJ);
  const int co0 = 64 * blockIdx.y;
  const float sgn = w & 1 ? -1.f : 1.f;
  int cd[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    cd[e] = V4 ? min(co0 + 4 * cq, f.Cout - 4) + e : min(co0 + 4 * cq + e, f.Cout - 1);
  v16f acc[JT][2];
#pragma unroll
  for (int i = 0; i < JT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  v4f tsum = {0.f, 0.f, 0.f, 0.f};
  Seen entries[JT], cols[2];  // (split.h)
  for (int64_t tile = (int64_t)blockIdx.x * WGW + w; tile < a.ntile;
       tile += (int64_t)gridDim.x * WGW) {
    Rows<SORTED> R;
    R.init(a, tile, lane);
    wave_sync();
    few_values<SORTED>(a, R, v, 1, LDJ, 32 * JT * LDJ, sgn, lane);
    struct Dy {
      v4f t[4], m[4];
    };
    auto load = [&](Dy& q, int st) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t p = min(R.row0 + 16 * st + 4 * pg + i, a.nrows - 1);
        const int64_t at = (SORTED ? (int64_t)a.fperm[p] : p) * f.Cout;
        if (V4) {
          q.t[i] = *reinterpret_cast<const v4f*>(f.dy + at + cd[0]);
          if (f.y) q.m[i] = *reinterpret_cast<const v4f*>(f.y + at + cd[0]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            q.t[i][e] = f.dy[at + cd[e]];
            if (f.y) q.m[i][e] = f.y[at + cd[e]];
          }
        }
      }
    };
    Dy q;
    load(q, 0);
#pragma unroll 1
    for (int st = 0; st < 4; ++st) {
      v4f d[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          d[i][e] = R.row0 + 16 * st + 4 * pg + i < a.nrows && (!f.y || q.m[i][e] > 0.f)
                        ? q.t[i][e] : 0.f;
      load(q, min(st + 1, 3));  // on its way during this stage's products
      // rows 16 st + 8 h + 0..7 of column 4 (m & 15) + 2 t + (m >> 4)
      v4u D[2][3];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          uint32_t p[3], u[3];
          split2(d[2 * j][2 * t], d[2 * j + 1][2 * t], p[0], p[1], p[2]);
          split2(d[2 * j][2 * t + 1], d[2 * j + 1][2 * t + 1], u[0], u[1], u[2]);
#pragma unroll
          for (int s = 0; s < 3; ++s) {
            const auto r = __builtin_amdgcn_permlane16_swap(p[s], u[s], false, false);
            D[t][s][j] = r[0];
            D[t][s][2 + j] = r[1];
          }
        }
#pragma unroll
      for (int i = 0; i < 4; ++i) tsum += d[i];
#pragma unroll
      for (int t = 0; t < 2; ++t) cols[t].add(D[t][0]);
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        const float* p = v + (32 * jt + n32) * LDJ + 16 * st + 8 * h;
        const v4f p0 = *reinterpret_cast<const v4f*>(p), p1 = *reinterpret_cast<const v4f*>(p + 4);
        const float e[8] = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
        const Frag3 X = split8(e);
        entries[jt].add(X.s[0]);
#pragma unroll
        for (int q = 0; q < SPLIT_PROD; ++q)
#pragma unroll
          for (int t = 0; t < 2; ++t)
            acc[jt][t] = mfma_bf16(X.s[split_a(q)], D[t][split_b(q)], acc[jt][t]);
      }
    }
  }
  // the four waves' sums, 32 reduction entries at a time
  float* const red = reinterpret_cast<float*>(smem);  // [4][32][64]
  float* const redT = red + 4 * 2048;                 // [4][64]
  float* const out = f.part + (int64_t)blockIdx.x * f.J * f.Cout;
  uint32_t* const seen = reinterpret_cast<uint32_t*>(redT + 256);  // [cols, entries][any, big][wave]
  bool odd = false;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float t1 = __shfl_xor(tsum[e], 16, 64);
    const float s1 = pg & 1 ? t1 + tsum[e] : tsum[e] + t1;
    const float t2 = __shfl_xor(s1, 32, 64);
    tsum[e] = s1 + t2;
  }
#pragma unroll
  for (int jt = 0; jt < JT; ++jt) {
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        red[w * 2048 + (8 * (r >> 2) + 4 * h + (r & 3)) * 64 + 4 * (n32 & 15) + 2 * t +
            (n32 >> 4)] = acc[jt][t][r];
    if (jt == 0 && pg == 0)
#pragma unroll
      for (int e = 0; e < 4; ++e) redT[w * 64 + 4 * cq + e] = tsum[e];
    if (jt == 0 && lane == 0) {
#pragma unroll
      for (int t = 0; t < 2 + JT; ++t) {
        seen[8 * t + w] = t < 2 ? cols[t & 1].any32() : entries[t < 2 ? 0 : t - 2].any32();
        seen[8 * t + 4 + w] = t < 2 ? cols[t & 1].big32() : entries[t < 2 ? 0 : t - 2].big32();
      }
    }
    __syncthreads();
    auto tiny = [&](int t) {
      const uint32_t* const sn = seen + 8 * t;
      return (sn[0] | sn[1] | sn[2] | sn[3]) & ~(sn[4] | sn[5] | sn[6] | sn[7]);
    };
    const bool tc = tiny(tid >> 1 & 1) >> (((tid & 63) >> 2) + 16 * (tid & 1)) & 1;
    const uint32_t te = tiny(2 + jt);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = u * 256 + tid, j = 32 * jt + e / 64, co = co0 + (tid & 63);
      const float t = (red[e] - red[2048 + e]) + (red[4096 + e] - red[6144 + e]);
      if (j < f.J && co < f.Cout) {
        // a sum to be redone is marked by a NaN
        const bool bad = !(t * 0.f == 0.f) || tc || (te >> e / 64 & 1);
        out[(int64_t)j * f.Cout + co] = bad ? __uint_as_float(0x7fc00000u) : t;
        odd = odd || bad;
      }
    }
    if (jt == 0 && tid < 64 && co0 + tid < f.Cout)
      f.partS[(int64_t)blockIdx.x * f.Cout + co0 + tid] =
          (redT[tid] + redT[64 + tid]) + (redT[128 + tid] + redT[192 + tid]);
  }
  // Sums of operands that the split cannot hold again, in fp32, a column per lane, from the rows that have the entry's offset.
  if (!__syncthreads_or(odd)) return;
  const int co = min(co0 + lane, f.Cout - 1);
#pragma unroll 1
  for (int jt = 0; jt < JT; ++jt) {
    float s[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) s[j] = 0.f;
#pragma unroll 1
    for (int64_t tile = (int64_t)blockIdx.x * WGW + w; tile < a.ntile;
         tile += (int64_t)gridDim.x * WGW) {
      Rows<SORTED> R;
      R.init(a, tile, lane);
      wave_sync();
      few_values<SORTED, true>(a, R, v, 1, LDJ, 32 * JT * LDJ, 1.f, lane);
      const int rows = (int)min<int64_t>(TILE, a.nrows - R.row0);
#pragma unroll 1
      for (int r = 0; r < rows; ++r) {
        const int64_t at = (SORTED ? (int64_t)a.fperm[R.row0 + r] : R.row0 + r) * f.Cout + co;
        const float d = !f.y || f.y[at] > 0.f ? f.dy[at] : 0.f;
        const float* const p = v + 32 * jt * LDJ + r;
#pragma unroll
        for (int j = 0; j < 32; ++j)
          s[j] = __float_as_uint(p[j * LDJ]) == ABSENT ? s[j] : fmaf(p[j * LDJ], d, s[j]);
      }
    }
    __syncthreads();  // every wave has read its values, or the sums before
#pragma unroll
    for (int j = 0; j < 32; ++j) red[w * 2048 + j * 64 + lane] = s[j];
    __syncthreads();
#pragma unroll 1
    for (int u = 0; u < 8; ++u) {
      const int e = u * 256 + tid, j = 32 * jt + e / 64, c = co0 + (tid & 63);
      if (j < f.J && c < f.Cout && !(out[(int64_t)j * f.Cout + c] * 0.f == 0.f))
        out[(int64_t)j * f.Cout + c] = (red[e] + red[2048 + e]) + (red[4096 + e] + red[6144 + e]);
    }
    __syncthreads();  // the next values are written where the sums stand
  }
}

// dW[j][co] = sum of the partials + g_in[c] u0[co].  A block covers FR_E
// elements; thread group g of FR_G sums the partials g (mod FR_G) in order,
// then the group sums are added in order, in 64 bits (up to 96 partials a
// thread: in 32 bits their roundings were most of dW's error on sums without
// cancellation, 7.0e-8 against 64-bit sums, 3.1e-8 now).
constexpr int FR_E = 32, FR_G = 8;
__global__ void __launch_bounds__(FR_E * FR_G) few_reduce_kernel(
    const float* __restrict__ part, int nwg, int64_t n, int Cout, int Cin,
    const float* __restrict__ g_in, const float* __restrict__ u0, float* __restrict__ dW) {
  __shared__ double sums[FR_G][FR_E];
  const int le = threadIdx.x % FR_E, g = threadIdx.x / FR_E;
  const int64_t i = (int64_t)blockIdx.x * FR_E + le;
  double d = 0.;
  if (i < n) {
#pragma unroll 4
    for (int c = g; c < nwg; c += FR_G) d += part[c * n + i];
  }
  sums[g][le] = d;
  __syncthreads();
  if (g || i >= n) return;
#pragma unroll
  for (int h = 1; h < FR_G; ++h) d += sums[h][le];
  dW[i] = (float)d + g_in[i / Cout % Cin] * u0[i % Cout];
}

typedef void (*TileFn)(TileArgs, int, int);

template <int TC, bool VEC>
TileFn pick_rows(bool sub, bool sorted, bool split) {
  if (sorted)
    return split ? tile_split_kernel<TC, VEC, true, true> : tile_wg_kernel<TC, VEC, true, true>;
  if (sub)
    return split ? tile_split_kernel<TC, VEC, true, false> : tile_wg_kernel<TC, VEC, true, false>;
  return split ? tile_split_kernel<TC, VEC, false, false> : tile_wg_kernel<TC, VEC, false, false>;
}

TileFn tile_fn(int tc, bool vec, bool sub, bool sorted, bool split) {
  if (tc == 1)
    return vec ? pick_rows<1, true>(sub, sorted, split) : pick_rows<1, false>(sub, sorted, split);
  return vec ? pick_rows<2, true>(sub, sorted, split) : pick_rows<2, false>(sub, sorted, split);
}

}  // namespace

int tile_steps(int Rk) { return (int)ceil_div(Rk, 16); }

// Split weights, then two words per column (wtiny).
static size_t pack_words(int K, int Rk, int Nc) {
  return (size_t)K * ceil_div(Nc, 64) * tile_steps(Rk) * 1536;
}
size_t tile_pack_bytes(int K, int Rk, int Nc) { return (pack_words(K, Rk, Nc) + 2 * Nc) * 4; }
const uint32_t* tile_wtiny(const uint32_t* Wp, int K, int Rk, int Nc) {
  return Wp + pack_words(K, Rk, Nc);
}

scn_status tile_pack(const float* W, int64_t wk, int64_t wj, int64_t wn, int K, int Rk, int Nc,
                     bool chunks, const float* g, int gm, const float* bias, int relu, uint32_t* Wp, float* sub,
                     float* g_pre, float* g_out, hipStream_t st) {
  const int nst = tile_steps(Rk), ncb = (int)ceil_div(Nc, 64);
  const int64_t n = std::max<int64_t>((int64_t)K * ncb * nst * 128, TILE_PAD);
  const int64_t np = ceil_div(n, NT), ng = ceil_div(Nc, PRE_COLS);
  hipLaunchKernelGGL(tile_pack_kernel, dim3((unsigned)(np + ng)), dim3(NT), 0, st, W, wk, wj, wn,
                     K, Rk, Nc, nst, ncb, Entries(Rk, chunks ? 16 * chunk_steps(Rk) : 1), g, gm, bias, relu, reinterpret_cast<v4u*>(Wp),
                     Wp + pack_words(K, Rk, Nc), sub, (int)np, g_pre, g_out);
  SCN_LAUNCH_CHECK();
  return SCN_OK;
}

scn_status launch_tile(const TileArgs& a, hipStream_t st) {
  if (a.nrows <= 0 || a.ntile <= 0) return SCN_OK;
  const int nst = tile_steps(a.Rk), ncb = (int)ceil_div(a.Nc, 64);
  // aligned pieces, and row starts in 16-byte units below 2^32 - 1
  const bool vec = (a.Rk & 3) == 0 && (reinterpret_cast<uintptr_t>(a.src) & 15) == 0 &&
                   a.nsrc * (a.Rk >> 2) < (int64_t)0xffffffff;
  const int64_t items = a.ntile * ncb;
  const bool split = items < TILE_SPLIT;
  const int tc = chunk_steps(a.Rk);
  // (split: g_in from 65536, the columns' limits from 66560)
  const size_t base = split ? 65536 : wg_lds(tc) + 64;
  const size_t smem = split ? base + 1024 + 512 : base + (size_t)nst * 64;
  TileFn fn = tile_fn(tc, vec, a.subtract, a.nb != nullptr, split);
  static LdsLimit limits[2][2][3][2];
  if (scn_status rc = allow_lds(reinterpret_cast<const void*>(fn),
                                limits[tc - 1][vec][a.nb ? 2 : a.subtract ? 1 : 0][split],
                                base + 1024 + 512))  // its largest size
    return rc;
  const int64_t nwg = split ? items : ceil_div(a.ntile, WGW) * ncb;
  hipLaunchKernelGGL(fn, dim3((unsigned)nwg), dim3(split ? NT : 64 * WGW), smem, st, a, nst / tc,
                     ncb);
  SCN_LAUNCH_CHECK();
  return SCN_OK;
}

bool few_channels(int K, int Cin) { return Cin <= FEW_C && K * Cin <= FEW_J; }

scn_status few_forward(const TileArgs& a, hipStream_t st) {
  if (a.nrows <= 0 || a.ntile <= 0) return SCN_OK;
  const int nst = tile_steps(a.K * a.Rk), ncb = (int)ceil_div(a.Nc, 64);
  const size_t smem = (size_t)WGW * few_lds(nst, ncb);  // at most 137 KB (6 steps)
  auto fn = a.nb ? few_fwd_kernel<true> : few_fwd_kernel<false>;
  static LdsLimit limits[2];
  if (scn_status rc = allow_lds(reinterpret_cast<const void*>(fn), limits[a.nb != nullptr], smem))
    return rc;
  hipLaunchKernelGGL(fn, dim3((unsigned)ceil_div(a.ntile, WGW)), dim3(64 * WGW), smem, st, a,
                     nst, ncb);
  SCN_LAUNCH_CHECK();
  return SCN_OK;
}

// Work-groups of the weight gradient, a tile per wave at least: three per CU for
// up to 32 entries (JT = 1); of the longer ones two run at once
int few_groups(int64_t nrows) {
  return (int)std::min<int64_t>(768, std::max<int64_t>(1, ceil_div(nrows, TILE * WGW)));
}

template <int JT>
static scn_status few_dw_launch(const FewArgs& f, bool v4, int nwg, hipStream_t st) {
  const size_t smem = std::max<size_t>((size_t)WGW * 32 * JT * 68 * 4,
                                       (4 * 2048 + 256 + 8 * (2 + JT)) * 4);
  auto fn = f.t.nb ? (v4 ? few_dw_kernel<JT, true, true> : few_dw_kernel<JT, true, false>)
                   : (v4 ? few_dw_kernel<JT, false, true> : few_dw_kernel<JT, false, false>);
  static LdsLimit limits[4];
  if (scn_status rc = allow_lds(reinterpret_cast<const void*>(fn),
                                limits[(f.t.nb ? 2 : 0) + (v4 ? 1 : 0)], smem))
    return rc;
  hipLaunchKernelGGL(fn, dim3((unsigned)nwg, (unsigned)ceil_div(f.Cout, 64)), dim3(64 * WGW), smem,
                     st, f);
  SCN_LAUNCH_CHECK();
  return SCN_OK;
}

scn_status few_partials(const TileArgs& a, const float* dy, const float* y, int Cout, float* part,
                        float* partS, hipStream_t st) {
  if (a.nrows <= 0) return SCN_OK;
  FewArgs f{a, dy, y, Cout, a.K * a.Rk, part, partS};
  const bool v4 = (Cout & 3) == 0 && ((reinterpret_cast<uintptr_t>(dy) |
                                       reinterpret_cast<uintptr_t>(y)) & 15) == 0;
  const int nwg = few_groups(a.nrows);
  if (f.J <= 32) return few_dw_launch<1>(f, v4, nwg, st);
  if (f.J <= 64) return few_dw_launch<2>(f, v4, nwg, st);
  return few_dw_launch<3>(f, v4, nwg, st);
}

scn_status few_reduce(const TileArgs& a, int Cout, const float* part, const float* u0, float* dW,
                      hipStream_t st) {
  const int64_t n = (int64_t)a.K * a.Rk * Cout;
  hipLaunchKernelGGL(few_reduce_kernel, dim3((unsigned)ceil_div(n, FR_E)), dim3(FR_E * FR_G), 0, st,
                     part, a.nrows > 0 ? few_groups(a.nrows) : 0, n, Cout, a.Rk, a.sub, u0, dW);
  SCN_LAUNCH_CHECK();
  return SCN_OK;
}

}  // namespace scn
