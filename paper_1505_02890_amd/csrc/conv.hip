// Sparse convolution, steps 2 and 3 of section 1.3 (gather the rows of Q, then
// Q W + B) and the gradients: the entry points, the contractions on the fp32
// matrix instruction (v_mfma_f32_16x16x4f32), and the weight gradient on the
// bf16 one (split.h).
//
// Q is never formed.  Its row for output o holds, per offset k, either an
// input row or the ground state g_in.  Writing v_k(o) = g_in + (x[r] - g_in)
// when site s*o+k is active,
//     Q W + B = g_pre + sum_{pairs (r, o) of offset k} (x[r] - g_in) W_k,
//     g_pre   = B + sum_k g_in W_k,
// so only the active blocks are gathered and multiplied.
//
// Most stride-1 layers go to tile.hip (fwd_route, tile_dx); the others take the
// gather kernel or, with the mask-sorted view, the dense-block forward.
//
// Gather kernel (forward and input gradient of strided rulebooks, forwards of
// sparse lists).  A work-group of four waves owns a tile of accumulator rows (output rows for the forward, input ranks for the
// input gradient) and 64 columns; the accumulators live in LDS and each wave
// owns 16 of the columns.  For each offset k the tile's pairs form one
// contiguous range of list k (lists ascend by output row and by input key).
// The tile's ranges are read once into lanes; the work-group walks them in
// stages of 32 pairs of one offset.  Per stage it gathers the 32 rows into an
// LDS buffer (one gather per row, shared by the four waves), each wave
// multiplies them by its slice of W_k on the matrix cores and adds the
// products into the LDS rows named by the pairs.  Rows, row indices and
// weights are fetched two stages ahead, and a stage's products are added one
// stage later, so no wave waits for memory or for its own matrix-core
// results in steady state.  A wave is the only writer of its columns and pair
// rows are distinct within an offset, so the scatter needs no atomics and the
// summation order is fixed.
//
// Weight gradient.  dW_k = X_k^T dY_k over the P_k pairs of offset k is a
// contraction along the pair axis: split into fixed chunks, each chunk's
// partial product goes to the workspace, and a reduction sums the chunks in
// index order (deterministic).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "scn_internal.h"
#include "split.h"
#include "tile.h"

namespace scn {
namespace {

constexpr int NT = 256;     // threads per work-group (4 waves)
constexpr int CB = 64;      // columns per work-group
constexpr int ACC_LD = CB + 4;

__device__ inline v4f mfma4(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Work-groups are dispatched round-robin over the 8 XCDs; give each XCD a
// contiguous range of work items so neighbouring tiles share its L2.
__device__ inline int64_t xcd_remap(int64_t b, int64_t n) {
  const int64_t x = b & 7, j = b >> 3, base = n >> 3, rem = n & 7;
  return x * base + min(x, rem) + j;
}

// ---------------------------------------------------------------------------
// Ground-state terms of the convolution.
//   gw[k][co]  = sum_ci g_in[ci] W[k][ci][co]       (what an inactive site at
//                offset k contributes; subtracted per pair in the residual form)
//   g_pre[co]  = B[co] + sum_k gw[k][co]
// ---------------------------------------------------------------------------
// One block per (k, 64 columns): thread (group g, column c) sums the input
// channels ci = g (mod GW_GROUPS) in ascending order, then the group sums are
// added in group order (fixed order, so the result is deterministic).
constexpr int GW_GROUPS = 4;
__global__ void __launch_bounds__(256) ground_w_kernel(const float* __restrict__ g_in,
                                                       const float* __restrict__ W, int K, int Cin,
                                                       int Cout, int ld, float* __restrict__ gw) {
  __shared__ float part[GW_GROUPS][64];
  const int nb = ld / 64;  // column blocks (ld is a multiple of 64)
  const int k = blockIdx.x / nb, c0 = (blockIdx.x - k * nb) * 64;
  const int c = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int co = c0 + c;
  float s = 0.f;
  if (co < Cout) {
    const float* wp = W + (int64_t)k * Cin * Cout + co;
#pragma unroll 4
    for (int ci = grp; ci < Cin; ci += GW_GROUPS) s = fmaf(g_in[ci], wp[(int64_t)ci * Cout], s);
  }
  part[grp][c] = s;
  __syncthreads();
  if (grp == 0) {
    float t = part[0][c];
#pragma unroll
    for (int g = 1; g < GW_GROUPS; ++g) t += part[g][c];
    gw[(int64_t)k * ld + co] = t;
  }
}

// g_pre (kept for the contraction's epilogue) and g_out = act(g_pre)
__global__ void ground_pre_kernel(const float* __restrict__ gw, int ld,
                                  const float* __restrict__ bias, int K, int Cout, int relu,
                                  float* __restrict__ g_pre, float* __restrict__ g_out) {
  const int co = blockIdx.x * blockDim.x + threadIdx.x;
  if (co >= Cout) return;
  float s = bias ? bias[co] : 0.f;
  for (int k = 0; k < K; ++k) s += gw[(int64_t)k * ld + co];
  g_pre[co] = s;
  g_out[co] = relu && !(s > 0.f) ? 0.f : s;
}

__global__ void zero_kernel(float* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// Packed weights for the gather kernel, in MFMA fragment order:
//   Wp[k][cb][w][t][lane][e] = W_k(j = 16t + 4q + e, n = 64cb + 16w + n16),
//   lane = n16 + 16q, zero outside j < Rk, n < Nc;  RkP = 16*NKT, NcP = 64*NCB.
//   forward:        W_k(j = ci, n = co) = W[k][ci][co]
//   input gradient: W_k(j = co, n = ci) = W[k][ci][co]
__global__ void __launch_bounds__(256) pack_w_kernel(const float* __restrict__ W, int K, int Cin,
                                                     int Cout, int transpose, int RkP, int NcP,
                                                     float* __restrict__ Wp) {
  const int Nc = transpose ? Cout : Cin, Rk = transpose ? Cin : Cout;
  const int nkt = RkP / 16, ncb = NcP / 64;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)K * NcP * RkP) return;
  const int e = (int)(i & 3), ln = (int)((i >> 2) & 63);
  const int64_t f = i >> 8;  // ((k*ncb + cb)*4 + w)*nkt + t
  const int t = (int)(f % nkt);
  const int64_t g = f / nkt;
  const int wv = (int)(g & 3);
  const int64_t h = g >> 2;
  const int cbk = (int)(h % ncb);
  const int64_t k = h / ncb;
  const int j = 16 * t + 4 * (ln >> 4) + e;
  const int n = 64 * cbk + 16 * wv + (ln & 15);
  float v = 0.f;
  if (j < Rk && n < Nc) {
    const int ci = transpose ? j : n, co = transpose ? n : j;
    v = W[(k * Cin + ci) * Cout + co];
  }
  Wp[i] = v;
}

// ---------------------------------------------------------------------------
// Gather -> MFMA -> LDS scatter
// ---------------------------------------------------------------------------
struct GatherArgs {
  const float* src;      // gathered rows [*][Rk]
  const int32_t* gidx;   // per pair: row of src
  const int32_t* aidx;   // per pair: accumulator row
  const int64_t* tpos;   // [K*ntile + 1] pair ranges per tile of TILE accumulator rows
  int64_t ntile;
  const float* Wp;       // W_k(j, n) = Wp[(k*NcP + n)*RkP + j], zero-padded (RkP = 16*ceil(Rk/16))
  const float* gwp;      // [K][NcP] subtracted from every pair's product (zeros if none)
  int NcP;               // Nc rounded up to 64
  int Rk;                // reduction length (channels of src)
  int Nc;                // output columns
  const float* add;      // [Nc] added to every accumulator row, or null
  int relu;
  float* dst;            // [nrows][Nc]
  const int32_t* wmap;   // dst row of accumulator row r (null = identity)
  int64_t nrows;
  int K;
  int vec_ok;            // rows of src are 16-byte aligned and Rk % 4 == 0
  int dvec_ok;           // rows of dst are 16-byte aligned and Nc % 4 == 0
};

// One pipeline stage covers up to 32 consecutive pairs of one offset (two
// 16-pair blocks).  The work-group gathers the stage's rows once into an LDS
// buffer (8 threads per row, float4 loads); each wave then reads MFMA
// fragments from LDS: lane (n16, q) takes channels 16t + 4q .. +3 of pair n16
// of each block, which is the B-operand layout of v_mfma_f32_16x16x4f32 when
// the contraction is computed transposed (R^T = W_k^T X^T).  The result holds
// pair n16, output columns 4q .. 4q+3 of the wave's 16 in one lane, so the
// lane adds one contiguous float4 into its pair's accumulator row.  The
// pair's accumulator row travels with its gathered row, in the padding word
// of the LDS row.
constexpr int SROWS = 32;  // pairs per stage

template <int NKT>
struct WFrag {
  float4 w[NKT];  // W_k(j = 16t + 4q + 0..3, column 16w + n16)
  float4 g;       // gw[k][16w + 4q .. +3]
};

// Weights in fragment order: Wp[k][cb][w][t][lane][e] = W_k(j = 16t + 4q + e,
// n = 64cb + 16w + n16) with lane = n16 + 16q, zero-padded to 16*NKT rows and
// NcP = 64*ceil(Nc/64) columns, so a wave's fragment is NKT contiguous 1 KB
// blocks.  gw is [K][NcP].
template <int NKT>
__device__ inline WFrag<NKT> load_w(const GatherArgs& a, int k, int cb, int w, int lane, int gcol) {
  WFrag<NKT> f;
  const float* wp =
      a.Wp + (((int64_t)k * (a.NcP >> 6) + cb) * 4 + w) * (int64_t)(NKT * 256) + lane * 4;
#pragma unroll
  for (int t = 0; t < NKT; ++t) f.w[t] = *reinterpret_cast<const float4*>(wp + 256 * t);
  f.g = *reinterpret_cast<const float4*>(a.gwp + (int64_t)k * a.NcP + gcol);
  return f;
}

// Per-thread share of one stage's gather: row tid/8, channel quads
// (tid%8) + 8u, and the row's accumulator index.  Positions past the stage's
// pairs are clamped to its last pair (loads stay in bounds; those rows are
// never scattered).  Reduction slots j >= Rk read some channel of the row and
// are stored as zero (the matching W entries are zero, but that channel may be
// infinite).
template <int NKT>
struct StageRegs {
  static constexpr int NQ = (4 * NKT + 7) / 8;  // float4 per thread
  v4f v[NQ];  // (arrays of HIP's float4 struct were left in scratch memory)
  int acc_row;
};

template <int NKT, bool VEC>
__device__ inline StageRegs<NKT> load_stage(const GatherArgs& a, int gi, int ai, int tid) {
  StageRegs<NKT> R;
  const float* rp = a.src + (int64_t)gi * a.Rk;
  const int part = tid & 7;
#pragma unroll
  for (int u = 0; u < StageRegs<NKT>::NQ; ++u) {
    const int c = 4 * (part + 8 * u);
    if (VEC) {
      const int cc = c < a.Rk ? c : 0;
      R.v[u] = *reinterpret_cast<const v4f*>(rp + cc);
    } else {
#pragma unroll
      for (int z = 0; z < 4; ++z) R.v[u][z] = rp[c + z < a.Rk ? c + z : 0];
    }
  }
  R.acc_row = ai;
  return R;
}

template <int NKT>
__device__ inline void store_stage(float* xs, int tid, int Rk, StageRegs<NKT> R) {
  constexpr int XLD = 16 * NKT + 4;
  const int row = tid >> 3, part = tid & 7;
#pragma unroll
  for (int u = 0; u < StageRegs<NKT>::NQ; ++u) {
    const int quad = part + 8 * u;
    if (8 * u + 7 >= 4 * (NKT - 1)) {  // the last 16 channels may end in the quad
#pragma unroll
      for (int z = 0; z < 4; ++z) R.v[u][z] = 4 * quad + z < Rk ? R.v[u][z] : 0.f;
    }
    if (quad < 4 * NKT) *reinterpret_cast<v4f*>(xs + row * XLD + 4 * quad) = R.v[u];
  }
  reinterpret_cast<int*>(xs)[row * XLD + 16 * NKT] = R.acc_row;  // same value from all 8
}

// Products of one stage held by a lane: pair n16 of each 16-pair block,
// output columns cq .. cq+3, already offset by -gw (the accumulator starts at
// -gw), and the accumulator rows they go to.
struct StageOut {
  v4f c0, c1;
  int i0, i1;
};

// Multiply one stage (cnt live pairs, possibly none) by the wave's W_k slice.
// Lanes past the live pairs target the spare row `spare` (never read), so
// the code has no branch.
template <int NKT>
__device__ inline StageOut stage_mfma(const float* xs, const WFrag<NKT>& B, int cnt, int spare,
                                      int n16, int q) {
  constexpr int XLD = 16 * NKT + 4;
  const float* r0 = xs + n16 * XLD + 4 * q;
  const float* r1 = xs + (16 + n16) * XLD + 4 * q;
  const int* ai = reinterpret_cast<const int*>(xs) + 16 * NKT;
  StageOut o;
  const int a0 = ai[n16 * XLD], a1 = ai[(16 + n16) * XLD];
  o.i0 = n16 < cnt ? a0 : spare;
  o.i1 = 16 + n16 < cnt ? a1 : spare;
  v4f c0v = {-B.g.x, -B.g.y, -B.g.z, -B.g.w}, c1v = c0v;
#pragma unroll
  for (int t = 0; t < NKT; ++t) {
    const float4 x0 = *reinterpret_cast<const float4*>(r0 + 16 * t);
    const float4 x1 = *reinterpret_cast<const float4*>(r1 + 16 * t);
    c0v = mfma4(B.w[t].x, x0.x, c0v);
    c1v = mfma4(B.w[t].x, x1.x, c1v);
    c0v = mfma4(B.w[t].y, x0.y, c0v);
    c1v = mfma4(B.w[t].y, x1.y, c1v);
    c0v = mfma4(B.w[t].z, x0.z, c0v);
    c1v = mfma4(B.w[t].z, x1.z, c1v);
    c0v = mfma4(B.w[t].w, x0.w, c0v);
    c1v = mfma4(B.w[t].w, x1.w, c1v);
  }
  o.c0 = c0v;
  o.c1 = c1v;
  return o;
}

// Add a stage's products into its accumulator rows (columns cq .. cq+3).
__device__ inline void stage_scatter(const StageOut& o, float* acc, int cq) {
  float4* r = reinterpret_cast<float4*>(&acc[o.i0 * ACC_LD + cq]);
  float4 v = *r;
  v.x += o.c0[0];
  v.y += o.c0[1];
  v.z += o.c0[2];
  v.w += o.c0[3];
  *r = v;
  r = reinterpret_cast<float4*>(&acc[o.i1 * ACC_LD + cq]);
  v = *r;
  v.x += o.c1[0];
  v.y += o.c1[1];
  v.z += o.c1[2];
  v.w += o.c1[3];
  *r = v;
}

// Stage schedule of one tile.  Lane k (< K) of every wave holds the tile's
// pair range of list k: start P and length N (at most TM*64: one pair per
// accumulator row and offset); `live` has bit k set when N > 0.  Stages are
// stepped with readlane, so the main loop makes no memory access to find its
// next stage.
struct Sched {
  int64_t P;
  int N;
  uint64_t live;
  int K;
};

__device__ inline int64_t lane64(int64_t v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// A stage position: offset k, pairs [p, p + min(n, 32)) of list k; k == K
// (n == 0) past the tile's last stage.
struct Pos {
  int k, n;
  int64_t p;
};

__device__ inline Pos jump(const Sched& s, uint64_t m) {
  Pos x;
  if (!m) {
    x.k = s.K;
    x.n = 0;
    x.p = 0;
    return x;
  }
  x.k = __builtin_ctzll(m);
  x.p = lane64(s.P, x.k);
  x.n = __builtin_amdgcn_readlane(s.N, x.k);
  return x;
}

__device__ inline Pos next_stage(const Sched& s, Pos x) {
  if (x.k >= s.K) return x;
  x.p += SROWS;
  x.n -= SROWS;
  if (x.n > 0) return x;
  return jump(s, s.live & ~((2ull << x.k) - 1ull));
}

// Main loop, unrolled by two so that the register sets of the software
// pipeline keep fixed names (X = iteration parity); a tile with an odd number
// of stages ends with one empty stage.  Iteration i computes
// stage s_i; in flight meanwhile: the rows of s_{i+1} (landed, stored to LDS
// at the top of the iteration), the rows of s_{i+2} and s_{i+3}, the row
// indices of s_{i+4} and s_{i+5}, and the weights of s_{i+1} and s_{i+2}.
// The row and index loads of an iteration are unconditional; the weights are
// loaded only when the offset changes.
template <int NKT, bool VEC, int TM, int MINB>
__global__ void __launch_bounds__(NT, MINB) gather_mfma_kernel(GatherArgs a) {
  extern __shared__ float smem[];
  constexpr int T = TM * TILE;
  constexpr int XLD = 16 * NKT + 4;
  float* acc = smem;                      // [T + 1][ACC_LD], row T is the spare row
  float* xsb = smem + (T + 1) * ACC_LD;   // [2][SROWS][XLD]
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const int n16 = lane & 15, q = lane >> 4;
  const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t t0 = tile * TM;
  const int64_t t1 = min(t0 + TM, a.ntile);
  const int64_t row0 = t0 * TILE;
  const int cb = blockIdx.y;
  const int c0 = cb * CB;
  const int cq = 16 * w + 4 * q;      // tile-local columns this lane accumulates
  const int lrow = tid >> 3;          // stage row this thread gathers

  for (int i = tid; i < T * ACC_LD / 4; i += NT)
    reinterpret_cast<float4*>(acc)[i] = make_float4(0.f, 0.f, 0.f, 0.f);

  Sched sc;
  sc.K = a.K;
  {
    const int k = lane < a.K ? lane : 0;
    sc.P = a.tpos[(int64_t)k * a.ntile + t0];
    sc.N = lane < a.K ? (int)(a.tpos[(int64_t)k * a.ntile + t1] - sc.P) : 0;
    sc.live = __ballot(sc.N > 0);
  }
  Pos s0 = jump(sc, sc.live);
  if (s0.k < a.K) {
    const Pos first = s0;
    // loads for a position past the last stage use the first stage (in
    // bounds, never scattered)
    auto real = [&](const Pos x) -> Pos { return x.k < a.K ? x : first; };
    auto gidx_of = [&](const Pos x) -> int {
      const Pos r = real(x);
      return a.gidx[r.p + min(lrow, r.n - 1)];
    };
    auto aidx_of = [&](const Pos x) -> int {
      const Pos r = real(x);
      return (int)(a.aidx[r.p + min(lrow, r.n - 1)] - row0);
    };
    auto wk = [&](const Pos x) { return load_w<NKT>(a, real(x).k, cb, w, lane, c0 + cq); };
    Pos s1 = next_stage(sc, s0), s2 = next_stage(sc, s1), s3 = next_stage(sc, s2);
    Pos s4 = next_stage(sc, s3), s5 = next_stage(sc, s4);

    store_stage<NKT>(xsb, tid, a.Rk, load_stage<NKT, VEC>(a, gidx_of(s0), aidx_of(s0), tid));
    StageRegs<NKT> R0 = load_stage<NKT, VEC>(a, gidx_of(s1), aidx_of(s1), tid);
    StageRegs<NKT> R1 = load_stage<NKT, VEC>(a, gidx_of(s2), aidx_of(s2), tid);
    int G0 = gidx_of(s3), G1 = gidx_of(s4);
    WFrag<NKT> B0 = wk(s0), B1 = wk(s1);
    // drain the prologue's loads once per tile, so that the wait counts in
    // the loop follow from the loop's own loads
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // one iteration: parity X selects the register sets.  The products of
    // s_i are added to the accumulators one iteration later, so the wave
    // never waits for its own matrix-core results.
    auto step = [&](StageRegs<NKT>& R, int& G, WFrag<NKT>& B, StageOut& Onew, const StageOut& Oprev,
                    float* xs_cur, float* xs_nxt) {
      // s_i is past the last stage (no live pairs) only in the second half
      // of the final pair
      Onew = stage_mfma<NKT>(xs_cur, B, min(s0.n, SROWS), T, n16, q);
      stage_scatter(Oprev, acc, cq);
      // rows of s_{i+1} -> the other buffer
      store_stage<NKT>(xs_nxt, tid, a.Rk, R);
      // rows of s_{i+3} (index loaded two iterations ago), index of s_{i+5}
      R = load_stage<NKT, VEC>(a, G, aidx_of(s3), tid);
      G = gidx_of(s5);
      // weights of s_{i+2} into the set just used, unless that set already
      // holds them (s_{i+2} continues s_i's offset: a full 128-row tile has
      // four stages per offset).  The branch tightens the compiler's wait
      // counts; fewer weight loads still win (input gradient 2.35 -> 2.26 ms)
      if (s2.k != s0.k) B = wk(s2);
    };
    auto shift = [&]() {
      s0 = s1;
      s1 = s2;
      s2 = s3;
      s3 = s4;
      s4 = s5;
      s5 = next_stage(sc, s5);
    };
    float* const xa = xsb;
    float* const xb = xsb + SROWS * XLD;
    // stages in pairs; the only exit is after the second of a pair, behind
    // its barrier (every path through the loop issues the same loads)
    StageOut O0, O1;
    O1.c0 = v4f{0.f, 0.f, 0.f, 0.f};
    O1.c1 = O1.c0;
    O1.i0 = O1.i1 = T;
    while (true) {
      step(R0, G0, B0, O0, O1, xa, xb);
      __syncthreads();
      shift();
      step(R1, G1, B1, O1, O0, xb, xa);
      __syncthreads();
      shift();
      if (s0.k >= a.K) break;
    }
    stage_scatter(O1, acc, cq);
  }
  __syncthreads();
  // epilogue: dst[row] = act(acc + add)
  const int ncols = min(CB, a.Nc - c0);
  for (int i = tid; i < T * (CB / 4); i += NT) {
    const int r = i / (CB / 4), cc = (i - r * (CB / 4)) * 4;
    const int64_t grow = row0 + r;
    if (cc >= ncols || grow >= a.nrows) continue;
    float4 v = *reinterpret_cast<const float4*>(&acc[r * ACC_LD + cc]);
    float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (a.add && cc + u < ncols) e[u] += a.add[c0 + cc + u];
      if (a.relu) e[u] = e[u] > 0.f ? e[u] : 0.f;
    }
    const int64_t drow = a.wmap ? (int64_t)a.wmap[grow] : grow;
    float* dp = a.dst + drow * a.Nc + c0 + cc;
    if (a.dvec_ok && cc + 3 < ncols) {
      *reinterpret_cast<float4*>(dp) = make_float4(e[0], e[1], e[2], e[3]);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (cc + u < ncols) dp[u] = e[u];
    }
  }
}

typedef void (*GatherFn)(GatherArgs);

// Tile rows (TM * 64) and work-groups per CU: the accumulators and the two
// stage buffers must fit the 160 KB of LDS.  Reductions over up to 160
// channels use 128-row tiles, three work-groups per CU up to 64 channels and
// two past that (several work-groups per CU hide the gather latency); longer
// reductions use 256-row tiles, one work-group per CU.
template <int NKT>
constexpr int gather_tm() {
  return NKT > 10 ? 4 : 2;
}

template <int NKT>
GatherFn pick_gather(bool vec) {
  constexpr int TM = gather_tm<NKT>(), MINB = NKT > 10 ? 1 : (NKT > 4 ? 2 : 3);
  return vec ? gather_mfma_kernel<NKT, true, TM, MINB> : gather_mfma_kernel<NKT, false, TM, MINB>;
}

GatherFn gather_fn(int nkt, bool vec) {
  switch (nkt) {
    case 1: return pick_gather<1>(vec);
    case 2: return pick_gather<2>(vec);
    case 3: return pick_gather<3>(vec);
    case 4: return pick_gather<4>(vec);
    case 5: return pick_gather<5>(vec);
    case 6: return pick_gather<6>(vec);
    case 7: return pick_gather<7>(vec);
    case 8: return pick_gather<8>(vec);
    case 9: return pick_gather<9>(vec);
    case 10: return pick_gather<10>(vec);
    case 11: return pick_gather<11>(vec);
    case 12: return pick_gather<12>(vec);
    case 13: return pick_gather<13>(vec);
    case 14: return pick_gather<14>(vec);
    case 15: return pick_gather<15>(vec);
    default: return pick_gather<16>(vec);
  }
}

scn_status launch_gather(GatherArgs a, hipStream_t st) {
  if (a.nrows <= 0) return SCN_OK;
  a.vec_ok = ((a.Rk & 3) == 0) && ((reinterpret_cast<uintptr_t>(a.src) & 15) == 0);

  a.dvec_ok = ((a.Nc & 3) == 0) && ((reinterpret_cast<uintptr_t>(a.dst) & 15) == 0);
  const int nkt = (int)ceil_div(a.Rk, 16);
  const int TM = nkt > 10 ? gather_tm<11>() : gather_tm<1>();
  const int64_t nwg = ceil_div(a.ntile, TM);
  const unsigned ncb = (unsigned)ceil_div(a.Nc, CB);
  const size_t smem =
      ((size_t)(TM * TILE + 1) * ACC_LD + 2 * (size_t)SROWS * (16 * nkt + 4)) * sizeof(float);
  const bool vec = a.vec_ok;
  GatherFn fn = gather_fn(nkt, vec);
  static LdsLimit limits[2][17];
  if (scn_status rc = allow_lds(reinterpret_cast<const void*>(fn), limits[vec][nkt], smem))
    return rc;
  hipLaunchKernelGGL(fn, dim3((unsigned)nwg, ncb), dim3(NT), smem, st, a);
  SCN_LAUNCH_CHECK();
  return SCN_OK;
}

// ---------------------------------------------------------------------------
// Dense-block forward (narrow layers with the mask-sorted view)
// ---------------------------------------------------------------------------
// The rulebook sorts the output rows by neighbour mask; cut into blocks of 32
// (DENSE_ROWS) the rows of a block mostly share one mask.  One wave owns a
// block and 64 output columns, with its 32 x 64 accumulators in registers:
// for each offset k of the union of the block's masks it gathers the block's
// 32 input rows (a row without offset k contributes zero) and multiplies them
// by W_k, 64 input channels at a time.  Lane (n16, q) gathers block rows n16
// and 16 + n16; a row's input at offset k is entry popcount(mask & (2^k - 1))
// of its output-major neighbour list.  There is no scatter: the rows of a
// block are distinct outputs, and the epilogue writes each once.  Rows hold
// x - g_in, so y = g_pre + sum over active offsets of (x - g_in) W_k.  The
// next (offset, channel chunk)'s rows are loaded while the current one is
// multiplied.
struct DenseArgs {
  const float* x;          // [a_in][Cin]
  const float* g_in;       // [Cin]
  const float* Wp;         // packed like GatherArgs::Wp (fragment order, transposed W)
  const float* add;        // [Cout] g_pre
  const int32_t* nb;       // rulebook fnb
  const uint32_t* nb_off;  // rulebook fnb_off
  const int32_t* fperm;    // rulebook fperm
  const uint32_t* fmask;   // rulebook fmask
  float* y;                // [a_out][Cout]
  int64_t a_out, nblk;
  int K, Cin, Cout, NcP, relu, dvec_ok;
};

// One block row as the lane sees it: its mask and the start of its list.
struct DRow {
  uint32_t m, off;
};

// The rows of one (offset, 64-channel chunk) item: lane (n16, q) holds
// channels 64ch + 16t + 4q .. +3 of block rows n16 and 16 + n16.
template <int TC>
struct DRows {
  float4 v[2][TC];
  int r0, r1;
};

__device__ inline int dense_src(const DenseArgs& a, const DRow& w, int k) {
  // the list entry is read unconditionally (the list has a spare entry)
  const int r = a.nb[w.off + __popc(w.m & ((1u << k) - 1u))];
  return (w.m >> k) & 1u ? r : -1;
}

// Channels past Cin read channel 0 (multiply takes zeros in their place: their
// weights are zero, but channel 0 may be infinite).
template <int NKT, bool VEC>
__device__ inline DRows<(NKT < 4 ? NKT : 4)> dense_rows_i(const DenseArgs& a, int r0, int r1,
                                                          int ch, int q) {
  constexpr int TC = NKT < 4 ? NKT : 4;
  DRows<TC> R;
  R.r0 = r0;
  R.r1 = r1;
  const float* p0 = a.x + (int64_t)(r0 >= 0 ? r0 : 0) * a.Cin;
  const float* p1 = a.x + (int64_t)(r1 >= 0 ? r1 : 0) * a.Cin;
#pragma unroll
  for (int t = 0; t < TC; ++t) {
    const int c = 64 * ch + 16 * t + 4 * q;
    if (VEC) {
      const int cc = c < a.Cin ? c : 0;
      R.v[0][t] = *reinterpret_cast<const float4*>(p0 + cc);
      R.v[1][t] = *reinterpret_cast<const float4*>(p1 + cc);
    } else {
      float e0[4], e1[4];
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        const int cz = c + z < a.Cin ? c + z : 0;
        e0[z] = p0[cz];
        e1[z] = p1[cz];
      }
      R.v[0][t] = make_float4(e0[0], e0[1], e0[2], e0[3]);
      R.v[1][t] = make_float4(e1[0], e1[1], e1[2], e1[3]);
    }
  }
  return R;
}

template <int NKT, bool VEC>
__global__ void __launch_bounds__(NT) dense_fwd_kernel(DenseArgs a) {
  constexpr int TC = NKT < 4 ? NKT : 4;        // 16-channel steps per chunk
  constexpr int NCH = (NKT + 3) / 4;           // 64-channel chunks
  __shared__ float gsh[16 * NKT];  // g_in, zero past Cin (those weights are zero)
  for (int c = threadIdx.x; c < 16 * NKT; c += NT) gsh[c] = c < a.Cin ? a.g_in[c] : 0.f;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int64_t b = (int64_t)blockIdx.x * (NT / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (b >= a.nblk) return;
  const int cb = blockIdx.y;
  // Two lane layouts.  MFMA layout: lane (n16, q) = n16 + 16q holds row n16
  // (and 16 + n16), channels 4q .. 4q + 3 of each 16; the operand fixes it.
  // Load layout: lane (rl, cq) = 4rl + cq loads row rl (and 16 + rl),
  // channels 4cq .. 4cq + 3, so four adjacent lanes read one row's 64
  // contiguous bytes (in the MFMA layout four adjacent lanes read four
  // rows, and the L1 serves each 16-byte piece on its own).  The rows are
  // gathered in the load layout and moved to the MFMA layout by ds_bpermute.
  const int n16 = lane & 15, q = lane >> 4;
  const int rl = lane >> 2, cq = lane & 3;
  const int from = (n16 * 4 + q) * 4;  // bpermute address: MFMA lane <- load lane 4 n16 + q
  const int ncb = a.NcP >> 6;
  const int64_t pos0 = b * DENSE_ROWS + n16, pos1 = pos0 + 16;      // MFMA layout
  const int64_t lpos0 = b * DENSE_ROWS + rl, lpos1 = lpos0 + 16;    // load layout
  const int o0 = pos0 < a.a_out ? a.fperm[pos0] : 0, o1 = pos1 < a.a_out ? a.fperm[pos1] : 0;
  const int lo0 = lpos0 < a.a_out ? a.fperm[lpos0] : 0, lo1 = lpos1 < a.a_out ? a.fperm[lpos1] : 0;
  DRow w0, w1;
  w0.m = lpos0 < a.a_out ? a.fmask[lpos0] : 0u;
  w1.m = lpos1 < a.a_out ? a.fmask[lpos1] : 0u;
  w0.off = a.nb_off[lo0];
  w1.off = a.nb_off[lo1];
  uint32_t u = w0.m | w1.m;
#pragma unroll
  for (int d = 4; d < 64; d <<= 1) u |= (uint32_t)__shfl_xor((int)u, d, 64);
  const uint32_t U = (uint32_t)__builtin_amdgcn_readfirstlane((int)u);
  v4f acc[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[r][g] = v4f{0.f, 0.f, 0.f, 0.f};
  if (U) {
    // item = (offset k, channel chunk ch), in order; `rest` holds the offsets
    // after k; past the last item an item stays where it is (its loads are in
    // bounds and unused)
    struct Item {
      int k, ch;
      uint32_t rest;
    };
    auto advance = [&](Item& t) {
      if (t.ch + 1 < NCH) {
        ++t.ch;
      } else if (t.rest) {
        t.k = __builtin_ctz(t.rest);
        t.rest &= t.rest - 1;
        t.ch = 0;
      }
    };
    Item c{__builtin_ctz(U), 0, U & (U - 1)};
    Item n = c;
    advance(n);
    Item nn = n;
    advance(nn);
    const int nit = __builtin_popcount(U) * NCH;
    int n0 = dense_src(a, w0, n.k), n1 = dense_src(a, w1, n.k);
    DRows<TC> cur = dense_rows_i<NKT, VEC>(a, dense_src(a, w0, c.k), dense_src(a, w1, c.k), 0, cq);
    DRows<TC> nxt;
    int nn0 = 0, nn1 = 0;
    for (int it = 0; it < nit; ++it) {
      const int ch = c.ch;
      const float* wp = a.Wp + (((int64_t)c.k * ncb + cb) * 4) * (NKT * 256) + lane * 4;
      auto wload = [&](int t, float4 (&A)[4]) {
        const int tg = 4 * ch + t < NKT ? 4 * ch + t : NKT - 1;  // past NKT: never used
#pragma unroll
        for (int g = 0; g < 4; ++g)
          A[g] = *reinterpret_cast<const float4*>(wp + (int64_t)g * (NKT * 256) + tg * 256);
      };
      // the next item's rows and the indices after it: issued after this
      // item's last weight load, so the waits for the weights leave them in
      // flight
      auto prefetch = [&]() {
        nxt = dense_rows_i<NKT, VEC>(a, n0, n1, n.ch, cq);
        nn0 = dense_src(a, w0, nn.k);
        nn1 = dense_src(a, w1, nn.k);
      };
      auto mult = [&](int t, const float4 (&A)[4]) {
        const int tg = 4 * ch + t;
        // x - g_in, zero for an absent row, in the load layout; then to the
        // MFMA layout
        const float4 gq = *reinterpret_cast<const float4*>(&gsh[16 * tg + 4 * cq]);
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 d0 = cur.v[0][t], d1 = cur.v[1][t];
        if (!VEC) {  // one piece, cut short
          if (a.Cin < 2) d0.y = d1.y = 0.f;
          if (a.Cin < 3) d0.z = d1.z = 0.f;
          if (a.Cin < 4) d0.w = d1.w = 0.f;
        }
        d0.x -= gq.x; d0.y -= gq.y; d0.z -= gq.z; d0.w -= gq.w;
        d1.x -= gq.x; d1.y -= gq.y; d1.z -= gq.z; d1.w -= gq.w;
        const int left = a.Cin - (16 * tg + 4 * cq);  // channels of the lane's piece and after
        const float4 L0 = cur.r0 >= 0 && left > 0 ? d0 : z, L1 = cur.r1 >= 0 && left > 0 ? d1 : z;
        auto perm = [&](float v) {
          return __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(v)));
        };
        const float4 B0 = make_float4(perm(L0.x), perm(L0.y), perm(L0.z), perm(L0.w));
        const float4 B1 = make_float4(perm(L1.x), perm(L1.y), perm(L1.z), perm(L1.w));
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          acc[0][g] = mfma4(A[g].x, B0.x, acc[0][g]);
          acc[1][g] = mfma4(A[g].x, B1.x, acc[1][g]);
          acc[0][g] = mfma4(A[g].y, B0.y, acc[0][g]);
          acc[1][g] = mfma4(A[g].y, B1.y, acc[1][g]);
          acc[0][g] = mfma4(A[g].z, B0.z, acc[0][g]);
          acc[1][g] = mfma4(A[g].z, B1.z, acc[1][g]);
          acc[0][g] = mfma4(A[g].w, B0.w, acc[0][g]);
          acc[1][g] = mfma4(A[g].w, B1.w, acc[1][g]);
        }
      };
      // weights two 16-channel steps ahead of their products (two register
      // sets, alternating)
      float4 A0[4], A1[4];
      wload(0, A0);
      if (TC > 1) wload(1, A1);
      if (TC <= 2) prefetch();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < TC; ++t) {
        if (NCH > 1 && 4 * ch + t >= NKT) {
          // a last chunk shorter than the step that issues the prefetch
          // (t = TC - 3) issues it here, so the next item's rows are loaded
          if (t <= TC - 3) prefetch();
          break;
        }
        // step t's products, then step t + 2's weights into the set just read
        if (t & 1) mult(t, A1); else mult(t, A0);
        if (t + 2 < TC) {
          if (t & 1) wload(t + 2, A1); else wload(t + 2, A0);
          if (t + 2 == TC - 1) prefetch();
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      c = n;
      n = nn;
      advance(nn);
      n0 = nn0;
      n1 = nn1;
      cur = nxt;
    }
  }
  // epilogue: rows n16 and 16 + n16 of the block, columns 64cb + 16g + 4q .. +3
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int64_t pos = r ? pos1 : pos0;
    if (pos >= a.a_out) continue;
    float* dp = a.y + (int64_t)(r ? o1 : o0) * a.Cout;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int col = 64 * cb + 16 * g + 4 * q;
      if (col >= a.Cout) continue;
      float e[4] = {acc[r][g][0], acc[r][g][1], acc[r][g][2], acc[r][g][3]};
#pragma unroll
      for (int u2 = 0; u2 < 4; ++u2) {
        if (col + u2 < a.Cout) e[u2] += a.add[col + u2];
        if (a.relu) e[u2] = e[u2] > 0.f ? e[u2] : 0.f;
      }
      if (a.dvec_ok && col + 3 < a.Cout) {
        // a streaming store: y is read only by later calls (kernel 2.669 ->
        // 2.653 ms on the 1M-site layer)
        __builtin_nontemporal_store(v4f{e[0], e[1], e[2], e[3]}, reinterpret_cast<v4f*>(dp + col));
      } else {
#pragma unroll
        for (int u2 = 0; u2 < 4; ++u2)
          if (col + u2 < a.Cout) dp[col + u2] = e[u2];
      }
    }
  }
}

typedef void (*DenseFn)(DenseArgs);

constexpr int DENSE_STEPS = 7;  // 16-channel steps of the longest reduction (fwd_route)

DenseFn dense_fn(int nkt, bool vec) {
  switch (nkt) {
    case 1: return vec ? dense_fwd_kernel<1, true> : dense_fwd_kernel<1, false>;
    case 2: return dense_fwd_kernel<2, true>;
    case 3: return dense_fwd_kernel<3, true>;
    case 4: return dense_fwd_kernel<4, true>;
    case 5: return dense_fwd_kernel<5, true>;
    case 6: return dense_fwd_kernel<6, true>;
    case 7: return dense_fwd_kernel<7, true>;
    default: return nullptr;
  }
}

scn_status launch_dense(DenseArgs a, hipStream_t st) {
  if (a.a_out <= 0 || a.nblk <= 0) return SCN_OK;
  const bool vec = ((a.Cin & 3) == 0) && ((reinterpret_cast<uintptr_t>(a.x) & 15) == 0);
  a.dvec_ok = ((a.Cout & 3) == 0) && ((reinterpret_cast<uintptr_t>(a.y) & 15) == 0);
  const int nkt = (int)ceil_div(a.Cin, 16);
  const DenseFn fn = dense_fn(nkt, vec);
  if (!fn || (!vec && nkt > 1)) {
    set_error("dense-block forward of %d channels", a.Cin);
    return SCN_ERR_INVALID;
  }
  const int64_t nwg = ceil_div(a.nblk, NT / 64);
  hipLaunchKernelGGL(fn, dim3((unsigned)nwg, (unsigned)(a.NcP / 64)), dim3(NT), 0,
                     st, a);
  SCN_LAUNCH_CHECK();
  return SCN_OK;
}

// ---------------------------------------------------------------------------
// Backward helpers
// ---------------------------------------------------------------------------
constexpr int RB_ROWS = 1024;  // rows per column-sum block

// dyb = relu ? dy * (y > 0) : dy (written only under relu);  partS[blk][c] = sum of dyb rows
__global__ void __launch_bounds__(NT) colsum_kernel(const float* __restrict__ dy,
                                                    const float* __restrict__ y, int relu,
                                                    int64_t rows, int C, float* __restrict__ dyb,
                                                    float* __restrict__ partS) {
  __shared__ float red[NT];
  const int64_t r0 = (int64_t)blockIdx.x * RB_ROWS;
  const int64_t r1 = min<int64_t>(r0 + RB_ROWS, rows);
  const int rg = threadIdx.x >> 6, cl = threadIdx.x & 63;
  for (int cbase = 0; cbase < C; cbase += 64) {
    const int c = cbase + cl;
    float s = 0.f;
    if (c < C) {
      for (int64_t r = r0 + rg; r < r1; r += 4) {
        float v = dy[r * C + c];
        if (relu) {
          v = y[r * C + c] > 0.f ? v : 0.f;
          dyb[r * C + c] = v;
        }
        s += v;
      }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (rg == 0 && c < C)
      partS[(int64_t)blockIdx.x * C + c] = ((red[cl] + red[64 + cl]) + red[128 + cl]) + red[192 + cl];
    __syncthreads();
  }
}

// Four channels per thread (C % 4 == 0, 16-byte aligned rows): a block reads
// RB_ROWS rows as float4, `per` rows at a time, and combines the rows in a
// fixed order.
__global__ void __launch_bounds__(NT) colsum_vec_kernel(const float4* __restrict__ dy,
                                                        const float4* __restrict__ y, int relu,
                                                        int64_t rows, int nc4,
                                                        float4* __restrict__ dyb,
                                                        float4* __restrict__ partS) {
  __shared__ float4 red[NT];
  const int per = NT / nc4;
  const int rl = threadIdx.x / nc4, c4 = threadIdx.x - rl * nc4;
  const int64_t r0 = (int64_t)blockIdx.x * RB_ROWS;
  const int64_t r1 = min<int64_t>(r0 + RB_ROWS, rows);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (rl < per) {
    int64_t r = r0 + rl;
    // four rows in flight per thread
    for (; r + 3 * per < r1; r += 4 * per) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = dy[(r + u * per) * nc4 + c4];
      if (relu) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float4 m = y[(r + u * per) * nc4 + c4];
          v[u].x = m.x > 0.f ? v[u].x : 0.f;
          v[u].y = m.y > 0.f ? v[u].y : 0.f;
          v[u].z = m.z > 0.f ? v[u].z : 0.f;
          v[u].w = m.w > 0.f ? v[u].w : 0.f;
          dyb[(r + u * per) * nc4 + c4] = v[u];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        s.x += v[u].x;
        s.y += v[u].y;
        s.z += v[u].z;
        s.w += v[u].w;
      }
    }
    for (; r < r1; r += per) {
      float4 v = dy[r * nc4 + c4];
      if (relu) {
        const float4 m = y[r * nc4 + c4];
        v.x = m.x > 0.f ? v.x : 0.f;
        v.y = m.y > 0.f ? v.y : 0.f;
        v.z = m.z > 0.f ? v.z : 0.f;
        v.w = m.w > 0.f ? v.w : 0.f;
        dyb[r * nc4 + c4] = v;
      }
      s.x += v.x;
      s.y += v.y;
      s.z += v.z;
      s.w += v.w;
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (rl == 0) {
    for (int i = 1; i < per; ++i) {
      const float4 t = red[i * nc4 + c4];
      s.x += t.x;
      s.y += t.y;
      s.z += t.z;
      s.w += t.w;
    }
    partS[(int64_t)blockIdx.x * nc4 + c4] = s;
  }
}

// S, dḡ, dbias; u0 = S + dḡ.  One block per column: each thread sums a
// strided share of the partials, then a fixed-shape tree.
__global__ void __launch_bounds__(NT) finish_vec_kernel(const float* __restrict__ partS,
                                                        int64_t nblk, int C,
                                                        const float* __restrict__ g_out,
                                                        const float* __restrict__ dg_out, int relu,
                                                        float* __restrict__ S,
                                                        float* __restrict__ u0,
                                                        float* __restrict__ dbias) {
  __shared__ float red[NT];
  const int c = blockIdx.x;
  float s = 0.f;
  for (int64_t b = threadIdx.x; b < nblk; b += NT) s += partS[b * C + c];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = NT / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float t = red[0];
    float dg = dg_out ? dg_out[c] : 0.f;
    if (relu && dg_out) dg = g_out[c] > 0.f ? dg : 0.f;
    S[c] = t;
    u0[c] = t + dg;
    if (dbias) dbias[c] = t + dg;
  }
}

// Weight gradient partials.  A work-group accumulates one 64x64 block of
// dW_k = sum_pairs (x[r] - g_in)^T dy[o] over a fixed chunk of list k, on the
// bf16 matrix cores in three-way split fp32 (split.h).  Each of its four waves
// takes every fourth stage of 16 pairs on its own; nothing passes through LDS
// and nothing waits for another wave until the four sums are added at the end,
// in wave order.
//
// A load instruction reads four pairs' 64 channels as 16-byte pieces (with a
// float per lane and one pair per instruction the address unit takes as long
// per instruction, and the kernel four times as long for its gather): lane
// 16 pg + cq gets channels 4 cq .. + 3 of pairs 4 pg + i, i < 4.  After the
// split two pairs of a channel share a word, the order the MFMA wants along
// the pair axis; exchanging odd and even 16-lane rows between the words of
// neighbouring channels (v_permlane16_swap) then gives every lane 8 pairs of
// one channel: operand row m of tile t is channel 4 (m & 15) + 2 t + (m >> 4).
// Per stage a wave issues 24 MFMAs (768 clocks) against about 270 vector
// instructions (1080, most of them splits): the vector unit bounds it.
constexpr int DW_SC = 64;  // chunks are whole multiples: one stage per wave
constexpr int DW_ST = 16;  // pairs per stage
constexpr int DW_OCC = 2;  // work-groups per CU

struct DwArgs {
  const float* x;        // [a_in][Cin]
  const float* dyb;      // [a_out][Cout]
  const float* g_in;     // [Cin]
  const int32_t* in_rows;
  const int32_t* out_rows;
  const int64_t* off;    // [K+1]
  int K;
  int Cin, Cout;
  int nco;               // 64-column blocks of Cout
  int nblk;              // (Cin blocks) * nco
  int64_t chp;           // pairs per chunk
  int64_t maxc;          // chunks per offset (slot count)
  float* part;           // [K][maxc][Cin][Cout]
  float* partT;          // [K][maxc][Cout]
};

typedef int32_t v4i_any __attribute__((ext_vector_type(4), aligned(4)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

// A lane's four channels of a row of C: 4 cq .. + 3 of the block that starts at
// c0.  QUAD (C >= 4): the last ones of a layer start earlier, so that they are
// four in a row (of any alignment) and repeat channels of the quad before; past
// the layer they repeat its last four.  A block's slot (its row or column 0 ..
// 63) holds slot_channel, and is written unless another slot holds that.
template <bool QUAD>
__device__ inline int slot_channel(int slot, int c0, int C) {
  const int q = c0 + (slot & ~3);
  return QUAD ? min(q, C - 4) + (slot & 3) : min(q + (slot & 3), C - 1);
}
template <bool QUAD>
__device__ inline bool slot_live(int slot, int c0, int C) {
  return QUAD ? slot_channel<true>(slot, c0, C) >= c0 + (slot & ~3) : c0 + slot < C;
}

template <bool QUAD>
__global__ void __launch_bounds__(NT, DW_OCC) dw_partial_kernel(DwArgs a) {
  __shared__ __align__(16) float red[4 * 32 * 64];
  __shared__ float redT[4 * 64];
  __shared__ uint32_t seen[4][2][4];  // [x 0, x 1, dy 0, dy 1][any, big][wave]
  __shared__ uint32_t some[4];        // whether a wave saw a row without a large value
  // flattened (chunk, offset, block) work item, blocks then offsets fastest,
  // contiguous per XCD
  const int64_t item = xcd_remap(blockIdx.x, gridDim.x);
  const int blk = (int)(item % a.nblk);
  const int64_t ck = item / a.nblk;
  const int k = (int)(ck % a.K);
  const int64_t c = ck / a.K;
  const int64_t lb = a.off[k], le = a.off[k + 1];
  const int64_t p_begin = lb + c * a.chp;
  if (p_begin >= le) return;
  const int64_t p_end = min(le, p_begin + a.chp);
  const int ci0 = (blk / a.nco) * 64, co0 = (blk % a.nco) * 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pg = lane >> 4, cq = lane & 15;
  const int64_t ldx = a.Cin, ldd = a.Cout;
  const uint32_t bx = 4u * (uint32_t)a.Cin, bd = 4u * (uint32_t)a.Cout;  // bytes per row
  int cx[4], cd[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    cx[e] = slot_channel<QUAD>(4 * cq + e, ci0, a.Cin);
    cd[e] = slot_channel<QUAD>(4 * cq + e, co0, a.Cout);
  }
  // The matrix core drops the bits of small addends below its adder, always
  // downwards: over a million pairs the drift of every sum was 2.4e-6 of dW's
  // size (1.0e-6 in all on the fp32 instruction).  Odd waves sum the negated
  // products, and the drifts cancel where the waves' sums meet.
  const float sgn = w & 1 ? -1.f : 1.f;
  v4f gs;
#pragma unroll
  for (int e = 0; e < 4; ++e) gs[e] = -sgn * a.g_in[cx[e]];
  const float* const x = QUAD ? a.x + cx[0] : a.x;
  const float* const dyb = QUAD ? a.dyb + cd[0] : a.dyb;

  struct Idx {
    int r[4], o[4];
  };
  struct Stage {
    v4f x[4], d[4];
  };
  // rows of pairs 4 pg + i of the stage at p0; pairs past the chunk repeat its
  // last one
  auto load_idx = [&](Idx& I, int64_t p0) {
    const int64_t p = p0 + 4 * pg;
    if (p0 + DW_ST <= p_end) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        I.r[i] = (*reinterpret_cast<const v4i_any*>(a.in_rows + p))[i];
        I.o[i] = (*reinterpret_cast<const v4i_any*>(a.out_rows + p))[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        I.r[i] = a.in_rows[min(p + i, p_end - 1)];
        I.o[i] = a.out_rows[min(p + i, p_end - 1)];
      }
    }
  };
  auto load = [&](Stage& S, const Idx& I) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (QUAD) {
        S.x[i] = *reinterpret_cast<const v4f_any*>(reinterpret_cast<const char*>(x) +
                                                   (uint64_t)(uint32_t)I.r[i] * bx);
        S.d[i] = *reinterpret_cast<const v4f_any*>(reinterpret_cast<const char*>(dyb) +
                                                   (uint64_t)(uint32_t)I.o[i] * bd);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          S.x[i][e] = x[I.r[i] * ldx + cx[e]];
          S.d[i][e] = dyb[I.o[i] * ldd + cd[e]];
        }
      }
    }
  };
  // the MFMA operands of the two tiles
  Seen tiles[4];  // x's and dy's operand tiles (split.h)
  auto operands = [&](const v4f (&v)[4], v4u (&f)[2][3]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t p[3], q[3];
        split2(v[2 * j][2 * t], v[2 * j + 1][2 * t], p[0], p[1], p[2]);
        split2(v[2 * j][2 * t + 1], v[2 * j + 1][2 * t + 1], q[0], q[1], q[2]);
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const auto r = __builtin_amdgcn_permlane16_swap(p[s], q[s], false, false);
          f[t][s][j] = r[0];
          f[t][s][2 + j] = r[1];
        }
      }
  };
  v16f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  v4f tsum = {0.f, 0.f, 0.f, 0.f};  // the lane's channels of dy over its pairs
  int64_t p0 = p_begin + DW_ST * w;
  if (p0 < p_end) {
    constexpr int STEP = 4 * DW_ST;
    Stage S;
    Idx I;
    load_idx(I, p0);
    load(S, I);
    load_idx(I, min(p0 + STEP, p_end - 1));
    while (true) {
      v4u X[2][3], D[2][3];
      if (p0 + DW_ST > p_end) {  // the chunk's last stage: pairs past it are zero
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            S.d[i][e] = p0 + 4 * pg + i < p_end ? S.d[i][e] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          S.x[i][e] = fmaf(S.x[i][e], sgn, gs[e]);  // +-(x - g_in), rounded once
          tsum[e] += S.d[i][e];
        }
      operands(S.x, X);
      operands(S.d, D);
      // the next stage's rows, and the indices after them, are on their way
      // during this one's products (past the chunk: its last pairs, unused)
      load(S, I);
      p0 += STEP;
      load_idx(I, min(p0 + STEP, p_end - 1));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < SPLIT_PROD; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = mfma_bf16(X[i][split_a(q)], D[j][split_b(q)], acc[i][j]);
      // under the products (a branch before them would part the loads from the
      // splits)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        tiles[t].add(X[t][0]);
        tiles[2 + t].add(D[t][0]);
      }
      if (p0 >= p_end) break;
    }
  }
  // Add the four waves' blocks, tile row i of x at a time.  Register 4 v + z of
  // tile (i, j) holds operand row 8 v + 4 h + z of x and n32 of dy.
  float* const out = a.part + ((int64_t)k * a.maxc + c) * a.Cin * a.Cout;
  const int n32 = lane & 31, h = lane >> 5;
  // over the lanes of a channel quad (pairs in a fixed order)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float t1 = __shfl_xor(tsum[e], 16, 64);
    const float s1 = pg & 1 ? t1 + tsum[e] : tsum[e] + t1;
    const float t2 = __shfl_xor(s1, 32, 64);
    if (pg == 0) redT[w * 64 + 4 * cq + e] = s1 + t2;
  }
  if (lane == 0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      seen[t][0][w] = tiles[t].any32();
      seen[t][1][w] = tiles[t].big32();
    }
    some[w] = (tiles[0].any32() & ~tiles[0].big32()) | (tiles[1].any32() & ~tiles[1].big32()) |
              (tiles[2].any32() & ~tiles[2].big32()) | (tiles[3].any32() & ~tiles[3].big32());
  }
  auto put = [&](int i, int e, float v) {  // operand row e / 64 of tile i, column e % 64
    const int m = e / 64, sx = 4 * (m & 15) + 2 * i + (m >> 4);
    if (slot_live<QUAD>(sx, ci0, a.Cin) && slot_live<QUAD>(tid & 63, co0, a.Cout))
      out[(int64_t)slot_channel<QUAD>(sx, ci0, a.Cin) * a.Cout +
          slot_channel<QUAD>(tid & 63, co0, a.Cout)] = v;
  };
  uint32_t odd = 0;  // which of the thread's sums are not finite
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (i) __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        red[w * 2048 + (8 * (r >> 2) + 4 * h + (r & 3)) * 64 + 4 * (n32 & 15) + 2 * j +
            (n32 >> 4)] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = u * NT + tid;
      const float v = (red[e] - red[2048 + e]) + (red[4096 + e] - red[6144 + e]);
      odd |= v * 0.f == 0.f ? 0u : 1u << (8 * i + u);
      put(i, e, v);
    }
  }
  if (ci0 == 0 && tid < 64 && slot_live<QUAD>(tid, co0, a.Cout))
    a.partT[((int64_t)k * a.maxc + c) * a.Cout + slot_channel<QUAD>(tid, co0, a.Cout)] =
        ((redT[tid] + redT[64 + tid]) + redT[128 + tid]) + redT[192 + tid];
  // Sums of operands that the split cannot hold again, on the fp32 matrix
  // instruction: waves 0 and 1 take the columns' halves of the first half of the
  // pairs, 2 and 3 of the second.  (All of them NaN, 64 -> 64 on 90k sites: 395
  // us, 112 finite.)
  if (!__syncthreads_or(odd != 0 || (some[0] | some[1] | some[2] | some[3]) != 0)) return;
  auto tiny = [&](int t, int row) {  // row of operand tile t
    const uint32_t(&q)[2][4] = seen[t];
    return ((q[0][0] | q[0][1] | q[0][2] | q[0][3]) & ~(q[1][0] | q[1][1] | q[1][2] | q[1][3])) >>
               row & 1;
  };
  const bool td = tiny(2 + (tid >> 1 & 1), ((tid & 63) >> 2) + 16 * (tid & 1));
#pragma unroll 1
  for (int i = 0; i < 2; ++i) {
    const int64_t half = (p_end - p_begin + 1) / 2;
    const int64_t p1 = w >> 1 ? p_end : p_begin + half;
    const int ci = slot_channel<QUAD>(4 * (n32 & 15) + 2 * i + (n32 >> 4), ci0, a.Cin);
    const int co = slot_channel<QUAD>(32 * (w & 1) + n32, co0, a.Cout);
    const float g = a.g_in[ci];
    v16f s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll 1
    for (int64_t p = w >> 1 ? p_begin + half : p_begin; p < p1; p += 8) {
      float xv[4], dv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t q = p + 2 * u + h, qq = min(q, p1 - 1);
        xv[u] = a.x[a.in_rows[qq] * ldx + ci] - g;
        dv[u] = a.dyb[a.out_rows[qq] * ldd + co];
        xv[u] = q < p1 ? xv[u] : 0.f;
        dv[u] = q < p1 ? dv[u] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(xv[u], dv[u], s, 0, 0, 0);
    }
    __syncthreads();  // the sums before have been read
#pragma unroll
    for (int r = 0; r < 16; ++r)
      red[(w >> 1) * 2048 + (8 * (r >> 2) + 4 * h + (r & 3)) * 64 + 32 * (w & 1) + n32] = s[r];
    __syncthreads();
#pragma unroll 1
    for (int u = 0; u < 8; ++u) {
      const int e = u * NT + tid;
      if ((odd >> (8 * i + u) & 1) || td || tiny(i, e / 64)) put(i, e, red[e] + red[2048 + e]);
    }
  }
}

// dW[k][ci][co] = sum_c part + g_in[ci] * u0[co];  T[k][co] = sum_c partT.
// A block covers RED_E consecutive elements; thread group g (of RED_G) sums
// the chunks c = g (mod RED_G) in ascending order, and the group sums are
// added in group order (a fixed order, so the result is deterministic).
constexpr int RED_E = 32, RED_G = 8;
__global__ void __launch_bounds__(RED_E * RED_G) dw_reduce_kernel(
    const float* __restrict__ part, const float* __restrict__ partT,
    const int64_t* __restrict__ off, int K, int Cin, int Cout, int64_t chp, int64_t maxc,
    const float* __restrict__ g_in, const float* __restrict__ u0, float* __restrict__ dW,
    float* __restrict__ T) {
  __shared__ float red[2][RED_G][RED_E];
  const int le = threadIdx.x % RED_E, g = threadIdx.x / RED_E;
  const int64_t i = (int64_t)blockIdx.x * RED_E + le;
  const int64_t per = (int64_t)Cin * Cout;
  float s = 0.f, t = 0.f;
  if (i < (int64_t)K * per) {
    const int k = (int)(i / per);
    const int64_t e = i - k * per;
    const int64_t nch = ceil_div(off[k + 1] - off[k], chp);
    const float* p = part + (int64_t)k * maxc * per + e;
#pragma unroll 4
    for (int64_t c = g; c < nch; c += RED_G) s += p[c * per];
  }
  if (i < (int64_t)K * Cout) {
    const int k = (int)(i / Cout), co = (int)(i % Cout);
    const int64_t nch = ceil_div(off[k + 1] - off[k], chp);
    for (int64_t c = g; c < nch; c += RED_G) t += partT[((int64_t)k * maxc + c) * Cout + co];
  }
  red[0][g][le] = s;
  red[1][g][le] = t;
  __syncthreads();
  if (g != 0) return;
  s = red[0][0][le];
  t = red[1][0][le];
#pragma unroll
  for (int h = 1; h < RED_G; ++h) {
    s += red[0][h][le];
    t += red[1][h][le];
  }
  if (i < (int64_t)K * per && dW) {
    const int64_t e = i % per;
    const int ci = (int)(e / Cout), co = (int)(e - (int64_t)ci * Cout);
    dW[i] = s + g_in[ci] * u0[co];
  }
  if (i < (int64_t)K * Cout) T[i] = t;
}

// dg_in[ci] = sum_k sum_co W[k][ci][co] * (u0[co] - T[k][co]); one block per ci,
// fixed-order tree over the block.
__global__ void __launch_bounds__(256) dgin_kernel(const float* __restrict__ W,
                                                   const float* __restrict__ u0,
                                                   const float* __restrict__ T, int K, int Cin,
                                                   int Cout, float* __restrict__ dg_in) {
  __shared__ float red[256];
  const int ci = blockIdx.x;
  const int64_t n = (int64_t)K * Cout;
  float s = 0.f;
  for (int64_t i = threadIdx.x; i < n; i += 256) {
    const int k = (int)(i / Cout), co = (int)(i - (int64_t)k * Cout);
    s = fmaf(W[((int64_t)k * Cin + ci) * Cout + co], u0[co] - T[i], s);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) dg_in[ci] = red[0];
}

// Work-groups of the weight-gradient kernel that run at once on the current
// device (per-CU occupancy times CUs), cached per device.
int dw_slots() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (cached[dev]) return cached[dev];
  int per_cu = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &per_cu, reinterpret_cast<const void*>(dw_partial_kernel<true>), NT, 0) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus < 1)
    cus = 1;
  (void)hipGetLastError();
  cached[dev] = per_cu * cus;
  return cached[dev];
}

// The (offset, chunk, column block) work items fill DW_ROUNDS whole rounds of
// the concurrent work-groups: each offset's list is cut into at most
// DW_ROUNDS * slots / (K * blocks) chunks, so the last round is nearly full
// instead of holding a few stragglers that would take a round's time alone.
// Chunks of up to DW_SMALL pairs grow first until one round holds them all: a
// work-group's sums over its waves and its share of the reduction cost as much
// as four stages (3x3x3, 16 -> 32 channels, 14k outputs: 37 us in 64-pair
// chunks, 29 so; the whole gradient without dx).
constexpr int DW_ROUNDS = 4;
constexpr int64_t DW_SMALL = 256;

// Which kernel takes the input gradient: the tile kernels read rows of at least
// four channels.
bool tile_dx(const scn_rulebook* rb, int Cout) { return rb->s == 1 && Cout >= 4; }

struct BwdLayout {
  int64_t chp, maxc, nblk;
  size_t o_dyb, o_part, o_partT, o_partS, o_S, o_u0, o_T, o_wp, o_gz, o_few, total;
};

BwdLayout bwd_layout(const scn_rulebook* rb, int Cin, int Cout, uint32_t flags) {
  BwdLayout L{};
  int64_t pmax = 0;
  for (int k = 0; k < rb->K; ++k) pmax = std::max(pmax, rb->off_host[k + 1] - rb->off_host[k]);
  const int64_t blocks = ceil_div(Cin, 64) * ceil_div(Cout, 64);
  const int64_t target = std::max<int64_t>(1, DW_ROUNDS * (int64_t)dw_slots() / (rb->K * blocks));
  const int64_t per = ceil_div(std::max<int64_t>(pmax, 1), target);
  const int64_t fit = std::max<int64_t>(1, (int64_t)dw_slots() / (rb->K * blocks));
  const int64_t one = std::min(DW_SMALL, ceil_div(std::max<int64_t>(pmax, 1), fit));
  L.chp = ceil_div(std::max(per, one), DW_SC) * DW_SC;
  L.maxc = std::max<int64_t>(1, ceil_div(pmax, L.chp));
  L.nblk = std::max<int64_t>(1, ceil_div(rb->a_out, RB_ROWS));
  auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
  size_t cur = 0;
  L.o_dyb = cur;
  cur += (flags & SCN_RELU) ? al((size_t)rb->a_out * Cout * 4) : 0;
  L.o_part = cur;
  cur += al((size_t)rb->K * L.maxc * Cin * Cout * 4);
  L.o_partT = cur;
  cur += al((size_t)rb->K * L.maxc * Cout * 4);
  L.o_partS = cur;
  cur += al((size_t)L.nblk * Cout * 4);
  L.o_S = cur;
  cur += al((size_t)Cout * 4);
  L.o_u0 = cur;
  cur += al((size_t)Cout * 4);
  L.o_T = cur;
  cur += al((size_t)rb->K * Cout * 4);
  L.o_wp = cur;
  cur += al(tile_dx(rb, Cout) ? tile_pack_bytes(rb->K, Cout, Cin)
                       : (size_t)rb->K * ceil_div(Cin, 64) * 64 * ceil_div(Cout, 16) * 16 * 4);
  L.o_gz = cur;
  cur += al(std::max((size_t)rb->K * ceil_div(Cin, 64) * 64, (size_t)TILE_PAD) * 4);
  L.o_few = cur;
  if (rb->s == 1 && few_channels(rb->K, Cin))
    cur += al((size_t)few_groups(rb->a_out) * ((size_t)rb->K * Cin + 1) * Cout * 4);
  L.total = cur;
  return L;
}

}  // namespace
}  // namespace scn

using namespace scn;

// Measurement hook (scn_set_kernel_timer): per host thread, pairs of the
// caller's events recorded on the call's stream around the contraction
// kernels: [0, 1] the forward, [2, 3] the input gradient, [4, 5] the weight
// gradient's partial products.
enum TimedKernel { TK_FWD = 0, TK_DX = 1, TK_DW = 2 };
static thread_local hipEvent_t g_kernel_timer[6] = {};

static scn_status timer_mark(TimedKernel k, int end, hipStream_t st) {
  hipEvent_t e = g_kernel_timer[2 * k + end];
  if (e) SCN_HIP(hipEventRecord(e, st));
  return SCN_OK;
}

// The forward's scratch: gw [K][NcP] and g_pre [NcP] (256-byte aligned),
// then the packed weights [K][NcP][RkP].  Every element is written by the
// forward's first kernels before any is read.
// Which kernel takes a forward.
enum class Fwd { few, tile, dense, gather };

// The tile kernels multiply every row of a tile at every offset of any of its
// rows, on the split products; the fp32 kernels multiply fewer rows that lack
// the offset.  All lines below are measured, the tile kernels against the fp32
// kernels, on shells, walks, patches and pooled shells of 1k to 3.6M outputs.
// `fill` is the active share of the (output, offset) entries.
//  - few_forward: Cin <= 2 takes 0.39 to 0.98 of the fp32 kernels' time, but
//    with the mask-sorted view more channels win only where masks repeat (3 ->
//    32: 0.6 to 0.9 from a fill of 0.5, 1.07 to 1.18 below; past 64 entries its
//    window values leave one work-group per CU: 1.2 to 1.7).
//  - View: a tile's rows share their masks, so the tile kernel wins where it
//    has products to do (64 -> 64: 0.83 to 1.01, 96 -> 128: 0.66 to 0.82) or
//    a fill of 0.7 (0.6 to 0.99).  The 32-row fp32 kernel, without a barrier per
//    item, wins with one column block and little to multiply per item: items
//    of one step (16 -> 64: tile 1.04 to 1.24, 48 -> 64: 1.02 to 1.31, 20 -> 64:
//    1.2 to 1.5, 112 -> 64: 0.98 to 1.38), rows not on 64 bytes (56 -> 64: 0.9 to
//    1.14), 32 channels, few offsets and outputs (32 -> 32: 1.07 to 1.18, 1.02 to
//    1.05 at 27 offsets; 32 -> 64: 0.96 to 1.1).  It reads rows 16 bytes at a
//    time.
//  - Lists: tiles of consecutive outputs are about as full as the list, and the
//    gather kernel multiplies active pairs alone, at 0.4 of the rate.  What it
//    saves of the tile kernel's steps (64 rows x 64 columns x 16 channels) has
//    to pay its three more launches, about 5500 steps of full tiles.  3x3x3
//    shells (fill 0.22): 64 -> 64 on 453k outputs 547 us in tiles, 373 from
//    pairs; on 14k 49 and 69.
Fwd fwd_route(const scn_rulebook* rb, const float* x, int Cin, int Cout) {
  if (rb->s != 1) return Fwd::gather;
  const double fill = (double)rb->n_pairs / ((double)rb->K * std::max<int64_t>(rb->a_out, 1));
  const int nst = tile_steps(Cin);
  if (rb->fnb) {
    const bool vec = Cin % 4 == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0;
    if (few_channels(rb->K, Cin) && (Cin <= 2 || (fill >= 0.5 && rb->K * Cin <= 64)))
      return Fwd::few;
    // four channels at 27 offsets: one chain over all of a row's products rounds
    // more often than the fp32 kernel (9.8e-8 off 64-bit sums, 8.8e-8)
    if (Cin < 4 || (Cin == 4 && rb->K * Cin > 96 && vec)) return Fwd::dense;
    const bool thin = Cin < 32 || (Cin == 32 && rb->K < 16 && Cout <= 32) ||
                      (nst % 2 && nst <= DENSE_STEPS) || (nst == 4 && Cin < 64);
    return vec && thin && Cout <= 64 && fill < 0.7 ? Fwd::dense : Fwd::tile;
  }
  if (few_channels(rb->K, Cin)) return Fwd::few;
  const double steps = (double)ceil_div(rb->a_out, TILE) * ceil_div(Cout, 64) * rb->K * nst;
  return steps * (0.4 - fill) >= 5500. ? Fwd::gather : Fwd::tile;
}

struct FwdScratch {
  Fwd route;
  int RkP, NcP;
  size_t gw_bytes, total;
  size_t bound;  // what scn_conv_fwd_noalloc limits: fp32 weights on padded tiles
};

static FwdScratch fwd_scratch(const scn_rulebook* rb, const float* x, int Cin, int Cout) {
  FwdScratch f;
  f.RkP = (int)ceil_div(Cin, 16) * 16;
  f.NcP = (int)ceil_div(Cout, 64) * 64;
  f.gw_bytes = ((size_t)(rb->K + 1) * f.NcP * sizeof(float) + 255) & ~size_t(255);
  f.route = fwd_route(rb, x, Cin, Cout);
  f.total = f.bound = f.gw_bytes + (size_t)rb->K * f.NcP * f.RkP * sizeof(float);
  if (f.route == Fwd::few || f.route == Fwd::tile)
    f.total = f.gw_bytes + TILE_PAD * sizeof(float) +
              (f.route == Fwd::few ? tile_pack_bytes(1, rb->K * Cin, Cout)
                                   : tile_pack_bytes(rb->K, Cin, Cout));
  return f;
}

static scn_status fwd_check(const char* who, const scn_rulebook* rb, const float* x,
                            const float* g_in, const float* W, int32_t Cin, int32_t Cout,
                            float* y, float* g_out) {
  if (!rb || !g_in || !W || !g_out || Cin < 1 || Cout < 1 || (rb->a_in > 0 && !x) ||
      (rb->a_out > 0 && !y)) {
    set_error("%s: invalid argument", who);
    return SCN_ERR_INVALID;
  }
  if (Cin > 256) {
    set_error("%s: Cin %d > 256 is not supported", who, Cin);
    return SCN_ERR_UNSUPPORTED;
  }
  return SCN_OK;
}

// Steps 2-3 with the ground state, on a scratch block laid out as FwdScratch.
static scn_status fwd_run(const scn_rulebook* rb, const float* x, const float* g_in,
                          const float* W, const float* bias, int32_t Cin, int32_t Cout,
                          uint32_t flags, float* y, float* g_out, hipStream_t st,
                          const FwdScratch& fs, float* gw) {
  const int relu = (flags & SCN_RELU) ? 1 : 0;
  const int RkP = fs.RkP, NcP = fs.NcP;
  float* const gpre = gw + (size_t)rb->K * NcP;
  float* Wp = reinterpret_cast<float*>(reinterpret_cast<char*>(gw) + fs.gw_bytes);
  if (fs.route == Fwd::few || fs.route == Fwd::tile) {
    float* const sub = Wp;  // the shifted rows' g_in, then the split weights
    uint32_t* const Ws = reinterpret_cast<uint32_t*>(Wp + TILE_PAD);
    const bool few = fs.route == Fwd::few;
    if (scn_status rc = tile_pack(W, (int64_t)Cin * Cout, Cout, 1, few ? 1 : rb->K,
                                  few ? rb->K * Cin : Cin, Cout, !few, g_in, Cin, bias, relu, Ws,
                                  sub, gpre, g_out, st))
      return rc;
    TileArgs t{};
    t.src = x;
    t.sub = sub;
    t.subtract = 1;
    t.Wp = Ws;
    t.wtiny = tile_wtiny(Ws, few ? 1 : rb->K, few ? rb->K * Cin : Cin, Cout);
    t.W = W;
    t.wk = (int64_t)Cin * Cout;
    t.wj = Cout;
    t.wn = 1;
    t.gidx = rb->in_rows;
    t.aidx = rb->out_rows;
    t.tpos = rb->otile;
    t.nb = rb->fnb;
    t.nb_off = rb->fnb_off;
    t.fperm = rb->fperm;
    t.fmask = rb->fmask;
    t.nsrc = rb->a_in;
    t.npairs = rb->n_pairs;
    t.ntile = ceil_div(rb->a_out, TILE);
    t.nrows = rb->a_out;
    t.K = rb->K;
    t.Rk = Cin;
    t.Nc = Cout;
    t.add = gpre;
    t.relu = relu;
    t.dst = y;
    scn_status rc;
    if ((rc = timer_mark(TK_FWD, 0, st)) || (rc = few ? few_forward(t, st) : launch_tile(t, st)))
      return rc;
    return timer_mark(TK_FWD, 1, st);
  }
  hipLaunchKernelGGL(pack_w_kernel, dim3((unsigned)ceil_div((int64_t)rb->K * NcP * RkP, 256)),
                     dim3(256), 0, st, W, rb->K, Cin, Cout, 1, RkP, NcP, Wp);
  SCN_LAUNCH_CHECK();
  hipLaunchKernelGGL(ground_w_kernel, dim3((unsigned)(rb->K * (NcP / 64))), dim3(256), 0, st,
                     g_in, W, rb->K, Cin, Cout, NcP, gw);
  SCN_LAUNCH_CHECK();
  hipLaunchKernelGGL(ground_pre_kernel, dim3((unsigned)ceil_div(Cout, 64)), dim3(64), 0, st, gw,
                     NcP, bias, rb->K, Cout, relu, gpre, g_out);
  SCN_LAUNCH_CHECK();
  if (fs.route == Fwd::dense) {
    DenseArgs d{};
    d.x = x;
    d.g_in = g_in;
    d.Wp = Wp;
    d.add = gpre;
    d.nb = rb->fnb;
    d.nb_off = rb->fnb_off;
    d.fperm = rb->fperm;
    d.fmask = rb->fmask;
    d.y = y;
    d.a_out = rb->a_out;
    d.nblk = rb->n_fblocks;
    d.K = rb->K;
    d.Cin = Cin;
    d.Cout = Cout;
    d.NcP = NcP;
    d.relu = relu;
    scn_status rc;
    if ((rc = timer_mark(TK_FWD, 0, st)) || (rc = launch_dense(d, st))) return rc;
    return timer_mark(TK_FWD, 1, st);
  }
  GatherArgs a{};
  a.src = x;
  a.gidx = rb->in_rows;
  a.aidx = rb->out_rows;
  a.tpos = rb->otile;
  a.ntile = rb->n_otiles;
  a.Wp = Wp;
  a.gwp = gw;
  a.NcP = NcP;
  a.Rk = Cin;
  a.Nc = Cout;
  a.add = gpre;
  a.relu = relu;
  a.dst = y;
  a.wmap = nullptr;
  a.nrows = rb->a_out;
  a.K = rb->K;
  scn_status rc;
  if ((rc = timer_mark(TK_FWD, 0, st)) || (rc = launch_gather(a, st))) return rc;
  return timer_mark(TK_FWD, 1, st);
}

// Scratch of scn_conv_fwd_noalloc: one array per GPU the library runs on,
// held until the process ends.  In host code its name is not a device
// address; the address each device gives it (hipGetSymbolAddress, once per
// device) is what kernels and copies get.
constexpr size_t NOALLOC_MAX_BYTES = size_t(8) << 20;
constexpr size_t NOALLOC_SCRATCH_BYTES = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[64] = {};

static scn_status noalloc_scratch(void** out) {
  int dev = 0;
  SCN_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) {
    set_error("scn_conv_fwd_noalloc: device %d out of range", dev);
    return SCN_ERR_HIP;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    SCN_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) {
      set_error("scn_conv_fwd_noalloc: no device address for the scratch array");
      return SCN_ERR_HIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return SCN_OK;
}

extern "C" {

scn_status scn_conv_fwd(const scn_rulebook* rb, const float* x, const float* g_in,
                        const float* W, const float* bias, int32_t Cin, int32_t Cout,
                        uint32_t flags, float* y, float* g_out, hipStream_t st) {
  clear_error();
  if (scn_status rc0 = after_build(rb, st)) return rc0;
  if (scn_status rc0 = fwd_check("scn_conv_fwd", rb, x, g_in, W, Cin, Cout, y, g_out))
    return rc0;
  const FwdScratch fs = fwd_scratch(rb, x, Cin, Cout);
  float* gw = nullptr;
  const Allocator al = current_allocator();
  scn_status rc = dalloc(reinterpret_cast<void**>(&gw), fs.total, st, al);
  if (rc) return rc;
  struct Free {
    float* p;
    hipStream_t s;
    Allocator al;
    ~Free() { dfree(p, s, al); }
  } free_gw{gw, st, al};
  return fwd_run(rb, x, g_in, W, bias, Cin, Cout, flags, y, g_out, st, fs, gw);
}

size_t scn_conv_fwd_noalloc_max_bytes(void) { return NOALLOC_MAX_BYTES; }

scn_status scn_set_kernel_timer(const hipEvent_t* events) {
  for (int i = 0; i < 6; ++i) g_kernel_timer[i] = events ? events[i] : nullptr;
  return SCN_OK;
}

scn_status scn_conv_fwd_noalloc(const scn_rulebook* rb, const float* x, const float* g_in,
                                const float* W, const float* bias, int32_t Cin, int32_t Cout,
                                uint32_t flags, float* y, float* g_out, hipStream_t st) {
  clear_error();
  if (scn_status rc0 = after_build(rb, st)) return rc0;
  if (scn_status rc0 = fwd_check("scn_conv_fwd_noalloc", rb, x, g_in, W, Cin, Cout, y, g_out))
    return rc0;
  const FwdScratch fs = fwd_scratch(rb, x, Cin, Cout);
  if (fs.bound > NOALLOC_MAX_BYTES || fs.total > NOALLOC_SCRATCH_BYTES) {
    set_error("scn_conv_fwd_noalloc: K=%d Cin=%d Cout=%d needs %zu bytes of scratch, more than "
              "the %zu the library holds",
              rb->K, Cin, Cout, fs.bound, NOALLOC_MAX_BYTES);
    return SCN_ERR_WORKSPACE;
  }
  void* base = nullptr;
  if (scn_status rc0 = noalloc_scratch(&base)) return rc0;
  return fwd_run(rb, x, g_in, W, bias, Cin, Cout, flags, y, g_out, st, fs,
                 static_cast<float*>(base));
}

size_t scn_conv_bwd_workspace_bytes(const scn_rulebook* rb, int32_t Cin, int32_t Cout,
                                    uint32_t flags) {
  if (!rb || Cin < 1 || Cout < 1) return 0;
  return bwd_layout(rb, Cin, Cout, flags).total;
}

scn_status scn_conv_bwd(const scn_rulebook* rb, const float* x, const float* g_in,
                        const float* W, const float* y, const float* g_out, const float* dy,
                        const float* dg_out, int32_t Cin, int32_t Cout, uint32_t flags,
                        float* dx, float* dg_in, float* dW, float* dbias, void* ws,
                        size_t ws_bytes, hipStream_t st) {
  clear_error();
  if (scn_status rc0 = after_build(rb, st)) return rc0;
  const int relu = (flags & SCN_RELU) ? 1 : 0;
  if (!rb || !g_in || !W || Cin < 1 || Cout < 1 || (rb->a_out > 0 && !dy) ||
      (rb->a_in > 0 && !x) || (relu && rb->a_out > 0 && !y) || (relu && dg_out && !g_out)) {
    set_error("scn_conv_bwd: invalid argument");
    return SCN_ERR_INVALID;
  }
  if (Cin > 256 || Cout > 256) {
    set_error("scn_conv_bwd: channels > 256 are not supported");
    return SCN_ERR_UNSUPPORTED;
  }
  const BwdLayout L = bwd_layout(rb, Cin, Cout, flags);
  if (!ws || ws_bytes < L.total) {
    set_error("scn_conv_bwd: workspace of %zu bytes needed, %zu given", L.total, ws_bytes);
    return SCN_ERR_WORKSPACE;
  }
  char* base = static_cast<char*>(ws);
  float* dyb = relu ? reinterpret_cast<float*>(base + L.o_dyb) : const_cast<float*>(dy);
  float* part = reinterpret_cast<float*>(base + L.o_part);
  float* partT = reinterpret_cast<float*>(base + L.o_partT);
  float* partS = reinterpret_cast<float*>(base + L.o_partS);
  float* S = reinterpret_cast<float*>(base + L.o_S);
  float* u0 = reinterpret_cast<float*>(base + L.o_u0);
  float* T = reinterpret_cast<float*>(base + L.o_T);
  float* wpack = reinterpret_cast<float*>(base + L.o_wp);
  float* gzero = reinterpret_cast<float*>(base + L.o_gz);
  const int K = rb->K;

  // A first layer's weight and bias gradients (few channels, no dx, no dg_in)
  // read dy and y once, with no masked copy and no gathers of their rows.
  if (rb->s == 1 && dW && !dx && !dg_in && few_channels(K, Cin)) {
    TileArgs t{};
    t.src = x;
    t.sub = g_in;
    t.gidx = rb->in_rows;
    t.aidx = rb->out_rows;
    t.tpos = rb->otile;
    t.nb = rb->fnb;
    t.nb_off = rb->fnb_off;
    t.fperm = rb->fperm;
    t.fmask = rb->fmask;
    t.nsrc = rb->a_in;
    t.npairs = rb->n_pairs;
    t.ntile = ceil_div(rb->a_out, TILE);
    t.nrows = rb->a_out;
    t.K = K;
    t.Rk = Cin;
    t.Nc = Cout;
    const float* const mask = relu ? y : nullptr;
    float* const fpart = reinterpret_cast<float*>(base + L.o_few);
    float* const fS = fpart + (size_t)few_groups(rb->a_out) * K * Cin * Cout;
    scn_status rc;
    if ((rc = timer_mark(TK_DW, 0, st)) ||
        (rc = few_partials(t, dy, mask, Cout, fpart, fS, st)) || (rc = timer_mark(TK_DW, 1, st)))
      return rc;
    hipLaunchKernelGGL(finish_vec_kernel, dim3((unsigned)Cout), dim3(NT), 0, st, fS,
                       rb->a_out > 0 ? (int64_t)few_groups(rb->a_out) : 0, Cout, g_out, dg_out,
                       relu, S, u0, dbias);
    SCN_LAUNCH_CHECK();
    return few_reduce(t, Cout, fpart, u0, dW, st);
  }

  // dȳ and S (column sums over active outputs)
  if (rb->a_out > 0) {
    const bool v4 = (Cout % 4 == 0) && Cout <= 4 * NT &&
                    ((reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(y) |
                      reinterpret_cast<uintptr_t>(ws)) & 15) == 0;
    if (v4)
      hipLaunchKernelGGL(colsum_vec_kernel, dim3((unsigned)L.nblk), dim3(NT), 0, st,
                         reinterpret_cast<const float4*>(dy), reinterpret_cast<const float4*>(y),
                         relu, rb->a_out, Cout / 4, reinterpret_cast<float4*>(dyb),
                         reinterpret_cast<float4*>(partS));
    else
      hipLaunchKernelGGL(colsum_kernel, dim3((unsigned)L.nblk), dim3(NT), 0, st, dy, y, relu,
                         rb->a_out, Cout, dyb, partS);
    SCN_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(finish_vec_kernel, dim3((unsigned)Cout), dim3(NT), 0, st, partS,
                     rb->a_out > 0 ? L.nblk : 0, Cout, g_out, dg_out, relu, S, u0, dbias);
  SCN_LAUNCH_CHECK();

  // input gradient: accumulate over input ranks with W_k^T
  if (dx && rb->a_in > 0 && tile_dx(rb, Cout)) {
    scn_status rc = tile_pack(W, (int64_t)Cin * Cout, 1, Cout, K, Cout, Cin, true, nullptr,
                              1, nullptr, 0, reinterpret_cast<uint32_t*>(wpack), gzero, nullptr,
                              nullptr, st);
    if (rc) return rc;
    TileArgs a{};
    a.src = dyb;
    a.sub = gzero;
    a.Wp = reinterpret_cast<uint32_t*>(wpack);
    a.wtiny = tile_wtiny(a.Wp, K, Cout, Cin);
    a.W = W;
    a.wk = (int64_t)Cin * Cout;
    a.wj = 1;
    a.wn = Cout;
    a.gidx = rb->out_rows;
    a.aidx = rb->in_rank;
    a.tpos = rb->itile;
    a.nsrc = rb->a_out;
    a.npairs = rb->n_pairs;
    a.ntile = rb->n_itiles;
    a.nrows = rb->a_in;
    a.K = K;
    a.Rk = Cout;
    a.Nc = Cin;
    a.dst = dx;
    a.wmap = rb->input_sorted ? nullptr : rb->perm;
    if ((rc = timer_mark(TK_DX, 0, st)) || (rc = launch_tile(a, st)) ||
        (rc = timer_mark(TK_DX, 1, st)))
      return rc;
  } else if (dx && rb->a_in > 0) {
    GatherArgs a{};
    a.src = dyb;
    a.gidx = rb->out_rows;
    a.aidx = rb->in_rank;
    a.tpos = rb->itile;
    a.ntile = rb->n_itiles;
    const int RkP = (int)ceil_div(Cout, 16) * 16, NcP = (int)ceil_div(Cin, 64) * 64;
    hipLaunchKernelGGL(pack_w_kernel, dim3((unsigned)ceil_div((int64_t)K * NcP * RkP, 256)),
                       dim3(256), 0, st, W, K, Cin, Cout, 0, RkP, NcP, wpack);
    SCN_LAUNCH_CHECK();
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)ceil_div((int64_t)K * NcP, 256)), dim3(256), 0,
                       st, gzero, (int64_t)K * NcP);
    SCN_LAUNCH_CHECK();
    a.Wp = wpack;  // W_k(j = output channel, n = input channel) = W[k][n][j]
    a.gwp = gzero;
    a.NcP = NcP;
    a.Rk = Cout;
    a.Nc = Cin;
    a.add = nullptr;
    a.relu = 0;
    a.dst = dx;
    a.wmap = rb->input_sorted ? nullptr : rb->perm;
    a.nrows = rb->a_in;
    a.K = K;
    scn_status rc;
    if ((rc = timer_mark(TK_DX, 0, st)) || (rc = launch_gather(a, st)) ||
        (rc = timer_mark(TK_DX, 1, st)))
      return rc;
  }

  // weight gradient partials (also the per-offset column sums T_k)
  if (dW || dg_in) {
    DwArgs d{};
    d.x = x;
    d.dyb = dyb;
    d.g_in = g_in;
    d.in_rows = rb->in_rows;
    d.out_rows = rb->out_rows;
    d.off = rb->off_dev;
    d.K = K;
    d.Cin = Cin;
    d.Cout = Cout;
    d.nco = (int)ceil_div(Cout, 64);
    d.nblk = (int)ceil_div(Cin, 64) * d.nco;
    d.chp = L.chp;
    d.maxc = L.maxc;
    d.part = part;
    d.partT = partT;
    if (rb->n_pairs > 0) {
      const int64_t nwg = L.maxc * K * d.nblk;
      if (scn_status rc = timer_mark(TK_DW, 0, st)) return rc;
      if (Cin >= 4 && Cout >= 4)
        hipLaunchKernelGGL(dw_partial_kernel<true>, dim3((unsigned)nwg), dim3(NT), 0, st, d);
      else
        hipLaunchKernelGGL(dw_partial_kernel<false>, dim3((unsigned)nwg), dim3(NT), 0, st, d);
      SCN_LAUNCH_CHECK();
      if (scn_status rc = timer_mark(TK_DW, 1, st)) return rc;
    }
    const int64_t nred = std::max<int64_t>((int64_t)K * Cin * Cout, (int64_t)K * Cout);
    hipLaunchKernelGGL(dw_reduce_kernel, dim3((unsigned)ceil_div(nred, RED_E)),
                       dim3(RED_E * RED_G), 0, st,
                       part, partT, rb->off_dev, K, Cin, Cout, L.chp, L.maxc, g_in, u0, dW, T);
    SCN_LAUNCH_CHECK();
    if (dg_in) {
      hipLaunchKernelGGL(dgin_kernel, dim3((unsigned)Cin), dim3(256), 0, st, W, u0, T, K, Cin,
                         Cout, dg_in);
      SCN_LAUNCH_CHECK();
    }
  }
  return SCN_OK;
}

}  // extern "C"
