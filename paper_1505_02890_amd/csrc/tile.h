// The tile contraction (tile.hip): rows gathered through a rulebook times W,
// accumulated per destination row.  Serves the forward and the input gradient
// of stride-1 rulebooks.
#pragma once

#include "scn_internal.h"

namespace scn {

struct TileArgs {
  const float* src;      // gathered rows [nsrc][Rk], Rk >= 4 (launch_tile)
  const float* sub;      // [TILE_PAD] subtracted from every row (zero past Rk); 16-byte aligned
  const uint32_t* Wp;    // split weights (tile_pack)
  const uint32_t* wtiny; // ... per column whether it is tiny, then row_limit (tile_wtiny)
  const float* W;        // the weights themselves: W_k(j, n) = W[k*wk + j*wj + n*wn]
  int64_t wk, wj, wn;
  // Rows from pair lists (nb == null): list k of the rulebook ascends by
  // accumulator row, tpos[k*ntile + t] starts the part of the tile of rows
  // [64t, 64t + 64).
  const int32_t* gidx;   // per pair: row of src
  const int32_t* aidx;   // per pair: accumulator row
  const int64_t* tpos;   // [K*ntile + 1]; null beside the dense forward view
  // Rows from the dense forward view: position p of the mask-sorted order is
  // output row fperm[p], its inputs nb[nb_off[row] ..] in offset order.
  const int32_t* nb;
  const uint32_t* nb_off;
  const int32_t* fperm;
  const uint32_t* fmask;
  int64_t nsrc;          // rows of src
  int64_t npairs;        // pairs of all lists
  int64_t ntile;         // tiles of 64 rows
  int64_t nrows;         // accumulator rows
  int K, Rk, Nc;
  const float* add;      // [Nc] added to every row, or null
  int relu;
  int subtract;          // whether rows are shifted by sub (else sub is all zeros)
  float* dst;            // [nrows][Nc]
  const int32_t* wmap;   // dst row of accumulator row r (null = identity)
};

constexpr int TILE_PAD = 256;  // floats of TileArgs::sub (Rk <= 256, padded to whole chunks)

// 16-channel steps of a reduction of Rk channels, and the bytes of its split
// weights.
int tile_steps(int Rk);
size_t tile_pack_bytes(int K, int Rk, int Nc);
const uint32_t* tile_wtiny(const uint32_t* Wp, int K, int Rk, int Nc);

// Splits W_k(j, n) into a.Wp's layout; fills sub[0 .. TILE_PAD) with g[j % gm]
// (zeros if g is null or past Rk).  With g_pre (else null): g_pre = bias + sum_k g W_k and
// g_out = act(g_pre).  chunks: entries as launch_tile reads rows, else in
// channel order (few_forward).
scn_status tile_pack(const float* W, int64_t wk, int64_t wj, int64_t wn, int K, int Rk, int Nc,
                     bool chunks, const float* g, int gm, const float* bias, int relu,
                     uint32_t* Wp, float* sub, float* g_pre, float* g_out, hipStream_t st);

scn_status launch_tile(const TileArgs& a, hipStream_t st);

// Layers of few input channels, whose offsets join the reduction.  Arguments
// as for launch_tile, but Wp packed from W as one offset of K*Cin entries (gm = Cin).
bool few_channels(int K, int Cin);
scn_status few_forward(const TileArgs& a, hipStream_t st);
// The weight gradient without dx and dg_in, from dy (times y > 0 unless y is
// null): partials part [few_groups][K*Cin][Cout] and column sums partS
// [few_groups][Cout], then dW = their sum + g_in u0.
int few_groups(int64_t nrows);
scn_status few_partials(const TileArgs& a, const float* dy, const float* y, int Cout, float* part,
                        float* partS, hipStream_t st);
scn_status few_reduce(const TileArgs& a, int Cout, const float* part, const float* u0, float* dW,
                      hipStream_t st);

}  // namespace scn
