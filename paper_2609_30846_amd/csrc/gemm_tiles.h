// Tiles of the projection GEMMs: how a product's output is cut into tiles and in which
// order they are dealt, shared by the host, which plans a launch, and the kernel.
#pragma once

#include <math.h>
#include <stdint.h>

#include "ipk_internal.h"

namespace ipk {

// Epilogues of row-major outputs: the requantized int8 values themselves, the residual
// add of Eq. 2 (with z1 laid out as the output), or the integer Swish of Eq. 12 and
// its requantization, applied through a 256-entry table indexed by the biased code.
enum Epilogue { EPI_PLAIN = 0, EPI_RESID = 1, EPI_SWISH = 2 };

// Tiles of TN channels x TM tokens of a product of `nb` utterances x `rows` tokens and N
// channels; no tile straddles two utterances (a product whose utterances may share a tile
// passes all its tokens as one).  Logical order: bands of `band` token tiles,
// channels outer, tokens inner within a band.
struct TileGrid {
  int tiles_n, tiles_m;  // tiles along the channels and along all utterances' tokens
  int tiles_m_per;       // token tiles per utterance
  int band;
  // by band tiles_n, band, the last band's height, tiles_m_per; without the divisors
  // themselves, since every workgroup starts by reading its kernel's arguments: with them (352
  // bytes of arguments instead of 320) a 125-token product took 0.25 us longer
  DivM span, full, last, per;
};

inline TileGrid tile_grid(int nb, int rows, int N, int TN, int TM) {
  TileGrid g;
  g.tiles_n = (N + TN - 1) / TN;
  g.tiles_m_per = (rows + TM - 1) / TM;
  g.tiles_m = nb * g.tiles_m_per;
  const int tiles = g.tiles_n * g.tiles_m;
  // band height: an XCD's share of about tiles/8 tiles covers ~band token tiles and
  // ~share/band channel tiles; weight rows per channel tile (TN) are worth TN/TM
  // token tiles, so the square in bytes has band ~ sqrt(share * TN / TM)
  const double share = (tiles + 7) / 8;
  const int band = (int)(sqrt(share * TN / TM) + 0.5);
  g.band = band < 1 ? 1 : (band > g.tiles_m ? g.tiles_m : band);
  g.span = make_div((uint32_t)(g.band * g.tiles_n)).by;
  g.full = make_div((uint32_t)g.band).by;
  g.last = make_div((uint32_t)(g.tiles_m - (g.tiles_m - 1) / g.band * g.band)).by;
  g.per = make_div((uint32_t)g.tiles_m_per).by;
  return g;
}

// Logical tile `i`: channel tile, utterance, token tile within the utterance.
struct TilePos {
  int nt, ub, mt;
};
__host__ __device__ __forceinline__ TilePos tile_at(const TileGrid& g, int i) {
  const int band_idx = (int)div_u((uint32_t)i, g.span);
  const int in_band = i - band_idx * g.band * g.tiles_n;
  const int rest = g.tiles_m - band_idx * g.band;
  const int nt = (int)div_u((uint32_t)in_band, rest < g.band ? g.last : g.full);
  const int mt = band_idx * g.band + in_band - nt * (rest < g.band ? rest : g.band);
  const int ub = (int)div_u((uint32_t)mt, g.per);
  return TilePos{nt, ub, mt - ub * g.tiles_m_per};
}

// The tile shapes (channels x tokens; four waves, the first eight) and the time model that picks one
// for a launch: ceil(tiles / CUs) tiles pass through the busiest CU, each costing `fixed`
// (its first operands and the epilogue: plain, with the residual add, with the Swish) plus
// `per_k` per 1024 bytes of K, in microseconds fitted to launches of 16 .. 23000 tokens with
// K = 256 .. 4096 and N = 256 .. 4096 (median error 3 %, and nine picks of ten within 5 % of
// the fastest shape).  Large tiles re-use their operands best, small ones spread a short
// call over the chip: 125 tokens x 4096 -> 1024 take 7.8 us in 128 x 32 tiles and 27 us in
// 256 x 128 ones, 23000 tokens 88 us in the latter and 170 us in the former; 2500 tokens
// x 1024 -> 4096 are fastest in between (128 x 64, 15.9 us against 17.3 and 21.6 us).
struct TileShape {
  int tn, tm;
  double fixed[3], per_k;
};
constexpr TileShape kTiles[] = {{256, 256, {4.5, 7.0, 5.5}, 10.2},
                                {256, 128, {2.2, 4.1, 2.8}, 5.2},
                                {256, 64, {1.3, 2.1, 1.45}, 2.9},
                                {128, 64, {0.52, 0.78, 0.62}, 1.92},
                                {64, 64, {0.39, 0.46, 0.41}, 1.47},
                                {128, 32, {0.34, 0.43, 0.31}, 1.40}};
constexpr int kGemmCUs = 256;

// A product's utterances, tokens per utterance and channels.
struct GemmDims {
  int nb, rows, N;
};

// The cheapest shape for one launch of `n` products of contraction length K, among those of
// at least min_tm tokens.
inline int pick_shape(const GemmDims* dims, int n, int K, int min_tm, int epi) {
  int best = -1;
  double best_t = 0.0;
  for (int i = 0; i < (int)(sizeof kTiles / sizeof kTiles[0]); ++i) {
    const TileShape& s = kTiles[i];
    if (s.tm < min_tm) continue;
    long tiles = 0;
    for (int p = 0; p < n; ++p)
      tiles += (long)dims[p].nb * ((dims[p].rows + s.tm - 1) / s.tm) * ((dims[p].N + s.tn - 1) / s.tn);
    const long rounds = (tiles + kGemmCUs - 1) / kGemmCUs;
    // one 256 x 256 workgroup fills a CU: with more than one round its first fetch and
    // epilogue are uncovered (23000 tokens x 1024 -> 4096, six rounds: 120 us against 106 us)
    if (s.tm == 256 && rounds > 1) continue;
    const double t = (double)rounds * (s.fixed[epi] + s.per_k * K / 1024.0);
    if (best < 0 || t < best_t) {
      best = i;
      best_t = t;
    }
  }
  return best;
}

}  // namespace ipk
