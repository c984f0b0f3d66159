// Tiles of the projection GEMMs: how a product's output is cut into tiles and in which
// order they are dealt, shared by the host, which plans a launch, and the kernel.
#pragma once

#include <math.h>
#include <stdint.h>

#include "ipk_internal.h"

namespace ipk {

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

}  // namespace ipk
