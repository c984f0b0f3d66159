// Host-side access to the launch planning of the kernels, for the CPU tests (built by
// host_plans.py from the library's own headers).
#include <stdint.h>

#include <vector>

#include "gemm_tiles.h"

using namespace ipk;

// 0 if the tiles of a product cover its output once each, else 1 + the first logical tile
// whose position lies outside or was taken before.
extern "C" int64_t tile_grid_fault(int nb, int rows, int N, int TN, int TM) {
  const TileGrid g = tile_grid(nb, rows, N, TN, TM);
  const int per = (rows + TM - 1) / TM, tn = (N + TN - 1) / TN;
  const int64_t tiles = (int64_t)nb * per * tn;
  if ((int64_t)g.tiles_n * g.tiles_m != tiles) return 1;
  std::vector<bool> seen(tiles);
  for (int64_t i = 0; i < tiles; ++i) {
    const TilePos p = tile_at(g, (int)i);
    if (p.nt < 0 || p.nt >= tn || p.ub < 0 || p.ub >= nb || p.mt < 0 || p.mt >= per) return 1 + i;
    const int64_t at = ((int64_t)p.ub * per + p.mt) * tn + p.nt;
    if (seen[at]) return 1 + i;
    seen[at] = true;
  }
  return 0;
}

// The first x of `xs` whose quotient by d is wrong, or -1.
extern "C" int64_t div_fault(uint32_t d, const uint32_t* xs, int64_t n) {
  const DivU v = make_div(d);
  for (int64_t i = 0; i < n; ++i)
    if (div_u(xs[i], v) != xs[i] / d) return xs[i];
  return -1;
}

// The tile shape a launch of n products {nb, rows, N} of contraction length K takes.
extern "C" void gemm_shape(const int* dims, int n, int K, int min_tm, int epi, int* tn, int* tm) {
  const int i = pick_shape((const GemmDims*)dims, n, K, min_tm, epi);
  *tn = kTiles[i].tn;
  *tm = kTiles[i].tm;
}

// The attention core's plan for B x H (utterance, head) pairs of T frames: key splits, tiles per
// wave and query blocks of the first and the second shape, and whether two workgroups share a CU.
extern "C" void attn_shape(int d_k, int T, int64_t pairs, int* out) {
  const AttnPlan p = attn_plan(d_k, t_aligned(T), (long)pairs, T);
  const int v[7] = {p.c1.ksplit, p.c1.ntl, p.nqb1, p.c2.ksplit, p.c2.ntl, p.nqb2, p.dense};
  for (int i = 0; i < 7; ++i) out[i] = v[i];
}
