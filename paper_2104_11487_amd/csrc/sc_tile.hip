// Tile kernel builds for bf16 layers of 32, 64 or 128 input channels, and the
// choice, set-up and launch of every build (kernel: sc_tile_kernel.h).
#include "sc_tile_kernel.h"

namespace sc {

namespace {

const TileBuild kTileBuilds[] = {
#define SC_X(rows, cols, ntn, a, b, wm, wn, kr, zi, krt, occ, ki)                                 \
  {rows, cols, ntn, 64 * a * b, tile_kernel<a, b, wm, wn, kr, occ, ki, zi, false, false, 0, false>, \
   tile_kernel<a, b, wm, wn, krt, occ, ki, true, true, false, 0, false>,                            \
   tile_kernel<a, b, wm, wn, kr, occ, ki, zi, false, true, 0, false>,                               \
   tile_kernel<a, b, wm, wn, kr, occ, kLearnItems(rows, a * b), zi, false, false, 1, false>,        \
   tile_kernel<a, b, wm, wn, kr, occ, kLearnItems(rows, a * b), zi, false, false, 3, false>,        \
   tile_kernel<a, b, wm, wn, kr, occ, kLearnItems(rows, a * b), zi, false, true, 1, false>,         \
   tile_kernel<a, b, wm, wn, kr, occ, kLearnItems(rows, a * b), zi, false, true, 3, false>},
    SC_TILE_BUILDS(SC_X)
#undef SC_X
};

const TileBuild* tile_build(const HaloParams& hp, int ntn) {
  int count = (int)(sizeof(kTileBuilds) / sizeof(kTileBuilds[0]));
  const TileBuild* b = hp.tab_off ? tile_tab_builds(&count) : hp.parts ? tile_parts_builds(&count) : kTileBuilds;
  for (; count > 0; --count, ++b)
    if (b->rows == hp.rows && b->cols == hp.side && b->ntn == ntn) return b;
  return nullptr;
}

// rho halo, pixel statistics, the chunk table with its zero word, chunk sums
int tile_lds(const HaloParams& hp, int ksteps) {
  if (hp.part_off) return hp.part_off + hp.hh * hp.hw * (((hp.pstride - 16) / 16) | 1) * 4;
  return hp.tab_off ? hp.tab_off + (ksteps * 4 + 4) * 4 : hp.lds_bytes + (hp.hh * hp.hw * 4 + 15) / 16 * 16;
}

}  // namespace

bool tile_shape(HaloParams& hp, int ntiles_n, int ksteps, int c, int learned, int lds_limit) {
  hp.pstride = 2 * c + 16;
  hp.lds_bytes = hp.hh * hp.hw * hp.pstride;
  hp.tab_off = c == 32 || c == 64 || c == 128 ? 0 : hp.lds_bytes + (hp.hh * hp.hw * 4 + 15) / 16 * 16;
  hp.lg_group = 1;
  while ((c >> 3) > 1 << hp.lg_group) ++hp.lg_group;
  hp.part_off = hp.lg_group > 4 ? hp.tab_off + (ksteps * 4 + 4) * 4 : 0;
  const TileBuild* b = tile_build(hp, ntiles_n);
  if (!b || hp.lg_group > 5 || tile_lds(hp, ksteps) > lds_limit) return false;
  return !learned || (!hp.tab_off && c <= 64 && (learned == 1 || learned == 3) &&
                      (hp.hh * hp.hw) << hp.lg_group <= kLearnItems(hp.rows, b->threads / 64) * b->threads);
}

int tile_occupancy(const HaloParams& hp, int ntiles_n, int ksteps) {
  const TileBuild* b = tile_build(hp, ntiles_n);
  int blocks = 0;
  if (!b) return 0;
  const int lds = tile_lds(hp, ksteps);
  for (TileKernel f : {b->chain1, b->chain3, b->learned1, b->learned3, b->chain, b->trans, b->plain})
    if (f && (hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, lds) !=
                  hipSuccess ||
              hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, f, b->threads, lds) != hipSuccess))
      return 0;
  return blocks;
}

hipError_t launch_tile(const GateParams& g, const ConvParams& c, const HaloParams& hp, hipStream_t st) {
  const TileBuild* b = tile_build(hp, c.ntiles_n);
  if (!b) return hipErrorInvalidValue;
  TileKernel f = c.zsrc ? b->trans : (g.rin ? b->chain : b->plain);
  if (g.learned) {
    const bool one = g.learned == 1;
    f = c.zsrc || (!one && g.learned != 3) ? nullptr
                                           : (g.rin ? (one ? b->chain1 : b->chain3) : (one ? b->learned1 : b->learned3));
  }
  if (!f) return hipErrorInvalidValue;
  hipLaunchKernelGGL(f, dim3(g.n * g.tiles_y * g.tiles_x), dim3(b->threads), tile_lds(hp, c.ksteps),
                     st, g, c, hp);
  return hipGetLastError();
}

}  // namespace sc
