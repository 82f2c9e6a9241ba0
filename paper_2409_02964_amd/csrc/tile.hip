// The tile kernel's instances (tile_kernel.hpp).
#include "step_launch.hpp"

namespace vanse_dev {

template <typename S, typename T, bool SHIFT, int FEAT, bool PAIRS>
void launch_tile(const StepGeom& g, const StepPhys<T>& ph, int walls, int steps, int blocks, hipStream_t st) {
  constexpr int TY = tile_y(int(sizeof(T)));
  hipLaunchKernelGGL((vanse_tile_kernel<S, T, SHIFT, FEAT, PAIRS, TY>), dim3(blocks), dim3(TILE_X * TY), 0, st, g,
                     ph, walls, steps);
}

#define VANSE_TILE_ONE(S, T, H, F) \
  template void launch_tile<S, T, H, F, false>(const StepGeom&, const StepPhys<T>&, int, int, int, hipStream_t); \
  template void launch_tile<S, T, H, F, true>(const StepGeom&, const StepPhys<T>&, int, int, int, hipStream_t);
#define VANSE_TILES(S, T, H) \
  VANSE_TILE_ONE(S, T, H, 0) VANSE_TILE_ONE(S, T, H, FEAT_FORCE) VANSE_TILE_ONE(S, T, H, FEAT_DRAG) \
  VANSE_TILE_ONE(S, T, H, FEAT_FORCE | FEAT_DRAG) VANSE_TILE_ONE(S, T, H, FEAT_MASK) \
  VANSE_TILE_ONE(S, T, H, FEAT_MASK | FEAT_FORCE | FEAT_DRAG) \
  VANSE_TILE_ONE(S, T, H, FEAT_DYNPHI | FEAT_FORCE | FEAT_DRAG)
VANSE_TILES(double, double, false)
VANSE_TILES(float, float, false)
VANSE_TILES(float, float, true)
VANSE_TILES(_Float16, float, true)
#undef VANSE_TILES
#undef VANSE_TILE_ONE

}  // namespace vanse_dev
