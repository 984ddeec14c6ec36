// Forward steps of a gradient run (FP32), which store the Laplacian: one per
// tile shape, with streaming and with cache-resident load policies.
#include "wave_step.h"

namespace wavek {

#define INST(TXV, TY, RY)                                                   \
    template __global__ void step_tiled_lap<false, TXV, TY, RY>(StepArgs); \
    template __global__ void step_tiled_lap<true, TXV, TY, RY>(StepArgs);
WAVE_TILE_SHAPES(INST)
#undef INST

}  // namespace wavek
