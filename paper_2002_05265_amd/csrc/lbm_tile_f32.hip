#include "lbm_tile_kernel.hpp"

namespace lbm {
void launch_tile_f32(lbm_ctx* ctx, int model, const double* w, int nsteps, const void* src, void* dst, int step,
                     const TileKeep* keep) {
    launch_tile_p<kF32>(ctx, model, w, nsteps, src, dst, step, keep);
}
}  // namespace lbm
