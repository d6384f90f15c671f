#include "lbm_walk_kernel.hpp"

namespace lbm {
void launch_walk_f32(lbm_ctx* ctx, int model, const double* w, int depth, int hs, const void* src, void* dst, int step) {
    launch_walk_p<kF32>(ctx, model, w, depth, hs, src, dst, step);
}
}  // namespace lbm
