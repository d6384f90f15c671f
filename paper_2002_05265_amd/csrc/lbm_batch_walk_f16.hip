#include "lbm_batch_walk.hpp"

namespace lbm {
void launch_batch_walk_f16(const BatchPass& p, int depth, const WalkTask* tasks, int ntasks) {
    launch_batch_walk_p<kF16>(p, depth, tasks, ntasks);
}
}  // namespace lbm
