#include "lbm_batch_resident.hpp"

namespace lbm {
void launch_batch_resident_f32(const BatchPass& p, int nsteps, int most) {
    launch_batch_resident_p<kF32>(p, nsteps, most);
}
}  // namespace lbm
