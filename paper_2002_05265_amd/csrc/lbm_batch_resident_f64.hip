#include "lbm_batch_resident.hpp"

namespace lbm {
void launch_batch_resident_f64(const BatchPass& p, int nsteps, int most) {
    launch_batch_resident_p<kF64>(p, nsteps, most);
}
}  // namespace lbm
