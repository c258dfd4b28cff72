// resident_f32_var.hip -- instances of the on-chip PCG kernel.
#include "resident_kernel.hpp"

namespace pcgmi {

hipError_t launch_resident_f32_var(const ResPlan& p, const ResTask& a, hipStream_t s) {
    return resident::pick_shape<float, double, true>(p, a, s);
}

}  // namespace pcgmi
