// resident_f32.hip -- instances of the on-chip PCG kernel.
#include "resident_kernel.hpp"

namespace pcgmi {

hipError_t launch_resident_f32(const ResPlan& p, const ResTask& a, hipStream_t s) {
    return resident::pick_shape<float, double, false>(p, a, s);
}

}  // namespace pcgmi
