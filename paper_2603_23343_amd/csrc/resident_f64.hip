// resident_f64.hip -- instances of the on-chip PCG kernel.
#include "resident_kernel.hpp"

namespace pcgmi {

hipError_t launch_resident_f64(const ResLaunch& a, hipStream_t s) {
    return a.kc ? resident::pick_shape<double, double, true>(a, s) : resident::pick_shape<double, double, false>(a, s);
}

}  // namespace pcgmi
