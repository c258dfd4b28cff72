// resident_f64.hip -- instances of the on-chip PCG kernel.
#include "resident_kernel.hpp"

namespace pcgmi {

hipError_t launch_resident_f64(const ResPlan& p, const ResTask& a, hipStream_t s) {
    if (a.kc) return resident::pick_shape<double, double, true>(p, a, s);
    return resident::pick_shape<double, double, false>(p, a, s);
}

}  // namespace pcgmi
