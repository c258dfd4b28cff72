// resident_batch.hip -- many on-chip solves in one launch (batched.hip): a
// work-group takes boxes from its list one after another. All lists name the
// problems in the same order, so the boxes of a problem always come together.
#include "resident_kernel.hpp"

namespace pcgmi {

namespace {

__global__ void __launch_bounds__(resident::RT, 2) k_batch_resident(const ResBatchTask* __restrict__ tasks,
                                                                    const int2* __restrict__ work,
                                                                    const int* __restrict__ first) {
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
    __shared__ resident::SumLds L;
    const int hi = first[blockIdx.x + 1];
    for (int i = first[blockIdx.x]; i < hi; ++i) {
        const int2 w = work[i];
        const ResTask& a = tasks[w.x].task;
        const int code = tasks[w.x].shape * 64 + tasks[w.x].V;
        bool ok = false;
        // every body inlined: called ones would each need the caller's registers saved
        auto one = [&]<int V, int SH>() __attribute__((always_inline)) {
            if (code == SH * 64 + V)
                ok = resident::solve_box<float, double, V, false, RES_SHAPES[SH][0], RES_SHAPES[SH][1]>(a, w.y, dyn, L);
        };
        auto run = [&]<int V, int... SH>(std::integer_sequence<int, SH...>) __attribute__((always_inline)) {
            (one.template operator()<V, SH>(), ...);
        };
        [&]<int... V>(std::integer_sequence<int, V...>) __attribute__((always_inline)) {
            (run.template operator()<V>(std::make_integer_sequence<int, RES_NSHAPES>{}), ...);
        }(ResBatchVs{});
        if (!ok) return;  // the others' waits run out too
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_batch_resident(const ResBatchTask* tasks, const int2* work, const int* first, int nwg, size_t lds,
                                 hipStream_t s) {
    if (nwg < 1 || nwg > RES_MAX_WG || lds > RES_MAX_LDS) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_batch_resident),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_batch_resident, dim3((unsigned)nwg), dim3(resident::RT), lds, s, tasks, work, first);
    return hipGetLastError();
}

}  // namespace pcgmi
