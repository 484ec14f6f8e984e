// The one-workgroup RK4 runs of 1D states (sgn_batch.h) in mixed precision: kernel and launch.
#include "sgn_batch.h"

namespace sgn {

template <>
hipError_t launch_batch_rk4_kernel<BATCH_MIXED>(int n, int grid, int cus, hipStream_t stream, const StepItem* items,
                                               int nitems, const StepShared* shared, StepResult* res, int* queue) {
    const int nt = batch_threads_for(n);
    const size_t lds = batch_lds_bytes(n);
    const hipError_t e = batch_grid(k_batch_rk4<BATCH_MIXED>, nt, lds, cus, nitems, grid);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_batch_rk4<BATCH_MIXED>, dim3(grid), dim3(nt), lds, stream, items, nitems, shared, res, queue);
    return hipGetLastError();
}

}  // namespace sgn
