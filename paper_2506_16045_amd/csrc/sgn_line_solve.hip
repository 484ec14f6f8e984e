// The one-workgroup 1D solves and right-hand sides (sgn_batch.h): kernels and launches.
#include "sgn_batch.h"

namespace sgn {

hipError_t launch_batch_solve_kernel(int mode, int n, int grid, int cus, hipStream_t stream, const BatchItem* items,
                                     int nitems, const SolveShared* shared, BatchResult* res, int* queue) {
    const int nt = batch_threads_for(n);
    const size_t lds = batch_lds_bytes(n);
    auto launch = [&](auto k) -> hipError_t {
        const hipError_t e = batch_grid(k, nt, lds, cus, nitems, grid);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3(grid), dim3(nt), lds, stream, items, nitems, shared, res, queue);
        return hipGetLastError();
    };
    return mode == BATCH_MIXED ? launch(k_batch_solve<BATCH_MIXED>) : launch(k_batch_solve<BATCH_FP64>);
}

hipError_t launch_rhs_1d_kernel(int n, hipStream_t stream, double L, const double* eta, const double* hx,
                                const double* u, double* eta_t, double* U_t, cpx<double>* spec, double* st,
                                const cpx<double>* tw) {
    const size_t lds = batch_lds_bytes(n);
    int grid = 1;
    auto launch = [&](auto k) -> hipError_t {
        const hipError_t e = batch_grid(k, batch_threads_for(n), lds, 1, 1, grid);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3(1), dim3(batch_threads_for(n)), lds, stream, n, L, eta, hx, u, eta_t, U_t, spec, st,
                           tw);
        return hipGetLastError();
    };
    return n < 2 * LINE_MMIN ? launch(k_rhs_1d<true>) : launch(k_rhs_1d<false>);
}

}  // namespace sgn
