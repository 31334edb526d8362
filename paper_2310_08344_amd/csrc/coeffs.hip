// Newton coefficients on the device (gfx950): the divided differences
// d_j = f[xi_0, ..., xi_j] of f(xi) = sigma phi_l(alpha h (c + gamma xi)) at
// the Leja points (Sec. 2.1, Eq. (2)), in double-double, for the outputs of
// one Leja loop or for every instance of a batch.
//
// A launch advances some columns of the tables (coef_device.h), one workgroup
// per series.  A loop on register tiles asks for its first columns this way
// and forms the others beside its windows (rtile.hip).
#include <hip/hip_runtime.h>

#include "coef_device.h"
#include "lx_device.h"

namespace lx {
namespace {

using namespace dev;

// The outputs of one Leja loop: workgroup k forms output k's coefficients.
// With ctl (the loop's first launch) also sets the loop's initial state, which
// saves the copy of it.
__global__ __launch_bounds__(64 * kCoefWaves) void coef_kernel(const CoefArgs a, const double* __restrict__ xi,
                                                               double* __restrict__ state, double* __restrict__ coef,
                                                               const int ld, const int rows, const int j0,
                                                               const int j1, LoopCtl* __restrict__ ctl) {
    const int k = static_cast<int>(blockIdx.x);
    if (ctl != nullptr && k == 0 && threadIdx.x == 0) {
        LoopCtl c{};
        c.rtol = a.rtol;
        c.atol = a.atol;
        c.fp32_switch = a.fp32_switch;
        c.max_iters = a.max_iters;
        c.slot[0].out32 = a.out32;
        for (int i = 0; i < kKMax; ++i)
            if (i < a.K) {
                c.slot[0].active[i] = 1;
                c.slot[0].iters[i] = a.max_iters;
            }
        *ctl = c;
    }
    advance_columns<true>(a.s[k], xi, state + static_cast<long>(k) * 2 * ld, coef + static_cast<long>(k) * ld, ld, rows, j0,
                    j1);
}

__global__ __launch_bounds__(64 * kCoefWaves) void batch_coef_kernel(const BatchInst* insts,
                                                                     const double* __restrict__ xi,
                                                                     double* __restrict__ state,
                                                                     double* __restrict__ coef, const int ld,
                                                                     const int rows, const int j0, const int j1) {
    const BatchInst& I = insts[blockIdx.x];
    const CoefSeries s{1.0, 1.0, I.h, I.c, I.gamma, I.l};
    advance_columns<true>(s, xi, state + static_cast<long>(blockIdx.x) * 2 * ld, coef + static_cast<long>(blockIdx.x) * ld,
                    ld, rows, j0, j1);
}

bool valid_span(int rows, int j0, int j1) {
    return rows >= 1 && rows <= kMaxCoefRows && j0 >= 0 && j0 < j1 && j1 <= rows;
}

}  // namespace

hipError_t launch_coeffs(const CoefArgs& a, const double* xi, double* state, double* coef, int ld, int rows, int j0,
                         int j1, LoopCtl* ctl, hipStream_t s) {
    if (!valid_span(rows, j0, j1) || j1 > ld || a.K < 1 || a.K > kKMax) return hipErrorInvalidValue;
    hipLaunchKernelGGL(coef_kernel, dim3(a.K), dim3(((rows + 63) / 64) * 64), 0, s, a, xi, state, coef, ld, rows, j0,
                       j1, ctl);
    return hipGetLastError();
}

hipError_t launch_batch_coeffs(const BatchInst* insts, int n_inst, const double* xi, double* state, double* coef,
                               int ld, int rows, int j0, int j1, hipStream_t s) {
    if (!valid_span(rows, j0, j1) || j1 > ld || n_inst < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(batch_coef_kernel, dim3(n_inst), dim3(((rows + 63) / 64) * 64), 0, s, insts, xi, state, coef,
                       ld, rows, j0, j1);
    return hipGetLastError();
}

}  // namespace lx
