// Newton coefficients on the device (gfx950): the divided differences
// d_j = f[xi_0, ..., xi_j] of f(xi) = sigma phi_l(alpha h (c + gamma xi)) at
// the Leja points (Sec. 2.1, Eq. (2)), in double-double, for the outputs of
// one Leja loop or for every instance of a batch.
//
// The table is formed column by column, a thread per row:
//     t_k <- (t_k - t_{k-1}) / (xi_k - xi_{k-j}),   k >= j,   j = 1, 2, ...
// after column j row j holds d_j for good.  A launch advances the columns
// [j0, j1) and keeps the rows in memory, so a loop asks for the columns its
// next launches read and pays for no others; the rows past the last column
// ride along in other wavefronts.  One workgroup per series; the previous
// row comes from the lane below (lane 0: from the wavefront below, through
// LDS, one barrier per column).
//
// What bounds a launch is the chain of dependent FP64 operations of each
// column.  The reciprocal of xi_k - xi_{k-j} does not depend on the table
// and stays off the chain, the three quotient digits of the double-double
// division are products with it, and the series of the function values take
// 1/k! from a table: 0.2 us per column, where three divisions per column and
// per series term took 0.5 us per column of 64 rows.  On the host, one
// thread took 0.87 ms for the 3 x 73 coefficients of a 60-iteration solve
// with three outputs, which left the GPU idle for 0.4 ms at 1024^2 (805 us per solve, 600 after).
#include <hip/hip_runtime.h>

#include "dd_math.h"
#include "lx_device.h"
#include "sweep_device.h"
#include "window_device.h"

namespace lx {
namespace {

using namespace dev;

constexpr int kCoefWaves = 16;   // rows / 64, at most (kMaxCoefRows)

// Rows of one series in `state` ([2][ld]: hi, lo) advanced over the columns
// [j0, j1); j0 = 0 starts from the function values.
__device__ __forceinline__ void advance_columns(const CoefSeries& s, const double* __restrict__ xi,
                                                double* __restrict__ state, double* __restrict__ coef, const int ld,
                                                const int rows, const int j0, const int j1) {
    __shared__ double2 edge[2][kCoefWaves];
    const int k = threadIdx.x, lane = k & 63, wave = k >> 6;
    const bool live = k < rows;
    const double xk = live ? xi[k] : 0.0;
    dd t{0.0, 0.0};
    if (live) {
        if (j0 == 0) t = dd_phi_at_fast(s.l, s.alpha, s.sigma, s.h, s.c, s.gamma, xk);
        else t = dd{state[k], state[ld + k]};
    }
    for (int j = j0 > 1 ? j0 : 1; j < j1; ++j) {
        // the last row of every wavefront, for the first row of the next
        if (lane == 63) edge[j & 1][wave] = double2{t.hi, t.lo};
        const bool act = live && k >= j;
        const dd den = two_sum(xk, act ? -xi[k - j] : 1.0);
        const double rcp = 1.0 / den.hi;
        __syncthreads();
        double2 below{0.0, 0.0};
        if (lane == 0 && wave > 0) below = edge[j & 1][wave - 1];
        const dd prev{lane_neighbour<true>(t.hi, below.x), lane_neighbour<true>(t.lo, below.y)};
        const dd q = dd_div_rcp(dd_sub(t, prev), den, rcp);
        if (act) t = q;
    }
    if (live) {
        state[k] = t.hi;
        state[ld + k] = t.lo;
        if (k >= j0 && k < j1) coef[k] = t.hi + t.lo;
    }
}

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
    advance_columns(a.s[k], xi, state + static_cast<long>(k) * 2 * ld, coef + static_cast<long>(k) * ld, ld, rows, j0,
                    j1);
}

__global__ __launch_bounds__(64 * kCoefWaves) void batch_coef_kernel(const BatchInst* insts,
                                                                     const double* __restrict__ xi,
                                                                     double* __restrict__ state,
                                                                     double* __restrict__ coef, const int ld,
                                                                     const int rows, const int j0, const int j1) {
    const BatchInst& I = insts[blockIdx.x];
    const CoefSeries s{1.0, 1.0, I.h, I.c, I.gamma, I.l};
    advance_columns(s, xi, state + static_cast<long>(blockIdx.x) * 2 * ld, coef + static_cast<long>(blockIdx.x) * ld,
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
