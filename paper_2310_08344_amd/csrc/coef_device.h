// Device code of the Newton coefficients, for a launch of their own
// (coeffs.hip) or beside the windows of a loop (rtile.hip).
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
#pragma once

#include <hip/hip_runtime.h>

#include "dd_math.h"
#include "lx_device.h"
#include "sweep_device.h"
#include "window_device.h"

namespace lx {
namespace dev {

constexpr int kCoefWaves = 16;   // rows / 64, at most (kMaxCoefRows)

// Rows of one series in `state` ([2][ld]: hi, lo) advanced over the columns
// [j0, j1) by a workgroup of at least `rows` threads; kStart: j0 may be 0, which
// starts from the function values.
template <bool kStart>
__device__ __forceinline__ void advance_columns(const CoefSeries& s, const double* __restrict__ xi,
                                                double* __restrict__ state, double* __restrict__ coef, const int ld,
                                                const int rows, const int j0, const int j1) {
    __shared__ double2 edge[2][kCoefWaves];
    const int k = threadIdx.x, lane = k & 63, wave = k >> 6;
    const bool live = k < rows;
    const double xk = live ? xi[k] : 0.0;
    dd t{0.0, 0.0};
    if (live) {
        if (kStart && j0 == 0) t = dd_phi_at_fast(s.l, s.alpha, s.sigma, s.h, s.c, s.gamma, xk);
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

}  // namespace dev
}  // namespace lx
