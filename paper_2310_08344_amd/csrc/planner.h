// Host planner of the Leja phi-action library (plain C++, no HIP).
#pragma once

#include <cmath>

namespace lx {

constexpr int kMaxPoints = 1024;   // LX_MAX_ITERS + 24: windows of D iterations read up to d_{max_iters+D}

// The power of two 2^e that brings the Gershgorin bound g of an operator into
// [1/2, 1).  Several sweeps of power iteration without a normalisation between
// them grow or shrink the vector like powers of the operator; scaled by 2^e
// they stay in range for operators of any size, and as the scaling is exact,
// the estimate, scaled back by 2^-e, has the same bits.
inline int power_exponent(double g) {
    if (!(g > 0.0) || !std::isfinite(g)) return 0;
    const int e = -std::ilogb(g) - 1;
    return e < -1022 ? -1022 : e;
}

// The launches of a loop that have started, by its progress word: launch L of
// the loop that was given `base` stores base + L + 1, and every later loop gets
// a base beyond those.  A launch that an earlier loop left on the stream may
// still store its own number: that counts as none.
inline int launches_started(unsigned word, unsigned base) {
    const int n = static_cast<int>(word - base);
    return n > 0 ? n : 0;
}

// Whether windows of depth da at a us per iteration end a loop sooner than
// windows of depth db at b us.  A loop of m iterations forms about m + D levels
// in windows of D: half a window past its last term, and half a window again
// for the output that stopped in it.  Taken for m = 50.  Third-order upwind at
// 16384^2, 55 iterations: windows of six on register tiles 640 us per iteration
// and 40.2 ms, windows of four on LDS tiles 653 us and 39.0 ms.
inline bool windows_faster(double a, int da, double b, int db) {
    constexpr double m = 50.0;
    return a * (m + da) < b * (m + db);
}

// Whether the tuner takes marching windows of FP32 sweeps of depth da at a us per
// iteration instead of depth db at b.  The two go over to FP32 at different
// iterations, so the choice shows in the results (by about 1e-9 at rtol 1e-6):
// deeper windows are taken up to 1 % slower, the spread of these timings, so that
// it turns on their noise for fewer grids (five-point operator, depth six over
// depth four, five timings each: 980^2 1.00 to 1.01, 1024^2 0.98 to 1.01, 1200^2 0.98
// to 1.00; elsewhere the two differ by more, 512^2 1.27, 2048^2 0.89).
inline bool fp32_marching_taken(double a, int da, double b, int db) { return a < (da > db ? 1.01 * b : b); }

// phi_l(z) for real z (Sec. 1 recursion; Taylor series near 0).
double phi_scalar(int l, double z);

// First M Leja points of [-2, 2] (Sec. 2.1), generated once per process and
// extended on demand; thread-safe.  Returns false for M outside 1..kMaxPoints.
bool leja_points(int M, double* out);

// Divided differences of f(xi) = sigma*phi_l(alpha*h*(c + gamma*xi)) at the
// points xi[0], xi[1], ... (Sec. 2.1, Eq. (2)), produced one at a time in
// double-double arithmetic and rounded to FP64: next() returns d_J and costs
// O(J).  xi must stay valid while the series is used.
class NewtonSeries {
public:
    NewtonSeries();
    ~NewtonSeries();
    NewtonSeries(const NewtonSeries&) = delete;
    NewtonSeries& operator=(const NewtonSeries&) = delete;
    void reset(int l, double alpha, double sigma, double h, double c, double gamma, const double* xi);
    double next();
    int count() const { return count_; }

private:
    struct Impl;
    Impl* impl_;
    const double* xi_ = nullptr;
    int count_ = 0;
};

// d_0..d_{M-1} of the series above at the points xi[0..M-1].
bool newton_coeffs(int l, double alpha, double sigma, double h, double c, double gamma,
                   int M, const double* xi, double* d);

}  // namespace lx
