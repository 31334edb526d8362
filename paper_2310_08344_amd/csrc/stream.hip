// Windows of D Leja iterations per launch by register streaming (gfx950),
// for the diffusion-advection operators and the Burgers Jacobian, FP64 or (not
// the third-order upwind operator) FP32 levels; and power iteration with many sweeps per launch in
// the same way.
//
// The window semantics are those of leja_block (window_device.h): every
// output takes the one-iteration loop's terms in the same order, and the
// stop rule (Sec. 2.2) is applied at every term m+1 .. m+D from the sums of
// squares the window records.  Only the way the levels are formed differs.
//
// Every wavefront works alone on an item: a strip of 128 columns (64 lanes,
// a column pair each) and a band of rows, marched from top to bottom with no
// barrier.  Its 128 columns are the item's output columns and D columns on
// each side; level j (the basis vector y_{m+j}) is valid on the strip minus
// j columns on each side, so after D levels the output columns remain.
// Rows are staged from D above the band to D below it.  At step t the
// wavefront takes row t of y_m (level 0) and then forms level j at row t - j
// for j = 1..D from the two rows of level j-1 it kept in registers and the
// row of level j-1 it just formed (the Newton recurrence of Sec. 2.1,
// Eq. (2)).  The side neighbours of a column pair come from the neighbouring
// lanes (DPP wavefront shifts).  Nothing is formed twice along y (the
// LDS-tile kernel forms up to 1.7 points per output point at D = 6 on 8-row
// tiles); along x the strip's side columns are formed by two wavefronts
// (128 columns per at most 128 - 2D outputs).
//
// The outputs: for the diffusion-advection operators (ring windows, stream_device.h)
// every level also goes into a small ring in LDS and the outputs of row
// t - D take all their terms at step t; otherwise (the Burgers Jacobian) an
// output row enters the registers when level 0 reaches it, takes term j
// when level j does, and leaves after its last term, D + 1 rows of every
// output in flight.  Rings of depth 7 or 8 (28 KB or 35 KB per wavefront),
// and of depth 6 with radius 2 (38 KB),
// leave room in LDS for one wavefront per SIMD: those windows have a kernel
// of their own, allowed the registers of a single wavefront.
//
// Each wavefront's items are a contiguous run of bands of one XCD, so the
// side columns a neighbouring strip also loads come from that XCD's L2.
#include <hip/hip_runtime.h>

#include "lx_device.h"
#include "stream_device.h"

namespace lx {
namespace {

using namespace dev;

template <int OP, int K, int D, bool F32>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void leja_stream(SweepArgs a,
                                                                                                const int L) {
    leja_stream_body<OP, K, D, F32>(a, L, static_cast<int>(blockIdx.x), nullptr);
}

// The same at one wavefront per SIMD (kDeepRing), with its registers; launch
// 0 (the first window) has a kernel of its own, since the registers of a
// kernel are allocated over all its forms and the first window's form,
// compiled beside the others, cost the full windows 12 % (and, in its
// general form with a start row per output, took half as long again as a
// full window itself).
template <int OP, int K, int D, bool F32>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void leja_stream_deep(
    SweepArgs a, const int L) {
    leja_stream_body<OP, K, D, F32>(a, L, static_cast<int>(blockIdx.x), nullptr);
}

template <int OP, int K, int D, bool F32>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void leja_stream_deep_first(
    SweepArgs a) {
    leja_stream_body<OP, K, D, F32, true>(a, 0, static_cast<int>(blockIdx.x), nullptr);
}

// ---------------------------------------------------------------------------
// Power iteration, up to DP sweeps per launch: level j = A^j (x / ||x||)
// formed by the same streaming (no shift), the sums of squares of every
// level recorded, the last level written; the next launch scales by its norm.
// The directions are those of the normalised iteration x_{k+1} = A x_k /
// ||A x_k||, and rho_hat = ||level nlev|| / ||level nlev-1|| of the last
// launch (level 0 has norm 1).  The host bounds nlev so that the unnormalised
// levels (at most rho^j) stay far from overflow.  With raw0 the first launch
// takes the start vector x as it is (levels A^j x, the same directions) and
// records ||x||^2 itself, which saves a pass over x; the final launch then
// reports a NaN estimate unless ||x||^2 lay in [1e-200, 1e20], where the
// unscaled levels keep the margin of the scaled ones, and the host repeats
// the iteration with x scaled first.
// Partial sums: the start vector's (power_norm_kernel, or launch 0 with
// raw0) at partials[nb + i], launch b's at partials[2 nb + (b & 1) nb DP +
// i DP + j].
// ---------------------------------------------------------------------------

// Launch b makes nlev levels from `in`, scaled by the norm of the last level
// of launch b - 1 (which made prev levels) or of the start vector (b = 0:
// unscaled with raw0, which needs nlev = DP).
template <int DP>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void power_stream(
    PowerArgs a, const double* in, double* out, const int b, const int nlev, const int prev, const int raw0) {
    const int wg = static_cast<int>(blockIdx.x);
    const bool lev0 = b == 0 && raw0 != 0;
    double scale = 1.0;
    if (b == 0) {
        if (!lev0) {
            double tot[1];
            sum_partials<1>(a.partials + a.nb, a.nb, tot);
            scale = 1.0 / sqrt(tot[0]);
        }
    } else {
        double tot[DP];
        sum_partials<DP>(a.partials + 2L * a.nb + static_cast<long>((b - 1) & 1) * a.nb * DP, a.nb, tot);
        double last = tot[DP - 1];
#pragma unroll
        for (int j = 0; j < DP; ++j)
            if (j == prev - 1) last = tot[j];
        scale = 1.0 / sqrt(last);
    }
    const int nl = __builtin_amdgcn_readfirstlane(nlev);
    // the plain operator (no shift)
    const StenT<double> st{a.cW, a.cE, a.cS, a.cN};
    double sy[DP];
#pragma unroll
    for (int j = 0; j < DP; ++j) sy[j] = 0.0;
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int items = a.tiles_x * a.tiles_y, G = a.nb * kStreamWaves;
    const int unit = strip_unit(a.nx, DP);
    double sy0 = 0.0;
    if (nl == DP) {
        const unsigned bytes = static_cast<unsigned>(a.nx) * static_cast<unsigned>(a.ny) * 8u;
        const Rsrc rin = make_rsrc(in, bytes), rout = make_rsrc(out, bytes);
        if (lev0) {
            for (int i = stream_wave(wg, a.nb); i < items; i += G)
                stream_power_item<DP, true>(st, a.cC, a.nx, a.ny, rin, rout, scale,
                                            stream_geom(i, a.nx, a.ny, a.tiles_x, a.tiles_y, unit), lane, sy, sy0);
        } else {
            for (int i = stream_wave(wg, a.nb); i < items; i += G)
                stream_power_item<DP, false>(st, a.cC, a.nx, a.ny, rin, rout, scale,
                                             stream_geom(i, a.nx, a.ny, a.tiles_x, a.tiles_y, unit), lane, sy, sy0);
        }
    } else {
        const Sten sa{a.cW, a.cE, a.cS, a.cN, a.cC, 0.0, 0.0, 0.0, 0.0};
        for (int i = stream_wave(wg, a.nb); i < items; i += G)
            stream_power_item_any<DP>(sa, a.nx, a.ny, in, out, scale, nl,
                                      stream_geom(i, a.nx, a.ny, a.tiles_x, a.tiles_y, unit), lane, sy);
    }
    block_sum<DP>(sy);
    if (lev0) {
        double s0[1] = {sy0};
        block_sum<1>(s0);
        sy0 = s0[0];
    }
    if (flat_tid() == 0) {
        double* __restrict__ Pp = a.partials + 2L * a.nb + static_cast<long>(b & 1) * a.nb * DP + static_cast<long>(wg) * DP;
#pragma unroll
        for (int j = 0; j < DP; ++j) Pp[j] = sy[j];
        if (lev0) a.partials[a.nb + wg] = sy0;
    }
}

// rho_hat = ||level nlev|| / ||level nlev-1|| of the last launch b; NaN
// after an unscaled first launch (raw0) whose ||x||^2 left [1e-200, 1e20]
template <int DP>
__global__ __launch_bounds__(kBlockThreads) void power_stream_final(PowerArgs a, const int b, const int nlev,
                                                                    const int raw0) {
    double tot[DP];
    sum_partials<DP>(a.partials + 2L * a.nb + static_cast<long>(b & 1) * a.nb * DP, a.nb, tot);
    double x2[1] = {1.0};
    if (raw0) sum_partials<1>(a.partials + a.nb, a.nb, x2);
    if (flat_tid() == 0) {
        double last = 0.0, prev = 1.0;
#pragma unroll
        for (int j = 0; j < DP; ++j) {
            if (j == nlev - 1) last = tot[j];
            if (j == nlev - 2) prev = tot[j];
        }
        const bool safe = x2[0] >= 1e-200 && x2[0] <= 1e20;
        publish_rho(a.rho, safe ? sqrt(last / prev) : __builtin_nan(""));
    }
}

// The register-marching window kernels there are: the five-point
// diffusion-advection operator at depth 4 (K <= 4), 6 (K <= 3) and 8 (K <= 3)
// in FP64, the Burgers Jacobian at depth 4 (K <= 2) and 6 (K = 1), and the
// third-order upwind operator at depths 4 and 6 (K = 1); FP32 sweeps of the
// first two for K <= 2 at depths 4 and 6 (K = 1).
#define LX_STREAM_KERNELS(X)                                                                              \
    X(kOpDiffAdv, 1, 4, false) X(kOpDiffAdv, 2, 4, false) X(kOpDiffAdv, 3, 4, false)                      \
    X(kOpDiffAdv, 4, 4, false) X(kOpDiffAdv, 1, 6, false) X(kOpDiffAdv, 2, 6, false)                      \
    X(kOpDiffAdv, 3, 6, false) X(kOpDiffAdv, 1, 8, false) X(kOpDiffAdv, 2, 8, false)                      \
    X(kOpDiffAdv, 3, 8, false) X(kOpBurgersJ, 1, 4, false) X(kOpBurgersJ, 2, 4, false)                    \
    X(kOpBurgersJ, 1, 6, false) X(kOpDiffAdv, 1, 4, true) X(kOpDiffAdv, 2, 4, true)                       \
    X(kOpDiffAdv, 1, 6, true) X(kOpBurgersJ, 1, 4, true) X(kOpBurgersJ, 2, 4, true)                       \
    X(kOpBurgersJ, 1, 6, true) X(kOpDiffAdv3, 1, 4, false) X(kOpDiffAdv3, 1, 6, false)

// the kernel of a (operator, K, depth, precision) combination, and its launch
template <int OP, int K, int D, bool F32>
const void* stream_fn() {
    if constexpr (kDeepRing<OP, D>) return reinterpret_cast<const void*>(leja_stream_deep<OP, K, D, F32>);
    else return reinterpret_cast<const void*>(leja_stream<OP, K, D, F32>);
}

template <int OP, int K, int D, bool F32>
void stream_launch(const SweepArgs& a, const int L, hipStream_t s) {
    if constexpr (kDeepRing<OP, D>) {
        if (L == 0) hipLaunchKernelGGL((leja_stream_deep_first<OP, K, D, F32>), dim3(a.nb), dim3(kBlockThreads), 0, s, a);
        else hipLaunchKernelGGL((leja_stream_deep<OP, K, D, F32>), dim3(a.nb), dim3(kBlockThreads), 0, s, a, L);
    } else
        hipLaunchKernelGGL((leja_stream<OP, K, D, F32>), dim3(a.nb), dim3(kBlockThreads), 0, s, a, L);
}

const void* stream_kernel(int op, int K, int depth, bool f32) {
#define LX_STREAM_PICK(O, KK, DD, F)                                                    \
    if (op == (O) && K == (KK) && depth == (DD) && f32 == (F)) return stream_fn<(O), (KK), (DD), (F)>();
    LX_STREAM_KERNELS(LX_STREAM_PICK)
#undef LX_STREAM_PICK
    return nullptr;
}

}  // namespace

int stream_strips(int nx, int halo) {
    const int unit = strip_unit(nx, halo);
    const int out_units = (128 - 2 * halo) / unit;   // column units a strip outputs
    return ((nx / unit) + out_units - 1) / out_units;
}

bool stream_has(int op, int K, int depth, bool fp32) { return stream_kernel(op, K, depth, fp32) != nullptr; }

hipError_t launch_leja_stream(int op, int K, int depth, bool fp32, const SweepArgs& a, int L, hipStream_t s) {
    const int halo = depth * (op == kOpDiffAdv3 ? 2 : 1);
    if (!stream_has(op, K, depth, fp32) || a.nb < 1 || a.nx % 2 != 0 || a.nx < halo || a.ny < halo)
        return hipErrorInvalidValue;
    if (op == kOpBurgersJ && (a.u == nullptr || (fp32 && a.u32 == nullptr))) return hipErrorInvalidValue;
    if (a.tiles_x != stream_strips(a.nx, halo) || a.tiles_y < 1 || a.tiles_y > a.ny) return hipErrorInvalidValue;
    if (static_cast<long>(a.nx) * a.ny * 8 > static_cast<long>(kFar)) return hipErrorInvalidValue;
#define LX_STREAM_LAUNCH(O, KK, DD, F)                                                                         \
    if (op == (O) && K == (KK) && depth == (DD) && fp32 == (F)) {                                              \
        stream_launch<(O), (KK), (DD), (F)>(a, L, s);                                                          \
        return hipGetLastError();                                                                              \
    }
    LX_STREAM_KERNELS(LX_STREAM_LAUNCH)
#undef LX_STREAM_LAUNCH
    return hipErrorInvalidValue;
}

int stream_resident(int op, int K, int depth, bool fp32, int power) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    const void* k = power ? reinterpret_cast<const void*>(power_stream<kPowerStreamDepth>)
                          : stream_kernel(op, K, depth, fp32);
    if (k == nullptr) return 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kBlockThreads, 0);
    return e == hipSuccess ? per_cu * cus : 0;
}

hipError_t launch_power_stream(const PowerArgs& a, const double* in, double* out, int b, int nlev, int prev,
                               bool raw0, hipStream_t s) {
    constexpr int DP = kPowerStreamDepth;
    if (a.nb < 1 || a.nx % 2 != 0 || a.nx < DP || a.ny < DP || nlev < 1 || nlev > DP || prev < 1 || prev > DP)
        return hipErrorInvalidValue;
    if (raw0 && b == 0 && nlev != DP) return hipErrorInvalidValue;
    if (a.tiles_x != stream_strips(a.nx, DP) || a.tiles_y < 1 || a.tiles_y > a.ny) return hipErrorInvalidValue;
    if (static_cast<long>(a.nx) * a.ny * 8 > static_cast<long>(kFar)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((power_stream<DP>), dim3(a.nb), dim3(kBlockThreads), 0, s, a, in, out, b, nlev, prev,
                       raw0 ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_power_stream_final(const PowerArgs& a, int b, int nlev, bool raw0, hipStream_t s) {
    hipLaunchKernelGGL((power_stream_final<kPowerStreamDepth>), dim3(1), dim3(kBlockThreads), 0, s, a, b, nlev,
                       raw0 ? 1 : 0);
    return hipGetLastError();
}

}  // namespace lx
