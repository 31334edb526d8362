// Batched register marching (gfx950): the windows and the power iteration of
// stream.hip for many independent instances, one launch for the whole batch.
//
// Every workgroup serves one instance (block_inst[blockIdx.x]); its four
// wavefronts each march items of that instance, a strip of 128 columns by a
// band of rows (stream_device.h), with the instance's own loop control,
// partial sums and stop decision, as in the LDS-tile form of the batch
// (batch_block_kernel).  Windows of six iterations (the Burgers Jacobian:
// four, or six in large batches) move a quarter to a third fewer bytes per
// iteration than LDS-tile windows of four and form nothing twice along y;
// wavefronts that meet at no barrier keep the memory system busy where the
// tiles, at two or three workgroups per CU with a barrier per level, did not.
// Measured on 256 diffusion-advection instances of 64^2 to 512^2 (22 M points,
// all of them at work): a window 241 us for six iterations (225 us for four on
// LDS tiles), ten power sweeps 160 us (1000 us one by one); the whole call
// 1.66 ms, before 3.74.  1024 instances of 256^2, half of them Burgers: 4.8 ms
// instead of 7.3; 16 of 128^2: 0.37 ms instead of 1.8.
#include <hip/hip_runtime.h>

#include "lx_device.h"
#include "stencil_coeffs.h"
#include "stream_device.h"

namespace lx {
namespace {

using namespace dev;

// A value that is the same in all lanes, as a scalar: instance descriptors
// are read through a uniform address, but buffer resources and addresses
// made from them have to be in scalar registers.
__device__ __forceinline__ int uniform(const int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ double uniform(const double v) {
    return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}

template <typename T>
__device__ __forceinline__ T* uniform(T* p) {
    const unsigned long long a = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = static_cast<unsigned>(uniform(static_cast<int>(a)));
    const unsigned hi = static_cast<unsigned>(uniform(static_cast<int>(a >> 32)));
    return gptr(reinterpret_cast<T*>((static_cast<unsigned long long>(hi) << 32) | lo));
}

// DA, DB: window depth of the diffusion-advection and of the Burgers
// instances (0: the batch has none).
template <int DA, int DB>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void batch_stream_kernel(
    const BatchInst* __restrict__ insts, LoopCtl* ctls, const int* __restrict__ block_inst, double* partials,
    const double* coef, const int ld, const double* xi, unsigned* done, const int L) {
    const int i = uniform(block_inst[blockIdx.x]);
    const BatchInst& I = insts[i];
    SweepArgs a{};
    a.nx = uniform(I.nx);
    a.ny = uniform(I.ny);
    a.tiles_x = uniform(I.tiles_x);
    a.tiles_y = uniform(I.tiles_y);
    a.nb = uniform(I.nb);
    a.ld = ld;
    a.inv_sqrtN = 1.0 / sqrt(static_cast<double>(a.nx) * a.ny);
    a.v = uniform(I.v);
    a.ybuf[0] = uniform(I.y[0]);
    a.ybuf[1] = uniform(I.y[1]);
    a.p[0] = uniform(I.out);
    a.p2[0] = uniform(I.out2);
    a.coef = coef + static_cast<long>(i) * ld;
    a.xi = xi;
    a.partials = partials + I.part_off;
    a.ctl = ctls + i;
    const int wg = static_cast<int>(blockIdx.x) - uniform(I.wg_begin);
    if (DB == 0 || uniform(I.kind) == kOpDiffAdv) {
        a.aE = uniform(I.st[0]);
        a.aW = uniform(I.st[1]);
        a.aN = uniform(I.st[2]);
        a.aS = uniform(I.st[3]);
        a.aC = uniform(I.st[4]);
        leja_stream_body<kOpDiffAdv, 1, DA, false>(a, L, wg, done);
    } else if constexpr (DB != 0) {
        a.u = uniform(I.u);
        a.kx = uniform(I.st[0]);
        a.ky = uniform(I.st[1]);
        a.gx = uniform(I.st[2]);
        a.gy = uniform(I.st[3]);
        a.kC = uniform(I.st[4]);
        leja_stream_body<kOpBurgersJ, 1, DB, false>(a, L, wg, done);
    }
}

// Power launch b of the diffusion-advection instances (power_stream's
// arithmetic): nlev levels of 2^e A (power_exponent: levels of an operator of
// any size stay in range), scaled by the norm of the prev levels of launch
// b - 1.  Launch 0 scales a given start vector by its norm
// (batch_power_norm_kernel) and takes the library's own as it is: its values
// lie in [-1, 1).
// Partial sums in the instance's record: the start vector's norm at [nb + j],
// launch b's at [2 nb + (b & 1) nb DP + j DP].
template <int DP>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void batch_power_stream_kernel(
    const BatchInst* __restrict__ insts, const int* __restrict__ block_inst, double* partials, const int b,
    const int nlev, const int prev, const int scale_own) {
    const int i = uniform(block_inst[blockIdx.x]);
    const BatchInst& I = insts[i];
    if (I.kind != kOpDiffAdv) return;
    const int nx = uniform(I.nx), ny = uniform(I.ny), nb = uniform(I.nb);
    const int wg = static_cast<int>(blockIdx.x) - uniform(I.wg_begin);
    double* __restrict__ P = gptr(partials) + I.part_off;
    double scale = 1.0;
    if (b == 0) {
        if (I.has_x0 || scale_own) {
            double tot[1];
            sum_partials<1>(P + nb, nb, tot);
            scale = 1.0 / sqrt(tot[0]);
        }
    } else {
        double tot[DP];
        sum_partials<DP>(P + 2L * nb + static_cast<long>((b - 1) & 1) * nb * DP, nb, tot);
        double last = tot[DP - 1];
#pragma unroll
        for (int j = 0; j < DP; ++j)
            if (j == prev - 1) last = tot[j];
        scale = 1.0 / sqrt(last);
    }
    const double* x0 = I.has_x0 ? I.x0 : I.y[1];
    const double* in = uniform(b == 0 ? x0 : const_cast<const double*>((b & 1) ? I.y[0] : I.y[1]));
    double* out = uniform((b & 1) ? I.y[1] : I.y[0]);
    const double cE = uniform(I.pw[0]), cW = uniform(I.pw[1]), cN = uniform(I.pw[2]), cS = uniform(I.pw[3]);
    const double cC = uniform(I.pw[4]);
    const StenT<double> st{cW, cE, cS, cN};
    double sy[DP], sy0 = 0.0;
#pragma unroll
    for (int j = 0; j < DP; ++j) sy[j] = 0.0;
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int strips = uniform(I.ptiles_x), bands = uniform(I.ptiles_y);
    const int items = strips * bands, G = nb * kStreamWaves, unit = strip_unit(nx, DP);
    if (nlev == DP) {
        const unsigned bytes = static_cast<unsigned>(nx) * static_cast<unsigned>(ny) * 8u;
        const Rsrc rin = make_rsrc(in, bytes), rout = make_rsrc(out, bytes);
        for (int k = stream_wave(wg, nb); k < items; k += G)
            stream_power_item<DP, false>(st, cC, nx, ny, rin, rout, scale,
                                         stream_geom(k, nx, ny, strips, bands, unit), lane, sy, sy0);
    } else {
        const Sten sa{cW, cE, cS, cN, cC, 0.0, 0.0, 0.0, 0.0};
        for (int k = stream_wave(wg, nb); k < items; k += G)
            stream_power_item_any<DP>(sa, nx, ny, in, out, scale, nlev, stream_geom(k, nx, ny, strips, bands, unit),
                                      lane, sy);
    }
    block_sum<DP>(sy);
    if (flat_tid() == 0) {
        double* __restrict__ Pp = P + 2L * nb + static_cast<long>(b & 1) * nb * DP + static_cast<long>(wg) * DP;
#pragma unroll
        for (int j = 0; j < DP; ++j) Pp[j] = sy[j];
    }
}

// The spectral estimate of every diffusion-advection instance from the last
// power launch b, rho = ||level nlev|| / ||level nlev-1|| (level 0 has norm
// 1), and its shift and scale (Listing 7); one workgroup per instance
template <int DP>
__global__ __launch_bounds__(kBlockThreads) void batch_power_stream_final_kernel(BatchInst* insts,
                                                                                 const double* partials, const int b,
                                                                                 const int nlev, const double safety) {
    BatchInst& I = insts[blockIdx.x];
    if (I.kind != kOpDiffAdv) return;
    double tot[DP];
    sum_partials<DP>(partials + I.part_off + 2L * I.nb + static_cast<long>(b & 1) * I.nb * DP, I.nb, tot);
    if (flat_tid() == 0) {
        double last = 0.0, prev = 1.0;
#pragma unroll
        for (int j = 0; j < DP; ++j) {
            if (j == nlev - 1) last = tot[j];
            if (j == nlev - 2) prev = tot[j];
        }
        const double rho = sqrt(last / prev) * I.pscale;
        const double lam = -safety * rho;
        I.rho = rho;
        I.c = lam / 2.0;
        I.gamma = -lam / 4.0;
        stencil_coeffs(0, I.dx, I.dy, I.D, I.vx, I.vy, I.nu, I.c, I.gamma, I.st);
    }
}

}  // namespace

hipError_t launch_batch_stream(const BatchInst* insts, LoopCtl* ctls, const int* block_inst, int nblocks, int da,
                               int db, double* partials, const double* coef, int ld, const double* xi, unsigned* done,
                               int L, hipStream_t s) {
    const dim3 grid(nblocks), block(kBlockThreads);
    if (da == 6 && db == 0)
        hipLaunchKernelGGL((batch_stream_kernel<6, 0>), grid, block, 0, s, insts, ctls, block_inst, partials, coef, ld,
                           xi, done, L);
    else if (da == 6 && db == 4)
        hipLaunchKernelGGL((batch_stream_kernel<6, 4>), grid, block, 0, s, insts, ctls, block_inst, partials, coef, ld,
                           xi, done, L);
    else if (da == 6 && db == 6)
        hipLaunchKernelGGL((batch_stream_kernel<6, 6>), grid, block, 0, s, insts, ctls, block_inst, partials, coef, ld,
                           xi, done, L);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_batch_power_stream(const BatchInst* insts, const int* block_inst, int nblocks, double* partials,
                                     int b, int nlev, int prev, bool scale_own, hipStream_t s) {
    constexpr int DP = kPowerStreamDepth;
    if (nlev < 1 || nlev > DP || prev < 1 || prev > DP) return hipErrorInvalidValue;
    hipLaunchKernelGGL(batch_power_stream_kernel<DP>, dim3(nblocks), dim3(kBlockThreads), 0, s, insts, block_inst,
                       partials, b, nlev, prev, scale_own ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_batch_power_stream_final(BatchInst* insts, int n_inst, const double* partials, int b, int nlev,
                                           double safety, hipStream_t s) {
    hipLaunchKernelGGL(batch_power_stream_final_kernel<kPowerStreamDepth>, dim3(n_inst), dim3(kBlockThreads), 0, s,
                       insts, partials, b, nlev, safety);
    return hipGetLastError();
}

}  // namespace lx
