// Register tiles (gfx950): windows of D Leja iterations, and power iteration
// with several sweeps per launch, on tiles whose levels stay in registers, for
// grids too small to keep a register-marching launch busy and for every odd
// grid.
//
// A workgroup of eight wavefronts holds 128 columns (a column pair per lane)
// by 8 RW rows (RW rows per lane): its output tile and the D radius cells on
// each side that the window needs.  A level is formed in place: the row
// neighbours are the lane's own rows, but for the first and last rows of a
// wavefront, which go through LDS (one barrier per level); the side neighbours
// come from the neighbouring lanes.  Cells near the edge of the 128 x 8 RW
// block go invalid by one radius per level, as the halo of any tile does.
//
// Window semantics, stop rule and results are those of leja_block and
// leja_stream (window_device.h): every output takes the one-iteration loop's
// terms in the same order, with the same operations.
//
// Why: on a small grid a launch is a chain of latencies.  A marching wavefront
// forms its D levels one after another at every row step; here the rows of a
// level are independent, and a level of the whole tile takes 0.3 us (RW = 4)
// or 0.5 (RW = 8).  The price is the halo formed twice (112 x 16 outputs of
// 128 x 32 cells at D = 8, RW = 4; 112 x 48 of 128 x 64 at RW = 8), which is
// what bounds larger grids: vector FP64 work and LDS row exchange.
// us per iteration, against the fastest other kernel: 64 x 64 1.64 (2.24),
// 1024 x 1024 with three outputs 3.9 (5.2), 2049 x 2047 11.4 (one iteration per
// launch, 42), FP32 sweeps of the Burgers Jacobian at 512 x 512 1.95 (4.7).
#include <hip/hip_runtime.h>

#include "coef_device.h"
#include "lx_device.h"
#include "stream_device.h"
#include "tile_device.h"
#include "window_device.h"

namespace lx {
namespace {

using namespace dev;

constexpr int kRtWaves = 8;
constexpr int kRtThreads = 64 * kRtWaves;
constexpr int kRtCols = 128;

// Tile t of a grid of sx by sy tiles: columns [xs, xs + ws), rows [yb, yb + hb);
// column edges are multiples of `unit` (2 where pairs are loaded whole).
struct RtGeom {
    int xs, ws, yb, hb;
};

__device__ __forceinline__ RtGeom rt_geom(const int t, const int nx, const int ny, const int sx, const int sy,
                                          const int unit) {
    const int b = t / sx, s = t - b * sx;
    const long units = nx / unit;
    RtGeom g;
    g.xs = unit * static_cast<int>((s * units) / sx);
    g.ws = unit * static_cast<int>(((s + 1) * units) / sx) - g.xs;
    g.yb = static_cast<int>((static_cast<long>(b) * ny) / sy);
    g.hb = static_cast<int>((static_cast<long>(b + 1) * ny) / sy) - g.yb;
    return g;
}

// This workgroup's tiles: a contiguous band of its XCD's (workgroup b runs on
// XCD b % 8) once the grid has a multiple of eight.
struct RtSpan {
    int first, step, end;
};

__device__ __forceinline__ RtSpan rt_span(const int wg, const int nb, const int T) {
    if (nb >= 8 && (nb & 7) == 0) {
        const int x = wg & 7;
        return {static_cast<int>((static_cast<long>(x) * T) >> 3) + (wg >> 3), nb >> 3,
                static_cast<int>((static_cast<long>(x + 1) * T) >> 3)};
    }
    return {wg, nb, T};
}

// A lane's place in a tile: its columns, and its share of the outputs.
template <int H, int RW>
struct RtLane {
    int c0, c1;      // grid columns of the pair
    bool o0, o1;     // output columns
    int er0;         // first row of the wavefront within the tile's rows
    int rows;        // rows the tile needs: hb + 2 H
    int ytop;
    __device__ __forceinline__ RtLane(const RtGeom& g, const int nx) {
        const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int rc = 2 * lane - H;
        c0 = wrap(g.xs + rc, nx);
        c1 = c0 + 1 < nx ? c0 + 1 : 0;
        o0 = rc >= 0 && rc < g.ws;
        o1 = rc + 1 >= 0 && rc + 1 < g.ws;
        er0 = wave * RW;
        rows = g.hb + 2 * H;
        ytop = g.yb - H;
    }
    __device__ __forceinline__ bool out_row(const int r) const { return er0 + r >= H && er0 + r < rows - H; }
    __device__ __forceinline__ bool any_out() const { return er0 + RW > H && er0 < rows - H; }
    // whether level j is formed on rows of this wavefront that a later level
    // or an output needs (radius R)
    __device__ __forceinline__ bool at_work(const int jr) const { return er0 + RW > jr && er0 < rows - jr; }
    __device__ __forceinline__ long row(const int r, const int nx, const int ny) const {
        return static_cast<long>(wrap(ytop + er0 + r, ny)) * nx;
    }
};

// A column pair of a row: one access where pairs are whole and aligned (kVec),
// else two.
template <bool kVec, typename S>
__device__ __forceinline__ P2<S> rt_ld(const S* __restrict__ p, const long row, const int c0, const int c1) {
    if constexpr (kVec) return *reinterpret_cast<const P2<S>*>(p + row + c0);
    else return P2<S>{p[row + c0], p[row + c1]};
}

template <bool kVec, typename S>
__device__ __forceinline__ void rt_st(S* __restrict__ p, const long row, const int c0, const int c1, const bool o0,
                                      const bool o1, const P2<S> v) {
    if constexpr (kVec) {
        if (o0) *reinterpret_cast<P2<S>*>(p + row + c0) = v;
    } else {
        if (o0) p[row + c0] = v.x;
        if (o1) p[row + c1] = v.y;
    }
}

// Sten in the arithmetic of the levels.
template <typename T>
struct RtSten {
    T c0, c1, c2, c3, e0, e1, e2, e3;
    __device__ __forceinline__ explicit RtSten(const Sten& s)
        : c0(static_cast<T>(s.c0)), c1(static_cast<T>(s.c1)), c2(static_cast<T>(s.c2)), c3(static_cast<T>(s.c3)),
          e0(static_cast<T>(s.e0)), e1(static_cast<T>(s.e1)), e2(static_cast<T>(s.e2)), e3(static_cast<T>(s.e3)) {}
};

// The next level of a wavefront's rows, in place: y, with the R rows above
// (up, nearest last) and below (dn, nearest first); for the Burgers Jacobian
// u on the same rows and one above and below.
template <int OP, int RW, typename T>
__device__ __forceinline__ void rt_level(const RtSten<T>& st, const T cc, P2<T> (&y)[RW],
                                         const P2<T> (&up)[OP == kOpDiffAdv3 ? 2 : 1],
                                         const P2<T> (&dn)[OP == kOpDiffAdv3 ? 2 : 1],
                                         const P2<T> (&u)[OP == kOpBurgersJ ? RW + 2 : 1]) {
    if constexpr (OP == kOpDiffAdv3) {
        P2<T> a2 = up[0], a1 = up[1];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const P2<T> C = y[r];
            const P2<T> n1 = r + 1 < RW ? y[r + 1 < RW ? r + 1 : 0] : dn[0];
            const P2<T> n2 = r + 2 < RW ? y[r + 2 < RW ? r + 2 : 0] : dn[r + 2 - RW < 0 ? 0 : r + 2 - RW];
            const T wy = nbr<true>(C.y), wx = nbr<true>(C.x), ex = nbr<false>(C.x), ey = nbr<false>(C.y);
            y[r].x = stencil_d3(st.c0, st.c1, st.c2, st.c3, cc, st.e0, st.e1, st.e2, st.e3, wy, C.y, a1.x, n1.x, C.x,
                                wx, ex, a2.x, n2.x);
            y[r].y = stencil_d3(st.c0, st.c1, st.c2, st.c3, cc, st.e0, st.e1, st.e2, st.e3, C.x, ex, a1.y, n1.y, C.y,
                                wy, ey, a2.y, n2.y);
            a2 = a1;
            a1 = C;
        }
    } else {
        P2<T> above = up[0];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const P2<T> C = y[r];
            const P2<T> N = r + 1 < RW ? y[r + 1 < RW ? r + 1 : 0] : dn[0];
            const T w = nbr<true>(C.y), e = nbr<false>(C.x);
            if constexpr (OP == kOpDiffAdv) {
                y[r].x = stencil_da(st.c0, st.c1, st.c2, st.c3, cc, w, C.y, above.x, N.x, C.x);
                y[r].y = stencil_da(st.c0, st.c1, st.c2, st.c3, cc, C.x, e, above.y, N.y, C.y);
            } else {
                const P2<T> uS = u[r], uC = u[r + 1], uN = u[r + 2];
                const T uw = nbr<true>(uC.y), ue = nbr<false>(uC.x);
                y[r].x = stencil_bu(st.c0, st.c1, st.c2, st.c3, cc, w, C.y, above.x, N.x, C.x, uw, uC.y, uS.x, uN.x);
                y[r].y = stencil_bu(st.c0, st.c1, st.c2, st.c3, cc, C.x, e, above.y, N.y, C.y, uC.x, ue, uS.y, uN.y);
            }
            above = C;
        }
    }
}

// The same in FP32, of FP64 values that are FP32 ones.
template <int OP, int RW>
__device__ __forceinline__ void rt_level_fp32(const RtSten<float>& st, const float cc, double2 (&y)[RW],
                                              const double2 (&up)[OP == kOpDiffAdv3 ? 2 : 1],
                                              const double2 (&dn)[OP == kOpDiffAdv3 ? 2 : 1],
                                              const double2 (&u)[OP == kOpBurgersJ ? RW + 2 : 1]) {
    constexpr int R = OP == kOpDiffAdv3 ? 2 : 1, U = OP == kOpBurgersJ ? RW + 2 : 1;
    P2<float> yf[RW], uf[U], upf[R], dnf[R];
#pragma unroll
    for (int r = 0; r < RW; ++r) yf[r] = as_t2<float>(y[r]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        upf[r] = as_t2<float>(up[r]);
        dnf[r] = as_t2<float>(dn[r]);
    }
    if constexpr (OP == kOpBurgersJ) {
#pragma unroll
        for (int r = 0; r < U; ++r) uf[r] = as_t2<float>(u[r]);
    }
    rt_level<OP, RW, float>(st, cc, yf, upf, dnf, uf);
#pragma unroll
    for (int r = 0; r < RW; ++r) y[r] = as_d2<float>(yf[r]);
}

// A wavefront's first and last R rows of a level, for its neighbours in the
// tile; two buffers, so one barrier per level is enough.
template <int R, typename T = double>
struct RtExchange {
    P2<T> row[2][kRtWaves][2 * R][64];
};

// Writes this wavefront's edge rows, waits, and reads the neighbours' (the
// tile's first and last wavefront read their own: such rows are invalid).
template <int R, int RW, typename T>
__device__ __forceinline__ void rt_exchange(RtExchange<R, T>& ex, const int buf, const P2<T> (&y)[RW], P2<T> (&up)[R],
                                            P2<T> (&dn)[R]) {
    const int lane = static_cast<int>(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        ex.row[buf][wave][i][lane] = y[i];
        ex.row[buf][wave][R + i][lane] = y[RW - R + i];
    }
    __syncthreads();
    const int a = wave > 0 ? wave - 1 : 0, b = wave < kRtWaves - 1 ? wave + 1 : wave;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        up[i] = ex.row[buf][a][R + i][lane];
        dn[i] = ex.row[buf][b][i][lane];
    }
}

template <int OP>
__device__ __forceinline__ Sten sweep_sten(const SweepArgs& a) {
    if constexpr (OP == kOpDiffAdv) return Sten{a.aW, a.aE, a.aS, a.aN, a.aC, 0.0, 0.0, 0.0, 0.0};
    else if constexpr (OP == kOpDiffAdv3) return Sten{a.aW, a.aE, a.aS, a.aN, a.aC, a.aW2, a.aE2, a.aS2, a.aN2};
    else return Sten{a.kx, a.ky, a.gx, a.gy, a.kC, 0.0, 0.0, 0.0, 0.0};
}

// The tiles of this workgroup in a window launch, the levels in T (FP32 levels
// of FP32 sweeps: the basis and the stencil arithmetic; outputs, terms and sums
// stay FP64).  s_d[k][j] = d_{m+j} of output k (0 past its last term), s_cc[j-1]
// the centre of level j.  kMixed (T FP64): the window that switches to FP32,
// with the precisions of one iteration at a time: w.lev64 levels in FP64, the
// next one formed in FP64 and rounded, the others in FP32.
template <int OP, int K, int D, int RW, bool kVec, typename T, bool kMixed = false>
__device__ __forceinline__ void rt_window(const SweepArgs& a, const WindowPlan<K>& w, const Sten& sten, const int wg,
                                          const double (&s_d)[K][D + 1], const double (&s_cc)[D],
                                          RtExchange<radius<OP>(), T>& ex, double (&sy)[D], double (&sp)[K][D]) {
    constexpr int R = radius<OP>(), H = D * R;
    const RtSten<T> st(sten);
    const int nx = a.nx, ny = a.ny, unit = kVec ? 2 : 1;
    const bool store_y = !w.redo, first = w.win == 0;
    const RtSpan span = rt_span(wg, a.nb, a.tiles_x * a.tiles_y);
    int buf = 0;
    for (int t = span.first; t < span.end; t += span.step) {
        const RtGeom g = rt_geom(t, nx, ny, a.tiles_x, a.tiles_y, unit);
        const RtLane<H, RW> ln(g, nx);
        const bool outs = ln.any_out();
        P2<T> y[RW], u[OP == kOpBurgersJ ? RW + 2 : 1];
        double2 p[K][RW];
        constexpr bool kF = sizeof(T) == sizeof(float);   // never a first window: its y_0 is FP64
        if (w.jmax > 0) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
                y[r] = rt_ld<kVec>(reinterpret_cast<const T*>(w.yin), ln.row(r, nx, ny), ln.c0, ln.c1);
            if constexpr (OP == kOpBurgersJ) {
                const T* __restrict__ us;
                if constexpr (kF) us = a.u32;
                else us = a.u;
#pragma unroll
                for (int r = 0; r < RW + 2; ++r) u[r] = rt_ld<kVec>(us, ln.row(r - 1, nx, ny), ln.c0, ln.c1);
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            // the first window starts from p_0 = d_0 y_0 (also when it is
            // re-executed); a copy reads the window's own result
            const bool rd = outs && (w.nt[k] > 0 || w.copy[k]) && !(first && !w.copy[k]);
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                p[k][r] = double2{0.0, 0.0};
                if (rd && ln.out_row(r) && (ln.o0 || ln.o1)) p[k][r] = rt_ld<kVec>(w.pin[k], ln.row(r, nx, ny), ln.c0, ln.c1);
            }
        }
        double fr[RW];   // 1 for output rows
#pragma unroll
        for (int r = 0; r < RW; ++r) fr[r] = ln.out_row(r) ? 1.0 : 0.0;
#pragma unroll
        for (int j = 1; j <= D; ++j) {
            if (j > w.jmax) continue;
            P2<T> up[R], dn[R];
            rt_exchange<R, RW, T>(ex, buf, y, up, dn);
            buf ^= 1;
            if (!kF && j == 1 && first) {
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (!w.copy[k]) {
                        const double d0 = s_d[k][0];
#pragma unroll
                        for (int r = 0; r < RW; ++r) {
                            const double2 v = as_d2<T>(y[r]);
                            p[k][r].x = d0 * v.x;
                            p[k][r].y = d0 * v.y;
                        }
                    }
            }
            if (!ln.at_work(j * R)) continue;
            if (kMixed && j > w.lev64 + 1) {
                if constexpr (kMixed)
                    rt_level_fp32<OP, RW>(RtSten<float>(sten), static_cast<float>(s_cc[j - 1]), y, up, dn, u);
            } else {
                rt_level<OP, RW, T>(st, static_cast<T>(s_cc[j - 1]), y, up, dn, u);
                if (kMixed && j == w.lev64 + 1) {
#pragma unroll
                    for (int r = 0; r < RW; ++r) {
                        y[r].x = static_cast<float>(y[r].x);
                        y[r].y = static_cast<float>(y[r].y);
                    }
                }
            }
            if (!outs) continue;
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const double2 v = as_d2<T>(y[r]);
                const double y1 = kVec ? v.y : (ln.o1 ? v.y : 0.0);
                s = fma(fr[r], fma(y1, y1, v.x * v.x), s);
            }
            sy[j - 1] += ln.o0 ? s : 0.0;   // lanes outside the output columns count for nothing
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double d = s_d[k][j];
                double q = 0.0;
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    const double2 v = as_d2<T>(y[r]);
                    p[k][r].x = fma(d, v.x, p[k][r].x);
                    p[k][r].y = fma(d, v.y, p[k][r].y);
                    const double p1 = kVec ? p[k][r].y : (ln.o1 ? p[k][r].y : 0.0);
                    q = fma(fr[r], fma(p1, p1, p[k][r].x * p[k][r].x), q);
                }
                sp[k][j - 1] += ln.o0 ? q : 0.0;
            }
        }
        if (outs) {
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                if (!ln.out_row(r)) continue;
                const long row = ln.row(r, nx, ny);
                if (store_y) {
                    if constexpr (kMixed)
                        rt_st<kVec>(reinterpret_cast<float*>(w.yout), row, ln.c0, ln.c1, ln.o0, ln.o1,
                                    as_t2<float>(as_d2<T>(y[r])));
                    else rt_st<kVec>(reinterpret_cast<T*>(w.yout), row, ln.c0, ln.c1, ln.o0, ln.o1, y[r]);
                }
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (w.nt[k] > 0 || w.copy[k]) rt_st<kVec>(w.pout[k], row, ln.c0, ln.c1, ln.o0, ln.o1, p[k][r]);
            }
        }
    }
}

// Launch L of the window loop: a.tiles_x by a.tiles_y tiles, a.nb workgroups.
// F32: FP32 sweeps (the switch to FP32 levels is decided on the device, and
// falls on the same iteration as one at a time; window_enter).
template <int OP, int K, int D, int RW, bool kVec, bool F32, int kEu>
__global__ __launch_bounds__(kRtThreads, kEu) void leja_rtile(SweepArgs a, const int L, const CoefJob job) {
    constexpr int R = radius<OP>(), H = D * R;
    static_assert(RW >= R && kRtWaves * RW > 2 * H && kRtCols > 2 * H, "a tile has outputs");
    __shared__ RtExchange<R> ex;
    __shared__ double s_d[K][D + 1], s_cc[D];
    const int wg = static_cast<int>(blockIdx.x), tid = static_cast<int>(threadIdx.x);
    if (wg >= a.nb) {
        // the workgroups past the tiles': output wg - nb's next coefficients,
        // unless the loop has ended.  Eight columns take 4 to 6 us, less than a
        // window; in launches of their own, 6 us for every second window, a
        // solve of 64 x 64 took 149 us, now 127 (333 x 250 197, now 167).
        // One thread reads the end flag for all: workgroup 0 of this launch may
        // set it meanwhile, and advance_columns has barriers.
        const int k = wg - a.nb;
        __shared__ int s_ended;
        if (tid == 0)
            s_ended = L > 0 && __hip_atomic_load(&a.ctl->slot[2].done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (s_ended) return;
        advance_columns<false>(job.s[k], a.xi, job.state + static_cast<long>(k) * 2 * a.ld,
                               job.coef + static_cast<long>(k) * a.ld, a.ld, job.rows, job.j0, job.j1);
        return;
    }
    WindowPlan<K> w;
    if (!window_enter<OP, K, D, true, F32, kRtWaves, F32>(a, L, wg, nullptr, w)) return;
    const Sten st = sweep_sten<OP>(a);
    if (tid < 64 * K && (tid & 63) <= D) {
        const int k = tid >> 6, j = tid & 63;
        // an output's terms end at nt (term 0 only starts it)
        int nt = 0;
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (i == k) nt = w.nt[i];
        s_d[k][j] = j == 0 || j <= nt ? a.coef[k * a.ld + w.m + j] : 0.0;
    }
    if (tid >= kRtThreads - 64 && tid - (kRtThreads - 64) < D) {
        const int j = tid - (kRtThreads - 64);
        s_cc[j] = st.c4 - a.xi[w.m + j];
    }
    double sy[D], sp[K][D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        sy[j] = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) sp[k][j] = 0.0;
    }
    if constexpr (F32) {
        if (w.win32) {
            if (w.in32)
                rt_window<OP, K, D, RW, kVec, float>(a, w, st, wg, s_d, s_cc,
                                                     reinterpret_cast<RtExchange<R, float>&>(ex), sy, sp);
            else rt_window<OP, K, D, RW, kVec, double, true>(a, w, st, wg, s_d, s_cc, ex, sy, sp);
            window_exit<K, D, kRtWaves>(a, L, wg, sy, sp);
            return;
        }
    }
    rt_window<OP, K, D, RW, kVec, double>(a, w, st, wg, s_d, s_cc, ex, sy, sp);
    window_exit<K, D, kRtWaves>(a, L, wg, sy, sp);
}

// ---------------------------------------------------------------------------
// Power iteration, up to DP sweeps per launch on the same tiles; the levels,
// sums and records of power_stream (stream.hip).
// ---------------------------------------------------------------------------

template <int OP, int DP, int RW, bool kVec, int kEu>
__global__ __launch_bounds__(kRtThreads, kEu) void power_rtile(PowerArgs a, const double* __restrict__ in,
                                                          double* __restrict__ out, const int b, const int nlev,
                                                          const int prev, const int raw0) {
    constexpr int R = radius<OP>(), H = DP * R;
    __shared__ RtExchange<R> ex;
    const int wg = static_cast<int>(blockIdx.x), tid = static_cast<int>(threadIdx.x);
    const bool lev0 = b == 0 && raw0 != 0;
    __shared__ double s_scale;
    if (!lev0) {
        // the norm of the last level before
        if (b == 0) {
            const double t = record_totals<1, kRtWaves>(a.partials + a.nb, a.nb);
            if (tid == 0) s_scale = 1.0 / sqrt(t);
        } else {
            const double t = record_totals<DP, kRtWaves>(
                a.partials + 2L * a.nb + static_cast<long>((b - 1) & 1) * a.nb * DP, a.nb);
            if (tid == prev - 1) s_scale = 1.0 / sqrt(t);
        }
        __syncthreads();
    }
    const double scale = lev0 ? 1.0 : s_scale;
    Sten st;
    if constexpr (OP == kOpDiffAdv) st = Sten{a.cW, a.cE, a.cS, a.cN, a.cC, 0.0, 0.0, 0.0, 0.0};
    else if constexpr (OP == kOpDiffAdv3) st = Sten{a.cW, a.cE, a.cS, a.cN, a.cC, a.cW2, a.cE2, a.cS2, a.cN2};
    else st = Sten{a.kx, a.ky, a.gx, a.gy, -2.0 * a.kx - 2.0 * a.ky, 0.0, 0.0, 0.0, 0.0};
    const RtSten<double> rst(st);
    double sy[DP + 1];   // [DP]: level 0
#pragma unroll
    for (int j = 0; j <= DP; ++j) sy[j] = 0.0;
    const int nx = a.nx, ny = a.ny, unit = kVec ? 2 : 1;
    const RtSpan span = rt_span(wg, a.nb, a.tiles_x * a.tiles_y);
    int buf = 0;
    for (int t = span.first; t < span.end; t += span.step) {
        const RtGeom g = rt_geom(t, nx, ny, a.tiles_x, a.tiles_y, unit);
        const RtLane<H, RW> ln(g, nx);
        const bool outs = ln.any_out();
        double2 y[RW], u[OP == kOpBurgersJ ? RW + 2 : 1];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            y[r] = rt_ld<kVec>(in, ln.row(r, nx, ny), ln.c0, ln.c1);
            y[r].x *= scale;
            y[r].y *= scale;
        }
        if constexpr (OP == kOpBurgersJ) {
#pragma unroll
            for (int r = 0; r < RW + 2; ++r) u[r] = rt_ld<kVec>(a.u, ln.row(r - 1, nx, ny), ln.c0, ln.c1);
        }
        double fr[RW];
#pragma unroll
        for (int r = 0; r < RW; ++r) fr[r] = ln.out_row(r) ? 1.0 : 0.0;
        auto sum = [&]() {
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const double y1 = kVec ? y[r].y : (ln.o1 ? y[r].y : 0.0);
                s = fma(fr[r], fma(y1, y1, y[r].x * y[r].x), s);
            }
            return ln.o0 && outs ? s : 0.0;
        };
        if (lev0) sy[DP] += sum();
#pragma unroll
        for (int j = 1; j <= DP; ++j) {
            if (j > nlev) continue;
            double2 up[R], dn[R];
            rt_exchange<R, RW, double>(ex, buf, y, up, dn);
            buf ^= 1;
            if (!ln.at_work(j * R)) continue;
            rt_level<OP, RW, double>(rst, st.c4, y, up, dn, u);
            sy[j - 1] += sum();
        }
        if (outs) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
                if (ln.out_row(r)) rt_st<kVec>(out, ln.row(r, nx, ny), ln.c0, ln.c1, ln.o0, ln.o1, y[r]);
        }
    }
    const double s = block_sums<DP + 1, kRtWaves>(sy);
    if (tid < DP) a.partials[2L * a.nb + static_cast<long>(b & 1) * a.nb * DP + static_cast<long>(wg) * DP + tid] = s;
    if (lev0 && tid == DP) a.partials[a.nb + wg] = s;
}

// rho_hat = ||level nlev|| / ||level nlev-1|| of the last launch b; NaN after
// an unscaled first launch whose ||x||^2 left [1e-200, 1e20]
template <int DP>
__global__ __launch_bounds__(kBlockThreads) void power_rtile_final(PowerArgs a, const int b, const int nlev,
                                                                   const int raw0) {
    double tot[DP], x2[1] = {1.0};
    sum_partials<DP>(a.partials + 2L * a.nb + static_cast<long>(b & 1) * a.nb * DP, a.nb, tot);
    if (raw0) sum_partials<1>(a.partials + a.nb, a.nb, x2);
    if (flat_tid() == 0) {
        double last = 0.0, prev = raw0 && b == 0 ? x2[0] : 1.0;   // level 0 has norm 1 unless it was taken unscaled
#pragma unroll
        for (int j = 0; j < DP; ++j) {
            if (j == nlev - 1) last = tot[j];
            if (j == nlev - 2) prev = tot[j];
        }
        const bool safe = x2[0] >= 1e-200 && x2[0] <= 1e20;
        publish_rho(a.rho, safe ? sqrt(last / prev) : __builtin_nan(""));
    }
}

// the register-tile kernels there are: (operator, outputs, depth), the
// radius-1 operators also for FP32 sweeps
#define LX_RTILE_KERNELS(X)                                                                     \
    X(kOpDiffAdv, 1, 8) X(kOpDiffAdv, 2, 8) X(kOpDiffAdv, 3, 8) X(kOpBurgersJ, 1, 8)            \
    X(kOpBurgersJ, 2, 8) X(kOpDiffAdv3, 1, 6)

// Launches of more than one round of workgroups of 8 rows per lane run the
// kernels bounded to 128 registers, two workgroups per CU, so that one loads
// while the other forms levels, where that costs few spills: power iteration
// (us for 20 sweeps, one / two per CU: Burgers 1400^2 133 / 118, 2048^2 210 / 174;
// third-order upwind 2048^2 240 / 186, 4095^2 535 / 447; five-point 2049^2 175 /
// 139; within one round it costs 2 %) and the windows of the third-order upwind
// operator (us per iteration 1201 x 1100 6.8 / 5.6, 2049 x 2047 13.9 / 10.7, 4095^2
// 48 / 35).  The other windows spill in their levels (five-point 2048^2 10.5 /
// 21.3).
constexpr int kRtRound = 256;

template <int OP, int K, int D, bool F32>
void rtile_launch(const SweepArgs& a, const int rw, const bool vec, const int L, const CoefJob& job, hipStream_t s) {
    const dim3 grid(a.nb + (job.j1 > job.j0 ? K : 0)), block(kRtThreads);
    if (rw == 4 && vec) hipLaunchKernelGGL((leja_rtile<OP, K, D, 4, true, F32, 2>), grid, block, 0, s, a, L, job);
    else if (rw == 4) hipLaunchKernelGGL((leja_rtile<OP, K, D, 4, false, F32, 2>), grid, block, 0, s, a, L, job);
    else if (OP == kOpDiffAdv3 && a.nb > kRtRound) {
        constexpr int kEu = OP == kOpDiffAdv3 ? 4 : 2;
        if (vec) hipLaunchKernelGGL((leja_rtile<OP, K, D, 8, true, F32, kEu>), grid, block, 0, s, a, L, job);
        else hipLaunchKernelGGL((leja_rtile<OP, K, D, 8, false, F32, kEu>), grid, block, 0, s, a, L, job);
    } else if (vec) hipLaunchKernelGGL((leja_rtile<OP, K, D, 8, true, F32, 2>), grid, block, 0, s, a, L, job);
    else hipLaunchKernelGGL((leja_rtile<OP, K, D, 8, false, F32, 2>), grid, block, 0, s, a, L, job);
}

template <int OP, int DP>
void power_rtile_launch(const PowerArgs& a, const double* in, double* out, const int rw, const bool vec, const int b,
                        const int nlev, const int prev, const int raw0, hipStream_t s) {
    const dim3 grid(a.nb), block(kRtThreads);
#define LX_POWER_RTILE(RW, VEC, EU) \
    hipLaunchKernelGGL((power_rtile<OP, DP, RW, VEC, EU>), grid, block, 0, s, a, in, out, b, nlev, prev, raw0)
    if (rw == 4 && vec) LX_POWER_RTILE(4, true, 2);
    else if (rw == 4) LX_POWER_RTILE(4, false, 2);
    else if (a.nb > kRtRound && vec) LX_POWER_RTILE(8, true, 4);
    else if (a.nb > kRtRound) LX_POWER_RTILE(8, false, 4);
    else if (vec) LX_POWER_RTILE(8, true, 2);
    else LX_POWER_RTILE(8, false, 2);
#undef LX_POWER_RTILE
}

}  // namespace

int rtile_depth(int op, int K) {
#define LX_RTILE_DEPTH(O, KK, DD) \
    if (op == (O) && K == (KK)) return DD;
    LX_RTILE_KERNELS(LX_RTILE_DEPTH)
#undef LX_RTILE_DEPTH
    return 0;
}

RtileGrid rtile_grid(int op, int depth, int nx, int ny, bool vec) {
    const int H = depth * (op == kOpDiffAdv3 ? 2 : 1), unit = vec ? 2 : 1;
    const int out_units = (kRtCols - 2 * H) / unit;
    RtileGrid g;
    g.tiles_x = (nx / unit + out_units - 1) / out_units;
    g.rw = 4;
    int th = kRtWaves * g.rw - 2 * H;
    if (g.tiles_x * ((ny + th - 1) / th) > 256) {
        g.rw = 8;
        th = kRtWaves * g.rw - 2 * H;
    }
    g.tiles_y = (ny + th - 1) / th;
    const int tiles = g.tiles_x * g.tiles_y;
    g.nb = tiles <= 1024 ? tiles : 512;
    return g;
}

static bool rtile_fits(int op, int depth, int nx, int ny, int tiles_x, int tiles_y, int nb, int rw, bool vec) {
    const int H = depth * (op == kOpDiffAdv3 ? 2 : 1), unit = vec ? 2 : 1;
    if (depth < 1 || nx <= H || ny <= H || (rw != 4 && rw != 8) || nb < 1 || tiles_x < 1 || tiles_y < 1) return false;
    if (vec && nx % 2 != 0) return false;
    // no tile wider or taller than a workgroup's cells hold
    const int units = nx / unit, w = ((units + tiles_x - 1) / tiles_x) * unit, h = (ny + tiles_y - 1) / tiles_y;
    return w <= kRtCols - 2 * H && h <= kRtWaves * rw - 2 * H;
}

hipError_t launch_leja_rtile(int op, int K, int rw, bool vec, bool fp32, const SweepArgs& a, int L,
                             const CoefJob& job, hipStream_t s) {
    if (job.j1 > job.j0 && (job.j0 < 1 || job.j1 > job.rows || job.rows > kCoefJobRows || job.rows > a.ld))
        return hipErrorInvalidValue;
    if (!rtile_fits(op, rtile_depth(op, K), a.nx, a.ny, a.tiles_x, a.tiles_y, a.nb, rw, vec)) return hipErrorInvalidValue;
    if (op == kOpBurgersJ && (a.u == nullptr || (fp32 && a.u32 == nullptr))) return hipErrorInvalidValue;
    if (fp32 && op == kOpDiffAdv3) return hipErrorInvalidValue;
#define LX_RTILE_LAUNCH(O, KK, DD)                                                          \
    if (op == (O) && K == (KK)) {                                                           \
        if (fp32) rtile_launch<(O), (KK), (DD), ((O) != kOpDiffAdv3)>(a, rw, vec, L, job, s); \
        else rtile_launch<(O), (KK), (DD), false>(a, rw, vec, L, job, s);                    \
        return hipGetLastError();                                                           \
    }
    LX_RTILE_KERNELS(LX_RTILE_LAUNCH)
#undef LX_RTILE_LAUNCH
    return hipErrorInvalidValue;
}

hipError_t launch_power_rtile(int op, int rw, bool vec, const PowerArgs& a, const double* in, double* out, int b,
                              int nlev, int prev, bool raw0, hipStream_t s) {
    const int dp = rtile_power_depth(op);
    if (!rtile_fits(op, dp, a.nx, a.ny, a.tiles_x, a.tiles_y, a.nb, rw, vec) || nlev < 1 || nlev > dp || prev < 1 ||
        prev > dp)
        return hipErrorInvalidValue;
    if (op == kOpBurgersJ && a.u == nullptr) return hipErrorInvalidValue;
    const int raw = raw0 ? 1 : 0;
    if (op == kOpDiffAdv) power_rtile_launch<kOpDiffAdv, 8>(a, in, out, rw, vec, b, nlev, prev, raw, s);
    else if (op == kOpBurgersJ) power_rtile_launch<kOpBurgersJ, 4>(a, in, out, rw, vec, b, nlev, prev, raw, s);
    else power_rtile_launch<kOpDiffAdv3, 4>(a, in, out, rw, vec, b, nlev, prev, raw, s);
    return hipGetLastError();
}

hipError_t launch_power_rtile_final(int op, const PowerArgs& a, int b, int nlev, bool raw0, hipStream_t s) {
    const int raw = raw0 ? 1 : 0;
    if (rtile_power_depth(op) == 8)
        hipLaunchKernelGGL(power_rtile_final<8>, dim3(1), dim3(kBlockThreads), 0, s, a, b, nlev, raw);
    else
        hipLaunchKernelGGL(power_rtile_final<4>, dim3(1), dim3(kBlockThreads), 0, s, a, b, nlev, raw);
    return hipGetLastError();
}

}  // namespace lx
