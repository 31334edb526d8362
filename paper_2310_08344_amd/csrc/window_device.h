// The window loop's control, shared by its kernels: leja_block (LDS tiles,
// block.hip), leja_stream (register marching, stream.hip) and leja_rtile
// (register tiles, rtile.hip).
//
// Launch w of the plain loop advances the Newton recurrence (Sec. 2.1,
// Eq. (2)) from y_m (m = wD) through y_{m+1} .. y_{m+D}.  The stop rule
// (Sec. 2.2) for term m+j needs norms of y_{m+j} and of p_{m+j} over the
// whole grid, which exist only after the launch; a window therefore adds all
// D terms speculatively to every output still iterating and records, for
// every j, the sums of squares of y_{m+j} and of each output as it stands
// after term m+j.  The next launch applies the stop rule at m+1, .., m+D in
// turn and, if an output stopped inside the window, re-executes the window
// for the stopped outputs only, with exactly the terms they take.
#pragma once

#include <hip/hip_runtime.h>

#include "lx_device.h"
#include "sweep_device.h"
#include "tile_device.h"

namespace lx {
namespace dev {

// v of lane l - 1 (kFromBelow: DPP wave_shr:1) or of lane l + 1 (wave_shl:1);
// the lane with no such neighbour keeps `old`.  Every lane of the wavefront
// must be active.
template <bool kFromBelow>
__device__ __forceinline__ double lane_neighbour(const double v, const double old) {
    constexpr int ctrl = kFromBelow ? 0x138 : 0x130;
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), ctrl, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), ctrl, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// What the stop rule says about a window, from its norms: the term at which
// each output stops (D: it may go on, or stops there), with its last error
// estimate and norm.
template <int K>
struct WindowVerdict {
    bool nonfinite, any_stop, capped;
    bool stop[K];
    int j[K];
    double err[K], pnorm[K], ynorm;
    int fp32_after;   // kSwitch: the first term after which FP32 sweeps start (D: with the next window), 0: none
};

// Applies the stop rule at the terms m+1 .. m+D of a window, one lane per
// norm: lane q holds norm q = (j-1)(1+K) + r of the window, r = 0: y_{m+j},
// r = 1+k: output k after term m+j.  Taken in order, an output is tested at
// j = 1, 2, .. until it stops (its estimate passes, or m + j reaches
// max_iters); a non-finite norm or estimate at a tested term ends the loop.
// Every lane of the wavefront must be active; all receive the verdict.
//
// kSwitch: also the term after which FP32 sweeps start, as the one-iteration
// loop finds it: the first at which some output goes on and every one that
// does has |d| ||y|| <= fp32_switch * (rtol ||p|| + atol).
template <int K, int D, bool kSwitch = false>
__device__ __forceinline__ WindowVerdict<K> window_verdict(const LoopCtl& ctl, const int m, const int (&active)[K],
                                                           const double norm, const double coef) {
    constexpr int R = 1 + K;
    const int lane = flat_tid() & 63, j = lane / R + 1;
    const bool live = lane < D * R && lane % R != 0;
    const double yn = __shfl(norm, (j - 1) * R & 63, 64);
    const double e = fabs(coef) * yn;
    const double thr = ctl.rtol * norm + ctl.atol;
    const bool fin = isfinite(norm) && isfinite(e);
    const bool pass = live && fin && e <= thr;
    const bool cap = live && fin && !(e <= thr) && m + j >= ctl.max_iters;
    const unsigned long long b_pass = __ballot(pass), b_cap = __ballot(cap), b_bad = __ballot(live && !fin);
    WindowVerdict<K> v;
    v.nonfinite = v.any_stop = v.capped = false;
    int last = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        unsigned long long mine = 0;   // the lanes of output k
#pragma unroll
        for (int i = 0; i < D; ++i) mine |= 1ull << (i * R + 1 + k);
        const unsigned long long ends = (b_pass | b_cap) & mine;
        const int q = ends != 0 ? __ffsll(static_cast<long long>(ends)) - 1 : (D - 1) * R + 1 + k;
        v.j[k] = q / R + 1;
        v.stop[k] = active[k] && ends != 0;
        v.err[k] = __shfl(e, q, 64);
        v.pnorm[k] = __shfl(norm, q, 64);
        if (active[k]) {
            if ((b_bad & mine & ((2ull << q) - 1)) != 0) v.nonfinite = true;
            if (ends != 0) v.any_stop = true;
            if (((b_cap >> q) & 1) != 0) v.capped = true;
            last = v.j[k] > last ? v.j[k] : last;
        }
    }
    v.ynorm = __shfl(norm, last > 0 ? (last - 1) * R : 0, 64);
    v.fp32_after = 0;
    if constexpr (kSwitch) {
        const unsigned long long b_small =
            __ballot(live && fin && ctl.fp32_switch >= 0.0 && e <= ctl.fp32_switch * thr);
        bool ended = false;   // a non-finite value at a tested term
#pragma unroll
        for (int i = 1; i <= D; ++i) {
            bool goes_on = false, small = true;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (!active[k]) continue;
                const int q = (i - 1) * R + 1 + k;
                if (v.j[k] >= i && ((b_bad >> q) & 1) != 0) ended = true;
                if (v.stop[k] && v.j[k] <= i) continue;
                goes_on = true;
                if (((b_small >> q) & 1) == 0) small = false;
            }
            if (v.fp32_after == 0 && !ended && goes_on && small) v.fp32_after = i;
        }
    }
    return v;
}

// The state entering a launch from the state of the previous launch and, if
// that was a window, the verdict on it.
//
// kFp32 (FP32 sweeps): a window forms its levels and writes y_{m+D} in FP32
// (out32) once, at the last term of the window before it, every output
// still iterating has |d| ||y|| <= fp32_switch * (rtol ||p|| + atol); from
// then on every window does.  in32: the window's y_m is stored in FP32.  A
// re-execution keeps the precision of the window it repeats.
//
// kSwitch: FP32 sweeps start after the very term (fp32_after) at which they
// do one iteration at a time.  Where that is not the window's last, the
// window is formed again with lev64 levels in FP64 and the others in FP32,
// and its stops are taken from that.
template <int K, int D, bool kFp32 = false, bool kSwitch = false>
__device__ __forceinline__ SweepState block_decide(const LoopCtl& ctl, const SweepState& prev,
                                                   const WindowVerdict<K>& v) {
    SweepState nx = prev;
    if (prev.blk_mode == 1) {
        // the window was re-executed with its stops: the outputs that took all
        // D terms go on from y_{m+D}
        nx.blk_mode = 0;
        nx.iter = prev.iter + D;
        nx.in32 = prev.out32;
        if (kSwitch && prev.lev64 < 0) {
            nx.out32 = 1;
            nx.lev64 = 0;
        }
        bool any = false;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            nx.active[k] = (prev.active[k] && prev.nt[k] == D) ? 1 : 0;
            nx.nt[k] = nx.active[k] ? D : 0;
            any = any || nx.active[k];
        }
        if (!any) nx.done = 1;
        return nx;
    }
    const int m = prev.iter;
    const int after = kSwitch && !prev.out32 ? v.fp32_after : 0;
    if (after > 0 && after < D) {
        nx.out32 = 1;
        nx.lev64 = after;
        return nx;
    }
    bool any_active = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (!prev.active[k]) continue;
        any_active = true;
        nx.err[k] = v.err[k];
        nx.pnorm[k] = v.pnorm[k];
        if (v.stop[k]) nx.iters[k] = m + v.j[k];
    }
    if (any_active) nx.ynorm = v.ynorm;
    if (v.nonfinite) {
        nx.status = 4;   // LX_ENONFINITE
        nx.done = 1;
        return nx;
    }
    if (v.any_stop) {
        // re-execute the window with the stops: nt[k] = -j for an output
        // that stopped after term m+j, D for one that goes on, 0 otherwise
        nx.blk_mode = 1;
#pragma unroll
        for (int k = 0; k < K; ++k) nx.nt[k] = !prev.active[k] ? 0 : (v.stop[k] ? -v.j[k] : D);
        if (v.capped) nx.status = 3;   // LX_ENOTCONV
        if (after == D) nx.lev64 = -1;
    } else {
        nx.iter = m + D;
        nx.in32 = prev.out32;
        if (after == D) {
            nx.out32 = 1;
            nx.lev64 = 0;
        }
        if (kFp32 && !kSwitch && !prev.out32 && ctl.fp32_switch >= 0.0) {
            bool small = true;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (prev.active[k] &&
                    !(nx.err[k] <= ctl.fp32_switch * (ctl.rtol * nx.pnorm[k] + ctl.atol)))
                    small = false;
            if (small) nx.out32 = 1;
        }
    }
    return nx;
}

// What launch L of a window loop does, decided at its entry.
template <int K>
struct WindowPlan {
    int m;                  // the window's first term index
    int win;                // window number, m / D
    bool redo;              // re-execution of a window in which an output stopped
    int nt[K];              // terms each output takes in this launch
    int jmax;               // levels this launch forms
    bool win32;             // levels formed, and y_{m+D} written, in FP32
    int lev64;              // kSwitch, win32 and not in32: but for the first lev64 (the next is formed in FP64 and rounded)
    bool in32;              // y_m is stored in FP32
    bool copy[K];           // a re-execution copies this output unchanged (pin to pout)
    const double* pin[K];   // outputs as the window finds them
    double* pout[K];        // and where it leaves them
    const double* yin;      // y_m
    double* yout;           // y_{m+D}
};

// Entry of launch L of the window loop as workgroup `wg` of the a.nb that
// serve this grid (at most NW wavefronts each): the decision from the previous
// launch's partial sums.  Workgroup 0 records the state; when the loop has
// ended it publishes slot[2] and, if `done` is given, counts the grid as
// finished.  Returns false when this launch has nothing to do (the same in
// every thread), also once the loop has ended.
//
// Every workgroup of every launch pays for this before its first level, so it
// is a short chain: the end flag, the state, the partial sums and the
// coefficients are loaded at once, the norms and their tests take a lane each.
// Before, one thread tested term after term behind a butterfly per value: a
// window of four on a 64^2 grid, all latency, went from 14.6 to 10.3 us, the
// windows of eight of 4096^2 (three outputs) from 215 to 196.
//
// kEndCopy: in a re-execution, an output that stopped after the window's
// last term (j = D) is not recomputed: the window's own result is exact.
// An odd window wrote it to the caller's buffer already (nothing to do); an
// even window's result is copied there (WindowPlan::copy).
//
// Buffers: window w reads y_m from v (w = 0) or ybuf[(w-1) & 1] and writes
// y_{m+D} to ybuf[w & 1]; it reads the outputs from p (w even) or p2 (w odd)
// and writes them to the other; a re-execution writes stopped outputs to p,
// the caller's buffer, so every final result lands there.
template <int OP, int K, int D, bool kEndCopy = false, bool kFp32 = false, int NW = kBlockThreads / 64,
          bool kSwitch = false>
__device__ __forceinline__ bool window_enter(const SweepArgs& a, const int L, const int wg, unsigned* done,
                                             WindowPlan<K>& w) {
    LoopCtl* __restrict__ ctl = gptr(a.ctl);
    constexpr int NV = D * (1 + K);
    __shared__ SweepState s_cur;
    const int tid = flat_tid();
    if (wg == 0 && tid == 0) report_progress(a, L);
    if (L == 0) {
        if (tid == 0) {
            SweepState st = ctl->slot[0];
            st.blk_mode = 0;
            st.iter = 0;
            for (int k = 0; k < kKMax; ++k) st.nt[k] = (k < K && st.active[k]) ? D : 0;
            st.n_work = 1;
            st.n_levels = D;
            st.in32 = 0;
            if (!kFp32) st.out32 = 0;
            st.n_fp32 = st.out32 ? D : 0;
            // v in, y_D out, the Burgers state, each output written
            double b = 8.0 + (st.out32 ? 4.0 : 8.0) + (OP == kOpBurgersJ ? (st.out32 && !kSwitch ? 4.0 : 8.0) : 0.0);
            for (int k = 0; k < K; ++k) b += st.nt[k] ? 8.0 : 0.0;
            st.bytes_pp = b;
            s_cur = st;
            if (wg == 0) ctl->slot[0] = st;
        }
    } else {
        // wavefront 0 decides; its lanes load what they need before the sums
        const SweepState* __restrict__ ps = &ctl->slot[(L - 1) & 1];
        const int lane = tid & 63;
        int ended = 0, m = 0, active[K];
        double cf = 0.0;
        if (tid < 64) {
            if (tid == 0) ended = __hip_atomic_load(&ctl->slot[2].done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            m = ps->iter;
#pragma unroll
            for (int k = 0; k < K; ++k) active[k] = ps->active[k];
            // (past the end of the loop m may lie beyond the last window)
            const int r = lane % (1 + K), j = m + lane / (1 + K) + 1;
            if (lane < NV && r > 0) cf = gptr(a.coef)[(r - 1) * a.ld + (j < a.ld ? j : a.ld - 1)];
        }
        const double tot = record_totals<NV, NW>(gptr(a.partials) + static_cast<long>((L - 1) & 1) * a.nb * NV, a.nb);
        if (tid < 64) {
            const double norm = lane < NV ? sqrt(tot) * a.inv_sqrtN : 0.0;
            const WindowVerdict<K> v = window_verdict<K, D, kSwitch>(*ctl, m, active, norm, cf);
            if (tid == 0) {
                SweepState st = block_decide<K, D, kFp32, kSwitch>(*ctl, *ps, v);
                if (ended) st.done = 1;
                if (!st.done) {
                    // algorithmic bytes per point: y in (and out, unless a
                    // re-execution), and per output written p (in and out; the
                    // first window only writes it)
                    const bool rd = st.blk_mode == 1;
                    st.n_work += 1;
                    double b = 0.0;
                    int lev = rd ? 0 : D;
                    for (int k = 0; k < K; ++k) {
                        const bool end = kEndCopy && rd && st.nt[k] == -D;   // exact already: copied or kept
                        const bool w_k = rd ? (st.nt[k] < 0 && (!end || (st.iter / D) % 2 == 0)) : st.nt[k] != 0;
                        if (w_k) b += st.iter == 0 && !end ? 8.0 : 16.0;
                        if (rd && !end && -st.nt[k] > lev) lev = -st.nt[k];
                    }
                    // y in (and out), and u, when levels are formed
                    const double yb = st.in32 ? 4.0 : 8.0, ob = st.out32 ? 4.0 : 8.0;
                    const double ub = kSwitch && !st.in32 ? 8.0 : ob;
                    if (!rd || lev > 0) b += yb + (rd ? 0.0 : ob) + (OP == kOpBurgersJ ? ub : 0.0);
                    st.bytes_pp += b;
                    st.n_levels += lev;
                    if (!rd && st.out32) st.n_fp32 += D;
                }
                s_cur = st;
                if (wg == 0 && !ended) {
                    ctl->slot[L & 1] = st;
                    if (st.done) {
                        publish_final(ctl, a.pub, st);   // this launch does no work
                        if (done != nullptr) atomicAdd(done, 1u);
                    }
                }
            }
        }
    }
    __syncthreads();
    if (s_cur.done) return false;
    // every field below is the same in all threads of the grid
    w.m = __builtin_amdgcn_readfirstlane(s_cur.iter);
    w.win = w.m / D;
    w.redo = __builtin_amdgcn_readfirstlane(s_cur.blk_mode) == 1;
    w.win32 = kFp32 && __builtin_amdgcn_readfirstlane(s_cur.out32) != 0;
    w.in32 = kFp32 && __builtin_amdgcn_readfirstlane(s_cur.in32) != 0;
    w.lev64 = kSwitch ? __builtin_amdgcn_readfirstlane(s_cur.lev64) : 0;
    // terms each output takes in this launch.  A re-execution recomputes
    // only the outputs that stopped (their final buffer is p); the others,
    // and y_{m+D}, the window already wrote exactly.
    w.jmax = w.redo ? 0 : D;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = __builtin_amdgcn_readfirstlane(s_cur.nt[k]);
        const bool end = kEndCopy && w.redo && q == -D;
        w.nt[k] = (w.redo && !end) ? (q < 0 ? -q : 0) : (w.redo ? 0 : q);
        if (w.nt[k] > w.jmax) w.jmax = w.nt[k];
        // an even window wrote its outputs to p2, an odd one to p
        w.copy[k] = end && (w.win & 1) == 0;
        w.pin[k] = gptr(end ? a.p2[k] : ((w.win & 1) ? a.p2[k] : a.p[k]));
        w.pout[k] = gptr(w.redo ? a.p[k] : ((w.win & 1) ? a.p[k] : a.p2[k]));
    }
    // selects, not a[win & 1]: indexing would keep a batch's arguments in memory
    double* const y0 = static_cast<double*>(a.ybuf[0]);
    double* const y1 = static_cast<double*>(a.ybuf[1]);
    w.yin = gptr(w.win == 0 ? a.v : static_cast<const double*>((w.win & 1) ? y0 : y1));
    w.yout = gptr((w.win & 1) ? y1 : y0);
    return true;
}

// Exit of a window launch: the workgroup's sums of squares of every level
// (sy[j-1]: y_{m+j}) and of every output after each term (sp[k][j-1]), in a
// fixed order, into this workgroup's record of partials[L & 1].
template <int K, int D, int NW = kBlockThreads / 64>
__device__ __forceinline__ void window_exit(const SweepArgs& a, const int L, const int wg, const double (&sy)[D],
                                            const double (&sp)[K][D]) {
    constexpr int NV = D * (1 + K);
    double v[NV];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        v[j * (1 + K)] = sy[j];
#pragma unroll
        for (int k = 0; k < K; ++k) v[j * (1 + K) + 1 + k] = sp[k][j];
    }
    const double s = block_sums<NV, NW>(v);
    if (flat_tid() < NV)
        gptr(a.partials)[static_cast<long>(L & 1) * a.nb * NV + static_cast<long>(wg) * NV + flat_tid()] = s;
}

}  // namespace dev
}  // namespace lx
