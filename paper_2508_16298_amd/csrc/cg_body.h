// Conjugate gradient on O = M^dag M (Methods, Eq. pCG), started from x = 0,
// one kernel launch per iteration.
//
// The recursion is CG with a single global reduction phase per iteration
// (the Chronopoulos-Gear arrangement: s = O p carried as a recurrence):
//   beta_i  = gamma_i / gamma_{i-1}            (0 on the first iteration)
//   p_i = r_i + beta_i p_{i-1},  s_i = w_i + beta_i s_{i-1}     (s = O p)
//   alpha_i = gamma_i / <p_i, s_i>
//   x_{i+1} = x_i + alpha_i p_i,  r_{i+1} = r_i - alpha_i s_i
//   w_{i+1} = O r_{i+1}
// mathematically the same iterates as Eq. pCG without preconditioner.  The
// denominator is expanded over vectors the previous launch already holds,
//   <p_i, s_i> = <r_i,w_i> + beta_i (<r_i,s_{i-1}> + <p_{i-1},w_i>)
//                + beta_i^2 <p_{i-1},s_{i-1}>,
// so one launch computes all five inner products of the next iteration
// together.  (The textbook Chronopoulos-Gear denominator
// delta - beta gamma / alpha_{i-1} leans on an orthogonality identity that
// FP32 rounding breaks: in emulation it needed 15-23% more iterations and
// diverged on ill-conditioned systems, while the expansion tracks the
// two-reduction form iteration for iteration.)
// A launch boundary is the only grid-wide synchronisation: every workgroup
// (one per time slice) reduces the per-slice partials of the previous launch
// in a fixed order (bitwise reproducible), recomputes the recurrences on the
// two neighbouring slices it needs for the stencil, and applies O to its
// slice.  r, s and w alternate between two buffers by iteration parity; the
// device scalars alternate between two slots by launch parity, so no launch
// reads what a concurrent workgroup writes.  x takes two steps at a time, at
// every second iteration after an update and where the recursion stops in
// between (the launch past the last iteration always runs): alpha_{i-1} and
// p_{i-1} are at hand there, and 16 of 112 bytes a site and iteration go (FP32:
// r, w, s, p read and r, s, w, p written 64, the phases of both directions 16, x
// 32 every second time).
//
// Stop and pause: an iteration that finds gamma_i <= tol^2 |rhs|^2 turns
// itself and all later launches into no-ops (the host reads the flag once per
// chunk).  The mixed path (complex-FP32 r, p, s, w, O; FP64 x and reductions)
// also pauses when gamma has fallen by 100 since the last reliable update or
// 50 iterations have passed (Sleijpen and van der Vorst 1996): then
// r = rhs - O x is recomputed with the FP64 operator and copied into the FP32
// recursion, w = O r and s = O p are recomputed (s is otherwise only a
// recurrence and drifts; the drift turns the denominator <p, O p> =
// delta - beta gamma / alpha negative on ill-conditioned systems) and the
// iteration resumes with p kept.  A denominator that is not positive forces
// the same update with a restart (beta = 0).  At a stop the FP64 true
// residual decides: converged, or resume (the FP64 path restarts with p = r,
// as the oracle does).
#pragma once
#include <cmath>

#include "cg_common.h"

namespace qh {

// ---------------------------------------------------------------------------
// Start: r_0 = rhs, w_0 = O r_0, x = p = s = 0, partials of iteration 0,
// slot 0 initialised.
// ---------------------------------------------------------------------------
template <typename R, int MC, int NB>
__device__ __forceinline__ void cg_start_body(const Lat& lt, const CgBufs<R>& B, const cplx<R>* __restrict__ gauge,
                                              const Coef<R>& co, double* __restrict__ scal, int tau, bool lead,
                                              const Tile& tl) {
    cplx<R>* buf2 = reinterpret_cast<cplx<R>*>(tl.buf);
    SliceCtx<MC> c;
    slice_ctx<MC>(lt, c, tau, tl);
    const size_t Vs = lt.Vs;
    cplx<R> hm[MC][12], ht[MC][12];
    hops_of<R, MC>(gptr(gauge), lt, c.tm, c.idx, co, hm);
    hops_of<R, MC>(gptr(gauge), lt, c.tau, c.idx, co, ht);
    Cells<R, MC> vm, vt, vn, w;
    double b2 = 0.0, dummy = 0.0;
    load_cvt<R, MC>(vm, gptr(B.rhs) + c.tm * Vs, nullptr, c.g, c.own, dummy);
    load_cvt<R, MC>(vt, gptr(B.rhs) + c.tau * Vs, nullptr, c.g, c.own, b2);
    load_cvt<R, MC>(vn, gptr(B.rhs) + c.tp * Vs, nullptr, c.g, c.own, dummy);
    Cells<R, MC> zero;
    Cells<double, MC> zx;
#pragma unroll
    for (int m = 0; m < MC; m++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            zero.v[m][q] = mk<R>(0, 0);
            zx.v[m][q] = mk<double>(0, 0);
        }
    store_cells<R, MC>(vt, gptr(B.r[0]) + c.tau * Vs, c.g, c.own);
    store_cells<R, MC>(zero, gptr(B.s[0]) + c.tau * Vs, c.g, c.own);
    store_cells<R, MC>(zero, gptr(B.p) + c.tau * Vs, c.g, c.own);
    store_cells<double, MC>(zx, gptr(B.x) + c.tau * Vs, c.g, c.own);
    const Cells<R, MC> r0 = vt;
    mdagm_cells<R, MC, NB>(vm, vt, vn, hm, ht, c.g, c.own, co, c.tau == 0 ? R(-1) : R(1),
                           c.tau == lt.Nt - 1 ? R(-1) : R(1), buf2, lt.Vs, w);
    store_cells<R, MC>(w, gptr(B.w[0]) + c.tau * Vs, c.g, c.own);
    double v[kNP] = {dot_cells<R, MC>(r0, r0, c.own), dot_cells<R, MC>(w, r0, c.own), 0.0, 0.0, 0.0, b2};
    write_partials<kNP>(gptr(B.part), lt.Nt, c.tau, v, tl);  // parity 0
    if (lead && tl.ltid < S_NSLOT) {
        double v = 0.0;
        if (tl.ltid == S_FIRST) v = 1.0;
        if (tl.ltid == S_B2) v = -1.0;
        if (tl.ltid == S_GPREV || tl.ltid == S_APREV) v = 1.0;
        gptr(scal)[tl.ltid] = v;
    }
}

// x += a p in FP64
template <typename R, int MC>
__device__ __forceinline__ void add_scaled(Cells<double, MC>& x, double a, const Cells<R, MC>& p) {
#pragma unroll
    for (int m = 0; m < MC; m++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            x.v[m][q].re += a * (double)p.v[m][q].re;
            x.v[m][q].im += a * (double)p.v[m][q].im;
        }
}

// ---------------------------------------------------------------------------
// One CG iteration (workgroups of THREADS or more).  kpar: launch parity (slot in = kpar, slot out = kpar^1).
// ---------------------------------------------------------------------------
// HALO (workgroups of two and more groups, which hold n consecutive slices
// hl.lo + 1 ... hl.hi - 1 in their first n groups): every group reads and
// advances its own slice alone, the first two the slice before and the slice
// after as well, and the operator takes the neighbours' new r from LDS.
// Against three slices read and advanced by every group it halves the loads
// and, in FP32, brings 200 registers to 166, three workgroups a CU instead of
// two: a launch of 640 workgroups (16 right-hand sides at L = 16, N_tau = 160)
// is one round of them instead of two.
struct Halo {
    int g, n;            // this thread's group; the workgroup's slices
    int lo, hi;          // the slices before and after them
    unsigned char* buf;  // LDS: n + 2 slices of r, a cell's four sites together
};

template <typename R, int MC, int NB, int THREADS, bool HALO>
__device__ __forceinline__ void cg_iter_body(const Lat& lt, const CgBufs<R>& B, const cplx<R>* __restrict__ gauge,
                                             const Coef<R>& co, double* __restrict__ scal, int kpar, int ipar,
                                             double tol2, int mixed, int maxit, int tau, bool lead,
                                             const Tile& tl, const Halo& hl = Halo{}) {
    cplx<R>* buf2 = reinterpret_cast<cplx<R>*>(tl.buf);
    const double* sin_ = gptr(scal) + S_NSLOT * kpar;
    double* sout = gptr(scal) + S_NSLOT * (kpar ^ 1);
    // Every load of the launch is issued before the scalars arrive: the
    // buffer parity ipar comes from the host -- the parity of the number of
    // iterations since the last reliable update (the ping-pong of r, s, w
    // restarts at buffer 0 after every update, so a chunk that starts right
    // after one has ipar = launch index & 1 whatever the iteration count; after
    // a stop or pause inside a chunk the remaining launches are no-ops, so the
    // guess is never used wrongly) -- and the stop flag is looked at only
    // after the loads.  The partials come first: their sums are ready while the
    // vectors are on their way.  All loads are in bounds whatever the flag says.
    const double done = sin_[S_DONE];
    const int it = (int)sin_[S_ITERS];
    const int ip = ipar, nx = ip ^ 1;
    PartSum<THREADS> ps;
    ps.load(gptr(B.part) + kNP * (size_t)lt.Nt * ip, lt.Nt);
    SliceCtx<MC> c;
    slice_ctx<MC>(lt, c, tau, tl);
    const size_t Vs = lt.Vs;
    // (HALO: wm, sm, rm of the slice before or after the workgroup's)
    Cells<R, MC> wm, wt, wn, sm, st, sn, rm, rt, rn, pp;
    load_cells<R, MC>(wt, gptr(B.w[ip]) + c.tau * Vs, c.g);
    load_cells<R, MC>(st, gptr(B.s[ip]) + c.tau * Vs, c.g);
    load_cells<R, MC>(rt, gptr(B.r[ip]) + c.tau * Vs, c.g);
    load_cells<R, MC>(pp, gptr(B.p) + c.tau * Vs, c.g);
    if constexpr (HALO) {
        if (hl.g < 2) {
            const size_t ho = (size_t)(hl.g == 0 ? hl.lo : hl.hi) * Vs;
            load_cells<R, MC>(wm, gptr(B.w[ip]) + ho, c.g);
            load_cells<R, MC>(sm, gptr(B.s[ip]) + ho, c.g);
            load_cells<R, MC>(rm, gptr(B.r[ip]) + ho, c.g);
        }
    } else {
        load_cells<R, MC>(wm, gptr(B.w[ip]) + c.tm * Vs, c.g);
        load_cells<R, MC>(wn, gptr(B.w[ip]) + c.tp * Vs, c.g);
        load_cells<R, MC>(sm, gptr(B.s[ip]) + c.tm * Vs, c.g);
        load_cells<R, MC>(sn, gptr(B.s[ip]) + c.tp * Vs, c.g);
        load_cells<R, MC>(rm, gptr(B.r[ip]) + c.tm * Vs, c.g);
        load_cells<R, MC>(rn, gptr(B.r[ip]) + c.tp * Vs, c.g);
    }
    // (with the halo later, where s and w are gone from the registers: FP64 98.0
    // -> 88.9 ms, FP32 50.3 -> 49.4 ms a trajectory of 16 chains of 8 to 20 cells
    // a side.  FP64 with two cells a thread has no registers for the phases beside
    // the three slices, nor for x under the operator: 200 iterations of four
    // chains of 44 cells a side took 18.2 ms with both, 15.3 ms without, and
    // 16.1 ms with x read and written every time.  Workgroups of more than 512
    // threads have 128 registers: L = 48, N_tau = 480 62.3 -> 57.6 ms a 300
    // iterations)
    constexpr bool tight = sizeof(R) == 8 && (MC == 2 || THREADS > 512);
    constexpr bool late = HALO || tight;
    cplx<R> hm[MC][12], ht[MC][12];
    auto hops = [&]() {
        hops_of<R, MC>(gptr(gauge), lt, c.tm, c.idx, co, hm);
        hops_of<R, MC>(gptr(gauge), lt, c.tau, c.idx, co, ht);
    };
    if constexpr (!late) hops();
    // x is behind by alpha_{i-1} p_{i-1} at odd ip: only every second iteration
    // reads and writes it, and so does the launch that stops in between
    const double aprev = sin_[S_APREV];
    auto catch_up = [&]() {
        if (!ip) return;
        Cells<double, MC> xo;
        load_cells<double, MC>(xo, gptr(B.x) + c.tau * Vs, c.g);
        add_scaled<R, MC>(xo, aprev, pp);
        store_cells<double, MC>(xo, gptr(B.x) + c.tau * Vs, c.g, c.own);
    };
    if (done != 0.0 || it >= maxit) {
        // stopped or paused: carry the state over; a running solve that used
        // its iteration budget is marked for its final true residual (6)
        if (done == 0.0) catch_up();
        if (lead && tl.ltid < S_NSLOT) {
            double v = sin_[tl.ltid];
            if (tl.ltid == S_DONE && v == 0.0) v = 6.0;
            sout[tl.ltid] = v;
        }
        return;
    }

    double pr[kNP];
    ps.finish(tl.red, pr);
    const double gam = pr[0], del = pr[1], aux = pr[5];
    double b2 = sin_[S_B2], target = sin_[S_TARGET], rrupd = sin_[S_RRUPD];
    if (b2 < 0.0) {  // first iteration of the solve: the start kernel left |rhs|^2 partials in aux
        b2 = aux;
        target = tol2 * aux;
        rrupd = gam;
    }
    int stop = 0;
    if (!isfinite(gam) || !isfinite(del) || ((it - (int)sin_[S_ITUPD]) & 1) != ipar)
        stop = 4;  // breakdown: non-finite recursion (or a host/device parity mismatch)
    else if (gam <= target)
        stop = 1;
    else if (mixed && (gam <= kDecade2 * rrupd || it - (int)sin_[S_ITUPD] >= kCap))
        stop = 2;
    if (stop) {
        catch_up();
        if (lead && tl.ltid < S_NSLOT) {
            double v = sin_[tl.ltid];
            if (tl.ltid == S_DONE) v = (double)stop;
            if (tl.ltid == S_B2) v = b2;
            if (tl.ltid == S_TARGET) v = target;
            if (tl.ltid == S_RRUPD) v = rrupd;
            if (tl.ltid == S_GCUR) v = gam;
            sout[tl.ltid] = v;
        }
        return;
    }
    const bool first = sin_[S_FIRST] != 0.0;
    const double beta = first ? 0.0 : gam / sin_[S_GPREV];
    const double den = first ? del : del + beta * (pr[2] + pr[3]) + beta * beta * pr[4];  // <p_i, s_i>
    if (!(den > 0.0)) {
        catch_up();
        if (lead && tl.ltid < S_NSLOT) {
            double v = sin_[tl.ltid];
            if (tl.ltid == S_DONE) v = 3.0;
            if (tl.ltid == S_B2) v = b2;
            if (tl.ltid == S_TARGET) v = target;
            if (tl.ltid == S_RRUPD) v = rrupd;
            if (tl.ltid == S_GCUR) v = gam;
            sout[tl.ltid] = v;
        }
        return;
    }
    const double alpha = gam / den;
    const R b = (R)beta, a = (R)alpha;
    const Cells<R, MC> pold = pp;

    // s_i = w_i + beta s_{i-1};  r_{i+1} = r_i - alpha s_i on the three slices
#pragma unroll
    for (int m = 0; m < MC; m++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            st.v[m][q] = cfma(b, st.v[m][q], wt.v[m][q]);
            pp.v[m][q] = cfma(b, pp.v[m][q], rt.v[m][q]);  // p_i = r_i + beta p_{i-1}
            rt.v[m][q] = cfma(-a, st.v[m][q], rt.v[m][q]);
        }
    auto advance = [&](Cells<R, MC>& r, const Cells<R, MC>& s, const Cells<R, MC>& w) {
#pragma unroll
        for (int m = 0; m < MC; m++)
#pragma unroll
            for (int q = 0; q < 4; q++) r.v[m][q] = cfma(-a, cfma(b, s.v[m][q], w.v[m][q]), r.v[m][q]);
    };
    if constexpr (HALO) {
        cplx<R>* rs = reinterpret_cast<cplx<R>*>(hl.buf);
        auto at = [&](int slot, int m) { return rs + (slot * lt.ncell + c.g[m].c) * 4; };
        if (hl.g < 2) {
            advance(rm, sm, wm);
#pragma unroll
            for (int m = 0; m < MC; m++)
                if (tl.ltid + m * tl.G < lt.ncell)
#pragma unroll
                    for (int q = 0; q < 4; q++) at(hl.g == 0 ? 0 : hl.n + 1, m)[q] = rm.v[m][q];
        }
#pragma unroll
        for (int m = 0; m < MC; m++)
            if (c.own[m])
#pragma unroll
                for (int q = 0; q < 4; q++) at(hl.g + 1, m)[q] = rt.v[m][q];
        if constexpr (late) hops();
        __syncthreads();
        // (a padding group reads slots that may hold nothing, and uses none of it)
#pragma unroll
        for (int m = 0; m < MC; m++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                rm.v[m][q] = at(hl.g, m)[q];
                rn.v[m][q] = at(hl.g + 2, m)[q];
            }
    } else {
        advance(rm, sm, wm);
        advance(rn, sn, wn);
        if constexpr (late) hops();
    }
    store_cells<R, MC>(st, gptr(B.s[nx]) + c.tau * Vs, c.g, c.own);
    store_cells<R, MC>(rt, gptr(B.r[nx]) + c.tau * Vs, c.g, c.own);
    store_cells<R, MC>(pp, gptr(B.p) + c.tau * Vs, c.g, c.own);
    // x_{i+1} = x_{i-1} + alpha_{i-1} p_{i-1} + alpha_i p_i in FP64, on its way
    // while the operator runs (tight: before it)
    Cells<double, MC> xo;
    auto step_x = [&]() {
        if (!ip) return;
        add_scaled<R, MC>(xo, aprev, pold);
        add_scaled<R, MC>(xo, alpha, pp);
        store_cells<double, MC>(xo, gptr(B.x) + c.tau * Vs, c.g, c.own);
    };
    if (ip) load_cells<double, MC>(xo, gptr(B.x) + c.tau * Vs, c.g);
    if constexpr (tight) step_x();
    const Cells<R, MC> rnew = rt;
    Cells<R, MC> w;
    mdagm_cells<R, MC, NB>(rm, rt, rn, hm, ht, c.g, c.own, co, c.tau == 0 ? R(-1) : R(1),
                           c.tau == lt.Nt - 1 ? R(-1) : R(1), buf2, lt.Vs, w);
    store_cells<R, MC>(w, gptr(B.w[nx]) + c.tau * Vs, c.g, c.own);
    if constexpr (!tight) step_x();
    double v[kNP - 1] = {dot_cells<R, MC>(rnew, rnew, c.own), dot_cells<R, MC>(w, rnew, c.own),
                     dot_cells<R, MC>(rnew, st, c.own), dot_cells<R, MC>(pp, w, c.own),
                     dot_cells<R, MC>(pp, st, c.own)};
    write_partials<kNP - 1>(gptr(B.part) + kNP * (size_t)lt.Nt * nx, lt.Nt, c.tau, v, tl);
    if (lead && tl.ltid < S_NSLOT) {
        double v = sin_[tl.ltid];
        if (tl.ltid == S_GPREV) v = gam;
        if (tl.ltid == S_APREV) v = alpha;
        if (tl.ltid == S_ITERS) v = (double)(it + 1);
        if (tl.ltid == S_FIRST) v = 0.0;
        if (tl.ltid == S_B2) v = b2;
        if (tl.ltid == S_TARGET) v = target;
        if (tl.ltid == S_RRUPD) v = rrupd;
        if (tl.ltid == S_GCUR) v = gam;
        sout[tl.ltid] = v;
    }
}

// ---------------------------------------------------------------------------
// Reliable update / true residual: r_i = rhs - O x (FP64 O x given), w_i =
// O r_i in the working precision, partials of iteration i replaced; aux gets
// the FP64 |rhs - O x|^2.  Slot kpar is only read.
// ---------------------------------------------------------------------------
template <typename R, int MC, int NB>
__device__ __forceinline__ void cg_replace_body(const Lat& lt, const CgBufs<R>& B, const cplx<R>* __restrict__ gauge,
                                                const Coef<R>& co, const double* __restrict__ scal, int kpar,
                                                int tau, const Tile& tl) {
    cplx<R>* buf2 = reinterpret_cast<cplx<R>*>(tl.buf);
    const int ip = 0;  // the resumed recursion restarts its ping-pong at buffer 0
    SliceCtx<MC> c;
    slice_ctx<MC>(lt, c, tau, tl);
    const size_t Vs = lt.Vs;
    cplx<R> hm[MC][12], ht[MC][12];
    hops_of<R, MC>(gptr(gauge), lt, c.tm, c.idx, co, hm);
    hops_of<R, MC>(gptr(gauge), lt, c.tau, c.idx, co, ht);
    Cells<R, MC> vm, vt, vn, w;
    double t2 = 0.0, dummy = 0.0;
    load_cvt<R, MC>(vm, gptr(B.rhs) + c.tm * Vs, gptr(B.Ox) + c.tm * Vs, c.g, c.own, dummy);
    load_cvt<R, MC>(vt, gptr(B.rhs) + c.tau * Vs, gptr(B.Ox) + c.tau * Vs, c.g, c.own, t2);
    load_cvt<R, MC>(vn, gptr(B.rhs) + c.tp * Vs, gptr(B.Ox) + c.tp * Vs, c.g, c.own, dummy);
    store_cells<R, MC>(vt, gptr(B.r[ip]) + c.tau * Vs, c.g, c.own);
    const Cells<R, MC> r0 = vt;
    const R em = c.tau == 0 ? R(-1) : R(1), et = c.tau == lt.Nt - 1 ? R(-1) : R(1);
    mdagm_cells<R, MC, NB>(vm, vt, vn, hm, ht, c.g, c.own, co, em, et, buf2, lt.Vs, w);
    store_cells<R, MC>(w, gptr(B.w[ip]) + c.tau * Vs, c.g, c.own);
    // s_{i-1} = O p_{i-1}, recomputed
    Cells<R, MC> pm, pt_, pn, sp;
    load_cells<R, MC>(pm, gptr(B.p) + c.tm * Vs, c.g);
    load_cells<R, MC>(pt_, gptr(B.p) + c.tau * Vs, c.g);
    load_cells<R, MC>(pn, gptr(B.p) + c.tp * Vs, c.g);
    __syncthreads();  // LDS exchange buffers are reused
    mdagm_cells<R, MC, NB>(pm, pt_, pn, hm, ht, c.g, c.own, co, em, et, buf2, lt.Vs, sp);
    store_cells<R, MC>(sp, gptr(B.s[ip]) + c.tau * Vs, c.g, c.own);
    double v[kNP] = {dot_cells<R, MC>(r0, r0, c.own), dot_cells<R, MC>(w, r0, c.own),
                     dot_cells<R, MC>(r0, sp, c.own), dot_cells<R, MC>(pt_, w, c.own),
                     dot_cells<R, MC>(pt_, sp, c.own), t2};
    write_partials<kNP>(gptr(B.part) + kNP * (size_t)lt.Nt * ip, lt.Nt, c.tau, v, tl);
}


// After k_cg_replace: true |r|^2 into the slot; converged -> stop flag 1;
// otherwise clear the flag and resume (restart: beta = 0 on the next
// iteration, the FP64 path's p = r).
__device__ __forceinline__ void cg_check_body(double* __restrict__ scal, int kpar, const double* __restrict__ part,
                                              int Nt, int restart, double* red) {
    double* sl = scal + S_NSLOT * kpar;
    const int ip = 0;  // the replacement's partials
    double pr[kNP];
    reduce_partials(part + kNP * (size_t)Nt * ip, Nt, whole_block_tile(nullptr, red), pr);
    const double a = pr[0], c = pr[5];
    if (threadIdx.x == 0) {
        sl[S_TRUE] = c;
        if (c <= sl[S_TARGET]) {
            sl[S_DONE] = 1.0;
        } else {
            sl[S_DONE] = 0.0;
            if (restart) sl[S_FIRST] = 1.0;
            sl[S_ITUPD] = sl[S_ITERS];
            sl[S_RRUPD] = a;
        }
    }
}

}  // namespace qh
