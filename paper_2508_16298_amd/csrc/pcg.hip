// The paper's preconditioner (Methods, "CG method and preconditioner"; the
// banded structure of Fig. 3) and CG preconditioned with it.
//
// Construction (once per handle, on first use), following the paper's recipe
// as read for this build:
//   1. O_pi = M^dag M at pi flux (theta_x = 0, theta_y = pi x) on a build
//      lattice of kBuildL x kBuildL x kBuildNt, assembled column by column by
//      the library's own FP64 M^dag M kernel applied to unit vectors;
//   2. forward IC(0) on the host in the natural order n = tau*Vs + s,
//      O_pi ~ L L^dag on the pattern of O_pi (|O| > 1e-12 max|O|), with a
//      diagonal shift if a pivot is not positive;
//   3. the rows of G = L^{-1} at an interior site of a bulk slice, one per x
//      parity (the pi-flux unit cell), by one triangular solve each;
//   4. taps (dtau, dx, dy, g) with 0 <= dtau <= kCapTau and |g| >= kThresh
//      (the paper's matrix shows a band of 6 in tau; the reach here was
//      chosen by time to solution).
// Application: G[(tau,s),(tau-dtau, s+ds)] = g_{x(s) mod 2}(dtau, ds), with
// -1 when tau-dtau wraps (antiperiodic), and P = G^dag G as two stencil
// passes.  P is Hermitian positive definite whenever G is non-singular.
//
// PCG, one iteration = three launches in spectral form (every read of a
// neighbouring slice crosses a launch boundary, so no buffer is read and
// written in one launch):
//   k_pcg_upd       partial sums -> beta, alpha (single reduction phase as in
//                   the unpreconditioned solver, denominator <p,s> expanded);
//                   p = u + beta p, s = w + beta s, x += alpha p, r -= alpha s;
//                   the forward DFT of r
//   k_pcs_tsum_inv  u = P r (k_pcs_tsum and k_pcs_inv on large slices; two
//                   stencil passes where the spectral form is not built)
//   k_pcg_mv        w = O u and the partials <r,r>, <r,u>, <w,u>, <u,s>, <p,w>, <p,s>
// with gamma = <r, P r>; stopping and reliable updates on |r| as in cg.hip.
//
// Up to 512 cells per slice the same three launches also carry out the
// reliable updates (no gated launches beside them, and none wasted after a
// pause): an update kernel that pauses the recursion leaves its request in the
// slot; the matvec of that triple, which would have nothing to do, forms
// r = rhs - O x in FP64 and s = O p instead; the next update kernel decides on
// the true residual and, where the solve goes on, transforms the new r.  A
// solve starts as if it had just paused.
#include <algorithm>
#include <vector>

#include <cstdlib>
#include <cstring>
#include "cg_common.h"
#include "spectral.h"

namespace qh {

static constexpr int kBuildL = 8;
static constexpr int kBuildNt = 24;
static constexpr int kCapTau = QEDHMC_PC_TAU_REACH;  // tau reach of G (QEDHMC_PC_CAP overrides, up to kCapMax)
static constexpr int kCapMax = 12;
static constexpr double kThresh = 1e-3;
static constexpr int kNP6 = 6;  // PCG partials: <r,r>, <r,u>, <w,u>, <u,s>, <p,w>, <p,s>

static constexpr int kPcSlots = 16;  // tau offsets per stencil pass at most (0 <= dt <= kCapMax, plus spare)

// One stencil tap of a parity's list, q = parity + c - cmin: aidx = a - amin
// (its slice in the window ring), off = b * half + (q >> 1) and plane = q & 1
// (row, column pair and column parity of the source relative to the output).
template <typename R>
struct PTap {
    int aidx;
    int off;
    int plane;
    int pad;
    cplx<R> g;
};

// ---------------------------------------------------------------------------
// Builder
// ---------------------------------------------------------------------------
__global__ void k_unit(cplx<double>* __restrict__ e, size_t n, size_t k) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        e[i] = mk<double>(i == k ? 1.0 : 0.0, 0.0);
}

// ---------------------------------------------------------------------------
// Spectral form of P.  Both passes are gathers whose taps depend only on the
// output's x parity, with space periodic and one sign flip per wrap of tau
// (the antiperiodic extension itself once N_tau exceeds a pass's tau reach).
// So each pass commutes with translations by the two-site cell (2 in x, 1 in
// y) and by one slice, and on the cell momenta kx = 2 pi nx / (L/2),
// ky = 2 pi ny / L it acts on the pair (v_even, v_odd) of a slice as a 2x2
// matrix S(k, a) per tau offset a:
//   S[p][p'](k, a) = sum over the taps (a, b, c, g) of parity p with
//                    (p + c) mod 2 = p' of g exp(i (kx (p + c - p') / 2 + ky b)).
// P = S_1 S_0 has the blocks H(k, a) = sum_{a1 + a2 = a} S_1(k, a2) S_0(k, a1)
// for a in [amin_0 + amin_1, amax_0 + amax_1], and one application is a 2D DFT
// of every slice's two parity planes, the banded tau sum
// z^(k, tau) = sum_a sign H(k, a) v^(k, tau + a) (sign -1 per wrap), and the
// inverse DFT (its 1 / (L L/2) folded into H).  Same operator, far fewer
// operations than the taps at the sizes the stencil is latency-bound at.
// ---------------------------------------------------------------------------
static_assert(kCapMax == kSpTau, "the tau sum's registers hold kSpTau offsets either way");
static constexpr int kSpecMaxNK = 8192;  // momenta per parity plane at most (4096 in FP64)

// Blocks of 16 DFT outputs per axis (y, x): the kernels' instantiations
static void spec_blocks(int L, int& ny, int& nx) {
    const int b = (L / 2 + 1 + 15) / 16;
    ny = b <= 3 ? b : 5;
    nx = b <= 2 ? 1 : (b <= 3 ? 2 : 3);
}

static qedhmc_status build_spectral(qedhmc_ctx* h, const std::vector<HostTap> (&pass)[2][2]) {
    h->pc_spec_na = 0;
    const int L = h->lat.L, Lh = L / 2, nk = L * Lh;
    if (L % 2 || h->lat.Nt <= h->pc_cap || nk > kSpecMaxNK) return QEDHMC_OK;
    const int a0 = h->pc_pass[0].amin + h->pc_pass[1].amin, a1 = h->pc_pass[0].amax + h->pc_pass[1].amax;
    const int na = a1 - a0 + 1;
    if (a0 != -a1 || a1 > kSpTau) return QEDHMC_OK;
    // e^{+2 pi i j / n} by integer index, so every phase is one table entry
    auto unit = [](int n) {
        std::vector<cplx<double>> t(n);
        for (int j = 0; j < n; j++) t[j] = mk<double>(std::cos(2 * M_PI * j / n), std::sin(2 * M_PI * j / n));
        return t;
    };
    const std::vector<cplx<double>> ex = unit(Lh), ey = unit(L);
    auto pmod = [](int v, int n) { return ((v % n) + n) % n; };
    auto cmul = [](cplx<double> x, cplx<double> y) {
        return mk<double>(x.re * y.re - x.im * y.im, x.re * y.im + x.im * y.re);
    };
    std::vector<cplx<double>> H((size_t)na * 4 * nk, mk<double>(0.0, 0.0));  // [a][entry pp'][k]
    const int n0 = h->pc_pass[0].amax - h->pc_pass[0].amin + 1, n1 = h->pc_pass[1].amax - h->pc_pass[1].amin + 1;
    std::vector<cplx<double>> S0((size_t)n0 * 4), S1((size_t)n1 * 4);
    for (int ny = 0; ny < L; ny++)
        for (int nx = 0; nx < Lh; nx++) {
            const int k = ny * Lh + nx;
            for (int ps = 0; ps < 2; ps++) {
                std::vector<cplx<double>>& S = ps ? S1 : S0;
                std::fill(S.begin(), S.end(), mk<double>(0.0, 0.0));
                for (int p = 0; p < 2; p++)
                    for (const auto& t : pass[ps][p]) {
                        const int pp = pmod(p + t.dx, 2), m = (p + t.dx - pp) / 2;
                        const cplx<double> ph = cmul(ex[pmod(m * nx, Lh)], ey[pmod(t.dy * ny, L)]);
                        cplx<double>& e = S[(size_t)(t.dt - h->pc_pass[ps].amin) * 4 + 2 * p + pp];
                        const cplx<double> c = cmul(mk<double>(t.gre, t.gim), ph);
                        e.re += c.re;
                        e.im += c.im;
                    }
            }
            for (int i0 = 0; i0 < n0; i0++)
                for (int i1 = 0; i1 < n1; i1++) {
                    const int ia = h->pc_pass[0].amin + i0 + h->pc_pass[1].amin + i1 - a0;
                    for (int p = 0; p < 2; p++)
                        for (int pp = 0; pp < 2; pp++) {
                            cplx<double>& e = H[((size_t)ia * 4 + 2 * p + pp) * nk + k];
                            for (int q = 0; q < 2; q++) {
                                const cplx<double> c = cmul(S1[(size_t)i1 * 4 + 2 * p + q], S0[(size_t)i0 * 4 + 2 * q + pp]);
                                e.re += c.re;
                                e.im += c.im;
                            }
                        }
                }
        }
    // only the offsets a >= 0 are kept (H(k, -a) = H(k, a)^dagger), as
    // [a][row][k] pairs of a row's two entries, normalised for the DFT pair
    const double norm = 1.0 / nk;
    std::vector<cplx<double>> Hh((size_t)(a1 + 1) * 4 * nk);
    for (int a = 0; a <= a1; a++)
        for (int row = 0; row < 2; row++)
            for (int k = 0; k < nk; k++)
                for (int c = 0; c < 2; c++) {
                    const cplx<double> e = H[((size_t)(a - a0) * 4 + 2 * row + c) * nk + k];
                    Hh[((size_t)(2 * a + row) * nk + k) * 2 + c] = mk<double>(e.re * norm, e.im * norm);
                }
    int ny, nx;
    spec_blocks(L, ny, nx);
    const size_t ntab = sp_table(L, ny) + sp_table(Lh, nx);
    std::vector<double> tw(ntab);
    std::vector<float> tw32(ntab);
    sp_fill_table<double>(L, ny, tw.data());
    sp_fill_table<double>(Lh, nx, tw.data() + sp_table(L, ny));
    sp_fill_table<float>(L, ny, tw32.data());
    sp_fill_table<float>(Lh, nx, tw32.data() + sp_table(L, ny));
    std::vector<cplx<float>> H32(Hh.size());
    for (size_t i = 0; i < Hh.size(); i++) H32[i] = mk<float>((float)Hh[i].re, (float)Hh[i].im);
    QH_HIP(hipMalloc(&h->pc_spec64, Hh.size() * sizeof(cplx<double>)));
    QH_HIP(hipMalloc(&h->pc_spec32, H32.size() * sizeof(cplx<float>)));
    QH_HIP(hipMalloc(&h->pc_tw64, tw.size() * sizeof(double)));
    QH_HIP(hipMalloc(&h->pc_tw32, tw32.size() * sizeof(float)));
    QH_HIP(hipMemcpyAsync(h->pc_spec64, Hh.data(), Hh.size() * sizeof(cplx<double>), hipMemcpyHostToDevice, h->stream));
    QH_HIP(hipMemcpyAsync(h->pc_spec32, H32.data(), H32.size() * sizeof(cplx<float>), hipMemcpyHostToDevice, h->stream));
    QH_HIP(hipMemcpyAsync(h->pc_tw64, tw.data(), tw.size() * sizeof(double), hipMemcpyHostToDevice, h->stream));
    QH_HIP(hipMemcpyAsync(h->pc_tw32, tw32.data(), tw32.size() * sizeof(float), hipMemcpyHostToDevice, h->stream));
    // the host vectors die at return: wait for the copies
    QH_HIP(hipStreamSynchronize(h->stream));
    h->pc_spec_a0 = a0;
    h->pc_spec_na = na;
    return QEDHMC_OK;
}

static qedhmc_status build_paper_precond(qedhmc_ctx* h) {
    qedhmc_params bp = h->p;
    bp.L = kBuildL;
    bp.Nt = kBuildNt;
    qedhmc_ctx* b = nullptr;
    QH_TRY(qedhmc_init_lattice(&bp, h->stream, &b));
    const int L0 = kBuildL, Vs = L0 * L0, n = Vs * kBuildNt;
    std::vector<double> th(2 * (size_t)n, 0.0);
    for (int tau = 0; tau < kBuildNt; tau++)
        for (int y = 0; y < L0; y++)
            for (int x = 0; x < L0; x++) th[(size_t)(kBuildNt + tau) * Vs + y * L0 + x] = M_PI * x;
    double *dth = nullptr, *dcols = nullptr, *de = nullptr;
    std::vector<cplx<double>> O((size_t)n * n);  // column-major: O[k * n + i] = O_ik
    qedhmc_status st = QEDHMC_OK;
    auto fail = [&](hipError_t e, const char* w) { st = hip_fail(e, w); };
    hipError_t e = hipMalloc(&dth, th.size() * sizeof(double));
    if (e == hipSuccess) e = hipMalloc(&dcols, (size_t)n * n * sizeof(cplx<double>));
    if (e == hipSuccess) e = hipMalloc(&de, (size_t)n * sizeof(cplx<double>));
    if (e == hipSuccess) e = hipMemcpyAsync(dth, th.data(), th.size() * sizeof(double), hipMemcpyHostToDevice, h->stream);
    if (e != hipSuccess) fail(e, "preconditioner build allocation");
    if (st == QEDHMC_OK) st = ensure_gauge(b, dth, QEDHMC_FP64);
    for (int k = 0; k < n && st == QEDHMC_OK; k++) {
        hipLaunchKernelGGL(k_unit, dim3(8), dim3(256), 0, h->stream, (cplx<double>*)de, (size_t)n, (size_t)k);
        st = launch_mdagm(b, QEDHMC_FP64, de, dcols + (size_t)2 * k * n, nullptr);
    }
    if (st == QEDHMC_OK) {
        e = hipMemcpyAsync(O.data(), dcols, O.size() * sizeof(cplx<double>), hipMemcpyDeviceToHost, h->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) fail(e, "preconditioner build copy");
    }
    (void)hipFree(dth);
    (void)hipFree(dcols);
    (void)hipFree(de);
    qedhmc_destroy(b);
    if (st != QEDHMC_OK) return st;

    // IC(0), left-looking, dense storage of the lower factor (column-major)
    double omax = 0.0;
    for (const auto& z : O) omax = std::max(omax, std::hypot(z.re, z.im));
    const double cut = 1e-12 * omax;
    std::vector<cplx<double>> Lf((size_t)n * n, mk<double>(0.0, 0.0));
    double shift = 0.0;
    for (;;) {
        bool ok = true;
        std::fill(Lf.begin(), Lf.end(), mk<double>(0.0, 0.0));
        for (int k = 0; k < n && ok; k++) {
            // col[i] = A_ik - sum_{j<k} L_ij conj(L_kj), i >= k
            std::vector<cplx<double>> col(n - k);
            for (int i = k; i < n; i++) {
                cplx<double> a = O[(size_t)k * n + i];
                if (i == k) a.re += shift * O[(size_t)k * n + k].re;
                double sr = 0.0, si = 0.0;
                for (int j = 0; j < k; j++) {
                    const cplx<double> lij = Lf[(size_t)j * n + i], lkj = Lf[(size_t)j * n + k];
                    sr += lij.re * lkj.re + lij.im * lkj.im;
                    si += lij.im * lkj.re - lij.re * lkj.im;
                }
                col[i - k] = mk<double>(a.re - sr, a.im - si);
            }
            const double piv = col[0].re;
            if (!(piv > 0.0)) {
                ok = false;
                break;
            }
            const double d = std::sqrt(piv);
            Lf[(size_t)k * n + k] = mk<double>(d, 0.0);
            for (int i = k + 1; i < n; i++) {
                const cplx<double> a = O[(size_t)k * n + i];
                if (std::hypot(a.re, a.im) > cut) Lf[(size_t)k * n + i] = mk<double>(col[i - k].re / d, col[i - k].im / d);
            }
        }
        if (ok) break;
        shift = shift == 0.0 ? 1e-3 : 2 * shift;
        if (shift > 1.0) {
            set_error("preconditioner: IC(0) pivots stay non-positive");
            return QEDHMC_EUNSUPPORTED;
        }
    }
    // truncation of the taps: kThresh, or QEDHMC_PC_THRESH; tau reach:
    // kCapTau, or QEDHMC_PC_CAP (1 .. kCapMax) (both read when the
    // preconditioner is built; tuning knobs)
    double thresh = kThresh;
    if (const char* et = std::getenv("QEDHMC_PC_THRESH"); et && *et) thresh = std::atof(et);
    h->pc_cap = kCapTau;
    if (const char* ec = std::getenv("QEDHMC_PC_CAP"); ec && std::atoi(ec) > 0)
        h->pc_cap = std::min(kCapMax, std::atoi(ec));
    // rows of G = L^{-1}: x^T L = e_n0^T  <=>  L^T x = e_n0 (back substitution)
    const int tau0 = kBuildNt / 2 + 4, y0 = L0 / 2;
    for (int par = 0; par < 2; par++) {
        const int x0 = L0 / 2 + par, n0 = tau0 * Vs + y0 * L0 + x0;
        std::vector<cplx<double>> xr(n, mk<double>(0.0, 0.0));
        for (int i = n0; i >= 0; i--) {
            double re = (i == n0) ? 1.0 : 0.0, im = 0.0;
            for (int j = i + 1; j <= n0; j++) {
                const cplx<double> lji = Lf[(size_t)i * n + j], xj = xr[j];
                re -= lji.re * xj.re - lji.im * xj.im;
                im -= lji.re * xj.im + lji.im * xj.re;
            }
            const cplx<double> lii = Lf[(size_t)i * n + i];  // real positive
            xr[i] = mk<double>(re / lii.re, im / lii.re);
        }
        auto& taps = h->pc_taps[par];
        taps.clear();
        for (int m = 0; m <= n0; m++) {
            const double mag = std::hypot(xr[m].re, xr[m].im);
            if (!(mag >= thresh)) continue;
            const int tm = m / Vs, sm = m % Vs;
            const int dt = tau0 - tm;
            if (dt < 0 || dt > h->pc_cap) continue;
            const int dx = ((sm % L0 - x0 + L0 / 2) % L0 + L0) % L0 - L0 / 2;
            const int dy = ((sm / L0 - y0 + L0 / 2) % L0 + L0) % L0 - L0 / 2;
            taps.push_back({dt, dx, dy, xr[m].re, xr[m].im});
        }
        std::sort(taps.begin(), taps.end(), [](const HostTap& a, const HostTap& b) {
            if (a.dt != b.dt) return a.dt < b.dt;
            if (a.dy != b.dy) return a.dy < b.dy;
            return a.dx < b.dx;
        });
    }
    h->pc_shift = shift;
    // The two passes as gathers out(tau, y, x) = sum h in(tau + a, y + b, x + c)
    // over the tap list of the output's x parity (sign -1 where tau + a leaves
    // [0, Nt)): G takes (a, b, c, h) = (-dt, dy, dx, g) from its own parity's
    // taps; G^dag takes (dt, -dy, -dx, conj g) from every tap whose source
    // x - dx has the parity of the list it came from.
    std::vector<HostTap> pass[2][2];
    for (int par = 0; par < 2; par++) {
        for (const auto& t : h->pc_taps[par]) pass[0][par].push_back({-t.dt, t.dx, t.dy, t.gre, t.gim});
        for (int pp = 0; pp < 2; pp++)
            for (const auto& t : h->pc_taps[pp])
                if ((((par - t.dx) % 2) + 2) % 2 == pp) pass[1][par].push_back({t.dt, -t.dx, -t.dy, t.gre, -t.gim});
    }
    std::vector<PTap<double>> t64;
    std::vector<PTap<float>> t32;
    for (int ps = 0; ps < 2; ps++) {
        PcPass& g = h->pc_pass[ps];
        g.amin = g.bmin = g.cmin = 1 << 20;
        g.amax = g.bmax = g.cmax = -(1 << 20);
        for (int par = 0; par < 2; par++)
            for (const auto& t : pass[ps][par]) {
                g.amin = std::min(g.amin, t.dt);
                g.amax = std::max(g.amax, t.dt);
                g.bmin = std::min(g.bmin, t.dy);
                g.bmax = std::max(g.bmax, t.dy);
                g.cmin = std::min(g.cmin, t.dx);
                g.cmax = std::max(g.cmax, t.dx);
            }
        if (g.amin > g.amax) g.amin = g.amax = g.bmin = g.bmax = g.cmin = g.cmax = 0;
        const int half = (h->lat.L + g.cmax - g.cmin + 1) / 2;
        for (int par = 0; par < 2; par++) {
            auto& lst = pass[ps][par];
            std::stable_sort(lst.begin(), lst.end(), [](const HostTap& a, const HostTap& b) { return a.dt < b.dt; });
            g.first[par] = (int)t64.size();
            g.count[par] = (int)lst.size();
            // start of each tau-offset group (a = amin + k) within the list
            for (int k = 0; k <= kPcSlots; k++) {
                int n = 0;
                for (const auto& t : lst)
                    if (t.dt - g.amin < k) n++;
                g.gstart[par][k] = n;
            }
            for (const auto& t : lst) {
                const int aidx = t.dt - g.amin, q = par + t.dx - g.cmin;
                const int off = t.dy * half + (q >> 1), plane = q & 1;
                t64.push_back({aidx, off, plane, 0, mk<double>(t.gre, t.gim)});
                t32.push_back({aidx, off, plane, 0, mk<float>((float)t.gre, (float)t.gim)});
            }
        }
    }
    // the same passes grouped by spatial offset for the tau-rolling kernel
    // (a pass reaching exactly kRollNS tau offsets; otherwise rcount stays 0)
    std::vector<RTap<double>> r64;
    std::vector<RTap<float>> r32;
    for (int ps = 0; ps < 2; ps++) {
        PcPass& g = h->pc_pass[ps];
        const int half = (h->lat.L + g.cmax - g.cmin + 1) / 2;
        for (int par = 0; par < 2; par++) {
            g.rfirst[par] = (int)r64.size();
            g.rcount[par] = 0;
            if (g.amax - g.amin + 1 != kRollNS) continue;
            std::vector<std::pair<int, int>> offs;  // (dy, dx) in first-seen order of the sorted list
            for (const auto& t : pass[ps][par])
                if (std::find(offs.begin(), offs.end(), std::make_pair(t.dy, t.dx)) == offs.end())
                    offs.push_back({t.dy, t.dx});
            std::sort(offs.begin(), offs.end());
            for (const auto& od : offs) {
                const int q = par + od.second - g.cmin;
                RTap<double> a{od.first * half + (q >> 1), q & 1, 0, 0, {}};
                for (int k = 0; k < kRollNS; k++) a.g[k] = mk<double>(0.0, 0.0);
                for (const auto& t : pass[ps][par])
                    if (t.dy == od.first && t.dx == od.second) a.g[t.dt - g.amin] = mk<double>(t.gre, t.gim);
                RTap<float> b{a.off, a.plane, 0, 0, {}};
                for (int k = 0; k < kRollNS; k++) b.g[k] = mk<float>((float)a.g[k].re, (float)a.g[k].im);
                r64.push_back(a);
                r32.push_back(b);
            }
            g.rcount[par] = (int)offs.size();
        }
    }
    const size_t nr = r64.size();
    QH_HIP(hipMalloc(&h->pc_roll64, std::max<size_t>(nr, 1) * sizeof(RTap<double>)));
    QH_HIP(hipMalloc(&h->pc_roll32, std::max<size_t>(nr, 1) * sizeof(RTap<float>)));
    if (nr) {
        QH_HIP(hipMemcpyAsync(h->pc_roll64, r64.data(), nr * sizeof(RTap<double>), hipMemcpyHostToDevice, h->stream));
        QH_HIP(hipMemcpyAsync(h->pc_roll32, r32.data(), nr * sizeof(RTap<float>), hipMemcpyHostToDevice, h->stream));
    }
    const size_t nt = t64.size();
    QH_HIP(hipMalloc(&h->pc_dev64, std::max<size_t>(nt, 1) * sizeof(PTap<double>)));
    QH_HIP(hipMalloc(&h->pc_dev32, std::max<size_t>(nt, 1) * sizeof(PTap<float>)));
    if (nt) {
        QH_HIP(hipMemcpyAsync(h->pc_dev64, t64.data(), nt * sizeof(PTap<double>), hipMemcpyHostToDevice, h->stream));
        QH_HIP(hipMemcpyAsync(h->pc_dev32, t32.data(), nt * sizeof(PTap<float>), hipMemcpyHostToDevice, h->stream));
    }
    QH_TRY(build_spectral(h, pass));
    QH_HIP(hipStreamSynchronize(h->stream));
    h->pc_ready = true;
    return QEDHMC_OK;
}

qedhmc_status ensure_paper_precond(qedhmc_ctx* h) {
    if (h->pc_ready) return QEDHMC_OK;
    return build_paper_precond(h);
}

// ---------------------------------------------------------------------------
// Stencil application, streamed along tau.  A workgroup owns one x parity of
// a band of TY rows (all x) and a run of Tc slices.  Its LDS holds a ring of
// nslot = amax - amin + 1 input slices over the band plus the rows and columns
// the taps reach (periodic in y and x, sign-flipped where the slice index
// leaves [0, Nt)), each slice stored as two planes of even and odd window
// columns, and a copy of the parity's taps.  Each step reads one new slice
// into the ring (prefetched into registers during the previous step); each
// output site is formed by a quad of lanes that split its taps (tap j to lane
// j mod 4 within each tau-offset group: an LDS read of the tap, an LDS read of
// the input at a fixed offset and four FMAs) and add their partial sums by
// DPP.  Four lanes per site give the workgroup four times the wavefronts to
// hide LDS latency with.
// stop (nullable): a scalar slot's stop flag; non-zero makes the launch a no-op.
// ---------------------------------------------------------------------------
struct PcGeo {
    int L, Nt, Vs;
    int TY, nband, Tc, nrun;
    int rows, cols, half, bmin, cmin, amin, nslot;
    int first[2], count[2];
    int gstart[2][kPcSlots + 1];  // per parity: start of each tau-offset group in the parity's list
};

// window elements per thread at most (the plan keeps rows x cols within
// kPcElems x threads)
static constexpr int kPcElems = 4;

template <typename R>
struct STap {
    R re, im;
    int toff;  // plane * plane size + off
    int pad;
};

__device__ __forceinline__ float dpp_f32_quad(float v, int sel) {
    const int i = __float_as_int(v);
    const int r = sel == 0 ? __builtin_amdgcn_update_dpp(0, i, 0xB1, 0xF, 0xF, false)
                           : __builtin_amdgcn_update_dpp(0, i, 0x4E, 0xF, 0xF, false);
    return __int_as_float(r);
}

template <typename R>
__device__ __forceinline__ R quad_sum(R v) {
    if constexpr (sizeof(R) == 8) {
        v += dpp_f64<0xB1, 0xF>(v);  // quad_perm [1,0,3,2]
        v += dpp_f64<0x4E, 0xF>(v);  // quad_perm [2,3,0,1]
    } else {
        v += dpp_f32_quad(v, 0);
        v += dpp_f32_quad(v, 1);
    }
    return v;
}

template <typename R>
__global__ __launch_bounds__(1024, 2) void k_pc_stream(PcGeo g, const PTap<R>* __restrict__ taps,
                                                       const cplx<R>* __restrict__ in, cplx<R>* __restrict__ out,
                                                       const double* __restrict__ stop) {
    if (stop && *stop != 0.0) return;
    extern __shared__ __align__(16) unsigned char smem[];
    cplx<R>* win = reinterpret_cast<cplx<R>*>(smem);
    const int plane = g.rows * g.half;  // one column-parity plane of a slice
    const int slice_elems = 2 * plane;
    STap<R>* st = reinterpret_cast<STap<R>*>(win + (size_t)g.nslot * slice_elems);
    const int nwork = g.nband * g.nrun * 2;
    const int per = (nwork + 7) >> 3;
    const int w = (blockIdx.x & 7) * per + (blockIdx.x >> 3);  // runs of one XCD are contiguous
    if (w >= nwork) return;
    const int par = w & 1, band = (w >> 1) % g.nband, run = (w >> 1) / g.nband;
    const int y0 = band * g.TY;
    const int tau0 = run * g.Tc, tau1 = min(g.Nt, tau0 + g.Tc);
    const int hx = g.L / 2;
    const int q = threadIdx.x & 3, o = threadIdx.x >> 2;
    const int iy = o / hx, jx = o - iy * hx;
    const bool act = iy < g.TY && y0 + iy < g.L;
    const int base = act ? (iy - g.bmin) * g.half + jx : -g.bmin * g.half;  // idle lanes read the first site's window
    const int ntap = g.count[par];
    {
        const PTap<R>* tp = taps + g.first[par];
        for (int j = threadIdx.x; j < ntap; j += blockDim.x) {
            const PTap<R> t = tp[j];
            st[j] = STap<R>{t.g.re, t.g.im, t.plane * plane + t.off, 0};
        }
    }
    // this thread's window elements (the same for every slice): source site
    // inside a slice and LDS position inside a slot (-1: none)
    int soff[kPcElems], doff[kPcElems];
    {
        const int total = g.rows * g.cols;
#pragma unroll
        for (int k = 0; k < kPcElems; k++) {
            const int e = (int)threadIdx.x + k * (int)blockDim.x;
            doff[k] = -1;
            soff[k] = 0;
            if (e < total) {
                const int r = e / g.cols, c = e - r * g.cols;
                const int yy = (y0 + g.bmin + r + 8 * g.L) % g.L, xx = (g.cmin + c + 8 * g.L) % g.L;
                soff[k] = yy * g.L + xx;
                doff[k] = (c & 1) * plane + r * g.half + (c >> 1);
            }
        }
    }
    auto fetch = [&](int s, cplx<R> (&v)[kPcElems]) {
        const cplx<R>* src = in + (size_t)(((s % g.Nt) + g.Nt) % g.Nt) * g.Vs;
#pragma unroll
        for (int k = 0; k < kPcElems; k++) v[k] = src[soff[k]];  // unused entries read site 0
    };
    auto store = [&](int s, const cplx<R> (&v)[kPcElems]) {
        const R sg = (s < 0 || s >= g.Nt) ? R(-1) : R(1);
        cplx<R>* dst = win + (size_t)(((s % g.nslot) + g.nslot) % g.nslot) * slice_elems;
#pragma unroll
        for (int k = 0; k < kPcElems; k++)
            if (doff[k] >= 0) dst[doff[k]] = mk<R>(sg * v[k].re, sg * v[k].im);
    };
    cplx<R> nxt[kPcElems];
    for (int s = tau0 + g.amin; s < tau0 + g.amin + g.nslot - 1; s++) {
        fetch(s, nxt);
        store(s, nxt);
    }
    fetch(tau0 + g.amin + g.nslot - 1, nxt);
    const int* gs = g.gstart[par];
    for (int tau = tau0; tau < tau1; tau++) {
        store(tau + g.amin + g.nslot - 1, nxt);
        __syncthreads();
        if (tau + 1 < tau1) fetch(tau + g.amin + g.nslot, nxt);  // in flight during the taps
        const int r0 = (((tau + g.amin) % g.nslot) + g.nslot) % g.nslot;
        R ar = 0, ai = 0;
        for (int gg = 0; gg < g.nslot; gg++) {
            int sl = r0 + gg;
            sl = sl >= g.nslot ? sl - g.nslot : sl;
            const cplx<R>* ws = win + (size_t)sl * slice_elems + base;
            const int j1 = gs[gg + 1];
#pragma unroll 4
            for (int j = gs[gg] + q; j < j1; j += 4) {
                const STap<R> t = st[j];
                const cplx<R> v = ws[t.toff];
                // four FMAs into the running sums (a product formed first and
                // then added would cost two more instructions per tap)
                ar = fma(t.re, v.re, ar);
                ar = fma(-t.im, v.im, ar);
                ai = fma(t.re, v.im, ai);
                ai = fma(t.im, v.re, ai);
            }
        }
        ar = quad_sum(ar);
        ai = quad_sum(ai);
        if (act && q == 3) out[(size_t)tau * g.Vs + (y0 + iy) * g.L + 2 * jx + par] = mk<R>(ar, ai);
        __syncthreads();  // the next step overwrites the oldest slot
    }
}

// ---------------------------------------------------------------------------
// The same stencil pass rolled along tau.  The taps of a spatial offset
// (b, c) at the kRollNS tau offsets a = amin .. amax act on one input value
// in(s, y + b, x + c); a lane reads that value once per input slice s and
// adds its kRollNS products into the running sums of the outputs s - a, held
// in registers (output tau is complete once slice tau + amax has been read).
// A workgroup owns one x parity of a band of TY rows and a run of Tc output
// slices, reads Tc + kRollNS - 1 input slices one at a time into a double
// buffer in LDS (window of the band plus the rows and columns the taps reach,
// even and odd columns as two planes, sign-flipped where the slice index
// leaves [0, Nt)), and gives each output site Q lanes in Q different
// wavefronts, each taking every Q-th spatial offset: the offset index is
// uniform across a wavefront, so the taps come through scalar loads.  The
// Q partial sums of a completed output meet in LDS.  One barrier per slice.
// ---------------------------------------------------------------------------
struct PcRollGeo {
    int L, Nt, Vs;
    int TY, nband, Tc, nrun;
    int rows, cols, half, bmin, cmin, amin;
    int S, Q;  // lanes per copy of the band's sites (a multiple of 64) and copies
    int first[2], count[2];
};

static constexpr int kRollElems = 4;  // window elements per thread at most
// per application of G^dag G, FP32: L = 24 per-tap 53 us / rolled 63 us;
// L = 48 242 / 200 us; L = 66 603 / 450 us
static constexpr int kRollFromL = 40;

template <typename R>
__global__ __launch_bounds__(1024) void k_pc_roll(PcRollGeo g, const RTap<R>* __restrict__ taps,
                                                  const cplx<R>* __restrict__ in, cplx<R>* __restrict__ out,
                                                  const double* __restrict__ stop) {
    if (stop && *stop != 0.0) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int plane = g.rows * g.half, slice_elems = 2 * plane;
    cplx<R>* win = reinterpret_cast<cplx<R>*>(smem);  // [2][slice_elems]
    cplx<R>* red = win + 2 * slice_elems;             // [2][Q][S] partial sums of completed outputs
    const int nwork = g.nband * g.nrun * 2;
    const int per = (nwork + 7) >> 3;
    const int w = (blockIdx.x & 7) * per + (blockIdx.x >> 3);  // runs of one XCD are contiguous
    if (w >= nwork) return;
    const int par = w & 1, band = (w >> 1) % g.nband, run = (w >> 1) / g.nband;
    const int y0 = band * g.TY;
    const int tau0 = run * g.Tc, tau1 = min(g.Nt, tau0 + g.Tc);
    const int hx = g.L / 2;
    const int o = (int)threadIdx.x % g.S;
    const int q = __builtin_amdgcn_readfirstlane((int)threadIdx.x / g.S);
    const int iy = o / hx, jx = o - iy * hx;
    const bool act = iy < g.TY && y0 + iy < g.L;
    const int base = act ? (iy - g.bmin) * g.half + jx : 0;  // idle lanes read a valid element
    int soff[kRollElems], doff[kRollElems];
    {
        const int total = g.rows * g.cols;
#pragma unroll
        for (int k = 0; k < kRollElems; k++) {
            const int e = (int)threadIdx.x + k * (int)blockDim.x;
            doff[k] = -1;
            soff[k] = 0;
            if (e < total) {
                const int r = e / g.cols, c = e - r * g.cols;
                const int yy = (y0 + g.bmin + r + 8 * g.L) % g.L, xx = (g.cmin + c + 8 * g.L) % g.L;
                soff[k] = yy * g.L + xx;
                doff[k] = (c & 1) * plane + r * g.half + (c >> 1);
            }
        }
    }
    auto fetch = [&](int s, cplx<R> (&v)[kRollElems]) {
        const cplx<R>* src = in + (size_t)(((s % g.Nt) + g.Nt) % g.Nt) * g.Vs;
#pragma unroll
        for (int k = 0; k < kRollElems; k++) v[k] = src[soff[k]];  // unused entries read site 0
    };
    auto store = [&](int buf, int s, const cplx<R> (&v)[kRollElems]) {
        const R sg = (s < 0 || s >= g.Nt) ? R(-1) : R(1);
        cplx<R>* dst = win + (size_t)buf * slice_elems;
#pragma unroll
        for (int k = 0; k < kRollElems; k++)
            if (doff[k] >= 0) dst[doff[k]] = mk<R>(sg * v[k].re, sg * v[k].im);
    };
    const RTap<R>* tp = taps + g.first[par];
    const int ntap = g.count[par];
    const int nsteps = (tau1 - tau0) + kRollNS - 1;
    const int s0 = tau0 + g.amin;
    cplx<R> acc[kRollNS];
#pragma unroll
    for (int k = 0; k < kRollNS; k++) acc[k] = mk<R>(R(0), R(0));
    cplx<R> nxt[kRollElems];
    fetch(s0, nxt);
    store(0, s0, nxt);
    __syncthreads();
    for (int j0 = 0; j0 < nsteps; j0 += kRollNS) {
#pragma unroll
        for (int u = 0; u < kRollNS; u++) {
            const int j = j0 + u;
            if (j >= nsteps) break;
            if (j + 1 < nsteps) fetch(s0 + j + 1, nxt);  // in flight during the taps
            const cplx<R>* ws = win + (size_t)(j & 1) * slice_elems + base;
            // wavefronts past the Q copies only help load the window
            for (int k = q; k < (q < g.Q ? ntap : 0); k += g.Q) {
                const RTap<R> t = tp[k];
                const cplx<R> v = ws[t.plane * plane + t.off];
                // input slice s0 + j feeds output tau0 + j - kk through the
                // tap of tau offset amin + kk (products for outputs outside
                // the run land in slots that are cleared unwritten: skipping
                // them measured slower)
#pragma unroll
                for (int kk = 0; kk < kRollNS; kk++) {
                    cplx<R>& A = acc[(u - kk + kRollNS) % kRollNS];
                    A.re = fma(t.g[kk].re, v.re, A.re);
                    A.re = fma(-t.g[kk].im, v.im, A.re);
                    A.im = fma(t.g[kk].re, v.im, A.im);
                    A.im = fma(t.g[kk].im, v.re, A.im);
                }
            }
            // output tau0 + j - (kRollNS - 1) is complete in slot (u + 1) mod kRollNS
            const int cs = (u + 1) % kRollNS;
            cplx<R>* rb = red + (size_t)(j & 1) * g.Q * g.S;
            if (g.Q > 1 && q < g.Q) rb[q * g.S + o] = acc[cs];
            if (j + 1 < nsteps) store((j + 1) & 1, s0 + j + 1, nxt);
            __syncthreads();
            const int tau = tau0 + j - (kRollNS - 1);
            if (q == 0 && act && tau >= tau0) {
                cplx<R> sum = acc[cs];
                if (g.Q > 1) {
                    sum = rb[o];
                    for (int k = 1; k < g.Q; k++) {
                        sum.re += rb[k * g.S + o].re;
                        sum.im += rb[k * g.S + o].im;
                    }
                }
                out[(size_t)tau * g.Vs + (y0 + iy) * g.L + 2 * jx + par] = sum;
            }
            acc[cs] = mk<R>(R(0), R(0));
        }
    }
}

template <typename R>
static const RTap<R>* rtaps_for(qedhmc_ctx* h) {
    if constexpr (sizeof(R) == 8)
        return (const RTap<double>*)h->pc_roll64;
    else
        return (const RTap<float>*)h->pc_roll32;
}

// Plan: a band of TY rows whose TY * L/2 output sites fill whole wavefronts
// best (at most 256 lanes per copy), Q = 2 copies for 256-lane bands and 4
// below, runs of 12 slices (each run reads kRollNS - 1 slices more than it
// writes).  QEDHMC_PC_TY, QEDHMC_PC_TC and QEDHMC_PC_Q (read per call)
// override the plan.
template <typename R>
static qedhmc_status launch_pc_roll(qedhmc_ctx* h, int ps, const cplx<R>* in, cplx<R>* out, const double* stop) {
    const PcPass& pp = h->pc_pass[ps];
    const Lat& lt = h->lat;
    PcRollGeo g{};
    g.L = lt.L;
    g.Nt = lt.Nt;
    g.Vs = lt.Vs;
    g.bmin = pp.bmin;
    g.cmin = pp.cmin;
    g.amin = pp.amin;
    g.cols = lt.L + pp.cmax - pp.cmin;
    g.half = (g.cols + 1) / 2;
    for (int par = 0; par < 2; par++) {
        g.first[par] = pp.rfirst[par];
        g.count[par] = pp.rcount[par];
    }
    const int hx = lt.L / 2;
    auto pad64 = [](int n) { return ((n + 63) / 64) * 64; };
    int TY = 1;
    double best = -1.0;
    for (int ty = 1; ty <= lt.L && pad64(ty * hx) <= 256; ty++) {
        const double eff = (double)(ty * hx) / pad64(ty * hx);
        if (eff >= best - 1e-9) {
            best = eff;
            TY = ty;
        }
    }
    const char* ety = std::getenv("QEDHMC_PC_TY");
    const char* etc = std::getenv("QEDHMC_PC_TC");
    const char* eq = std::getenv("QEDHMC_PC_Q");
    if (ety && std::atoi(ety) > 0) TY = std::min(lt.L, std::atoi(ety));
    g.nband = (lt.L + TY - 1) / TY;
    g.TY = (lt.L + g.nband - 1) / g.nband;
    g.rows = g.TY + pp.bmax - pp.bmin;
    g.S = pad64(g.TY * hx);
    g.Q = g.S >= 256 ? 2 : 4;  // measured best at L = 48 (4) and 66 (2)
    if (eq && std::atoi(eq) > 0) g.Q = std::atoi(eq);
    while (g.Q > 1 && g.Q * g.S > 1024) g.Q--;
    if (g.S > 1024) {
        set_error("paper preconditioner: a band row exceeds one workgroup at this L");
        return QEDHMC_EUNSUPPORTED;
    }
    // every window element of a slice has a thread (kRollElems each at most):
    // whole wavefronts past the Q copies only load
    const int need = ((g.rows * g.cols + kRollElems - 1) / kRollElems + 63) / 64 * 64;
    const int threads = std::max(g.Q * g.S, need);
    if (threads > 1024) {
        set_error("paper preconditioner: the stencil window exceeds the rolling kernel's workgroup");
        return QEDHMC_EUNSUPPORTED;
    }
    g.Tc = 12;  // a sweep of 6, 12, 24 at L = 48 and 66 put 12 first or within 1 %
    if (etc && std::atoi(etc) > 0) g.Tc = std::atoi(etc);
    g.Tc = std::min(g.Tc, lt.Nt);
    g.nrun = (lt.Nt + g.Tc - 1) / g.Tc;
    const size_t lds = (size_t)2 * 2 * g.rows * g.half * sizeof(cplx<R>) +
                       (g.Q > 1 ? (size_t)2 * g.Q * g.S * sizeof(cplx<R>) : 0);
    if (lds > h->max_lds) {
        set_error("paper preconditioner: the rolling kernel's window exceeds the LDS");
        return QEDHMC_EUNSUPPORTED;
    }
    if (lds > 65536) QH_TRY(allow_lds((const void*)k_pc_roll<R>, h->max_lds));
    const int nwork = g.nband * g.nrun * 2;
    hipLaunchKernelGGL(k_pc_roll<R>, dim3(8 * ((nwork + 7) / 8)), dim3(threads), lds, h->stream, g, rtaps_for<R>(h),
                       in, out, stop);
    QH_HIP(hipGetLastError());
    return QEDHMC_OK;
}

template <typename R>
static const PTap<R>* taps_for(qedhmc_ctx* h) {
    if constexpr (sizeof(R) == 8)
        return (const PTap<double>*)h->pc_dev64;
    else
        return (const PTap<float>*)h->pc_dev32;
}

// Band height TY: four lanes per output site, about 448 lanes, and an LDS
// window within 64 KB (FP32) or 128 KB (FP64); runs of 2 .. 16 slices aiming
// at about 4096 workgroups.
template <typename R>
static qedhmc_status launch_pc(qedhmc_ctx* h, int ps, const cplx<R>* in, cplx<R>* out, const double* stop) {
    const PcPass& pp = h->pc_pass[ps];
    // the tau-rolling kernel from L = kRollFromL on (below it the per-tap
    // kernel measured as fast or faster: too few rolled work items to fill
    // the device); QEDHMC_PC_KERNEL=roll|stream (read per call) forces one
    const char* ek = std::getenv("QEDHMC_PC_KERNEL");
    const bool forced = ek && (std::strcmp(ek, "roll") == 0 || std::strcmp(ek, "stream") == 0);
    const bool roll = forced ? std::strcmp(ek, "roll") == 0 : h->lat.L >= kRollFromL;
    if (pp.rcount[0] > 0 && pp.rcount[1] > 0 && roll) return launch_pc_roll<R>(h, ps, in, out, stop);
    const Lat& lt = h->lat;
    PcGeo g{};
    g.L = lt.L;
    g.Nt = lt.Nt;
    g.Vs = lt.Vs;
    g.bmin = pp.bmin;
    g.cmin = pp.cmin;
    g.amin = pp.amin;
    g.nslot = pp.amax - pp.amin + 1;
    if (g.nslot > kPcSlots) {
        set_error("paper preconditioner: stencil reaches too many slices");
        return QEDHMC_EUNSUPPORTED;
    }
    g.cols = lt.L + pp.cmax - pp.cmin;
    g.half = (g.cols + 1) / 2;
    for (int par = 0; par < 2; par++) {
        g.first[par] = pp.first[par];
        g.count[par] = pp.count[par];
        for (int k = 0; k <= kPcSlots; k++) g.gstart[par][k] = pp.gstart[par][std::min(k, g.nslot)];
    }
    const int hx = lt.L / 2;
    const int maxtap = std::max(pp.count[0], pp.count[1]);
    const size_t tap_bytes = (size_t)maxtap * sizeof(STap<R>);
    const size_t budget = std::min<size_t>(sizeof(R) == 8 ? 131072 : 65536, h->max_lds);
    auto lds_of = [&](int ty) {
        return (size_t)g.nslot * (ty + pp.bmax - pp.bmin) * 2 * g.half * sizeof(cplx<R>) + tap_bytes;
    };
    // tuning overrides, read per call: QEDHMC_PC_TY (rows per band, at most
    // the plan's) and QEDHMC_PC_TC (slices per run); 0 or unset: automatic
    const char* ety = std::getenv("QEDHMC_PC_TY");
    const char* etc = std::getenv("QEDHMC_PC_TC");
    // about 448 lanes per workgroup: several small workgroups per compute
    // unit beat one large one (less barrier coupling; measured at L = 24,
    // 48, 66)
    int TY = std::max(1, std::min(lt.L, 448 / (4 * hx)));
    while (TY > 1 && lds_of(TY) > budget) TY--;
    if (ety && std::atoi(ety) > 0) TY = std::min(TY, std::atoi(ety));
    if (4 * hx > 1024 || lds_of(TY) > h->max_lds) {
        set_error("paper preconditioner: the stencil window exceeds one workgroup at this L");
        return QEDHMC_EUNSUPPORTED;
    }
    g.nband = (lt.L + TY - 1) / TY;
    g.TY = (lt.L + g.nband - 1) / g.nband;
    g.rows = g.TY + pp.bmax - pp.bmin;
    g.Tc = std::max(2, std::min(16, lt.Nt * g.nband * 2 / 4096));
    if (etc && std::atoi(etc) > 0) g.Tc = std::atoi(etc);
    g.Tc = std::min(g.Tc, lt.Nt);
    g.nrun = (lt.Nt + g.Tc - 1) / g.Tc;
    const size_t lds = lds_of(g.TY);
    int threads = ((4 * g.TY * hx + 63) / 64) * 64;
    // every window element of a slice has a thread (kPcElems each at most)
    const int need = (g.rows * g.cols + kPcElems - 1) / kPcElems;
    threads = std::max(threads, ((need + 63) / 64) * 64);
    if (threads > 1024) {
        set_error("paper preconditioner: stencil window too large for one workgroup at this L");
        return QEDHMC_EUNSUPPORTED;
    }
    const int nwork = g.nband * g.nrun * 2;
    if (lds > 65536) QH_TRY(allow_lds((const void*)k_pc_stream<R>, h->max_lds));
    hipLaunchKernelGGL(k_pc_stream<R>, dim3(8 * ((nwork + 7) / 8)), dim3(threads), lds, h->stream, g, taps_for<R>(h),
                       in, out, stop);
    QH_HIP(hipGetLastError());
    return QEDHMC_OK;
}

// ---------------------------------------------------------------------------
// Spectral application (the tables of build_spectral; spectral.h).  Momentum
// vectors use the memory of a site vector, [tau][ny][nx][parity].
// ---------------------------------------------------------------------------
// Workgroup size cap of the spectral kernels: FP64 takes at most 512
// threads (at 1024 its registers spill)
template <typename R>
constexpr int spec_max_threads() {
    return sizeof(R) == 8 ? 512 : 1024;
}

// Site vector -> momentum planes, a slice per workgroup.  With the transform
// on the matrix cores (spectral.h) against direct sums through LDS, which were
// bound by LDS reads: L = 24 5.3 -> 4.6 us, L = 66, N_tau = 660 83 -> 27 us
// (46 MB, 1.7 TB/s; the inverse the same).  What is left at L = 66 is the
// chain load, y products, barrier, x products, store of each workgroup, with
// two workgroups in a compute unit, and 7 us of FP32 products.
template <typename R, int NY, int NX, bool TL>
__global__ __launch_bounds__(spec_max_threads<R>()) void k_pcs_fwd(PcSpecGeo g, const R* __restrict__ tab,
                                                                  const cplx<R>* __restrict__ in,
                                                                  cplx<R>* __restrict__ out,
                                                                  const double* __restrict__ stop) {
    if (stop && *stop != 0.0) return;
    extern __shared__ __align__(32) unsigned char smem[];
    R* V = reinterpret_cast<R*>(smem);
    const int tau = slice_of_block(blockIdx.x, g.Nt);
    if (tau < 0) return;
    const R* tb = sp_tables<R, TL>(tab, V + g.L * g.ld, g);
    const cplx<R>* src = in + (size_t)tau * g.Vs;
    for (int e = threadIdx.x; e < g.Vs; e += blockDim.x) {
        const int y = e / g.L;
        *reinterpret_cast<cplx<R>*>(V + y * g.ld + 2 * (e - y * g.L)) = src[e];
    }
    sp_forward<R, NY, NX>(V, g, tb, out + (size_t)tau * g.Vs);
}

// Momentum planes -> site vector, a slice per workgroup.
template <typename R, int NY, int NX, bool TL>
__global__ __launch_bounds__(spec_max_threads<R>()) void k_pcs_inv(PcSpecGeo g, const R* __restrict__ tab,
                                                                  const cplx<R>* __restrict__ in,
                                                                  cplx<R>* __restrict__ out,
                                                                  const double* __restrict__ stop) {
    if (stop && *stop != 0.0) return;
    extern __shared__ __align__(32) unsigned char smem[];
    R* V = reinterpret_cast<R*>(smem);
    const int tau = slice_of_block(blockIdx.x, g.Nt);
    if (tau < 0) return;
    const R* tb = sp_tables<R, TL>(tab, V + g.L * g.ld, g);
    const cpair<R>* src = reinterpret_cast<const cpair<R>*>(in + (size_t)tau * g.Vs);
    for (int k = threadIdx.x; k < g.nk; k += blockDim.x) {
        const int y = k / g.Lh;
        *reinterpret_cast<cpair<R>*>(V + y * g.ld + 4 * (k - y * g.Lh)) = src[k];
    }
    sp_inverse<R, NY, NX>(V, g, tb, out + (size_t)tau * g.Vs);
}

// slice tau + a (|a| < N_tau) in [0, N_tau) and its sign (-1 where it wraps)
template <typename R>
__device__ __forceinline__ int sp_slice(int s, int Nt, R& sign) {
    sign = (s < 0 || s >= Nt) ? R(-1) : R(1);
    return s < 0 ? s + Nt : (s >= Nt ? s - Nt : s);
}

// z^(k, tau) = sum_a sign H(k, a) v^(k, tau + a): a thread per (momentum, run
// of T slices) holds the T + 2 kSpTau input slices it needs in registers and
// reads each block of H once for the run.  Bound by the FMAs (400 per
// momentum and slice: 15 us of the 28 at L = 66, N_tau = 660) with two
// wavefronts a SIMD.
// Workgroup i runs on XCD i mod 8: every XCD takes an eighth of the momenta
// for all slices, so the runs' windows, which overlap in 24 slices, come from
// its L2: P at L = 66 81.2 -> 77.7 us (FP32), 156 -> 145 us (FP64, N_tau = 640).
__host__ __device__ __forceinline__ int tsum_first(int nk, int xcd) { return (int)((long)nk * xcd / 8); }

template <typename R, int T>
__global__ __launch_bounds__(256) void k_pcs_tsum(PcSpecGeo g, const cpair<R>* __restrict__ H,
                                                  const cplx<R>* __restrict__ in, cplx<R>* __restrict__ out,
                                                  const double* __restrict__ stop) {
    if (stop && *stop != 0.0) return;
    const int nk = g.nk, nrun = (g.Nt + T - 1) / T;
    const int k0 = tsum_first(nk, blockIdx.x & 7), wk = tsum_first(nk, (blockIdx.x & 7) + 1) - k0;
    const int i = (blockIdx.x >> 3) * blockDim.x + threadIdx.x;
    if (i >= wk * nrun) return;
    const int k = k0 + i % wk, tau0 = (i / wk) * T;
    constexpr int NW = T + 2 * kSpTau;
    cpair<R> v[NW];
    // window slices past the last one needed read the run's first slice and
    // are not used: every load in flight together
#pragma unroll
    for (int j = 0; j < NW; j++) {
        const int a = j - kSpTau;
        R sg = R(1);
        const bool on = a >= -g.reach && a < T + g.reach && tau0 + a < g.Nt + g.reach;
        const int s = on ? sp_slice<R>(tau0 + a, g.Nt, sg) : tau0;
        v[j] = reinterpret_cast<const cpair<R>*>(in + (size_t)s * g.Vs)[k];
        v[j] = sp_signed(sg, v[j]);
    }
    // the far offsets first: H falls off with |a|, so the running sums stay
    // small for most of their roundings
    cpair<R> z[T];
#pragma unroll
    for (int t = 0; t < T; t++) z[t] = {mk<R>(0, 0), mk<R>(0, 0)};
#pragma unroll
    for (int a = kSpTau; a >= 1; a--)
        if (a <= g.reach) {
            const cpair<R> h0 = H[(size_t)(2 * a) * nk + k], h1 = H[(size_t)(2 * a + 1) * nk + k];
#pragma unroll
            for (int t = 0; t < T; t++) {
                sp_up<R>(z[t], h0, h1, v[t + kSpTau + a]);
                sp_down<R>(z[t], h0, h1, v[t + kSpTau - a]);
            }
        }
    {
        const cpair<R> h0 = H[k], h1 = H[nk + k];
#pragma unroll
        for (int t = 0; t < T; t++) sp_up<R>(z[t], h0, h1, v[t + kSpTau]);
    }
#pragma unroll
    for (int t = 0; t < T; t++)
        if (tau0 + t < g.Nt) reinterpret_cast<cpair<R>*>(out + (size_t)(tau0 + t) * g.Vs)[k] = z[t];
}

// The tau sum and the inverse DFT in one launch, a slice per workgroup: both
// parities of a momentum in one thread (each input value and each block of H
// is read once per slice, H once for the two slices it serves), straight into
// the LDS image that is transformed back.  Used where a slice is small.  A
// workgroup per (slice, parity) reading all 25 blocks of H took 14.3 us per
// launch at L = 24, N_tau = 240 (110 MB of L2 reads); this one 9.2 us (56 MB),
// of which about 1.6 us are the launch.
template <typename R, int NY, int NX, bool TL>
__global__ __launch_bounds__(512) void k_pcs_tsum_inv(PcSpecGeo g, const cpair<R>* __restrict__ H,
                                                      const R* __restrict__ tab, const cplx<R>* __restrict__ in,
                                                      cplx<R>* __restrict__ out, const double* __restrict__ stop) {
    extern __shared__ __align__(32) unsigned char smem[];
    R* V = reinterpret_cast<R*>(smem);
    const int tau = slice_of_block(blockIdx.x, g.Nt), nk = g.nk;
    if (tau < 0) return;
    // (looked at once the first momentum's sum is formed: one round trip less)
    const double done = stop ? *stop : 0.0;
    const R* tb = sp_tables<R, TL>(tab, V + g.L * g.ld, g);
    constexpr int CH = sizeof(R) == 8 ? 3 : 6;  // offsets per load batch
    static_assert(kSpTau % CH == 0, "whole batches");
    for (int k = threadIdx.x; k < nk; k += blockDim.x) {
        cpair<R> z{mk<R>(0, 0), mk<R>(0, 0)};
        const cpair<R> hc0 = H[k], hc1 = H[nk + k];
        const cpair<R> vc = reinterpret_cast<const cpair<R>*>(in + (size_t)tau * g.Vs)[k];
        // the far offsets first (as k_pcs_tsum)
#pragma unroll
        for (int c = kSpTau - CH + 1; c >= 1; c -= CH) {
            cpair<R> h0[CH], h1[CH], vu[CH], vd[CH];
            R su[CH], sd[CH];
#pragma unroll
            for (int i = 0; i < CH; i++) {
                // offsets past the reach read valid entries with sign 0
                const int a = c + i <= g.reach ? c + i : 0;
                const int u = sp_slice<R>(tau + a, g.Nt, su[i]), d = sp_slice<R>(tau - a, g.Nt, sd[i]);
                if (a == 0) su[i] = sd[i] = R(0);
                h0[i] = H[(size_t)(2 * a) * nk + k];
                h1[i] = H[(size_t)(2 * a + 1) * nk + k];
                vu[i] = reinterpret_cast<const cpair<R>*>(in + (size_t)u * g.Vs)[k];
                vd[i] = reinterpret_cast<const cpair<R>*>(in + (size_t)d * g.Vs)[k];
            }
#pragma unroll
            for (int i = CH - 1; i >= 0; i--) {
                sp_up<R>(z, h0[i], h1[i], sp_signed(su[i], vu[i]));
                sp_down<R>(z, h0[i], h1[i], sp_signed(sd[i], vd[i]));
            }
        }
        sp_up<R>(z, hc0, hc1, vc);
        const int y = k / g.Lh;
        *reinterpret_cast<cpair<R>*>(V + y * g.ld + 4 * (k - y * g.Lh)) = z;
        if (done != 0.0) break;
    }
    if (done != 0.0) return;  // every thread, those without a momentum too
    sp_inverse<R, NY, NX>(V, g, tb, out + (size_t)tau * g.Vs);
}

template <typename R>
static PcSpecGeo spec_geo(const qedhmc_ctx* h) {
    const Lat& lt = h->lat;
    PcSpecGeo g{lt.L, lt.L / 2, lt.Nt, lt.Vs, lt.L * (lt.L / 2), -h->pc_spec_a0, sp_ld(lt.L), 0, 0};
    int ny, nx;
    spec_blocks(lt.L, ny, nx);
    g.ty = sp_table(g.L, ny);
    g.tx = sp_table(g.Lh, nx);
    return g;
}

// LDS of a transform: the slice image, and the tables as long as two
// workgroups then fit a compute unit (tl)
template <typename R>
static size_t spec_lds(const PcSpecGeo& g, bool& tl) {
    const size_t image = (size_t)g.L * g.ld * sizeof(R), tabs = (size_t)(g.ty + g.tx) * sizeof(R);
    tl = image + tabs <= 79 * 1024;
    return image + (tl ? tabs : 0);
}

// whether apply_P_t takes the spectral form: built (L even, N_tau above the
// tau reach of a pass, L * L/2 <= 8192), at most 4096 momenta per plane in
// FP64 (whose slice image then fits the LDS), and not overridden by
// QEDHMC_PC_KERNEL=roll|stream (read per call)
template <typename R>
static bool use_spectral(const qedhmc_ctx* h) {
    if (h->pc_spec_na <= 0) return false;
    const PcSpecGeo g = spec_geo<R>(h);
    bool tl;
    // (room for the update kernel's static reduction scratch)
    if (g.nk > kSpecMaxNK / (sizeof(R) == 8 ? 2 : 1) || spec_lds<R>(g, tl) + 2048 > h->max_lds) return false;
    const char* ek = std::getenv("QEDHMC_PC_KERNEL");
    return !ek || !*ek || std::strcmp(ek, "spectral") == 0;
}

// The tau sum is fused into the inverse DFT on small slices (each workgroup then
// reads H and 2 reach + 1 input slices through the L2, in FP64 three offsets at
// a time).  P fused / separate, N_tau = 10 L: FP32 L = 24 15.2 / 18.9 us, L = 48
// 38.1 / 38.9, L = 52 55.0 / 51.5, L = 58 66.5 / 53.8; FP64 L = 24 17.3 / 21.0,
// L = 26 26.8 / 22.8, L = 40 50.9 / 46.5, L = 58 132 / 96.5.  A solve to 1e-8:
// mixed L = 48, N_tau = 200 4.09 / 4.14 ms, L = 50 3.75 / 3.66, L = 58 4.79 /
// 4.53; FP64 L = 24 2.25 / 2.44, L = 26, N_tau = 260 2.13 / 1.88, L = 40, N_tau =
// 200 3.62 / 3.46.
// The number of slices counts too.  The fused form is a workgroup a slice.  FP64
// in one round of one per compute unit: L = 26, N_tau = 100 17.2 / 20.4 us, L = 32,
// N_tau = 64 and 240 19.8 / 21.7 and 22.7 / 25.1, L = 36, N_tau = 64 and 240 24.6 /
// 23.6 and 26.3 / 27.3, L = 40, N_tau = 240 31.3 / 29.4 (solves to 1e-10, L = 28,
// N_tau = 64 and 240 1.28 / 1.32 and 2.85 / 3.09 ms).  Where that round is at least
// two thirds full and the separate sum's workgroups (256 threads of more than 256
// registers, three slices a thread: one to a unit) need a second one: L = 44,
// N_tau = 240 33.7 / 37.9 us (6.18 / 6.63 ms a solve), L = 58 52.0 / 54.5 (10.7 /
// 10.8 ms); less full: L = 54, N_tau = 160 43.3 / 40.9.  FP32 with too few slices
// for the chip, which the separate sum fills: L = 48, N_tau = 13, 64, 100, 240 20.3 /
// 19.9, 21.0 / 20.8, 21.0 / 21.5, 22.4 / 24.2 us (mixed solves to 1e-8 1.76 / 1.58,
// 2.38 / 2.23, 2.91 / 2.80, 4.86 / 4.83 ms), L = 44, N_tau = 13 18.5 / 19.8 us;
// L = 58, N_tau = 240 28.5 / 30.3 us, but 5.13 / 4.98 ms.
// QEDHMC_PC_FUSE=0|1 (read per call) forces either form.
template <typename R>
static bool spec_fused(const qedhmc_ctx* h) {
    const char* ef = std::getenv("QEDHMC_PC_FUSE");
    if (ef && *ef) return std::atoi(ef) != 0;
    const int L = h->lat.L, Nt = h->lat.Nt, cu = h->n_cu;
    if (sizeof(R) == 4) return L <= 44 || (L <= 48 && Nt >= 100);
    if (L <= 24 || Nt > cu) return L <= 24;
    const bool full = 3 * Nt >= 2 * cu, second = L * (L / 2) * ((Nt + 2) / 3) > 256 * cu;
    return L <= 32 || (full && (L <= 36 || (second && L <= 58)));
}

template <typename R>
static const R* spec_tab(const qedhmc_ctx* h) {
    return (const R*)(sizeof(R) == 8 ? h->pc_tw64 : h->pc_tw32);
}

template <typename R>
static const cpair<R>* spec_H(const qedhmc_ctx* h) {
    return (const cpair<R>*)(sizeof(R) == 8 ? h->pc_spec64 : h->pc_spec32);
}

// f.operator()<NY, NX, TL>() of this lattice's transform
template <typename R, typename F>
static qedhmc_status with_spec(const PcSpecGeo& g, F&& f) {
    bool tl;
    (void)spec_lds<R>(g, tl);
    int ny, nx;
    spec_blocks(g.L, ny, nx);
    if (ny == 1) return f.template operator()<1, 1, true>();
    if (ny == 2) return tl ? f.template operator()<2, 1, true>() : f.template operator()<2, 1, false>();
    if (ny == 3) return tl ? f.template operator()<3, 2, true>() : f.template operator()<3, 2, false>();
    if constexpr (sizeof(R) == 4) return f.template operator()<5, 3, false>();
    set_error("paper preconditioner: the spectral plan does not fit one workgroup");
    return QEDHMC_EUNSUPPORTED;
}

// threads of a transform's workgroup: a wavefront per 16 columns of reals
// (the y axis' share of one turn), at least enough to load n elements a few
// at a time
static int spec_threads(const PcSpecGeo& g, int n, int most) {
    const int t = std::max(64 * ((2 * g.L + 15) / 16), (n + 63) / 64 * 64);
    return std::min(t, most);
}

// where the forward transform of r should land for launch_pcs_rest(m0, z,
// m1) of the solver's buffers: tmp when the rest is fused (it reads
// neighbouring slices and writes z), z otherwise
template <typename R>
static cplx<R>* spec_vhat(const qedhmc_ctx* h, cplx<R>* z, cplx<R>* tmp) {
    return spec_fused<R>(h) ? tmp : z;
}

template <typename R>
static qedhmc_status launch_pcs_fwd(qedhmc_ctx* h, const cplx<R>* r, cplx<R>* vhat, const double* stop) {
    const PcSpecGeo g = spec_geo<R>(h);
    return with_spec<R>(g, [&]<int NY, int NX, bool TL>() -> qedhmc_status {
        bool tl;
        const size_t lds = spec_lds<R>(g, tl);
        if (lds > 65536) QH_TRY(allow_lds((const void*)k_pcs_fwd<R, NY, NX, TL>, h->max_lds));
        hipLaunchKernelGGL((k_pcs_fwd<R, NY, NX, TL>), dim3(slice_grid(g.Nt)),
                           dim3(spec_threads(g, g.Vs / 2, spec_max_threads<R>())), lds, h->stream, g, spec_tab<R>(h),
                           r, vhat, stop);
        QH_HIP(hipGetLastError());
        return QEDHMC_OK;
    });
}

// z = P r from vhat = the forward transform of r; m1: momentum scratch (not
// used when the tau sum is fused), may be neither vhat nor z
template <typename R>
static qedhmc_status launch_pcs_rest(qedhmc_ctx* h, const cplx<R>* vhat, cplx<R>* z, cplx<R>* m1,
                                     const double* stop) {
    const PcSpecGeo g = spec_geo<R>(h);
    if (!spec_fused<R>(h)) {
        // Runs of 6 slices (a run reads 24 slices more than it writes) once
        // they give a thread to every lane of the chip, of 3 below.  P at
        // L = 66, N_tau = 660 with runs of 3 / 4 / 5 / 6: FP32 77.9 / 76.7 /
        // 81.7 / 77.3 us, FP64 (N_tau = 640) 153 / 147 / 149 / 145 us.
        auto runs = [&]<int T>() {
            const int nth = (g.nk + 7) / 8 * ((g.Nt + T - 1) / T);  // of an XCD, at most
            hipLaunchKernelGGL((k_pcs_tsum<R, T>), dim3(8 * ((nth + 255) / 256)), dim3(256), 0, h->stream, g,
                               spec_H<R>(h), vhat, m1, stop);
        };
        if ((size_t)g.nk * g.Nt >= ((size_t)1 << 20))
            runs.template operator()<6>();
        else
            runs.template operator()<3>();
        QH_HIP(hipGetLastError());
    }
    return with_spec<R>(g, [&]<int NY, int NX, bool TL>() -> qedhmc_status {
        bool tl;
        const size_t lds = spec_lds<R>(g, tl);
        if (!spec_fused<R>(h)) {
            if (lds > 65536) QH_TRY(allow_lds((const void*)k_pcs_inv<R, NY, NX, TL>, h->max_lds));
            hipLaunchKernelGGL((k_pcs_inv<R, NY, NX, TL>), dim3(slice_grid(g.Nt)),
                               dim3(spec_threads(g, g.nk / 2, spec_max_threads<R>())), lds, h->stream, g,
                               spec_tab<R>(h), (const cplx<R>*)m1, z, stop);
            QH_HIP(hipGetLastError());
            return QEDHMC_OK;
        }
        if (lds > 65536) QH_TRY(allow_lds((const void*)k_pcs_tsum_inv<R, NY, NX, TL>, h->max_lds));
        const dim3 grid(slice_grid(g.Nt)), blk(spec_threads(g, g.nk, 512));
        hipEvent_t e0, e1;
        if (prof_sample(h, sizeof(R) == 4 ? QEDHMC_K_PC_SPEC_FP32 : QEDHMC_K_PC_SPEC_FP64, e0, e1))
            hipExtLaunchKernelGGL((k_pcs_tsum_inv<R, NY, NX, TL>), grid, blk, lds, h->stream, e0, e1, 0, g,
                                  spec_H<R>(h), spec_tab<R>(h), vhat, z, stop);
        else
            hipLaunchKernelGGL((k_pcs_tsum_inv<R, NY, NX, TL>), grid, blk, lds, h->stream, g, spec_H<R>(h),
                               spec_tab<R>(h), vhat, z, stop);
        QH_HIP(hipGetLastError());
        return QEDHMC_OK;
    });
}

// z = G^dag (G r); m0 and m1: scratch vectors of the same precision for the
// momentum form (r, z and m0 distinct; m1 distinct from r and m0; where the tau
// sum is not fused m0 may be z, if z is aligned to 32 bytes)
template <typename R>
static qedhmc_status apply_P_t(qedhmc_ctx* h, const cplx<R>* r, cplx<R>* z, cplx<R>* m0, cplx<R>* m1,
                               const double* stop) {
    if (use_spectral<R>(h)) {
        QH_TRY(launch_pcs_fwd<R>(h, r, m0, stop));
        return launch_pcs_rest<R>(h, m0, z, m1, stop);
    }
    QH_TRY(launch_pc<R>(h, 0, r, m1, stop));
    return launch_pc<R>(h, 1, m1, z, stop);
}

template <typename A, typename B>
__global__ void k_pc_convert(const cplx<A>* __restrict__ a, cplx<B>* __restrict__ b, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        b[i] = mk<B>((B)a[i].re, (B)a[i].im);
}

// out = P in on FP64 vectors with the stencil passes in FP32 (the input
// rounded once, the result widened): for flexible CG, which tolerates an
// inexact preconditioner.  Scratch: ws[8] and ws[9].
qedhmc_status launch_apply_precond_fp32(qedhmc_ctx* h, const double* in, double* out) {
    QH_TRY(ensure_paper_precond(h));
    const size_t N = (size_t)h->lat.Nt * h->lat.Vs;
    cplx<float>* r32 = reinterpret_cast<cplx<float>*>(h->ws[9]);
    cplx<float>* t32 = r32 + N;
    cplx<float>* z32 = reinterpret_cast<cplx<float>*>(h->ws[8]);
    const int grid = (int)std::min<size_t>((N + 255) / 256, 4096);
    hipLaunchKernelGGL((k_pc_convert<double, float>), dim3(grid), dim3(256), 0, h->stream,
                       reinterpret_cast<const cplx<double>*>(in), r32, N);
    QH_HIP(hipGetLastError());
    QH_TRY(apply_P_t<float>(h, r32, z32, t32, z32 + N, nullptr));
    hipLaunchKernelGGL((k_pc_convert<float, double>), dim3(grid), dim3(256), 0, h->stream, (const cplx<float>*)z32,
                       reinterpret_cast<cplx<double>*>(out), N);
    QH_HIP(hipGetLastError());
    return QEDHMC_OK;
}

qedhmc_status launch_apply_precond(qedhmc_ctx* h, qedhmc_precision prec, const void* in, void* out,
                                   const double* stop) {
    QH_TRY(ensure_paper_precond(h));
    // the caller's vectors are read and written element by element; the
    // momentum form lives in the handle's scratch
    if (prec == QEDHMC_FP64)
        return apply_P_t<double>(h, (const cplx<double>*)in, (cplx<double>*)out, (cplx<double>*)h->ws[9],
                                 (cplx<double>*)h->ws[8], stop);
    return apply_P_t<float>(h, (const cplx<float>*)in, (cplx<float>*)out, (cplx<float>*)h->ws[9],
                            (cplx<float>*)h->ws[8], stop);
}

// ---------------------------------------------------------------------------
// PCG kernels
// ---------------------------------------------------------------------------
template <typename R>
struct PcgBufs {
    cplx<R>* r;
    cplx<R>* p;
    cplx<R>* s;
    cplx<R>* u;
    cplx<R>* w;
    cplx<R>* t;
    cplx<double>* x;
    const cplx<double>* rhs;
    const cplx<double>* Ox;
    double* part;   // [kNP6][nparts]: per slice, or per (slice, tile) for the tiled matvec
    double* partb;  // [Nt]: |rhs|^2 or the FP64 true |r|^2
    int nparts;
};

// r = rhs (kept in B.rhs), x = p = s = 0; partb = |rhs|^2 per slice
template <typename R>
__global__ __launch_bounds__(256) void k_pcg_start(Lat lt, PcgBufs<R> B, const cplx<double>* __restrict__ rhs,
                                                   cplx<double>* __restrict__ keep) {
    __shared__ double red[64];
    const size_t base = (size_t)blockIdx.x * lt.Vs;
    double b2 = 0.0;
    for (int k = threadIdx.x; k < lt.Vs; k += blockDim.x) {
        const cplx<double> b = rhs[base + k];
        keep[base + k] = b;
        B.r[base + k] = mk<R>((R)b.re, (R)b.im);
        B.p[base + k] = mk<R>(0, 0);
        B.s[base + k] = mk<R>(0, 0);
        B.x[base + k] = mk<double>(0, 0);
        b2 += b.re * b.re + b.im * b.im;
    }
    double v[1] = {b2};
    block_sumk<1>(v, red);
    if (threadIdx.x == 0) B.partb[blockIdx.x] = v[0];
}

// slot 0 from the |rhs|^2 partials
__global__ void k_pcg_init_slot(double* __restrict__ scal, const double* __restrict__ partb, int Nt, double tol2,
                                int maxit) {
    __shared__ double red[64];
    double v[1] = {0.0};
    for (int t = threadIdx.x; t < Nt; t += blockDim.x) v[0] += partb[t];
    block_sumk<1>(v, red);
    if (threadIdx.x < S_NSLOT) {
        double val = 0.0;
        if (threadIdx.x == S_FIRST || threadIdx.x == S_GPREV || threadIdx.x == S_APREV) val = 1.0;
        if (threadIdx.x == S_MAXIT) val = maxit;
        scal[threadIdx.x] = val;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        scal[S_B2] = v[0];
        scal[S_TARGET] = tol2 * v[0];
        scal[S_RRUPD] = v[0];
    }
}

// The start of a solve whose reliable updates run inside the triples: B.rhs =
// rhs, r = rhs - O x0 (FP64; x0 null: zero start, r = rhs), x = x0, p = s = 0,
// partb = |r|^2 and part[0] = |rhs|^2 per slice, and a slot that looks like one
// that has just paused (S_B2 < 0: |rhs|^2 to be taken from part; S_TARGET
// holds tol^2 until then).  Budget and tolerance live in the slot, so that the
// graphs of the triples serve every solve of a handle.
template <typename R, int MC, int NB, int BS>
__global__ __launch_bounds__(BS) void k_pcg_begin(Lat lt, PcgBufs<R> B, const cplx<double>* __restrict__ gauge64,
                                                  Coef<double> co64, const cplx<double>* __restrict__ rhs,
                                                  cplx<double>* __restrict__ keep, const cplx<double>* __restrict__ x0,
                                                  double* __restrict__ scal, double tol2, int maxit) {
    extern __shared__ __align__(16) unsigned char smem[];
    cplx<double>* buf2 = reinterpret_cast<cplx<double>*>(smem);
    double* red = reinterpret_cast<double*>(smem + (size_t)NB * 2 * lt.Vs * sizeof(cplx<double>));
    const int tau = slice_of_block(blockIdx.x, lt.Nt);
    if (blockIdx.x == 0 && threadIdx.x < S_NSLOT) {
        const int k = threadIdx.x;
        double val = 0.0;
        if (k == S_DONE) val = 2.0;
        if (k == S_B2 || k == S_NREL) val = -1.0;
        if (k == S_GPREV || k == S_APREV) val = 1.0;
        if (k == S_TARGET) val = tol2;
        if (k == S_MAXIT) val = maxit;
        scal[k] = val;
    }
    if (tau < 0) return;
    SliceCtx<MC> c;
    slice_ctx<MC>(lt, c, tau, whole_block_tile(smem, red));
    const size_t Vs = lt.Vs;
    Cells<double, MC> b, o;
    load_cells<double, MC>(b, rhs + c.tau * Vs, c.g);
    store_cells<double, MC>(b, keep + c.tau * Vs, c.g, c.own);
    double v[2] = {0.0, dot_cells<double, MC>(b, b, c.own)};
    Cells<double, MC> xt;
#pragma unroll
    for (int m = 0; m < MC; m++)
#pragma unroll
        for (int q = 0; q < 4; q++) xt.v[m][q] = o.v[m][q] = mk<double>(0, 0);
    if (x0) {
        cplx<double> hm[MC][12], ht[MC][12];
        hops_of<double, MC>(gauge64, lt, c.tm, c.idx, co64, hm);
        hops_of<double, MC>(gauge64, lt, c.tau, c.idx, co64, ht);
        Cells<double, MC> xm, xn;
        load_cells<double, MC>(xm, x0 + c.tm * Vs, c.g);
        load_cells<double, MC>(xt, x0 + c.tau * Vs, c.g);
        load_cells<double, MC>(xn, x0 + c.tp * Vs, c.g);
        mdagm_cells<double, MC, NB>(xm, xt, xn, hm, ht, c.g, c.own, co64, c.tau == 0 ? -1.0 : 1.0,
                                    c.tau == lt.Nt - 1 ? -1.0 : 1.0, buf2, lt.Vs, o);
    }
    Cells<R, MC> r, zero;
#pragma unroll
    for (int m = 0; m < MC; m++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const double re = b.v[m][q].re - o.v[m][q].re, im = b.v[m][q].im - o.v[m][q].im;
            if (c.own[m]) v[0] += re * re + im * im;
            r.v[m][q] = mk<R>((R)re, (R)im);
            zero.v[m][q] = mk<R>(0, 0);
        }
    store_cells<double, MC>(xt, B.x + c.tau * Vs, c.g, c.own);
    store_cells<R, MC>(r, B.r + c.tau * Vs, c.g, c.own);
    store_cells<R, MC>(zero, B.p + c.tau * Vs, c.g, c.own);
    store_cells<R, MC>(zero, B.s + c.tau * Vs, c.g, c.own);
    block_sumk<2>(v, red);
    if (threadIdx.x == 0) {
        B.partb[c.tau] = v[0];
        B.part[c.tau] = v[1];
    }
}

// A wavefront's share of the sum of n partials, the same wherever it is taken
__device__ __forceinline__ double lane_sum(const double* __restrict__ src, int n) {
    double s = 0.0;
    for (int i0 = threadIdx.x & 63; i0 < n; i0 += 4 * 64) {
        double a[4];
#pragma unroll
        for (int u = 0; u < 4; u++) a[u] = i0 + 64 * u < n ? src[i0 + 64 * u] : 0.0;
#pragma unroll
        for (int u = 0; u < 4; u++) s += a[u];
    }
    return s;
}

// One slice per block (dealt to the XCDs as slice_of_block deals them):
// scalars from the partials, then the elementwise update.
// DFT (NY > 0): the block then also transforms the new r of its slice (both
// parity planes, through LDS) into vhat, the first step of the spectral P r;
// vhat may be u itself, whose slice only this block reads.
// updates: the reliable updates run inside the triples; a slot that asks for
// one is decided here (converged, failed with S_WHY, or resume), and a solve
// that resumes transforms the replaced r.
// Latency: every load (the partials first: each wavefront adds one of the
// sums, then the vectors of the thread's first kUpdPre sites) is requested
// before the slot is looked at, one round trip to memory for all of them, so
// that a launch of a finished solve costs as much as one that works; those are
// few where the updates run inside the triples.  8.5 -> 6.6 us at L = 24, N_tau
// = 240 (FP32).
// Large lattices: bound by the bytes, 88 a site on average in FP32 with the
// transform, 80 without (x, FP64, is read and written at every second
// iteration).  65 us at 104 a site at L = 66, N_tau = 660 (4.6 TB/s), 58 us now
// (4.4 TB/s); the sites past a thread's first kUpdPre
// are also requested kUpdPre at a time, and the launch without a transform has
// a thread for every four sites: CG at L = 80, N_tau = 200 43.9 -> 38.9 ms.
static constexpr int kUpdPre = 4;

template <typename R, int NY, int NX, bool TL>
__global__ __launch_bounds__(spec_max_threads<R>()) void k_pcg_upd(Lat lt, PcgBufs<R> B, double* __restrict__ scal, int kpar,
                                                  int mixed, int updates, PcSpecGeo sg,
                                                  const R* __restrict__ tab, cplx<R>* __restrict__ vhat) {
    constexpr bool DFT = NY > 0;
    __shared__ double red[8];
    extern __shared__ __align__(32) unsigned char smem[];
    R* V = reinterpret_cast<R*>(smem);  // the new r, as the transform reads it
    const double* sin_ = scal + S_NSLOT * kpar;
    double* sout = scal + S_NSLOT * (kpar ^ 1);
    const int tau = slice_of_block(blockIdx.x, lt.Nt);
    const size_t base = (size_t)(tau < 0 ? 0 : tau) * lt.Vs;
    if (!updates && sin_[S_DONE] != 0.0) {
        if (blockIdx.x == 0 && threadIdx.x < S_NSLOT) sout[threadIdx.x] = sin_[threadIdx.x];
        return;
    }
    double sl[S_NSLOT];
#pragma unroll
    for (int k = 0; k < S_NSLOT; k++) sl[k] = sin_[k];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
    // sum q over the partials: q < 6 the inner products, q = 6 partb
    auto partial = [&](int q) {
        return q < kNP6 ? lane_sum(B.part + (size_t)q * B.nparts, B.nparts) : lane_sum(B.partb, lt.Nt);
    };
    double sum = wave <= kNP6 ? partial(wave) : 0.0;
    // x is behind by alpha_{i-1} p_{i-1} after an odd number of iterations since
    // the last update: it takes two steps at every second iteration, and one
    // where the recursion stops in between
    const int it = (int)sl[S_ITERS];
    const bool behind = ((it - (int)sl[S_ITUPD]) & 1) != 0;
    const double aprev = sl[S_APREV];
    cplx<R> p0[kUpdPre], u0[kUpdPre], s0[kUpdPre], w0[kUpdPre], r0[kUpdPre];
    cplx<double> x0[kUpdPre];
    auto fetch = [&](int k0) {
        size_t i[kUpdPre];
#pragma unroll
        for (int j = 0; j < kUpdPre; j++) {
            const int k = k0 + j * (int)blockDim.x;
            i[j] = base + (k < lt.Vs ? k : 0);
            p0[j] = B.p[i[j]];
            u0[j] = B.u[i[j]];
            s0[j] = B.s[i[j]];
            w0[j] = B.w[i[j]];
            r0[j] = B.r[i[j]];
        }
        if (behind)
#pragma unroll
            for (int j = 0; j < kUpdPre; j++) x0[j] = B.x[i[j]];
    };
    fetch(threadIdx.x);
    const R* tb = nullptr;
    if constexpr (DFT) tb = sp_tables<R, TL>(tab, V + sg.L * sg.ld, sg);
    for (int q = wave; q <= kNP6; q += nw) {
        sum = wave_sum_f64(q == wave ? sum : partial(q));
        if (lane == 63) red[q] = sum;
    }
    __syncthreads();
    double pr[kNP6 + 1];
#pragma unroll
    for (int k = 0; k <= kNP6; k++) pr[k] = red[k];
    const double rr = pr[0], gam = pr[1], del = pr[2], done = sl[S_DONE];
    const int maxit = (int)sl[S_MAXIT];
    double alpha = 0.0, beta = 0.0;
    bool go = false, resume = false;
    if (done == 0.0) {
        int stop = 0;
        const bool first = sl[S_FIRST] != 0.0;
        if (!isfinite(rr) || !isfinite(gam) || !isfinite(del))
            stop = 4;
        else if (rr <= sl[S_TARGET])
            stop = 1;
        else if (it >= maxit)
            stop = 2;  // the budget is used: the update decides
        else if (mixed && (rr <= kDecade2 * sl[S_RRUPD] || it - (int)sl[S_ITUPD] >= kCap))
            stop = 2;
        else {
            beta = first ? 0.0 : gam / sl[S_GPREV];
            const double den = first ? del : del + beta * (pr[3] + pr[4]) + beta * beta * pr[5];
            if (!(den > 0.0))
                stop = 3;
            else
                alpha = gam / den;
        }
        go = stop == 0;
        sl[S_GCUR] = rr;
        if (stop) {
            sl[S_DONE] = (double)stop;
            if (stop == 4) sl[S_WHY] = WHY_BREAKDOWN;
        } else {
            sl[S_GPREV] = gam;
            sl[S_APREV] = alpha;
            sl[S_ITERS] = (double)(it + 1);
            sl[S_FIRST] = 0.0;
        }
    } else if (gate_open(done)) {
        // (updates) the replaced residual decides
        const double tr = pr[kNP6];
        const bool begin = sl[S_B2] < 0.0;
        if (begin) {
            sl[S_B2] = rr;  // the start kernel's |rhs|^2
            sl[S_TARGET] *= rr;  // tol^2 until here
        }
        const int stall = (it + 1 == (int)sl[S_LASTUP]) ? (int)sl[S_STALL] + 1 : 0;
        sl[S_STALL] = begin ? 0 : stall;
        sl[S_LASTUP] = begin ? 0 : it + 1;
        sl[S_NREL] += 1.0;
        sl[S_TRUE] = tr;
        sl[S_GCUR] = tr;
        if (!isfinite(tr) || !isfinite(sl[S_B2])) {
            sl[S_DONE] = 4.0;
            sl[S_WHY] = begin ? WHY_BREAKDOWN : WHY_NONFINITE;
        } else if (tr <= sl[S_TARGET]) {
            sl[S_DONE] = 5.0;
            if (begin) sl[S_NREL] = 1.0;  // the start was this solve's check
        } else if (!begin && (it >= maxit || stall >= 3)) {
            sl[S_DONE] = 4.0;
            sl[S_WHY] = it >= maxit ? WHY_BUDGET : WHY_STALL;
        } else {
            resume = true;
            sl[S_DONE] = 0.0;
            if (begin || !mixed || done == 3.0) sl[S_FIRST] = 1.0;
            sl[S_ITUPD] = it;
            sl[S_RRUPD] = tr;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0)
#pragma unroll
        for (int k = 0; k < S_NSLOT; k++) sout[k] = sl[k];
    if (tau < 0) return;
    // f(site, the site's vectors), the first kUpdPre sites of a thread from its
    // registers, the others as many at a time
    const int stride = kUpdPre * (int)blockDim.x;
    auto each = [&](auto&& f) {
        for (int k0 = threadIdx.x; k0 < lt.Vs; k0 += stride) {
#pragma unroll
            for (int j = 0; j < kUpdPre; j++) {
                const int k = k0 + j * (int)blockDim.x;
                if (k < lt.Vs) f(k, p0[j], u0[j], s0[j], w0[j], r0[j], x0[j]);
            }
            if (k0 + stride < lt.Vs) fetch(k0 + stride);
        }
    };
    auto step = [](cplx<double> x, double al, cplx<R> p) {
        x.re += al * (double)p.re;
        x.im += al * (double)p.im;
        return x;
    };
    if (!go && done == 0.0 && behind)
        each([&](int k, cplx<R> pk, cplx<R>, cplx<R>, cplx<R>, cplx<R>, cplx<double> xv) {
            B.x[base + k] = step(xv, aprev, pk);
        });
    if (!(go || resume)) return;
    if (resume) {
        if constexpr (DFT) {
            each([&](int k, cplx<R>, cplx<R>, cplx<R>, cplx<R>, cplx<R> rk, cplx<double>) {
                const int y = k / sg.L;
                *reinterpret_cast<cplx<R>*>(V + y * sg.ld + 2 * (k - y * sg.L)) = rk;
            });
            sp_forward<R, NY, NX>(V, sg, tb, vhat + base);
        }
        return;
    }
    const R a = (R)alpha, b = (R)beta;
    each([&](int k, cplx<R> pk, cplx<R> uk, cplx<R> sk, cplx<R> wk, cplx<R> rk, cplx<double> xv) {
        const size_t i = base + k;
        const cplx<R> pn = cfma(b, pk, uk);
        const cplx<R> sn = cfma(b, sk, wk);
        B.p[i] = pn;
        B.s[i] = sn;
        if (behind) B.x[i] = step(step(xv, aprev, pk), alpha, pn);
        const cplx<R> rn = cfma(-a, sn, rk);
        B.r[i] = rn;
        if (DFT) {
            const int y = k / sg.L;
            *reinterpret_cast<cplx<R>*>(V + y * sg.ld + 2 * (k - y * sg.L)) = rn;
        }
    });
    if constexpr (DFT) sp_forward<R, NY, NX>(V, sg, tb, vhat + base);
}

// w = O u (own slice) and the partials of the next iteration; or (UPD), where
// the slot asks for a reliable update, r = rhs - O x (FP64, partb its norm) and
// s = O p.  flag: the slot's stop flag (null: none).  Its own slice's vectors
// of the inner products are requested with u with one cell a thread and at
// most 512 threads (1024-thread workgroups would spill), else after the matvec;
// the slot is looked at once they are on their way.  A workgroup has a CU to
// itself here, so the time is one round trip to memory and the operator's chain
// of exchanges: 7.3 us at L = 24, N_tau = 240 (FP32).  No launch bound below 512
// registers is set: with 168 the FP32 form spills 184 and takes 15.7 us.
template <typename R, int MC, int NB, int BS, bool UPD>
__global__ __launch_bounds__(BS) void k_pcg_mv(Lat lt, PcgBufs<R> B, const cplx<R>* __restrict__ gauge, Coef<R> co,
                                               const cplx<double>* __restrict__ gauge64, Coef<double> co64,
                                               const double* __restrict__ flag) {
    extern __shared__ __align__(16) unsigned char smem[];
    cplx<R>* buf2 = reinterpret_cast<cplx<R>*>(smem);
    double* red = reinterpret_cast<double*>(smem + (size_t)NB * 2 * lt.Vs * sizeof(cplx<R>));
    const int tau = slice_of_block(blockIdx.x, lt.Nt);
    if (tau < 0) return;
    const double done = flag ? *flag : 0.0;
    if (!UPD && done != 0.0) return;
    SliceCtx<MC> c;
    slice_ctx<MC>(lt, c, tau, whole_block_tile(smem, red));
    const size_t Vs = lt.Vs;
    const R em = c.tau == 0 ? R(-1) : R(1), et = c.tau == lt.Nt - 1 ? R(-1) : R(1);
    cplx<R> hm[MC][12], ht[MC][12];
    hops_of<R, MC>(gauge, lt, c.tm, c.idx, co, hm);
    hops_of<R, MC>(gauge, lt, c.tau, c.idx, co, ht);
    Cells<R, MC> um, ut, un, w;
    load_cells<R, MC>(um, B.u + c.tm * Vs, c.g);
    load_cells<R, MC>(ut, B.u + c.tau * Vs, c.g);
    load_cells<R, MC>(un, B.u + c.tp * Vs, c.g);
    Cells<R, MC> rt, pt, st;
    constexpr bool early = MC == 1 && BS <= 512;
    if constexpr (early) {
        load_cells<R, MC>(rt, B.r + c.tau * Vs, c.g);
        load_cells<R, MC>(pt, B.p + c.tau * Vs, c.g);
        load_cells<R, MC>(st, B.s + c.tau * Vs, c.g);
    }
    if (UPD && done != 0.0) {
        if (!gate_open(done)) return;
        if constexpr (sizeof(R) == 8) {
            // x takes the place of u below (an FP64 solve restarts after every
            // update, so s is not needed)
            load_cells<R, MC>(um, reinterpret_cast<const cplx<R>*>(B.x) + c.tm * Vs, c.g);
            load_cells<R, MC>(ut, reinterpret_cast<const cplx<R>*>(B.x) + c.tau * Vs, c.g);
            load_cells<R, MC>(un, reinterpret_cast<const cplx<R>*>(B.x) + c.tp * Vs, c.g);
        } else if constexpr (UPD) {
            static_assert(NB == 2, "one FP64 exchange buffer fits the two FP32 ones");
            Cells<double, MC> b, o;
            load_cells<double, MC>(b, B.rhs + c.tau * Vs, c.g);
            {
                cplx<double> gm[MC][12], gt[MC][12];
                hops_of<double, MC>(gauge64, lt, c.tm, c.idx, co64, gm);
                hops_of<double, MC>(gauge64, lt, c.tau, c.idx, co64, gt);
                Cells<double, MC> xm, xt, xn;
                load_cells<double, MC>(xm, B.x + c.tm * Vs, c.g);
                load_cells<double, MC>(xt, B.x + c.tau * Vs, c.g);
                load_cells<double, MC>(xn, B.x + c.tp * Vs, c.g);
                mdagm_cells<double, MC, 1>(xm, xt, xn, gm, gt, c.g, c.own, co64, (double)em, (double)et,
                                            reinterpret_cast<cplx<double>*>(smem), lt.Vs, o);
            }
            double v[1] = {0.0};
            Cells<R, MC> r, pm, po, pn;
#pragma unroll
            for (int m = 0; m < MC; m++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const double re = b.v[m][q].re - o.v[m][q].re, im = b.v[m][q].im - o.v[m][q].im;
                    if (c.own[m]) v[0] += re * re + im * im;
                    r.v[m][q] = mk<R>((R)re, (R)im);
                }
            store_cells<R, MC>(r, B.r + c.tau * Vs, c.g, c.own);
            block_sumk<1>(v, red);
            if (threadIdx.x == 0) B.partb[c.tau] = v[0];
            load_cells<R, MC>(pm, B.p + c.tm * Vs, c.g);
            load_cells<R, MC>(po, B.p + c.tau * Vs, c.g);
            load_cells<R, MC>(pn, B.p + c.tp * Vs, c.g);
            // (fetched again rather than held across the FP64 operator)
            cplx<R> gm[MC][12], gt[MC][12];
            hops_of<R, MC>(gauge, lt, c.tm, c.idx, co, gm);
            hops_of<R, MC>(gauge, lt, c.tau, c.idx, co, gt);
            __syncthreads();  // the exchange buffers are reused
            mdagm_cells<R, MC, NB>(pm, po, pn, gm, gt, c.g, c.own, co, em, et, buf2, lt.Vs, w);
            store_cells<R, MC>(w, B.s + c.tau * Vs, c.g, c.own);
            return;
        }
    }
    mdagm_cells<R, MC, NB>(um, ut, un, hm, ht, c.g, c.own, co, em, et, buf2, lt.Vs, w);
    if constexpr (UPD && sizeof(R) == 8) {
        if (done != 0.0) {
            Cells<R, MC> b;
            load_cells<R, MC>(b, reinterpret_cast<const cplx<R>*>(B.rhs) + c.tau * Vs, c.g);
#pragma unroll
            for (int m = 0; m < MC; m++)
#pragma unroll
                for (int q = 0; q < 4; q++) b.v[m][q] = csub(b.v[m][q], w.v[m][q]);
            store_cells<R, MC>(b, B.r + c.tau * Vs, c.g, c.own);
            double v[1] = {dot_cells<R, MC>(b, b, c.own)};
            block_sumk<1>(v, red);
            if (threadIdx.x == 0) B.partb[c.tau] = v[0];
            return;
        }
    }
    store_cells<R, MC>(w, B.w + c.tau * Vs, c.g, c.own);
    if constexpr (!early) {
        load_cells<R, MC>(rt, B.r + c.tau * Vs, c.g);
        load_cells<R, MC>(pt, B.p + c.tau * Vs, c.g);
        load_cells<R, MC>(st, B.s + c.tau * Vs, c.g);
    }
    const Cells<R, MC>& u0 = ut;  // the matvec reads its own slice without changing it
    double v[kNP6] = {dot_cells<R, MC>(rt, rt, c.own), dot_cells<R, MC>(rt, u0, c.own),
                      dot_cells<R, MC>(w, u0, c.own),  dot_cells<R, MC>(u0, st, c.own),
                      dot_cells<R, MC>(pt, w, c.own),  dot_cells<R, MC>(pt, st, c.own)};
#pragma unroll
    for (int k = 0; k < kNP6; k++) v[k] = wave_sum_f64(v[k]);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 63)
#pragma unroll
        for (int k = 0; k < kNP6; k++) red[kNP6 * wv + k] = v[k];
    __syncthreads();
    if (threadIdx.x < kNP6) {
        double t = 0.0;
        const int nw = (int)(blockDim.x + 63) >> 6;
        for (int i = 0; i < nw; i++) t += red[kNP6 * i + threadIdx.x];
        B.part[(size_t)threadIdx.x * B.nparts + c.tau] = t;
    }
}

// r = rhs - O x from the FP64 O x; partb = FP64 |rhs - O x|^2 per slice
template <typename R>
__global__ __launch_bounds__(256) void k_pcg_rep(Lat lt, PcgBufs<R> B) {
    __shared__ double red[64];
    const size_t base = (size_t)blockIdx.x * lt.Vs;
    double t2 = 0.0;
    for (int k = threadIdx.x; k < lt.Vs; k += blockDim.x) {
        const cplx<double> b = B.rhs[base + k], o = B.Ox[base + k];
        const double re = b.re - o.re, im = b.im - o.im;
        B.r[base + k] = mk<R>((R)re, (R)im);
        t2 += re * re + im * im;
    }
    double v[1] = {t2};
    block_sumk<1>(v, red);
    if (threadIdx.x == 0) B.partb[blockIdx.x] = v[0];
}

// After a replacement: converged -> stop 1; otherwise resume (restart sets
// beta = 0 on the next iteration).  rr: the partials of the replaced r's
// <r, r> in the working precision, or null (the FP64 residual is taken); b2:
// at the start of a solve whose slot holds tol^2, the partials of |rhs|^2.
__global__ void k_pcg_check(double* __restrict__ scal, int kpar, const double* __restrict__ rr, int nparts,
                            const double* __restrict__ partb, int Nt, int restart, const double* __restrict__ b2) {
    __shared__ double red[3];
    const int wave = threadIdx.x >> 6;
    const double* src = wave == 0 ? partb : (wave == 1 ? rr : b2);
    const double s = wave_sum_f64(src ? lane_sum(src, wave == 1 ? nparts : Nt) : 0.0);
    if ((threadIdx.x & 63) == 63) red[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double* sl = scal + S_NSLOT * kpar;
        if (b2) {
            sl[S_B2] = red[2];
            sl[S_TARGET] *= red[2];
        }
        sl[S_TRUE] = red[0];
        if (red[0] <= sl[S_TARGET]) {
            sl[S_DONE] = 1.0;
        } else {
            sl[S_DONE] = 0.0;
            if (restart) sl[S_FIRST] = 1.0;
            sl[S_ITUPD] = sl[S_ITERS];
            sl[S_RRUPD] = rr ? red[1] : red[0];
        }
    }
}

// a slot to a solve's record in pinned host memory
__global__ void k_pcg_record(const double* __restrict__ sl, double* __restrict__ out) {
    if (threadIdx.x == 0) {
        out[CR_ITERS] = sl[S_ITERS];
        out[CR_TRUE] = sl[S_TRUE];
        out[CR_B2] = sl[S_B2];
        out[CR_NREL] = sl[S_NREL];
        out[CR_WHY] = sl[S_WHY];
        out[CR_EST] = sl[S_GCUR];
        out[CR_DONE] = sl[S_DONE];
    }
}

// ---------------------------------------------------------------------------
// Host driver
// ---------------------------------------------------------------------------
// The solver keeps its right-hand side and solution in the handle's workspace
// (ws[2], ws[7]), so captured graphs do not depend on a caller's buffers.
template <typename R>
static PcgBufs<R> pbufs_of(qedhmc_ctx* h) {
    PcgBufs<R> B;
    const size_t N = (size_t)h->lat.Nt * h->lat.Vs;
    cplx<R>* base = reinterpret_cast<cplx<R>*>(h->cg_arena);
    B.r = base;
    B.p = base + N;
    B.s = base + 2 * N;
    B.u = base + 3 * N;
    B.w = base + 4 * N;
    B.t = base + 5 * N;
    B.x = reinterpret_cast<cplx<double>*>(h->ws[7]);
    B.rhs = reinterpret_cast<const cplx<double>*>(h->ws[2]);
    B.Ox = reinterpret_cast<const cplx<double>*>(h->ws[3]);
    if (h->lat.ncell > 1024) {
        // the tiled matvec writes one partial tuple per (slice, tile)
        B.nparts = h->lat.Nt * mdagm_tiled_tiles(h->lat, sizeof(R) == 8);
        B.part = h->tpart;
        B.partb = h->tpart + kNP6 * (size_t)h->lat.Nt * h->tpart_tiles;
    } else {
        B.nparts = h->lat.Nt;
        B.part = h->partial;
        B.partb = h->partial + kNP6 * (size_t)h->lat.Nt;
    }
    return B;
}

// whether the reliable updates run inside the triples: slices of up to so many
// cells, one a thread, whose FP64 operator fits the matvec's registers (with
// 1024 threads a workgroup it has 128 of the 233 it takes)
static constexpr int kUpdCells = 512;

template <typename R>
static qedhmc_status launch_mv(qedhmc_ctx* h, const PcgBufs<R>& B, const double* stop, bool timed, bool updates) {
    if (h->lat.ncell > 1024) return launch_mdagm_tiled_parts<R>(h, B.u, B.w, B.r, B.p, B.s, B.part, stop);
    return with_shape<R>(h, [&]<int MC, int NB, int BS>(int nt, size_t lds) -> qedhmc_status {
        auto go = [&](auto kern) -> qedhmc_status {
            QH_TRY(lds_attr(h, kern, lds));
            hipEvent_t e0, e1;
            const int cls = sizeof(R) == 4 ? QEDHMC_K_PCG_MV_FP32 : QEDHMC_K_PCG_MV_FP64;
            if (timed && prof_sample(h, cls, e0, e1))
                hipExtLaunchKernelGGL(kern, dim3(slice_grid(h->lat.Nt)), dim3(nt), lds, h->stream, e0, e1, 0, h->lat, B,
                                      gauge_for<R>(h), coef_of<R>(h->p), (const cplx<double>*)h->gauge64,
                                      coef_of<double>(h->p), stop);
            else
                hipLaunchKernelGGL(kern, dim3(slice_grid(h->lat.Nt)), dim3(nt), lds, h->stream, h->lat, B,
                                   gauge_for<R>(h), coef_of<R>(h->p), (const cplx<double>*)h->gauge64,
                                   coef_of<double>(h->p), stop);
            QH_HIP(hipGetLastError());
            return QEDHMC_OK;
        };
        if constexpr (MC == 1 && BS <= 512 && (sizeof(R) == 8 || NB == 2))
            if (updates) return go(k_pcg_mv<R, MC, NB, BS, true>);
        return go(k_pcg_mv<R, MC, NB, BS, false>);
    });
}

// u = P r, w = O u, partials (stop: nullable slot flag); with the identity
// preconditioner u is r itself and only w = O r is launched
template <typename R>
static qedhmc_status pcg_tail(qedhmc_ctx* h, const PcgBufs<R>& B, const double* stop, bool identity,
                              bool updates = false) {
    if (!identity) QH_TRY(apply_P_t<R>(h, B.r, B.u, spec_vhat<R>(h, B.u, B.t), B.t, stop));
    return launch_mv<R>(h, B, stop, stop != nullptr, updates);
}

// n iterations from launch parity kpar: update, then preconditioner and
// matvec, each gated on the slot's stop flag.  decide: the update kernel also
// takes the decision after a reliable update.
template <typename R>
static qedhmc_status pcg_chunk(qedhmc_ctx* h, const PcgBufs<R>& B, int kpar, int n, bool mixed, bool identity,
                               bool decide) {
    const bool updates = !identity && h->lat.ncell <= kUpdCells;  // inside the triples
    // spectral P: the update kernel does its first step
    const bool fdft = !identity && use_spectral<R>(h);
    const PcSpecGeo sg = fdft ? spec_geo<R>(h) : PcSpecGeo{};
    cplx<R>* vhat = fdft ? spec_vhat<R>(h, B.u, B.t) : nullptr;
    for (int k = 0; k < n; k++) {
        if (fdft)
            QH_TRY(with_spec<R>(sg, [&]<int NY, int NX, bool TL>() -> qedhmc_status {
                bool tl;
                const size_t lds = spec_lds<R>(sg, tl);
                if (lds > 65536 - 2048) QH_TRY(allow_lds((const void*)k_pcg_upd<R, NY, NX, TL>, h->max_lds));
                hipLaunchKernelGGL((k_pcg_upd<R, NY, NX, TL>), dim3(slice_grid(h->lat.Nt)),
                                   dim3(spec_threads(sg, sg.Vs, spec_max_threads<R>())), lds, h->stream, h->lat, B,
                                   h->scal, kpar, mixed ? 1 : 0, decide ? 1 : 0, sg, spec_tab<R>(h), vhat);
                return QEDHMC_OK;
            }));
        else
            // (four sites a thread, as many as it requests at once)
            hipLaunchKernelGGL((k_pcg_upd<R, 0, 0, false>), dim3(slice_grid(h->lat.Nt)),
                               dim3(std::clamp((h->lat.Vs / kUpdPre + 63) / 64 * 64, 256, spec_max_threads<R>())), 0,
                               h->stream, h->lat, B, h->scal, kpar, mixed ? 1 : 0, decide ? 1 : 0, sg, (const R*)nullptr,
                               (cplx<R>*)nullptr);
        kpar ^= 1;
        const double* stop = h->scal + S_NSLOT * kpar + S_DONE;
        if (fdft) {
            QH_TRY(launch_pcs_rest<R>(h, vhat, B.u, B.t, stop));
            QH_TRY(launch_mv<R>(h, B, stop, true, updates));
        } else {
            QH_TRY(pcg_tail<R>(h, B, stop, identity, updates));
        }
    }
    QH_HIP(hipGetLastError());
    return QEDHMC_OK;
}

// the start of a solve on slices of up to kUpdCells cells (x0 null: from zero)
template <typename R>
static qedhmc_status launch_begin(qedhmc_ctx* h, const PcgBufs<R>& B, const double* rhs, const double* x0, double tol,
                                  int maxit) {
    return with_shape<double>(h, [&]<int MC, int NB, int BS>(int nt, size_t lds) -> qedhmc_status {
        if constexpr (MC == 1 && BS <= 512) {
            QH_TRY(lds_attr(h, k_pcg_begin<R, MC, NB, BS>, lds));
            hipLaunchKernelGGL((k_pcg_begin<R, MC, NB, BS>), dim3(slice_grid(h->lat.Nt)), dim3(nt), lds, h->stream,
                               h->lat, B, (const cplx<double>*)h->gauge64, coef_of<double>(h->p),
                               (const cplx<double>*)rhs, (cplx<double>*)h->ws[2], (const cplx<double>*)x0, h->scal,
                               tol * tol, maxit);
            QH_HIP(hipGetLastError());
        }
        return QEDHMC_OK;
    });
}

// Runs enqueue(), or replays it from the graph captured the first time this
// (mode, length, plan) combination is seen; the launch
// shapes and kernel attributes are set by an eager run before any capture.
template <typename F>
static qedhmc_status run_graph(qedhmc_ctx* h, qedhmc_ctx::PcgGraph& gr, const qedhmc_ctx::PcgGraph& key, F&& enqueue) {
    if (gr.exec && (gr.mixed != key.mixed || gr.count != key.count || gr.plan != key.plan)) {
        QH_HIP(hipGraphExecDestroy(gr.exec));
        gr.exec = nullptr;
    }
    if (!gr.exec) {
        if (!h->cap_stream) QH_HIP(hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking));
        hipStream_t user = h->stream;
        const int prof = h->prof_every;
        h->stream = h->cap_stream;
        h->prof_every = 0;  // no event launches inside a graph
        hipGraph_t g = nullptr;
        qedhmc_status st = QEDHMC_OK;
        hipError_t e = hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal);
        if (e == hipSuccess) {
            st = enqueue();
            e = hipStreamEndCapture(h->cap_stream, &g);
        }
        h->stream = user;
        h->prof_every = prof;
        if (st != QEDHMC_OK) {
            if (g) (void)hipGraphDestroy(g);
            return st;
        }
        QH_HIP(e);
        hipGraphExec_t exec = nullptr;
        e = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        QH_HIP(e);
        gr = key;
        gr.exec = exec;
    }
    QH_HIP(hipGraphLaunch(gr.exec, h->stream));
    return QEDHMC_OK;
}

// the launches a graph of the solver holds besides its length
template <typename R>
static int pcg_plan(const qedhmc_ctx* h, bool identity) {
    return identity ? 0 : (use_spectral<R>(h) ? 1 : 0) | (spec_fused<R>(h) ? 2 : 0);
}

// Triples per graph of the solver whose reliable updates run inside them (an
// even count: every graph starts at launch parity 0); the host reads the
// record of each.  The launches of the last graph past the end of a solve, and
// of one queued behind it in vain, do little but load (11 us a triple at L = 24
// in FP32 and at L = 12 in FP64, 9 of them inside the kernels; 13 at L = 40), and
// each graph costs about 8 us between the record and the next one's first
// launch: 4, 6, 8, 10 measured 7.69, 7.48, 7.61, 7.37 ms per trajectory at L =
// 24, N_tau = 240 (mixed) and 4.70, 4.57, 4.45, 4.34 ms at L = 12, N_tau = 120
// (FP64); 6, 10, 30 a solve at L = 24 to 1e-6 1.47, 1.47, 1.63 ms, to 1e-10 2.46,
// 2.32, 2.35 ms.
static constexpr int kPcgTriples = 10;

// The solve with every decision taken on the device: graphs of kPcgTriples
// triples and a record of the slot.  A reliable update is one triple (the stop,
// nothing, r = rhs - O x and s = O p in the matvec's launch) and the first of
// the next (the decision, and the transform of the new r): no launch waits for
// the host and none is wasted between a pause and its update.  Against whole
// rounds of 12 iterations with gated update launches, and a solve for the
// correction where a trajectory starts warm: 8.7 -> 7.4 ms per trajectory at
// L = 24, N_tau = 240, tol 1e-10 (mixed), 4.0 -> 3.0 ms per solve at tol 1e-12.
// The host keeps the next one queued behind the running one and holds it back
// only when the residual estimates of the
// last two, extrapolated geometrically, say that the running one converges (a
// wrong guess costs one host round trip).
template <typename R>
static qedhmc_status pcg_device(qedhmc_ctx* h, const PcgBufs<R>& B, const double* rhs, double* x, bool warm, double tol,
                                int maxit, qedhmc_precision prec, int* iters, double* true_rel, int* n_reliable,
                                long most) {
    const bool mixed = prec != QEDHMC_FP64;
    for (auto& e : h->cg_ev)
        if (!e) QH_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    QH_TRY(launch_begin<R>(h, B, rhs, warm ? x : nullptr, tol, maxit));
    auto& graphs = h->pcg_round[sizeof(R) == 8 ? 1 : 0];
    // the first launches of a handle's first solve set the kernel attributes
    const bool eager0 = !graphs[0].exec;
    qedhmc_ctx::PcgGraph key{};
    key.mixed = mixed ? 1 : 0;
    key.count = kPcgTriples;
    key.plan = pcg_plan<R>(h, false);
    auto round = [&](long n) -> qedhmc_status {
        const int par = (int)(n & 1);
        double* out = h->h_pinned + 32 + 16 * par;
        auto enqueue = [&]() -> qedhmc_status {
            QH_TRY(pcg_chunk<R>(h, B, 0, kPcgTriples, mixed, false, true));
            hipLaunchKernelGGL(k_pcg_record, dim3(1), dim3(64), 0, h->stream, (const double*)h->scal, out);
            QH_HIP(hipGetLastError());
            return QEDHMC_OK;
        };
        if (n == 0 && eager0)
            QH_TRY(enqueue());
        else
            QH_TRY(run_graph(h, graphs[par], key, enqueue));
        QH_HIP(hipEventRecord(h->cg_ev[par], h->stream));
        return QEDHMC_OK;
    };
    // a triple iterates, or belongs to an update; three updates without an
    // iteration between them end the solve
    const long max_rounds = most ? most : (9L * maxit + 32) / kPcgTriples + 4;
    long queued = 0;
    bool over = false;
    double prev = -1.0;
    const double* r = nullptr;
    QH_TRY(round(queued++));
    QH_TRY(round(queued++));
    for (long n = 0;; n++) {
        // queued: round n, and rounds n + 1 and n + 2 unless held back
        QH_HIP(hipEventSynchronize(h->cg_ev[n & 1]));
        r = h->h_pinned + 32 + 16 * (n & 1);
        if (r[CR_DONE] == 4.0 || r[CR_DONE] == 5.0) break;
        over = n + 2 >= max_rounds;
        if (over) break;
        if (queued < n + 2) QH_TRY(round(queued++));  // round n + 1 was held back wrongly
        const double tr = r[CR_EST], target = tol * tol * r[CR_B2];
        const bool last = prev > 0.0 && tr > 0.0 && tr * (tr / prev) <= target;
        prev = tr;
        if (!last && queued < n + 3) QH_TRY(round(queued++));
    }
    QH_HIP(hipMemcpyAsync(x, B.x, (size_t)h->lat.Nt * h->lat.Vs * sizeof(cplx<double>), hipMemcpyDeviceToDevice,
                          h->stream));
    QH_HIP(hipStreamSynchronize(h->stream));
    const double* rec = h->h_pinned + 32 + 16 * ((queued - 1) & 1);  // rounds past the end repeat the slot
    const int it = (int)rec[CR_ITERS];
    if (iters) *iters = it;
    // (a breakdown before the first update: the start's residual, 1 from zero)
    const double tr = rec[CR_TRUE], b2 = rec[CR_B2];
    double rel = b2 > 0.0 ? std::sqrt(tr / b2) : 0.0;
    if (warm && !(std::isfinite(tr) && std::isfinite(b2))) rel = HUGE_VAL;
    if (!warm && rec[CR_NREL] == 0.0) rel = 1.0;
    if (true_rel) *true_rel = rel;
    // (a warm start that meets the target has had no update)
    if (n_reliable) *n_reliable = warm && it == 0 && rec[CR_DONE] == 5.0 ? 0 : (int)rec[CR_NREL];
    if (rec[CR_DONE] == 5.0) return QEDHMC_OK;
    if (over) set_error("PCG did not end within " + std::to_string(max_rounds) + " rounds");
    switch ((int)rec[CR_WHY]) {
        case WHY_BREAKDOWN:
            set_error("PCG breakdown: non-finite inner products after " + std::to_string(it) + " iterations");
            break;
        case WHY_NONFINITE:
            set_error("PCG breakdown: non-finite true residual after " + std::to_string(it) + " iterations");
            break;
        case WHY_STALL:
            set_error("PCG made no progress across reliable updates at iteration " + std::to_string(it));
            break;
        default:
            break;
    }
    return QEDHMC_ENOCONV;
}

// identity = true: plain CG in the same two-launch form (update, then
// M^dag M with the partials), the form used for lattices whose slices hold
// more than 1024 cells: there the fused one-launch iteration would need two
// cells per thread and more registers than a 576-thread workgroup has.
template <typename R>
static qedhmc_status pcg_t(qedhmc_ctx* h, const double* rhs, double* x, double tol, int maxit, qedhmc_precision prec,
                           int* iters, double* true_rel, int* n_reliable, bool identity, bool warm = false,
                           long most = 0) {
    if (!identity) QH_TRY(ensure_paper_precond(h));
    const bool mixed = prec != QEDHMC_FP64;
    PcgBufs<R> B = pbufs_of<R>(h);
    if (identity) B.u = B.r;
    const int Nt = h->lat.Nt;
    // QEDHMC_NO_GRAPH (read per solve): no captured graphs, and every decision here
    const bool no_graph = std::getenv("QEDHMC_NO_GRAPH") != nullptr;
    const bool small = !identity && h->lat.ncell <= kUpdCells;
    if (small && !no_graph)
        return pcg_device<R>(h, B, rhs, x, warm, tol, maxit, prec, iters, true_rel, n_reliable, most);
    // iterations per host round trip: the plain recursion pauses after kCap at
    // most; with the paper's preconditioner a decade, and with it a pause, takes
    // about 9 to 30 iterations, and the launches past a pause are wasted.  Chunks
    // of 51 / 24 / 12, ms per solve: L = 46, N_tau = 200, tol 1e-8 5.55 / 3.78 /
    // 3.12, L = 66, N_tau = 200, 1e-4 3.43 / 2.76 / 2.58, L = 66, N_tau = 660,
    // 1e-12 31.5 / 29.0 / 28.6, L = 80, N_tau = 200, 1e-12 18.0 / 16.0 / 15.8
    // (small: every iteration by itself, its matvec carrying out an update)
    const int chunk = small ? 1 : (mixed ? (identity ? kCap + 1 : 12) : 64);
    int kpar = 0, nrel = 0, it = 0, stalled = 0, last_it = -1;
    double rel = 1.0;
    bool converged = false, broken = false;
    // the true residual's decision, into the slot and to the host
    auto check = [&](bool restart, bool begin) -> qedhmc_status {
        hipLaunchKernelGGL(k_pcg_check, dim3(1), dim3(192), 0, h->stream, h->scal, kpar,
                           (const double*)(small ? nullptr : B.part), B.nparts, (const double*)B.partb, Nt,
                           restart ? 1 : 0, (const double*)(begin ? B.part : nullptr));
        QH_HIP(hipGetLastError());
        QH_TRY(read_slot(h, kpar));
        const double b2 = h->h_pinned[S_B2];
        if (!std::isfinite(h->h_pinned[S_TRUE]) || !std::isfinite(b2)) {
            broken = true;
            set_error(begin ? "PCG breakdown: non-finite inner products after 0 iterations"
                            : "PCG breakdown: non-finite true residual after " + std::to_string(it) + " iterations");
        }
        converged = !broken && h->h_pinned[S_DONE] == 1.0;
        if (!begin || warm || converged) rel = b2 > 0.0 ? std::sqrt(h->h_pinned[S_TRUE] / b2) : 0.0;
        if (warm && broken) rel = HUGE_VAL;
        return QEDHMC_OK;
    };
    if (small) {
        QH_TRY(launch_begin<R>(h, B, rhs, warm ? x : nullptr, tol, maxit));
        QH_TRY(check(true, true));
        if (converged && !warm) nrel = 1;  // the start was this solve's check
        if (!broken && !converged) QH_TRY(pcg_tail<R>(h, B, nullptr, false, true));
    } else {
        hipLaunchKernelGGL(k_pcg_start<R>, dim3(Nt), dim3(256), 0, h->stream, h->lat, B, (const cplx<double>*)rhs,
                           (cplx<double>*)h->ws[2]);
        hipLaunchKernelGGL(k_pcg_init_slot, dim3(1), dim3(256), 0, h->stream, h->scal, (const double*)B.partb, Nt,
                           tol * tol, maxit);
        QH_HIP(hipGetLastError());
        QH_TRY(pcg_tail<R>(h, B, nullptr, identity));
    }
    while (!broken && !converged) {
        // one launch past the budget stops the recursion and brings x up to date
        const int n = std::min(maxit - it, chunk - 1) + 1;
        auto enqueue = [&]() { return pcg_chunk<R>(h, B, kpar, n, mixed, identity, false); };
        if (n == chunk && !no_graph) {
            qedhmc_ctx::PcgGraph key{};
            key.mixed = mixed ? 1 : 0;
            key.count = n;
            key.plan = pcg_plan<R>(h, identity);
            QH_TRY(run_graph(h, h->pcg_graph[sizeof(R) == 8 ? 1 : 0][identity ? 1 : 0][kpar], key, enqueue));
        } else {
            QH_TRY(enqueue());
        }
        if (n & 1) kpar ^= 1;
        QH_TRY(read_slot(h, kpar));
        it = (int)h->h_pinned[S_ITERS];
        const double flag = h->h_pinned[S_DONE];
        if (flag == 0.0) continue;
        if (flag == 4.0) {
            broken = true;
            set_error("PCG breakdown: non-finite inner products after " + std::to_string(it) + " iterations");
            break;
        }
        stalled = (it == last_it) ? stalled + 1 : 0;
        last_it = it;
        if (!small && stalled >= 3) {
            set_error("PCG made no progress across reliable updates at iteration " + std::to_string(it));
            break;
        }
        // FP64 true residual; r replaced, s = O p refreshed, u, w and partials recomputed
        const bool restart = !mixed || flag == 3.0;
        nrel++;
        if (small) {
            QH_TRY(check(restart, false));  // the matvec's launch has replaced r
            if (!broken && !converged && it < maxit && stalled >= 3) {
                set_error("PCG made no progress across reliable updates at iteration " + std::to_string(it));
                break;
            }
            if (!broken && !converged && it < maxit) QH_TRY(pcg_tail<R>(h, B, nullptr, false, true));
        } else {
            QH_TRY(launch_mdagm(h, QEDHMC_FP64, B.x, h->ws[3], nullptr));
            hipLaunchKernelGGL(k_pcg_rep<R>, dim3(Nt), dim3(256), 0, h->stream, h->lat, B);
            QH_HIP(hipGetLastError());
            QH_TRY(launch_mdagm(h, prec == QEDHMC_FP64 ? QEDHMC_FP64 : QEDHMC_FP32, B.p, B.s, nullptr));
            QH_TRY(pcg_tail<R>(h, B, nullptr, identity));
            QH_TRY(check(restart, false));
        }
        if (it >= maxit) break;
    }
    QH_HIP(hipMemcpyAsync(x, B.x, (size_t)Nt * h->lat.Vs * sizeof(cplx<double>), hipMemcpyDeviceToDevice, h->stream));
    QH_HIP(hipStreamSynchronize(h->stream));
    if (iters) *iters = it;
    if (true_rel) *true_rel = rel;
    if (n_reliable) *n_reliable = nrel;
    if (broken) return QEDHMC_ENOCONV;
    return converged ? QEDHMC_OK : QEDHMC_ENOCONV;
}

bool pcg_warm_ok(const qedhmc_ctx* h) { return h->lat.ncell <= kUpdCells; }

qedhmc_status pcg_solve_impl(qedhmc_ctx* h, const double* rhs, double* x, double tol, int maxit,
                             qedhmc_precision prec, int* iters, double* true_rel, int* n_reliable, bool warm,
                             long most) {
    if (prec == QEDHMC_FP64)
        return pcg_t<double>(h, rhs, x, tol, maxit, prec, iters, true_rel, n_reliable, false, warm, most);
    return pcg_t<float>(h, rhs, x, tol, maxit, prec, iters, true_rel, n_reliable, false, warm, most);
}

qedhmc_status cg2_solve_impl(qedhmc_ctx* h, const double* rhs, double* x, double tol, int maxit,
                             qedhmc_precision prec, int* iters, double* true_rel, int* n_reliable) {
    if (prec == QEDHMC_FP64) return pcg_t<double>(h, rhs, x, tol, maxit, prec, iters, true_rel, n_reliable, true);
    return pcg_t<float>(h, rhs, x, tol, maxit, prec, iters, true_rel, n_reliable, true);
}

}  // namespace qh
