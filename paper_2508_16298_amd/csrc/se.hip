// Stochastic estimation of fermionic observables (Methods, "Stochastic
// estimation of fermionic observables", Eq. Cij_est and the FFT translational
// average; Supplemental Material SIV for the spin correlator).
//
//   probes   xi_p, p < n_rv: complex Gaussian, E[xi^* xi^T] = 1 (Philox
//            purpose 4, element p N + n, index = the measurement index)
//   solve    X_p = (M^dag M)^{-1} M^dag xi_p = G xi_p for all p at once: a
//            batch of n_rv right-hand sides whose workgroups all read one
//            gauge field (the multi-RHS CG)
//   spin     C_S(Delta) = delta_{Delta,0} T1 - T2(Delta) with
//            T1 = (1/(n_rv N)) sum_p sum_i X_p,i conj(xi_p,i) and
//            T2 = 1/(n_rv (n_rv-1) N^2) sum_k S_k e^{+i k.Delta},
//            S_k = sum_{p<q} A_{-k} B_k + A_k B_{-k},
//            A = DFT[X_p conj(xi_q)], B = DFT[X_q conj(xi_p)]
//
// The three-dimensional DFTs are separable.  Forward, per pass of pairs: one
// kernel forms both products of a pair on a slice in LDS and transforms both
// spatial axes on the matrix cores (spectral.h: real products with paired
// points, FP64); one transforms tau the same way for a group of spatial
// frequencies k and the mirrored group -k, whose A_k, B_k, A_{-k}, B_{-k} then
// sit in the same lanes, multiplies them and adds over the pairs in registers:
// the transforms in tau are never written.  Backward, one vector: a spatial
// pass on the matrix cores and a direct tau pass.  All sums run in a fixed
// order.
#include <algorithm>
#include <cstdlib>
#include <new>
#include <vector>

#include "qedhmc_internal.h"
#include "rng.h"
#include "spectral.h"

struct qedhmc_se {
    qedhmc_params p{};
    int n_rv = 0;
    int64_t N = 0;
    int L = 0, Nt = 0, Vs = 0;
    hipStream_t stream = nullptr;
    qedhmc_batch* b = nullptr;     // n_rv right-hand sides sharing one gauge field
    qh::cplx<double>* rhs = nullptr;  // n_rv x N: M^dag xi_p
    qh::cplx<double>* ws = nullptr;   // spatial transforms of P pairs: 2 P vectors of [Nt][2][nrp]
    qh::cplx<double>* S = nullptr;    // 2 x N: the pair products summed in k-space, and its spatial transform
    qh::cplx<double>* Sp = nullptr;   // the same sum per chunk of pairs, [chunks][Nt][nrp]
    qh::cplx<double>* T = nullptr;    // N: the inverse transform
    double* tabL = nullptr;           // DFT weights of the spatial axes
    double* tabT = nullptr;           // ... and of tau
    int* cols = nullptr;              // [2][nrp] position in a slice's image of the columns' spatial frequencies
                                      // (representatives of the pairs {k, -k}, then their mirror images; padding: 0);
                                      // then [Vs] column of a frequency; then [npairs][2] the probe pairs
    qh::cplx<double>* twT = nullptr;  // Nt twiddles
    qh::cplx<double>* part = nullptr; // T1 partial sums
    int nrp = 0;                      // representatives, padded to whole groups of kCols
    int nchunk = 0, per = 0;          // chunks of pairs per pass, pairs per chunk
    int P = 0;                        // pairs per pass
    int n_part = 0;
};

namespace qh {

namespace {

constexpr int kBS = 256;
constexpr size_t kWorkBytes = (size_t)192 << 20;  // spatial transforms of a pass: they stay in the last-level cache

__device__ __forceinline__ cplx<double> cmul(cplx<double> a, cplx<double> b) {
    return mk<double>(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
__device__ __forceinline__ cplx<double> cmulc(cplx<double> a, cplx<double> b) {  // a conj(b)
    return mk<double>(a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im);
}

__global__ void k_se_probes(uint64_t seed, uint64_t meas, uint32_t total, cplx<double>* __restrict__ xi) {
    const double r2 = 0.70710678118654752440;
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        uint32_t x[4];
        double g1, g2;
        draw_block(seed, meas, RNG_PROBE, e, x);
        gauss_pair(x, g1, g2);
        xi[e] = mk<double>(r2 * g1, r2 * g2);
    }
}

__global__ void k_se_twiddle(int n, cplx<double>* __restrict__ tw) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    double s, c;
    sincospi(-2.0 * (double)k / (double)n, &s, &c);
    tw[k] = mk<double>(c, s);
}

// Reals per LDS row of a slice of L complex values: half a bank turn between
// two rows (the transforms read four or eight rows at once).
constexpr int se_ld(int L) { return 2 * L + (2 * L % 16 == 8 ? 0 : (24 - 2 * L % 16) % 16); }

// 16-output blocks of a DFT of n points
constexpr int se_blocks(int n) { return (n / 2 + 1 + 15) / 16; }

// Spatial DFT of the vectors of one pair (PROD: a = X_p conj(xi_q) and b =
// X_q conj(xi_p) of pairs[pair], formed on the way in) or of one vector,
// on one slice per workgroup, both axes in place in LDS.  PROD writes the
// frequencies in the order of cols ([tau][2][nrp], coalesced for the tau
// pass), otherwise [tau][ky][kx] with the inverse sign.  Slices of one tau are
// consecutive on one XCD, where the pairs re-read X and xi from the L2.
// 97 us per pass of 40 pairs at L = 24, N_tau = 240 (24 us of products, about
// 30 us each of LDS traffic and of vector instructions around them); direct
// sums took 255 us per 60 pairs.
template <int NB, bool PROD>
__global__ __launch_bounds__(512) void k_se_xy(int L, int ld, int Nt, int64_t N, const int2* __restrict__ pairs,
                                               int np, int nrp, const cplx<double>* __restrict__ X,
                                               const cplx<double>* __restrict__ xi, const double* __restrict__ tab,
                                               const int* __restrict__ cols, cplx<double>* __restrict__ out) {
    extern __shared__ __align__(32) unsigned char smem[];
    constexpr int NV = PROD ? 2 : 1;
    double* V = reinterpret_cast<double*>(smem);
    const int Vs = L * L, image = L * ld;
    const int j = (int)blockIdx.x >> 3, tau = ((int)blockIdx.x & 7) + 8 * (j / np), pair = j % np;
    if (tau >= Nt) return;
    const int64_t off = (int64_t)tau * Vs;
    // the weights, after the images
    double* w = V + NV * image;
    const int ntab = sp_table(L, NB);
    for (int i = threadIdx.x; i < ntab; i += blockDim.x) w[i] = tab[i];
    if constexpr (PROD) {
        const int p = pairs[pair].x, q = pairs[pair].y;
        const cplx<double>*Xp = X + (int64_t)p * N + off, *Xq = X + (int64_t)q * N + off;
        const cplx<double>*zp = xi + (int64_t)p * N + off, *zq = xi + (int64_t)q * N + off;
        for (int s = threadIdx.x; s < Vs; s += blockDim.x) {
            const int y = s / L, e = y * ld + 2 * (s - y * L);
            *reinterpret_cast<cplx<double>*>(V + e) = cmulc(Xp[s], zq[s]);
            *reinterpret_cast<cplx<double>*>(V + image + e) = cmulc(Xq[s], zp[s]);
        }
    } else {
        for (int s = threadIdx.x; s < Vs; s += blockDim.x) {
            const int y = s / L;
            *reinterpret_cast<cplx<double>*>(V + y * ld + 2 * (s - y * L)) = X[off + s];
        }
    }
    __syncthreads();
    const int nw = (int)blockDim.x >> 6, wave = (int)threadIdx.x >> 6;
    const int nty = (2 * L + 15) / 16, ntx = (L + 7) / 8;
    for (int t = wave; t < NV * nty; t += nw) {
        double* Vv = V + (t / nty) * image;
        sp_y_tile<double, NB, !PROD>(Vv, L, 2 * L, ld, t % nty, w, [&](int jj, int c, vec4<double> v) {
            *reinterpret_cast<vec4<double>*>(Vv + jj * ld + c) = v;
        });
    }
    __syncthreads();
    for (int t = wave; t < NV * ntx; t += nw) {
        double* Vv = V + (t / ntx) * image;
        sp_x_tile<double, NB, !PROD, 1>(Vv, L, L, ld, t % ntx, w, [&](int r, int jj, vec4<double> v) {
            *reinterpret_cast<cplx<double>*>(Vv + r * ld + 2 * jj) = mk<double>(v[0], v[1]);
            *reinterpret_cast<cplx<double>*>(Vv + (r + 1) * ld + 2 * jj) = mk<double>(v[2], v[3]);
        });
    }
    __syncthreads();
    if constexpr (PROD) {
        cplx<double>* dst = out + ((int64_t)(2 * pair) * Nt + tau) * 2 * nrp;
        for (int i = threadIdx.x; i < 2 * nrp; i += blockDim.x) {
            const int e = cols[i];
            const cplx<double> a = *reinterpret_cast<const cplx<double>*>(V + e);
            const cplx<double> b = *reinterpret_cast<const cplx<double>*>(V + image + e);
            dst[i] = a;
            dst[i + (int64_t)Nt * 2 * nrp] = b;
        }
    } else {
        for (int s = threadIdx.x; s < Vs; s += blockDim.x) {
            const int y = s / L;
            out[off + s] = *reinterpret_cast<const cplx<double>*>(V + y * ld + 2 * (s - y * L));
        }
    }
}

// The tau transforms of a pass of pairs and their products.  A workgroup owns
// kCols spatial frequencies and their mirror images, a chunk of `per` pairs
// and eight blocks of 16 tau frequencies, one per wavefront.  It walks the four
// tiles A_k, B_k, A_{-k}, B_{-k} of each pair, NTL at a time in LDS (kCols
// columns of N_tau values each; the next ones loaded into registers during the
// products), and adds
//   S_k(j) = A_{-k}(-j) B_k(j) + A_k(j) B_{-k}(-j)
// over its pairs in registers: a lane's two sums P and Q (spectral.h) give
// the frequencies j and -j.  The weights stream from the L2 once per NTL tiles
// (tile by tile they bounded the kernel).  At L = 24, N_tau = 240 a pass of 40
// pairs takes 159 us, 76 of them FP64 products (1984 per pair and group of 8
// frequencies); direct sums over LDS and a separate product pass took 1319 us
// for 60 pairs.
constexpr int kCols = 8;
typedef double vec2 __attribute__((ext_vector_type(2)));

template <int NTL, int PF>
__global__ __launch_bounds__(512) void k_se_t_acc(int Nt, int nrp, int np, int per, int first,
                                                  const double* __restrict__ tab,
                                                  const cplx<double>* __restrict__ F, cplx<double>* __restrict__ Sp) {
    extern __shared__ __align__(32) unsigned char smem[];
    double* buf = reinterpret_cast<double*>(smem);
    const int lane = threadIdx.x & 63, col = lane & 15, q4 = lane >> 4;
    const int b = (int)blockIdx.z * 8 + ((int)threadIdx.x >> 6), hn = Nt / 2, steps = sp_steps(Nt);
    const bool act = b < se_blocks(Nt);
    const int p0 = (int)blockIdx.y * per, p1 = min(np, p0 + per);
    if (p0 >= p1) return;
    const double* tb = tab + (act ? (size_t)b * steps * 2 * 64 : 0) + lane;
    const int rows = hn + 1, nel = rows * kCols;
    // group t of NTL tiles, counted over the chunk: tile u of pair p0 + NTL t / 4;
    // a thread takes the points k and N_tau - k of a column
    auto fetch = [&](int t, vec2 (&lo)[NTL * PF], vec2 (&hi)[NTL * PF]) {
        const int pair = p0 + NTL * t / 4, u0 = NTL * t % 4;
#pragma unroll
        for (int v = 0; v < NTL; v++) {
            const int u = u0 + v;
            const cplx<double>* src =
                F + (int64_t)(2 * pair + (u & 1)) * Nt * 2 * nrp + (u >> 1) * nrp + (int64_t)blockIdx.x * kCols;
#pragma unroll
            for (int i = 0; i < PF; i++) {
                const int e = min((int)threadIdx.x + i * (int)blockDim.x, nel - 1), k = e / kCols;
                lo[v * PF + i] = *reinterpret_cast<const vec2*>(src + (int64_t)k * 2 * nrp + e % kCols);
                hi[v * PF + i] = *reinterpret_cast<const vec2*>(src + (int64_t)(k ? Nt - k : 0) * 2 * nrp + e % kCols);
            }
        }
    };
    // the paired terms of the products: E_k = v_k + v_{n-k} and O_k = v~_k -
    // v~_{n-k} (spectral.h), formed once for the eight wavefronts
    auto stash = [&](const vec2 (&lo)[NTL * PF], const vec2 (&hi)[NTL * PF]) {
        vec2* dst = reinterpret_cast<vec2*>(buf);
#pragma unroll
        for (int v = 0; v < NTL; v++)
#pragma unroll
            for (int i = 0; i < PF; i++) {
                const int e = (int)threadIdx.x + i * (int)blockDim.x;
                if (e >= nel) continue;
                const vec2 a = lo[v * PF + i], c = hi[v * PF + i];
                dst[2 * v * nel + e] = a + c;
                dst[(2 * v + 1) * nel + e] = vec2{a.y - c.y, a.x - c.x};
            }
    };
    const double* pt = buf + sp_row<double>(col);
    cplx<double> sj[2], sm[2];  // S at j and -j of this lane's two frequencies
#pragma unroll
    for (int c = 0; c < 2; c++) sj[c] = sm[c] = mk<double>(0.0, 0.0);
    vec2 lo[NTL * PF], hi[NTL * PF];
    fetch(0, lo, hi);
    const int ngroup = (p1 - p0) * (4 / NTL);
    for (int t0 = 0; t0 < ngroup; t0 += 4 / NTL) {
        vec4<double> P[4], Q[4];
#pragma unroll
        for (int u0 = 0; u0 < 4; u0 += NTL) {
            const int t = t0 + u0 / NTL;
            __syncthreads();  // the last group's products are done with the buffer
            stash(lo, hi);
            __syncthreads();
            if (t + 1 < ngroup) fetch(t + 1, lo, hi);  // in flight during the products
            if (!act) continue;
#pragma unroll
            for (int v = 0; v < NTL; v++)
#pragma unroll
                for (int i = 0; i < 4; i++) P[u0 + v][i] = Q[u0 + v][i] = 0.0;
            // the operands of the next step load during this step's products
            double wc = tb[0], ws = tb[64], e[NTL], o[NTL];
            auto operands = [&](int s, double (&e)[NTL], double (&o)[NTL]) {
                const int k = min(4 * s + q4, hn);  // padding points carry zero weights
#pragma unroll
                for (int v = 0; v < NTL; v++) {
                    e[v] = pt[(2 * v * rows + k) * 2 * kCols];
                    o[v] = pt[((2 * v + 1) * rows + k) * 2 * kCols];
                }
            };
            operands(0, e, o);
            for (int s = 0; s < steps; s++) {
                const int sn = min(s + 1, steps - 1);
                const double nc = tb[sn * 128], ns = tb[sn * 128 + 64];
                double en[NTL], on[NTL];
                operands(sn, en, on);
#pragma unroll
                for (int v = 0; v < NTL; v++) {
                    P[u0 + v] = sp_mfma(e[v], wc, P[u0 + v]);
                    Q[u0 + v] = sp_mfma(o[v], ws, Q[u0 + v]);
                }
                wc = nc;
                ws = ns;
#pragma unroll
                for (int v = 0; v < NTL; v++) {
                    e[v] = en[v];
                    o[v] = on[v];
                }
            }
        }
        if (act)
#pragma unroll
            for (int c = 0; c < 2; c++) {
                cplx<double> f[4], g[4];  // the four transforms at j and at -j
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const double pr = P[u][2 * c], pi = P[u][2 * c + 1], qr = Q[u][2 * c], qi = Q[u][2 * c + 1];
                    f[u] = mk<double>(pr + qr, pi - qi);
                    g[u] = mk<double>(pr - qr, pi + qi);
                }
                const cplx<double> a1 = cmul(g[2], f[1]), a2 = cmul(f[0], g[3]);
                const cplx<double> b1 = cmul(f[2], g[1]), b2 = cmul(g[0], f[3]);
                sj[c].re += a1.re + a2.re;
                sj[c].im += a1.im + a2.im;
                sm[c].re += b1.re + b2.re;
                sm[c].im += b1.im + b2.im;
            }
    }
    const int j = 16 * b + col;
    if (!act || j > hn) return;
    cplx<double>* dst = Sp + (int64_t)blockIdx.y * Nt * nrp + (int64_t)blockIdx.x * kCols + 2 * q4;
#pragma unroll
    for (int c = 0; c < 2; c++) {
        cplx<double>* a = dst + (int64_t)j * nrp + c;
        *a = first ? sj[c] : cadd(*a, sj[c]);
        if (j && j != Nt - j) {
            cplx<double>* d = dst + (int64_t)(Nt - j) * nrp + c;
            *d = first ? sm[c] : cadd(*d, sm[c]);
        }
    }
}

// S_k: the chunks' sums in order; S_{-k} = S_k.
__global__ void k_se_fold(int Nt, int Vs, int nrp, int nchunk, const int* __restrict__ colof,
                          const cplx<double>* __restrict__ Sp, cplx<double>* __restrict__ S) {
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= (int64_t)Nt * Vs) return;
    const int kt = (int)(k / Vs), ks = (int)(k - (int64_t)kt * Vs), c = colof[ks];
    const int t = c < nrp || kt == 0 ? kt : Nt - kt, r = c < nrp ? c : c - nrp;
    cplx<double> s = mk<double>(0.0, 0.0);
    for (int i = 0; i < nchunk; i++) s = cadd(s, Sp[((int64_t)i * Nt + t) * nrp + r]);
    S[k] = s;
}

// Inverse DFT along tau of KT spatial columns, staged in LDS:
// out(kt, c) = sum_tau in(tau, c) conj(tw)^{tau kt}.
__global__ __launch_bounds__(kBS) void k_se_t(int Nt, int Vs, int KT, const cplx<double>* __restrict__ in,
                                              const cplx<double>* __restrict__ tw, cplx<double>* __restrict__ out) {
    extern __shared__ unsigned char smem[];
    cplx<double>* col = reinterpret_cast<cplx<double>*>(smem);  // [Nt][KT]
    cplx<double>* w = col + (size_t)Nt * KT;
    const int c0 = blockIdx.x * KT;
    const int nc = min(KT, Vs - c0);
    for (int k = threadIdx.x; k < Nt; k += blockDim.x) {
        const cplx<double> t = tw[k];
        w[k] = mk<double>(t.re, -t.im);
    }
    for (int e = threadIdx.x; e < Nt * KT; e += blockDim.x) {
        const int tau = e / KT, c = e - tau * KT;
        col[e] = c < nc ? in[(int64_t)tau * Vs + c0 + c] : mk<double>(0.0, 0.0);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < Nt * KT; e += blockDim.x) {
        const int kt = e / KT, c = e - kt * KT;
        if (c >= nc) continue;
        cplx<double> acc = mk<double>(0.0, 0.0);
        int idx = 0;
        for (int tau = 0; tau < Nt; tau++) {
            const cplx<double> a = col[tau * KT + c], t = w[idx];
            acc.re = fma(a.re, t.re, fma(-a.im, t.im, acc.re));
            acc.im = fma(a.re, t.im, fma(a.im, t.re, acc.im));
            idx += kt;
            if (idx >= Nt) idx -= Nt;
        }
        out[(int64_t)kt * Vs + c0 + c] = acc;
    }
}

// Partial sums of sum_p sum_i X_p,i conj(xi_p,i): one per workgroup.
__global__ __launch_bounds__(kBS) void k_se_t1(int64_t total, const cplx<double>* __restrict__ X,
                                               const cplx<double>* __restrict__ xi, cplx<double>* __restrict__ part) {
    __shared__ double red[2][kBS];
    double sx = 0.0, sy = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)kBS + threadIdx.x; e < total; e += (int64_t)gridDim.x * kBS) {
        const cplx<double> t = cmulc(X[e], xi[e]);
        sx += t.re;
        sy += t.im;
    }
    red[0][threadIdx.x] = sx;
    red[1][threadIdx.x] = sy;
    __syncthreads();
    for (int h = kBS / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            red[0][threadIdx.x] += red[0][threadIdx.x + h];
            red[1][threadIdx.x] += red[1][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = mk<double>(red[0][0], red[1][0]);
}

// C = -scale_T2 * T (T: the inverse transform of S); C(0) += T1, with T1 the
// partial sums added in order and divided by n_rv N.
__global__ void k_se_finish(int64_t N, double scale_T2, int n_part, const cplx<double>* __restrict__ part,
                            double inv_t1, const cplx<double>* __restrict__ T, cplx<double>* __restrict__ C) {
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= N) return;
    cplx<double> c = mk<double>(-scale_T2 * T[k].re, -scale_T2 * T[k].im);
    if (k == 0) {
        double sx = 0.0, sy = 0.0;
        for (int j = 0; j < n_part; j++) {
            sx += part[j].re;
            sy += part[j].im;
        }
        c.re += sx * inv_t1;
        c.im += sy * inv_t1;
    }
    C[k] = c;
}

// spatial columns per workgroup of the direct tau pass (it transforms a
// single vector: narrow tiles give the chip enough workgroups; 118 -> 37 us at
// L = 24, N_tau = 240 against 16 columns)
constexpr int kTauTile = 4;

size_t xy_lds(int L, int nv) { return ((size_t)nv * L * se_ld(L) + sp_table(L, se_blocks(L))) * sizeof(double); }
size_t t_lds(int Nt) { return (size_t)(Nt * kTauTile + Nt) * sizeof(cplx<double>); }

// f.operator()<NB>() for the spatial axes (L <= 44: one or two blocks)
template <typename F>
qedhmc_status with_xy(int L, F&& f) {
    return se_blocks(L) == 1 ? f.template operator()<1>() : f.template operator()<2>();
}
// f.operator()<NTL, PF>(lds) of the tau pass: the four tiles of a pair together
// while eight blocks of frequencies hold them all (N_tau <= 254; PF pairs of
// points per thread and tile), two of them while two fit the LDS (N_tau <=
// 510), else one
template <typename F>
qedhmc_status with_acc(int Nt, F&& f) {
    const int threads = 64 * std::min(8, se_blocks(Nt)), nel = (Nt / 2 + 1) * kCols;
    const int need = (nel + threads - 1) / threads;  // point pairs per thread and tile
    const size_t tile = (size_t)2 * nel * sizeof(cplx<double>);
    if (need <= 2) return f.template operator()<4, 2>(4 * tile);
    if (need <= 4) return f.template operator()<2, 4>(2 * tile);
    return f.template operator()<1, 9>(tile);
}

qedhmc_status set_lds_attr(const void* k, size_t bytes) {
    if (bytes > 65536) QH_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    return QEDHMC_OK;
}

qedhmc_status se_fail(qedhmc_se* se, qedhmc_status st) {
    qedhmc_se_destroy(se);
    return st;
}

}  // namespace

}  // namespace qh

using namespace qh;

extern "C" {

qedhmc_status qedhmc_se_create(const qedhmc_params* params, int32_t n_rv, void* stream, qedhmc_se_t* out) {
    if (!params || !out) {
        set_error("se: null argument");
        return QEDHMC_EINVAL;
    }
    *out = nullptr;
    QH_TRY(check_params(params));
    const int64_t N = (int64_t)params->L * params->L * params->Nt;
    if (n_rv < 2 || (int64_t)n_rv * N >= ((int64_t)1 << 32)) {
        set_error("se: need 2 <= n_rv and n_rv * L^2 * Nt < 2^32");
        return QEDHMC_EINVAL;
    }
    if (params->L > 44) {
        set_error("se: the multi-RHS CG holds a slice in one workgroup group of at most 256 threads (L <= 44)");
        return QEDHMC_EUNSUPPORTED;
    }
    qedhmc_se* se = new (std::nothrow) qedhmc_se{};
    if (!se) return QEDHMC_ENOMEM;
    se->p = *params;
    se->n_rv = n_rv;
    se->N = N;
    se->L = params->L;
    se->Nt = params->Nt;
    se->Vs = params->L * params->L;
    se->stream = (hipStream_t)stream;
    int dev = 0;
    int lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
        return se_fail(se, hip_fail(hipGetLastError(), "se: device attributes"));
    // (the tau pass keeps N_tau <= 1137: kCols columns of FP64 values and a
    // twiddle table within a workgroup's LDS)
    if (xy_lds(se->L, 2) > (size_t)lds || (size_t)(se->Nt * kCols + se->Nt) * sizeof(cplx<double>) > (size_t)lds) {
        set_error("se: transform tiles exceed the LDS of a workgroup");
        return se_fail(se, QEDHMC_EUNSUPPORTED);
    }
    qedhmc_status st = batch_create_shared(*params, n_rv, stream, &se->b);
    if (st != QEDHMC_OK) return se_fail(se, st);
    const int64_t npairs = (int64_t)n_rv * (n_rv - 1) / 2;
    // columns: representatives of {k, -k}, then the mirror images
    const int L = se->L, Vs = se->Vs, Nt = se->Nt;
    std::vector<int> rep;
    for (int k = 0; k < Vs; k++) {
        const int m = (L - k / L) % L * L + (L - k % L) % L;
        if (k <= m) rep.push_back(k);
    }
    se->nrp = ((int)rep.size() + kCols - 1) / kCols * kCols;
    const size_t pairs_at = (size_t)2 * se->nrp + Vs + (Vs & 1);
    std::vector<int> cols(pairs_at, 0);
    const int ld = se_ld(L);
    auto place = [&](int k) { return k / L * ld + 2 * (k % L); };
    for (size_t r = 0; r < rep.size(); r++) {
        const int k = rep[r], m = (L - k / L) % L * L + (L - k % L) % L;
        cols[r] = place(k);
        cols[se->nrp + r] = place(m);
        cols[2 * se->nrp + m] = se->nrp + (int)r;
        cols[2 * se->nrp + k] = (int)r;
    }
    for (int p = 0; p < n_rv; p++)
        for (int q = p + 1; q < n_rv; q++) {
            cols.push_back(p);
            cols.push_back(q);
        }
    // a pass: as many pairs as keep the spatial transforms within kWorkBytes,
    // in whole chunks
    int ncu = 256;
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    const int groups = se->nrp / kCols * ((se_blocks(Nt) + 7) / 8);
    const int64_t pair_bytes = (int64_t)2 * Nt * 2 * se->nrp * sizeof(cplx<double>);
    se->P = (int)std::max<int64_t>(1, std::min<int64_t>(npairs, kWorkBytes / pair_bytes));
    // QEDHMC_SE_PAIRS (tuning and tests): at most this many pairs per pass
    if (const char* e = std::getenv("QEDHMC_SE_PAIRS"))
        if (std::atoi(e) > 0) se->P = std::min(se->P, std::atoi(e));
    // (a workgroup fills a compute unit's LDS: the chunks that leave the
    // fewest units idle in the last of one to three rounds)
    double best = 0.0;
    for (int rounds = 1; rounds <= 3; rounds++) {
        const int c = std::max(1, rounds * ncu / groups);
        const double use = (double)c * groups / (((int64_t)c * groups + ncu - 1) / ncu * ncu);
        if (use > best + 0.01) {
            best = use;
            se->nchunk = c;
        }
    }
    se->nchunk = std::min(se->P, se->nchunk);
    se->per = se->P / se->nchunk;
    se->P = se->per * se->nchunk;
    se->n_part = 1024;
    const size_t nL = sp_table(L, se_blocks(L)), nT = sp_table(Nt, se_blocks(Nt));
    bool ok = hipMalloc(&se->rhs, (size_t)n_rv * N * sizeof(cplx<double>)) == hipSuccess;
    ok = ok && hipMalloc(&se->ws, (size_t)se->P * pair_bytes) == hipSuccess;
    ok = ok && hipMalloc(&se->S, (size_t)2 * N * sizeof(cplx<double>)) == hipSuccess;
    ok = ok && hipMalloc(&se->Sp, (size_t)se->nchunk * Nt * se->nrp * sizeof(cplx<double>)) == hipSuccess;
    ok = ok && hipMalloc(&se->T, (size_t)N * sizeof(cplx<double>)) == hipSuccess;
    ok = ok && hipMalloc(&se->tabL, nL * sizeof(double)) == hipSuccess;
    ok = ok && hipMalloc(&se->tabT, nT * sizeof(double)) == hipSuccess;
    ok = ok && hipMalloc(&se->cols, cols.size() * sizeof(int)) == hipSuccess;
    ok = ok && hipMalloc(&se->twT, (size_t)se->Nt * sizeof(cplx<double>)) == hipSuccess;
    ok = ok && hipMalloc(&se->part, (size_t)se->n_part * sizeof(cplx<double>)) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        set_error("se: device allocation failed");
        return se_fail(se, QEDHMC_ENOMEM);
    }
    std::vector<double> tab(std::max(nL, nT));
    hipError_t e = hipMemcpyAsync(se->cols, cols.data(), cols.size() * sizeof(int), hipMemcpyHostToDevice, se->stream);
    sp_fill_table<double>(L, se_blocks(L), tab.data());
    if (e == hipSuccess)
        e = hipMemcpyAsync(se->tabL, tab.data(), nL * sizeof(double), hipMemcpyHostToDevice, se->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(se->stream);  // the host tables are reused and die here
    sp_fill_table<double>(Nt, se_blocks(Nt), tab.data());
    if (e == hipSuccess)
        e = hipMemcpyAsync(se->tabT, tab.data(), nT * sizeof(double), hipMemcpyHostToDevice, se->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(se->stream);
    if (e != hipSuccess) return se_fail(se, hip_fail(e, "se: transform tables"));
    st = with_xy(L, [&]<int NB>() -> qedhmc_status {
        QH_TRY(set_lds_attr((const void*)k_se_xy<NB, true>, xy_lds(L, 2)));
        return set_lds_attr((const void*)k_se_xy<NB, false>, xy_lds(L, 1));
    });
    if (st == QEDHMC_OK)
        st = with_acc(Nt, [&]<int NTL, int PF>(size_t bytes) -> qedhmc_status {
            return set_lds_attr((const void*)k_se_t_acc<NTL, PF>, std::max<size_t>(bytes, 65537));
        });
    if (st == QEDHMC_OK) st = set_lds_attr((const void*)k_se_t, t_lds(Nt));
    if (st != QEDHMC_OK) return se_fail(se, st);
    hipLaunchKernelGGL(k_se_twiddle, dim3((se->Nt + 255) / 256), dim3(256), 0, se->stream, se->Nt, se->twT);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(se->stream) != hipSuccess)
        return se_fail(se, hip_fail(hipGetLastError(), "se: twiddle tables"));
    *out = se;
    return QEDHMC_OK;
}

qedhmc_status qedhmc_se_destroy(qedhmc_se_t se) {
    if (!se) return QEDHMC_OK;
    if (se->b) qedhmc_batch_destroy(se->b);
    for (void* ptr : {(void*)se->rhs, (void*)se->ws, (void*)se->S, (void*)se->Sp, (void*)se->T, (void*)se->tabL,
                      (void*)se->tabT, (void*)se->cols, (void*)se->twT, (void*)se->part})
        if (ptr) (void)hipFree(ptr);
    delete se;
    return QEDHMC_OK;
}

qedhmc_status qedhmc_se_probes(qedhmc_se_t se, uint64_t meas_index, double* xi_all) {
    if (!se || !xi_all) {
        set_error("se: null argument");
        return QEDHMC_EINVAL;
    }
    const uint32_t total = (uint32_t)((int64_t)se->n_rv * se->N);
    const int grid = (int)std::min<int64_t>(((int64_t)total + 255) / 256, 8192);
    hipLaunchKernelGGL(k_se_probes, dim3(grid), dim3(256), 0, se->stream, se->p.seed, meas_index, total,
                       reinterpret_cast<cplx<double>*>(xi_all));
    QH_HIP(hipGetLastError());
    return QEDHMC_OK;
}

qedhmc_status qedhmc_se_solve(qedhmc_se_t se, const double* theta, const double* xi_all, double* X_all, double tol,
                              int32_t maxit, qedhmc_precision prec, int32_t* iters, double* true_rel) {
    if (!se || !theta || !xi_all || !X_all || !iters || !true_rel) {
        set_error("se: null argument");
        return QEDHMC_EINVAL;
    }
    if (xi_all == X_all) {
        set_error("se: xi and X alias");
        return QEDHMC_EINVAL;
    }
    if (!(tol > 0.0) || maxit < 1 || (prec != QEDHMC_FP64 && prec != QEDHMC_FP32)) {
        set_error("se: bad solver arguments");
        return QEDHMC_EINVAL;
    }
    // R_p = M^dag xi_p on the batch's stream (ordered after the caller's work)
    QH_TRY(batch_enter(se->b));
    qedhmc_ctx* h0 = batch_ctx0(se->b);
    QH_TRY(ensure_gauge(h0, theta, QEDHMC_FP64));
    for (int k = 0; k < se->n_rv; k++)
        QH_TRY(launch_apply_M(h0, QEDHMC_FP64, xi_all + 2 * se->N * k, se->rhs + se->N * k, 1));
    return batch_solve_shared(se->b, theta, reinterpret_cast<const double*>(se->rhs), X_all, tol, maxit, prec, iters,
                              true_rel);
}

qedhmc_status qedhmc_se_spin_correlator(qedhmc_se_t se, const double* xi_all, const double* X_all, double* C_out) {
    if (!se || !xi_all || !X_all || !C_out) {
        set_error("se: null argument");
        return QEDHMC_EINVAL;
    }
    const int64_t N = se->N;
    const int n = se->n_rv;
    const cplx<double>* xi = reinterpret_cast<const cplx<double>*>(xi_all);
    const cplx<double>* X = reinterpret_cast<const cplx<double>*>(X_all);
    cplx<double>* C = reinterpret_cast<cplx<double>*>(C_out);
    const int eg = (int)((N + 255) / 256);
    hipLaunchKernelGGL(k_se_t1, dim3(se->n_part), dim3(kBS), 0, se->stream, (int64_t)n * N, X, xi, se->part);
    QH_HIP(hipGetLastError());
    const int L = se->L, Nt = se->Nt, Vs = se->Vs, nrp = se->nrp, ld = se_ld(L);
    const int2* pairs = reinterpret_cast<const int2*>(se->cols + 2 * nrp + Vs + (Vs & 1));
    const int npairs = n * (n - 1) / 2;
    const int nty = (2 * L + 15) / 16;
    auto spatial = [&]<bool PROD>(int t0, int np, const cplx<double>* in, cplx<double>* out) -> qedhmc_status {
        return with_xy(L, [&]<int NB>() -> qedhmc_status {
            const int nv = PROD ? 2 : 1;
            hipLaunchKernelGGL((k_se_xy<NB, PROD>), dim3(8 * ((Nt + 7) / 8) * np), dim3(64 * std::min(8, nv * nty)),
                               xy_lds(L, nv), se->stream, L, ld, Nt, N, pairs + t0, np, nrp, in, xi, se->tabL,
                               se->cols, out);
            QH_HIP(hipGetLastError());
            return QEDHMC_OK;
        });
    };
    int nchunk = 0;
    for (int t0 = 0; t0 < npairs; t0 += se->P) {
        const int np = std::min(se->P, npairs - t0);
        QH_TRY(spatial.template operator()<true>(t0, np, X, se->ws));
        const int nc = (np + se->per - 1) / se->per;
        nchunk = std::max(nchunk, nc);
        QH_TRY(with_acc(Nt, [&]<int NTL, int PF>(size_t bytes) -> qedhmc_status {
            hipLaunchKernelGGL((k_se_t_acc<NTL, PF>), dim3(nrp / kCols, nc, (se_blocks(Nt) + 7) / 8),
                               dim3(64 * std::min(8, se_blocks(Nt))), bytes, se->stream, Nt, nrp, np, se->per,
                               t0 == 0 ? 1 : 0, se->tabT, se->ws, se->Sp);
            QH_HIP(hipGetLastError());
            return QEDHMC_OK;
        }));
    }
    hipLaunchKernelGGL(k_se_fold, dim3(eg), dim3(256), 0, se->stream, Nt, Vs, nrp, nchunk, se->cols + 2 * nrp, se->Sp,
                       se->S);
    // T(Delta) = sum_k S_k e^{+i k.Delta}
    QH_TRY(spatial.template operator()<false>(0, 1, se->S, se->S + N));
    hipLaunchKernelGGL(k_se_t, dim3((Vs + kTauTile - 1) / kTauTile), dim3(kBS), t_lds(Nt), se->stream, Nt, Vs, kTauTile,
                       se->S + N, se->twT, se->T);
    QH_HIP(hipGetLastError());
    const double scale = 1.0 / ((double)n * (double)(n - 1) * (double)N * (double)N);
    hipLaunchKernelGGL(k_se_finish, dim3(eg), dim3(256), 0, se->stream, N, scale, se->n_part, se->part,
                       1.0 / ((double)n * (double)N), se->T, C);
    QH_HIP(hipGetLastError());
    return QEDHMC_OK;
}

}  // extern "C"
