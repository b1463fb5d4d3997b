// DFTs on the matrix cores (the paper preconditioner's spectral form, pcg.hip;
// the spin correlator's transforms, se.hip) and the preconditioner's banded
// tau sum.
//
// A slice of a site vector is a matrix of L rows (y) of 2 L reals (x, re/im
// interleaved).  Its momentum form on the two-site cell (2 in x, 1 in y) is
// [ny][nx][parity] complex: the two parity values of a momentum are adjacent,
// as the 2x2 blocks of the tau sum read them.  Both axes are direct DFTs
// written as real matrix products:
//   out(j) = sum_k v_k (cos(2 pi j k / n) -+ i sin(2 pi j k / n)),
// with the terms k and n - k added before the product (cos is even in k, sin
// odd) and the outputs j and n - j formed from the same two sums,
//   P(j) = sum_{k <= n/2} C(j,k) (v_k + v_{n-k}),
//   Q(j) = sum_{k <= n/2} S(j,k) w_k,  w = v~_k - v~_{n-k}, v~ = (im, re),
//   out(j) = P + s Q, out(n - j) = P - s Q, s = + for re and - for im
// (forward e^{-i}; opposite for the inverse), a quarter of the products of
// the plain DFT matrix.  Self-paired k (0, and n/2 for even n) carry half the
// weight in C.  The products are v_mfma_f32_16x16x4f32 and
// v_mfma_f64_16x16x4f64 (full precision operands and accumulation): the data
// is the A operand (16 reals along the untransformed axis x 4 points), the
// weights the B operand (4 points x 16 outputs), packed in fragment order.
#pragma once
#include <cmath>
#include <vector>

#include "qedhmc_internal.h"

namespace qh {

template <typename R>
struct vec4_of;
template <>
struct vec4_of<float> {
    typedef float type __attribute__((ext_vector_type(4)));
};
template <>
struct vec4_of<double> {
    typedef double type __attribute__((ext_vector_type(4)));
};
template <typename R>
using vec4 = typename vec4_of<R>::type;

// D += A B (16x4 by 4x16).  Lane l holds A[sp_row(l % 16)][l / 16],
// B[l / 16][l % 16] and, in element i, D[4 (l / 16) + i][l % 16]: the FP64
// instruction keeps row 4 i + l / 16 in element i, so its A rows are dealt
// out permuted (sp_row) and both precisions read the same layout.
__device__ __forceinline__ vec4<float> sp_mfma(float a, float b, vec4<float> c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ vec4<double> sp_mfma(double a, double b, vec4<double> c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <typename R>
__device__ __forceinline__ int sp_row(int m) {
    return sizeof(R) == 8 ? (m & 3) * 4 + (m >> 2) : m;
}

constexpr int kSpTau = QEDHMC_PC_TAU_REACH;  // tau offsets of P at most, either way

// fragments of a table of n points in NT blocks of 16 outputs: [block][step][C, S][lane]
__host__ __device__ constexpr int sp_steps(int n) { return n / 2 / 4 + 1; }
__host__ __device__ constexpr int sp_table(int n, int nt) { return nt * sp_steps(n) * 2 * 64; }

// Weights of n points in nt blocks in the fragment order of sp_tile: cos and
// sin of 2 pi j k / n at k = 4 step + lane / 16, j = 16 block + lane % 16, both
// up to n / 2 (zero beyond); half the cosine at a k paired with itself.  The
// angles are formed in extended precision and every FP64 entry is rounded once: with
// angles rounded to FP64 the correlator's error was up to 1.24 times that of
// direct sums over such twiddles (22 x 22 x 101, 10 probes: 3.6e-15 of its RMS
// away from the coincident point), now it is below it (1.9e-15, direct 3.0e-15).
template <typename R>
inline void sp_fill_table(int n, int nt, R* t) {
    const int steps = sp_steps(n);
    std::vector<double> cs(n), sn(n);
    for (int m = 0; m < n; m++) {
        const long double a = 8 * std::atan(1.0L) * m / n;
        cs[m] = (double)std::cos(a);
        sn[m] = (double)std::sin(a);
    }
    for (int b = 0; b < nt; b++)
        for (int s = 0; s < steps; s++)
            for (int l = 0; l < 64; l++) {
                const int k = 4 * s + l / 16, j = 16 * b + l % 16;
                const bool on = k <= n / 2 && j <= n / 2;
                const int m = on ? (int)((long)j * k % n) : 0;
                const double w = (k == 0 || 2 * k == n) ? 0.5 : 1.0;
                R* f = t + (size_t)((b * steps + s) * 2) * 64 + l;
                f[0] = on ? (R)(w * cs[m]) : R(0);
                f[64] = on && w == 1.0 ? (R)sn[m] : R(0);
            }
}

struct PcSpecGeo {
    int L, Lh, Nt, Vs, nk;
    int reach;  // tau offsets of P: -reach .. reach
    int ld;     // reals per row of the LDS image of a slice
    int ty, tx; // reals of the y and the x table
};

// Reals per LDS row of a slice of 2 L reals: a multiple of 4 (whole quads)
// that puts four consecutive rows into different quarters of the banks (the A
// operand reads 16 reals of four rows at once).
__host__ __device__ inline int sp_ld(int L) {
    int s = (2 * L + 15) / 16 * 16;
    return (s / 16) % 2 ? s : s + 16;
}

// P and Q of one tile of 16 reals: pt points at this lane's complex value of
// point 0 (its row permuted by sp_row), consecutive points `stride` reals
// apart; part: the lane's real is the imaginary one.
template <typename R, int NT>
__device__ __forceinline__ void sp_tile(const R* pt, int stride, int n, int part, const R* tab, vec4<R> (&P)[NT],
                                        vec4<R> (&Q)[NT]) {
    const int lane = threadIdx.x & 63, g = lane >> 4, hn = n >> 1, steps = sp_steps(n);
#pragma unroll
    for (int b = 0; b < NT; b++)
#pragma unroll
        for (int i = 0; i < 4; i++) P[b][i] = Q[b][i] = R(0);
    // (one step at a time: batches of four steps measured 91 against 81 us for
    // P at L = 66, where the padding of the last batch costs LDS reads)
    for (int s = 0; s < steps; s++) {
        int k = 4 * s + g;
        k = k <= hn ? k : 0;  // padding points carry zero weights
        const int m = k ? n - k : 0;
        const cplx<R> a = *reinterpret_cast<const cplx<R>*>(pt + k * stride);
        const cplx<R> c = *reinterpret_cast<const cplx<R>*>(pt + m * stride);
        const R e = part ? a.im + c.im : a.re + c.re;
        const R o = part ? a.re - c.re : a.im - c.im;
#pragma unroll
        for (int b = 0; b < NT; b++) {
            const R* t = tab + (size_t)((b * steps + s) * 2) * 64 + lane;
            P[b] = sp_mfma(e, t[0], P[b]);
            Q[b] = sp_mfma(o, t[64], Q[b]);
        }
    }
}

// One tile along the rows of an image with n rows of `cols` reals, `ld` reals
// apart: 16 columns, V[k][c] -> j.  emit(j, c, quad) takes four consecutive
// reals of output row j (default: back into the image).
template <typename R, int NT, bool INV, typename Emit>
__device__ __forceinline__ void sp_y_tile(const R* V, int n, int cols, int ld, int t, const R* tab, Emit emit) {
    const int lane = threadIdx.x & 63, q = lane >> 4, col = lane & 15;
    const int c = min(16 * t + sp_row<R>(col), cols - 1);
    vec4<R> P[NT], Q[NT];
    sp_tile<R, NT>(V + (c & ~1), ld, n, c & 1, tab, P, Q);
    const int c0 = 16 * t + 4 * q;  // this lane's four consecutive outputs start at an even real
    if (c0 < cols)
#pragma unroll
        for (int b = 0; b < NT; b++) {
            const int j = 16 * b + col;
            if (j > n / 2) continue;
            vec4<R> u, w;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const R s = ((i & 1) != 0) != INV ? -Q[b][i] : Q[b][i];
                u[i] = P[b][i] + s;
                w[i] = P[b][i] - s;
            }
            emit(j, c0, u);
            if (j && j != n - j) emit(n - j, c0, w);
        }
}

// One tile along a row: G interleaved sequences of n complex values (the
// parity planes, G = 2, or a plain row, G = 1), 8 / G rows.  emit(r, j, quad)
// takes the four reals of (row r, point j) for G = 2, of (rows r and r + 1,
// point j) for G = 1.
template <typename R, int NT, bool INV, int G, typename Emit>
__device__ __forceinline__ void sp_x_tile(const R* V, int n, int rows, int ld, int t, const R* tab, Emit emit) {
    const int lane = threadIdx.x & 63, q = lane >> 4, col = lane & 15;
    const int m = sp_row<R>(col);
    const int r = min((8 / G) * t + m / (2 * G), rows - 1);
    vec4<R> P[NT], Q[NT];
    sp_tile<R, NT>(V + r * ld + (m & (2 * G - 2)), 2 * G, n, m & 1, tab, P, Q);
    const int ro = (8 / G) * t + q * 2 / G;
    if (ro < rows)
#pragma unroll
        for (int b = 0; b < NT; b++) {
            const int j = 16 * b + col;
            if (j > n / 2) continue;
            vec4<R> u, w;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const R s = ((i & 1) != 0) != INV ? -Q[b][i] : Q[b][i];
                u[i] = P[b][i] + s;
                w[i] = P[b][i] - s;
            }
            emit(ro, j, u);
            if (j && j != n - j) emit(ro, n - j, w);
        }
}

// All tiles of a slice image by the workgroup's wavefronts in turn.  A tile
// reads and writes its own columns (rows) alone, so in-place emits need no
// barrier within an axis.
template <typename R, int NT, bool INV, typename Emit>
__device__ __forceinline__ void sp_dft_y(const R* V, const PcSpecGeo& g, const R* tab, Emit emit) {
    const int nw = (int)blockDim.x >> 6, cols = 2 * g.L, ntile = (cols + 15) >> 4;
    for (int t = (int)threadIdx.x >> 6; t < ntile; t += nw) sp_y_tile<R, NT, INV>(V, g.L, cols, g.ld, t, tab, emit);
}
template <typename R, int NT, bool INV, typename Emit>
__device__ __forceinline__ void sp_dft_x(const R* V, const PcSpecGeo& g, const R* tab, Emit emit) {
    const int nw = (int)blockDim.x >> 6, ntile = (g.L + 3) >> 2;
    for (int t = (int)threadIdx.x >> 6; t < ntile; t += nw)
        sp_x_tile<R, NT, INV, 2>(V, g.Lh, g.L, g.ld, t, tab, emit);
}

// The slice image V (sites) to momentum planes at dst ([ny][nx][parity], 16
// byte aligned scratch).  The workgroup has stored V and not yet synchronised.
template <typename R, int NY, int NX>
__device__ __forceinline__ void sp_forward(R* V, const PcSpecGeo& g, const R* tabs, cplx<R>* dst) {
    __syncthreads();
    sp_dft_y<R, NY, false>(V, g, tabs, [&](int j, int c, vec4<R> v) {
        *reinterpret_cast<vec4<R>*>(V + j * g.ld + c) = v;
    });
    __syncthreads();
    sp_dft_x<R, NX, false>(V, g, tabs + g.ty, [&](int r, int j, vec4<R> v) {
        *reinterpret_cast<vec4<R>*>(dst + 2 * (r * g.Lh + j)) = v;
    });
}

// The momentum image V back to the sites of a slice at dst (element aligned:
// a caller's vector).
template <typename R, int NY, int NX>
__device__ __forceinline__ void sp_inverse(R* V, const PcSpecGeo& g, const R* tabs, cplx<R>* dst) {
    __syncthreads();
    sp_dft_x<R, NX, true>(V, g, tabs + g.ty, [&](int r, int j, vec4<R> v) {
        *reinterpret_cast<vec4<R>*>(V + r * g.ld + 4 * j) = v;
    });
    __syncthreads();
    sp_dft_y<R, NY, true>(V, g, tabs, [&](int j, int c, vec4<R> v) {
        cplx<R>* o = dst + (size_t)j * g.L + (c >> 1);
        o[0] = mk<R>(v[0], v[1]);
        o[1] = mk<R>(v[2], v[3]);
    });
}

// The tables: staged in LDS (TL; before the first barrier) or read through
// the caches.
template <typename R, bool TL>
__device__ __forceinline__ const R* sp_tables(const R* __restrict__ tab, R* lds, const PcSpecGeo& g) {
    if constexpr (TL) {
        const int n4 = (g.ty + g.tx) / 4;
        for (int i = threadIdx.x; i < n4; i += blockDim.x)
            reinterpret_cast<vec4<R>*>(lds)[i] = reinterpret_cast<const vec4<R>*>(tab)[i];
        return lds;
    } else {
        return tab;
    }
}

// acc += m v and acc += conj(m) v (complex), four FMAs
template <typename R>
__device__ __forceinline__ void v_cmac(cplx<R>& acc, cplx<R> m, cplx<R> v) {
    acc.re = fma(m.re, v.re, acc.re);
    acc.re = fma(-m.im, v.im, acc.re);
    acc.im = fma(m.re, v.im, acc.im);
    acc.im = fma(m.im, v.re, acc.im);
}
template <typename R>
__device__ __forceinline__ void v_cmacc(cplx<R>& acc, cplx<R> m, cplx<R> v) {
    acc.re = fma(m.re, v.re, acc.re);
    acc.re = fma(m.im, v.im, acc.re);
    acc.im = fma(m.re, v.im, acc.im);
    acc.im = fma(-m.im, v.re, acc.im);
}

// The two parity values of a momentum.
template <typename R>
struct alignas(16) cpair {
    cplx<R> a, b;
};

// H is Hermitian block by block (H(k, -a) = H(k, a)^dagger), so only the
// offsets a = 0 .. reach are kept, H[a][row][k] = (H_row0, H_row1): one block
// serves the slices tau + a and tau - a.
// z += H v (slice tau + a)
template <typename R>
__device__ __forceinline__ void sp_up(cpair<R>& z, const cpair<R>& h0, const cpair<R>& h1, const cpair<R>& v) {
    v_cmac(z.a, h0.a, v.a);
    v_cmac(z.a, h0.b, v.b);
    v_cmac(z.b, h1.a, v.a);
    v_cmac(z.b, h1.b, v.b);
}
// z += H^dagger v (slice tau - a)
template <typename R>
__device__ __forceinline__ void sp_down(cpair<R>& z, const cpair<R>& h0, const cpair<R>& h1, const cpair<R>& v) {
    v_cmacc(z.a, h0.a, v.a);
    v_cmacc(z.a, h1.a, v.b);
    v_cmacc(z.b, h0.b, v.a);
    v_cmacc(z.b, h1.b, v.b);
}
template <typename R>
__device__ __forceinline__ cpair<R> sp_signed(R s, const cpair<R>& v) {
    return {mk<R>(s * v.a.re, s * v.a.im), mk<R>(s * v.b.re, s * v.b.im)};
}

}  // namespace qh
