// Training kernels of the learned preconditioner on the matrix cores, FP32
// operands and accumulation throughout (v_mfma_f32_16x16x4f32): forward of
// every layer, data gradient of the hidden layers, weight gradients.
//
// Convolutions: per tap the product [16 sites x Cin] x [Cin x Cout].  The lane
// of k-group q holds channels q Cin/4 + kk of its site at K step kk, and the
// weights are packed in the matching fragment order, frag[k][ob][kk / 4][lane]
// [kk % 4] (Cin = 32; [k][ob][lane][kk] for the 8 channels of the feature
// map) = Wt_k[q Cin/4 + kk][16 ob + lane % 16], Wt_k = W_k ([in][out], forward)
// or W_k^T (data gradient, whose tap offsets are mirrored).  One workgroup of
// 16 wavefronts per compute unit stages a layer's weights in LDS once and
// walks tiles of 16 sites, dealt to the XCDs in contiguous ranges; a tile's 27
// taps are unrolled, the rows of the next tap in flight during the products.
//
// Weight gradients: dW_k = A_k^T G with K = sites.  A workgroup stages a brick
// of sites of one slice (the input with a halo of one site all round, the
// output gradient without) in LDS, so a tap is a constant LDS offset, and adds
// the products of its bricks in registers; one partial per workgroup, summed
// in a fixed order.
#include <algorithm>

#include "net_internal.h"

namespace qh {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

static constexpr int kConvThreads = 1024;
static constexpr int kAhead = 2;  // taps whose rows are requested ahead

// floats of a packed layer
static constexpr size_t conv_frag(int cin, int coutb) { return (size_t)27 * coutb * (cin / 4) * 64; }
// first layer, four hidden layers forward, last layer, four hidden layers transposed
static constexpr size_t kFragFirst = conv_frag(8, 2), kFragHidden = conv_frag(32, 2), kFragLast = conv_frag(32, 1);
static constexpr int kHidden = 4;

size_t net_f32_weight_elems() { return kFragFirst + 2 * kHidden * kFragHidden + kFragLast; }

static size_t frag_at(int l, bool transpose) {
    if (l == 0) return 0;
    if (transpose) return kFragFirst + (kHidden + l - 1) * kFragHidden;
    if (l < kNetLayers - 1) return kFragFirst + (l - 1) * kFragHidden;
    return kFragFirst + 2 * kHidden * kFragHidden;
}

// W: device layout [27][cin][cout] of one layer; CIN the padded input channels
template <int CIN>
__global__ void k_pack_conv(const float* __restrict__ W, int cin, int cout, int coutb, int transpose,
                            float* __restrict__ out) {
    constexpr int KK = CIN / 4, V = KK < 4 ? KK : 4;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 27 * coutb * KK * 64) return;
    const int kk = i % V + V * ((i / (V * 64)) % (KK / V)), lane = (i / V) % 64;
    const int ob = (i / (64 * KK)) % coutb, k = i / (64 * KK * coutb);
    const int row = KK * (lane >> 4) + kk, col = 16 * ob + (lane & 15);
    const int ci = transpose ? col : row, co = transpose ? row : col;
    out[i] = ci < cin && co < cout ? W[((size_t)k * cin + ci) * cout + co] : 0.0f;
}

enum { CONV_HIDDEN = 0, CONV_FIRST = 1, CONV_LAST = 2, CONV_DGRAD = 3 };

// CONV_HIDDEN / FIRST: pre = conv(in) + b (nullable), out = SiLU(pre); FIRST
// reads the feature map [N][8], its residual channels 4 and 5 sign-flipped
// where the tap wraps in tau.  LAST: out = pre = conv(in) + b, two channels.
// DGRAD: out = conv^T(in = the output gradient) * SiLU'(pre_prev).
//
// Bound by the products (a hidden layer at N = 138240: 7.6 GFLOP, 50 us at the
// FP32 matrix rate; 83 us measured, of which about 15 are the launch, the
// weights and the last tiles, and 10 loads from the L2).  Two 16-site tiles per
// wavefront and 512 sites per workgroup gave 270 workgroups to 256 compute
// units, two rounds for 1.05: 167 us.  First layer 69 us on the vector ALUs,
// 31 us here; last layer 73 and 61 us.
template <int MODE>
__global__ __launch_bounds__(kConvThreads) void k_conv_train(NetGeo g, int ntile, const float* __restrict__ in,
                                                             const float* __restrict__ wfrag,
                                                             const float* __restrict__ bias,
                                                             const float* __restrict__ pre_prev,
                                                             float* __restrict__ pre, float* __restrict__ out) {
    constexpr int CIN = MODE == CONV_FIRST ? 8 : 32, OB = MODE == CONV_LAST ? 1 : 2, KK = CIN / 4;
    constexpr int NV = CIN == 32 ? 2 : 1;  // vector loads per site and lane
    constexpr int FR = 27 * OB * KK * 64;
    extern __shared__ __align__(16) float sW[];
    {
        constexpr int N4 = FR / 4, IT = (N4 + kConvThreads - 1) / kConvThreads;
        f32x4 v[IT];
#pragma unroll
        for (int i = 0; i < IT; i++) {
            const int e = (int)threadIdx.x + i * kConvThreads;
            v[i] = reinterpret_cast<const f32x4*>(wfrag)[e < N4 ? e : 0];
        }
#pragma unroll
        for (int i = 0; i < IT; i++) {
            const int e = (int)threadIdx.x + i * kConvThreads;
            if (e < N4) reinterpret_cast<f32x4*>(sW)[e] = v[i];
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane & 15, kq = lane >> 4;
    const int wgs = (int)gridDim.x >> 3, per = (ntile + 7) >> 3, xcd = (int)blockIdx.x & 7;
    for (int t = wave * wgs + ((int)blockIdx.x >> 3); t < per; t += wgs * (kConvThreads / 64)) {
        const int tile = xcd * per + t;
        if (tile >= ntile) break;
        const int site0 = 16 * tile;
        // this lane's A row: its neighbours' slice, row and column offsets per
        // direction (d = 0, 1, 2 for the tap's -1, 0, +1)
        int ot[3], oy[3], ox[3];
        float sg[3];
        {
            int st, sy, sx;
            site_of(g, min(site0 + row, g.N - 1), st, sy, sx);
#pragma unroll
            for (int d = 0; d < 3; d++) {
                const int s = MODE == CONV_DGRAD ? 1 - d : d - 1;
                ot[d] = wrap(st + s, g.Nt) * g.Vs;
                oy[d] = wrap(sy + s, g.L) * g.L;
                ox[d] = wrap(sx + s, g.L);
                sg[d] = MODE == CONV_FIRST && kq == 2 && (st + s < 0 || st + s >= g.Nt) ? -1.0f : 1.0f;
            }
        }
        const float* inq = in + KK * kq;
        float a[kAhead + 1][KK];
        auto load = [&](int k, float (&v)[KK]) {
            const unsigned m = (unsigned)(ot[k / 9] + oy[k / 3 % 3] + ox[k % 3]);
            const float* src = inq + (size_t)m * CIN;
            if constexpr (CIN == 32) {
                const f32x4 x = reinterpret_cast<const f32x4*>(src)[0], y = reinterpret_cast<const f32x4*>(src)[1];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    v[i] = x[i];
                    v[4 + i] = y[i];
                }
            } else {
                const f32x2 x = *reinterpret_cast<const f32x2*>(src);
                v[0] = sg[k / 9] * x[0];
                v[1] = sg[k / 9] * x[1];
            }
        };
        f32x4 acc[OB];
#pragma unroll
        for (int ob = 0; ob < OB; ob++) acc[ob] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < kAhead; k++) load(k, a[k]);
#pragma unroll
        for (int k = 0; k < 27; k++) {
            if (k + kAhead < 27) load(k + kAhead, a[(k + kAhead) % (kAhead + 1)]);  // in flight during the products
#pragma unroll
            for (int h = 0; h < NV; h++) {
                constexpr int V = KK / NV;
                float b[OB][V];
#pragma unroll
                for (int ob = 0; ob < OB; ob++) {
                    const float* w = sW + ((size_t)(k * OB + ob) * NV + h) * 64 * V + lane * V;
#pragma unroll
                    for (int i = 0; i < V; i++) b[ob][i] = w[i];
                }
#pragma unroll
                for (int i = 0; i < V; i++)
#pragma unroll
                    for (int ob = 0; ob < OB; ob++)
                        acc[ob] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k % (kAhead + 1)][h * V + i], b[ob][i], acc[ob], 0, 0, 0);
            }
        }
        // D fragment: lane holds sites 4 (lane / 16) + i, channel 16 ob + lane % 16
#pragma unroll
        for (int ob = 0; ob < OB; ob++) {
            const int c = 16 * ob + row;
            if (MODE == CONV_LAST && c >= 2) continue;
            const float bc = MODE == CONV_DGRAD ? 0.0f : bias[c];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int site = site0 + 4 * kq + i;
                if (site >= g.N) continue;
                const size_t e = (size_t)site * (MODE == CONV_LAST ? 2 : 32) + c;
                const float v = acc[ob][i] + bc;
                if constexpr (MODE == CONV_DGRAD) {
                    out[e] = v * dsilu_f(pre_prev[e]);
                } else {
                    if (pre) pre[e] = v;
                    out[e] = MODE == CONV_LAST ? v : silu_f(v);
                }
            }
        }
    }
}

qedhmc_status net_pack_f32(qedhmc_net* n) {
    if (n->wf32_ready) return QEDHMC_OK;
    hipStream_t st = n->h->stream;
    for (int l = 0; l < kNetLayers; l++) {
        const int cin = kNetCh[l], cout = kNetCh[l + 1], ob = l == kNetLayers - 1 ? 1 : 2;
        const float* W = n->params + n->woff[l];
        float* dst = n->wf32 + frag_at(l, false);
        const int total = (int)conv_frag(l ? 32 : 8, ob);
        if (l == 0)
            hipLaunchKernelGGL(k_pack_conv<8>, dim3((total + 255) / 256), dim3(256), 0, st, W, cin, cout, ob, 0, dst);
        else
            hipLaunchKernelGGL(k_pack_conv<32>, dim3((total + 255) / 256), dim3(256), 0, st, W, cin, cout, ob, 0, dst);
        if (l > 0 && l < kNetLayers - 1)
            hipLaunchKernelGGL(k_pack_conv<32>, dim3((total + 255) / 256), dim3(256), 0, st, W, cin, cout, ob, 1,
                               n->wf32 + frag_at(l, true));
    }
    QH_HIP(hipGetLastError());
    n->wf32_ready = true;
    return QEDHMC_OK;
}

template <int MODE>
static qedhmc_status launch_conv(qedhmc_net* n, const float* in, const float* wfrag, const float* bias,
                                 const float* pre_prev, float* pre, float* out) {
    const NetGeo& g = n->g;
    const int ntile = (g.N + 15) / 16, per = (ntile + 7) / 8;
    // (a tile to every compute unit before a second wavefront gets one)
    const int wgs = std::max(1, std::min(n->h->n_cu / 8, per));
    const size_t lds = sizeof(float) * conv_frag(MODE == CONV_FIRST ? 8 : 32, MODE == CONV_LAST ? 1 : 2);
    if (lds > 65536) QH_TRY(allow_lds((const void*)k_conv_train<MODE>, n->h->max_lds));
    hipEvent_t e0, e1;
    if (MODE == CONV_HIDDEN && prof_sample(n->h, QEDHMC_K_NET_FP32, e0, e1))
        hipExtLaunchKernelGGL(k_conv_train<MODE>, dim3(8 * wgs), dim3(kConvThreads), lds, n->h->stream, e0, e1, 0, g,
                              ntile, in, wfrag, bias, pre_prev, pre, out);
    else
        hipLaunchKernelGGL(k_conv_train<MODE>, dim3(8 * wgs), dim3(kConvThreads), lds, n->h->stream, g, ntile, in,
                           wfrag, bias, pre_prev, pre, out);
    QH_HIP(hipGetLastError());
    return QEDHMC_OK;
}

// layer l forward in FP32 on the matrix cores (l = 0: in is the feature map)
qedhmc_status launch_fwd_mfma32(qedhmc_net* n, int l, const float* in, float* pre, float* act) {
    QH_TRY(net_pack_f32(n));
    const float* wf = n->wf32 + frag_at(l, false);
    const float* b = n->params + n->boff[l];
    if (l == 0) return launch_conv<CONV_FIRST>(n, in, wf, b, nullptr, pre, act);
    if (l == kNetLayers - 1) return launch_conv<CONV_LAST>(n, in, wf, b, nullptr, pre, act);
    return launch_conv<CONV_HIDDEN>(n, in, wf, b, nullptr, pre, act);
}

// data gradient through hidden layer l (1 .. 4): gin = W_l^T * gout, times SiLU'(pre of layer l - 1)
qedhmc_status launch_dgrad_mfma32(qedhmc_net* n, int l, const float* gout, const float* pre_prev, float* gin) {
    QH_TRY(net_pack_f32(n));
    return launch_conv<CONV_DGRAD>(n, gout, n->wf32 + frag_at(l, true), nullptr, pre_prev, nullptr, gin);
}

// ---------------------------------------------------------------------------
// Weight gradients
// ---------------------------------------------------------------------------
// Bricks of BX x BY sites of a slice (ragged at the far edges)
struct Brick {
    int BX, BY, nbx, nby, total;
    int wx, wy;  // window: BX + 2, BY + 2
};

static constexpr int kBrickSites = 96;

static Brick brick_of(const NetGeo& g) {
    Brick b;
    b.nbx = (g.L + 23) / 24;
    b.BX = (g.L + b.nbx - 1) / b.nbx;
    const int by = std::max(1, std::min(g.L, kBrickSites / b.BX));
    b.nby = (g.L + by - 1) / by;
    b.BY = (g.L + b.nby - 1) / b.nby;
    b.total = b.nbx * b.nby * g.Nt;
    b.wx = b.BX + 2;
    b.wy = b.BY + 2;
    return b;
}

// channels of a site padded to the vectors of 4 (or the pairs) they load as
template <int C>
constexpr int wg_vec() { return C % 4 == 0 ? 4 : 2; }

// The brick at (tau, y0, x0) with a halo of one site into dst [3][wy][wx][C]
// (SIGN: channels 4 and 5 negated where the slice wraps in tau).
template <int C, bool SIGN>
__device__ __forceinline__ void wg_window(const NetGeo& g, const Brick& b, int tau, int y0, int x0,
                                          const float* __restrict__ src, float* dst) {
    constexpr int V = wg_vec<C>(), Q = C / V;
    typedef float vec __attribute__((ext_vector_type(V)));
    const int plane = b.wy * b.wx;
    for (int e = threadIdx.x; e < 3 * plane * Q; e += blockDim.x) {
        const int s = e / Q, c = e - s * Q;
        const int d = s / plane, p = s - d * plane, ry = p / b.wx, rx = p - ry * b.wx;
        const int t = tau + d - 1;
        const int m = wrap(t, g.Nt) * g.Vs + wrap(y0 + ry - 1, g.L) * g.L + wrap(x0 + rx - 1, g.L);
        vec v = *reinterpret_cast<const vec*>(src + (size_t)m * C + V * c);
        if (SIGN && c == 1 && (t < 0 || t >= g.Nt)) {
            v[0] = -v[0];
            v[1] = -v[1];
        }
        *reinterpret_cast<vec*>(dst + (size_t)s * C + V * c) = v;
    }
}

// The brick's own sites into dst [sites, padded to 4][C], zero outside the lattice.
template <int C>
__device__ __forceinline__ void wg_sites(const NetGeo& g, const Brick& b, int tau, int y0, int x0,
                                         const float* __restrict__ src, float* dst) {
    constexpr int V = wg_vec<C>(), Q = C / V;
    typedef float vec __attribute__((ext_vector_type(V)));
    const int ns = b.BX * b.BY, np = (ns + 3) & ~3;
    for (int e = threadIdx.x; e < np * Q; e += blockDim.x) {
        const int s = e / Q, c = e - s * Q, r = s / b.BX, x = x0 + s - r * b.BX, y = y0 + r;
        vec v;
#pragma unroll
        for (int i = 0; i < V; i++) v[i] = 0.0f;
        if (s < ns && y < g.L && x < g.L)
            v = *reinterpret_cast<const vec*>(src + ((size_t)tau * g.Vs + (size_t)y * g.L + x) * C + V * c);
        *reinterpret_cast<vec*>(dst + (size_t)s * C + V * c) = v;
    }
}

// LAYER 0: first (feature map [N][8], 6 channels used, to 32), 1: hidden (32 to
// 32), 2: last (32 to 2).  Products per step of 4 sites (a lane's site is
// 4 step + lane / 16):
//   hidden  per tap a 32 x 32 block; wavefront w has taps 7 w .. 7 w + 6, the
//           28th slot is the bias gradient (A = 1)
//   first   rows (tap, channel) = 162 and the bias row (A = 1), 11 blocks of
//           16, dealt to the wavefronts; the columns are the 32 outputs
//   last    with the roles shifted, dW_k = sum_m in[m] g[m - d_k]: rows the 32
//           channels, columns (tap, output) = 54, a block of 16 per wavefront
// Bound by the products in the hidden layers (50 us at N = 138240, as the
// forward); the end layers by staging the bricks.  Before, every wavefront
// fetched each site's neighbours from memory with its own index arithmetic:
// 208 us hidden, 182 us first, 168 us last; now 113, 31 and 18 us.
template <int LAYER>
__global__ __launch_bounds__(256) void k_wgrad_brick(NetGeo g, Brick b, const float* __restrict__ in,
                                                     const float* __restrict__ gout, float* __restrict__ part) {
    constexpr int CIN = LAYER == 0 ? 8 : 32, COUT = LAYER == 2 ? 2 : 32;
    constexpr int RA = LAYER == 1 ? 7 : (LAYER == 0 ? 3 : 1);    // A operands per step (taps, row blocks)
    constexpr int NA = LAYER == 0 ? 1 : 2, NB = LAYER == 2 ? 1 : 2;  // blocks of 16 in A and B per operand
    constexpr int CW = LAYER == 2 ? COUT : CIN, CS = LAYER == 2 ? CIN : COUT;  // channels of the window, of the sites
    extern __shared__ __align__(16) float smem[];
    const int plane = b.wy * b.wx, ns = b.BX * b.BY;
    float* win = smem;
    float* sites = smem + ((3 * plane * CW + 3) & ~3);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int c16 = lane & 15, kq = lane >> 4;
    auto tap = [&](int k) { return ((k / 9 - 1) * plane + (k / 3 % 3 - 1) * b.wx + k % 3 - 1) * CW; };
    // this lane's window offsets from the centre of its site
    int off[RA];
    bool one[RA];  // the operand is the constant 1 (bias)
#pragma unroll
    for (int j = 0; j < RA; j++) {
        one[j] = false;
        off[j] = 0;
        if constexpr (LAYER == 1) {
            const int k = 7 * wave + j;
            one[j] = k == 27;
            off[j] = one[j] ? 0 : tap(k) + c16;
        } else if constexpr (LAYER == 0) {
            const int r = 16 * (wave + 4 * j) + c16;
            one[j] = r == 162;
            off[j] = r < 162 ? tap(r / 6) + r % 6 : 0;
        } else {
            const int q = 16 * wave + c16;
            off[j] = q < 54 ? -tap(q / 2) + q % 2 : 0;
        }
    }
    f32x4 acc[RA][NA][NB], accb = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int j = 0; j < RA; j++)
#pragma unroll
        for (int u = 0; u < NA; u++)
#pragma unroll
            for (int v = 0; v < NB; v++) acc[j][u][v] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int nwg = (int)gridDim.x >> 3, per = (b.total + 7) >> 3, xcd = (int)blockIdx.x & 7;
    for (int t = (int)blockIdx.x >> 3; t < per; t += nwg) {
        const int id = xcd * per + t;
        if (id >= b.total) break;
        const int tau = id / (b.nbx * b.nby), q = id - tau * (b.nbx * b.nby);
        const int y0 = q / b.nbx * b.BY, x0 = q % b.nbx * b.BX;
        __syncthreads();  // the last brick's products are done with the LDS
        if constexpr (LAYER == 2) {
            wg_window<2, false>(g, b, tau, y0, x0, gout, win);
            wg_sites<32>(g, b, tau, y0, x0, in, sites);
        } else {
            wg_window<CIN, LAYER == 0>(g, b, tau, y0, x0, in, win);
            wg_sites<32>(g, b, tau, y0, x0, gout, sites);
        }
        __syncthreads();
        // this lane's site: row r, column c of the brick
        int r = 0, c = kq;
        while (c >= b.BX) {
            c -= b.BX;
            r++;
        }
        for (int s0 = 0; s0 < ns; s0 += 4) {
            const int s = s0 + kq;
            const bool on = s < ns;
            const float* ctr = win + ((b.wy + (on ? r : 0) + 1) * b.wx + (on ? c : 0) + 1) * CW;
            const float* own = sites + s * CS + c16;
            if constexpr (LAYER == 2) {
                const float a0 = own[0], a1 = own[16], bw = ctr[off[0]];
                acc[0][0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, bw, acc[0][0][0], 0, 0, 0);
                acc[0][1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, bw, acc[0][1][0], 0, 0, 0);
                // the centre tap's columns with A = 1 on the lattice's sites: the bias gradient
                const float a2 = on && y0 + r < g.L && x0 + c < g.L ? 1.0f : 0.0f;
                if (wave == 1) accb = __builtin_amdgcn_mfma_f32_16x16x4f32(a2, bw, accb, 0, 0, 0);
            } else {
                const float b0 = own[0], b1 = own[16];
#pragma unroll
                for (int j = 0; j < RA; j++)
#pragma unroll
                    for (int u = 0; u < NA; u++) {
                        const float a = one[j] ? 1.0f : ctr[off[j] + 16 * u];
                        acc[j][u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b0, acc[j][u][0], 0, 0, 0);
                        acc[j][u][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b1, acc[j][u][1], 0, 0, 0);
                    }
            }
            c += 4;
            while (c >= b.BX) {
                c -= b.BX;
                r++;
            }
        }
    }
    // D fragment: lane holds rows 4 (lane / 16) + i, column lane % 16; partial
    // layout [27][cin][cout], then the bias
    constexpr int CI = LAYER == 0 ? 6 : 32, EK = CI * COUT, E = 27 * EK;
    float* out = part + (size_t)blockIdx.x * (E + COUT);
#pragma unroll
    for (int j = 0; j < RA; j++)
#pragma unroll
        for (int u = 0; u < NA; u++)
#pragma unroll
            for (int v = 0; v < NB; v++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float x = acc[j][u][v][i];
                    if constexpr (LAYER == 1) {
                        const int k = 7 * wave + j, ci = 16 * u + 4 * kq + i, o = 16 * v + c16;
                        if (k < 27)
                            out[(size_t)k * EK + ci * COUT + o] = x;
                        else if (ci == 0)
                            out[E + o] = x;
                    } else if constexpr (LAYER == 0) {
                        const int row = 16 * (wave + 4 * j) + 4 * kq + i, o = 16 * v + c16;
                        if (row <= 162) out[row * COUT + o] = x;  // row 162 is the bias, right after the taps
                    } else {
                        const int ci = 16 * u + 4 * kq + i, q = 16 * wave + c16;
                        if (q < 54) out[(size_t)(q / 2) * EK + ci * COUT + q % 2] = x;
                    }
                }
    if (LAYER == 2 && wave == 1 && kq == 0) {
        const int q = 16 + c16;
        if (q / 2 == 13) out[E + q % 2] = accb[0];
    }
}

// Workgroups (one partial each) of layer l's weight gradient; every lattice has
// at least one brick.  A workgroup's FP32 sums run over all its bricks, so the
// chip is filled as many times over as keeps them to 288 sites, 256 more for
// every 2^19 sites; the partials are added in FP64.  Filled once at every size
// the sums grew to 1500 sites: error against 64 bits in the hidden layers, in
// units of the sum's own random size, at N = 262144, 524288, 1048576 4.4e-7,
// 5.7e-7, 6.9e-7; now 2.8e-7, 2.9e-7, 4.0e-7 (chunks of 256, 256, 512 sites, the
// partials added in FP32: 3.1e-7, 3.3e-7, 3.9e-7).  Step at L = 48, N_tau = 228
// 4.77 -> 4.99 ms, at L = 64, N_tau = 256 10.1 -> 9.6 ms.
int wgrad_parts(const qedhmc_net* n, int l) {
    const Brick b = brick_of(n->g);
    const int slots = n->h->n_cu * (l > 0 && l < kNetLayers - 1 ? 2 : 4);
    const int most = (288 + (n->g.N - 1) / (1 << 19) * 256) / (b.BX * b.BY);  // bricks per workgroup
    const int fills = (b.total + slots * most - 1) / (slots * most);
    return 8 * std::max(1, std::min(slots * fills / 8, (b.total + 7) / 8));
}

qedhmc_status launch_wgrad_mfma(qedhmc_net* n, int l, const float* in, const float* gout) {
    const Brick b = brick_of(n->g);
    const int grid = wgrad_parts(n, l);
    const int plane = b.wy * b.wx, np = (b.BX * b.BY + 3) & ~3;
    auto go = [&](auto kern, int cw, int cs) -> qedhmc_status {
        const size_t lds = sizeof(float) * (((size_t)3 * plane * cw + 3) / 4 * 4 + (size_t)np * cs);
        if (lds > n->h->max_lds) {
            set_error("net: a weight-gradient brick exceeds the LDS");
            return QEDHMC_EUNSUPPORTED;
        }
        if (lds > 65536) QH_TRY(allow_lds((const void*)kern, n->h->max_lds));
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, n->h->stream, n->g, b, in, gout, n->wpart);
        QH_HIP(hipGetLastError());
        return QEDHMC_OK;
    };
    if (l == 0) return go(k_wgrad_brick<0>, 8, 32);
    if (l == kNetLayers - 1) return go(k_wgrad_brick<2>, 2, 32);
    return go(k_wgrad_brick<1>, 32, 32);
}

}  // namespace qh
