// backward.hip -- backward of the masked k x k convolution layer on gfx950,
// for training on the negative log-likelihood (Sec. 3 NLL equation; the
// appendix's training details reset the masked weights' gradients to zero
// after every step), behind finc_backward of include/finc.h.
//
// y = layer(x) sends x[ci, i + a - oh, j + b - ow] to y[co, i, j] with weight
// K[co][ci][a][b] (zero at the masked self-tap entries ci > co), so for an
// output gradient dy:
//   dx[ci, s, t] = sum_{co, a, b} K[co][ci][a][b] dy[co, s - a + oh, t - b + ow]
//     -- a convolution of dy with the kernel transposed over channels and
//     flipped in space: the forward of that kernel with the opposite corner
//     (layer_grads of finc_detail.h), or an implicit GEMM where that is faster
//     or does not fit (gemm_grad_kernel);
//   dK[co][ci][a][b] = sum over images and pixels of dy[co, i, j] times the
//     input the tap read (zero outside the image) -- a GEMM with
//     M = C_out, N = C_in k^2 and a reduction over the B H W positions, in
//     parts of the positions (dk_tile.h), which dk_reduce_kernel adds in
//     order, sets the masked entries to 0 and adds the log|det| term
//     gld H W / K[c][c][self] on the self diagonal.
// Both run in one launch, or dK in one of its own (dk_kernel) where dx is not
// wanted.
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>
#include <type_traits>

#include "conv_gemm.h"
#include "dk_tile.h"
#include "finc.h"
#include "finc_detail.h"

namespace {

inline size_t up256b(size_t n) { return (n + 255) & ~(size_t)255; }
inline size_t imax_sz(size_t a, size_t b) { return a > b ? a : b; }
inline bool overlapb(const void *a, size_t na, const void *b, size_t nb) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb && y < x + na;
}

// dK's blocks alone (dK without dx, and images of 2 GB or more).
template <int K, int FORM, bool BIG>
__global__ __launch_bounds__(256) void dk_kernel(DkArgs a) {
    __shared__ __attribute__((aligned(16))) float lds[dk_lds_floats<K, FORM>()];
    dk_tile<K, FORM, BIG>(a, blockIdx.x, lds);
}

// dK = the sum of the parts, in a fixed order: of the eight groups of 32 threads
// of a block, group g adds parts g, g + 8, g + 16, ... of 32 neighbouring
// entries in turn, then the groups' sums in order.
__global__ __launch_bounds__(256) void dk_reduce_kernel(const float *partial, int parts,
                                                        const float *K, float *dK, double gld,
                                                        int C, int k, int H, int W, int oh,
                                                        int ow) {
    __shared__ float red[8][33];
    const int N = C * k * k, n = C * N;
    const int l = threadIdx.x & 31, g = threadIdx.x >> 5, e = blockIdx.x * 32 + l;
    const int ec = e < n ? e : n - 1;
    float v = 0.0f;
    for (int z = g; z < parts; z += 64) {
        float p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            p[u] = partial[(long long)min(z + 8 * u, parts - 1) * n + ec];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v += z + 8 * u < parts ? p[u] : 0.0f;
    }
    red[g][l] = v;
    __syncthreads();
    if (g != 0 || e >= n)
        return;
#pragma unroll
    for (int u = 1; u < 8; ++u)
        v += red[u][l];
    const int co = e / N, col = e - co * N, ci = col / (k * k), t = col - ci * k * k;
    dK[e] = dk_entry(v, co, ci, t, K, gld, C, k, H, W, oh, ow);
}

// The most parts of the position reduction, whose sums the workspace holds: of
// 128 positions and more each, 512 for each 64 columns of C k^2 and 16 rows of C
// together, and at most 16 M floats of partial sums.  (A part has nt^2 blocks for
// each nine taps, fewer than that for several channel tiles: 48 x 8 x 8, batch
// 64 runs 198.)
int dk_parts(int B, int C, int H, int W, int k) {
    const long long nchunk = ((long long)B * H * W + 63) / 64;
    const long long tiles = (long long)((C * k * k + 63) / 64) * ((C + 15) / 16);
    long long parts = 512 / (tiles > 0 ? tiles : 1);
    if (parts > nchunk / 2)
        parts = nchunk / 2;
    const long long cap = (16ll << 20) / ((long long)C * C * k * k);
    if (parts > cap)
        parts = cap;
    return (int)(parts < 1 ? 1 : parts);
}

// dK's bands: 32 columns (more where there are less than eight rows), and rows,
// or whole images, up to kDkPos positions and dk_x pixels with the halo; of
// these, cut from the most, the ones that take the blocks (tiles of them a part,
// `most` parts) the least time.  A band's time is that of its positions, while
// every compute unit has a block or less however few blocks there are, of the
// pixels it stages, about a third of a position each, and of its latencies, about
// 64 positions; a cut has to gain 15%.  us, dK alone, one image a band of whole
// rows -> these: 12 x 4 x 4, batch 96 16.0 -> 9.6; 12 x 16 x 16, batch 64 10.5 ->
// 9.3; 12 x 2 x 2, batch 4096 46 -> 12; 12 x 1 x 1, batch 4096 175 -> 11.
void dk_bands(DkArgs &a, int B, int H, int W, int k, bool big, int tiles, int most) {
    // (rows of more than a band: the halo that cropping saves is not worth it)
    const bool crop = !big && W <= 32;
    a.pr = H < k && crop ? H - 1 : k - 1;
    a.pc = W < k && crop ? W - 1 : k - 1;
    int wb = 32;
    if (H < kDkPos / wb) {
        const int x = dk_x(k, false) / (H + a.pr) - a.pc;
        wb = kDkPos / H < x ? kDkPos / H : x;
    }
    if (wb > W)
        wb = W;
    const int rows = dk_x(k, false) / (wb + a.pc) - a.pr;
    int rb = kDkPos / wb < rows ? kDkPos / wb : rows, ni = 1;
    if (rb >= H) {
        rb = H;
        const int x = dk_x(k, true) / ((H + a.pr) * (W + a.pc));
        if (wb == W && x > 1)
            ni = kDkPos / (H * W) < x ? kDkPos / (H * W) : x;
    }
    double best = 0.0;
    for (;;) {
        const long long nb = (long long)cdiv(B, ni) * cdiv(H, rb) * cdiv(W, wb);
        const long long bpp = (nb + most - 1) / most, blocks = (nb + bpp - 1) / bpp * tiles;
        const double pos = (double)ni * rb * wb, x = (double)ni * (rb + a.pr) * (wb + a.pc);
        const double t = bpp * (64.0 + pos * (blocks > 256 ? blocks / 256.0 : 1.0) + 0.3 * x);
        if (best == 0.0 || t < 0.85 * best) {
            best = t;
            a.ni = ni;
            a.RB = rb;
            a.WB = wb;
        }
        const int each = cdiv(B, most);   // images of a part
        if (ni > 1)
            ni = ni > each ? each : (ni + 1) / 2;
        else if (rb > 1)
            rb = (rb + 1) / 2;
        else if (wb > 32)
            wb = wb > 64 ? (wb + 1) / 2 : 32;
        else
            break;
    }
    a.bx = cdiv(W, a.WB);
    a.form = a.pr < k - 1 || a.pc < k - 1 ? kDkCrop : a.ni > 1 ? kDkMulti : kDkOne;
}

bool valid_bwd_shape(int B, int C, int H, int W, int k) {
    if (B < 0 || C < 1 || C > FINC_MAX_C || H < 1 || W < 1 || k < 1 || k > FINC_MAX_K)
        return false;
    return (long long)B * C * H * W < (1ll << 31);
}

// Both gradients where layer_grads refuses (one or two taps, images of a few
// pixels, rows that do not fit in LDS): dx as the implicit GEMM of conv_gemm.h on
// K read transposed and flipped, beside dK's blocks (da.blocks of them, or none).  dx in tiles of 64 c_out x 64 pixels at 64 channels, else
// 16 x 128, or 16 x 64 while there are fewer than two blocks a compute unit.
template <int R, int WCO, int NS, int FORM>
__global__ __launch_bounds__(256) void gemm_grad_kernel(ConvArgs ca, int gx, DkArgs da) {
    constexpr int nc = conv_lds_floats<WCO, NS>(), nd = dk_lds_floats<R, FORM>();
    __shared__ __attribute__((aligned(16))) float lds[nc > nd ? nc : nd];
    if ((int)blockIdx.x < da.blocks) {
        dk_tile<R, FORM, false>(da, blockIdx.x, lds);
        return;
    }
    const int b = blockIdx.x - da.blocks;
    conv_tile<R, WCO, NS, 4>(ca, b % gx, b / gx, 0, lds);
}
template <int R>
void launch_gemm_grad(const ConvArgs &a, const DkArgs &da, hipStream_t st) {
    const long long Q = (long long)a.B * a.H * a.W;
    const int gy = cdiv(a.Co, 16);
    auto go = [&](auto wco, auto ns) {
        constexpr int WCO = decltype(wco)::value, NS = decltype(ns)::value;
        const int gx = cdiv(Q, 16 * NS * (4 / WCO)), g = gx * cdiv(a.Co, 16 * WCO);
        auto *kernel = da.form == kDkCrop    ? gemm_grad_kernel<R, WCO, NS, kDkCrop>
                       : da.form == kDkMulti ? gemm_grad_kernel<R, WCO, NS, kDkMulti>
                                             : gemm_grad_kernel<R, WCO, NS, kDkOne>;
        hipLaunchKernelGGL(kernel, dim3(da.blocks + g), dim3(kConvThreads), 0, st, a, gx, da);
    };
    if (a.Co >= 64 && cdiv(Q, 64) >= 256)
        go(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{});
    else if ((long long)cdiv(Q, 128) * gy >= 512)
        go(std::integral_constant<int, 1>{}, std::integral_constant<int, 2>{});
    else
        go(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
}

// f(integral constant k) for 1 <= k <= 7.
template <typename F>
void for_k(int k, F f) {
    switch (k) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    default: f(std::integral_constant<int, 7>{}); break;
    }
}

// Both gradients of one layer whose images lie img floats apart in x, dy and
// dx (C H W for a whole tensor, more for a channel slice of a wider one);
// partial: dk_parts(B, C, H, W, k) C^2 k^2 floats.  Arguments checked by
// the caller.
int launch_layer_backward(const float *x, const float *dy, const float *K, float *dx, float *dK,
                          double gld, int B, int C, int H, int W, int k, int corner,
                          long long img, float *partial, hipStream_t stream) {
    const int oh = (corner == FINC_TL || corner == FINC_TR) ? k - 1 : 0;
    const int ow = (corner == FINC_TL || corner == FINC_BL) ? k - 1 : 0;
    const int n = C * C * k * k;
    const bool big = (long long)C * H * W * 4 >= (1ll << 31);
    // dK, in partial sums over parts of the positions
    int parts = 0;
    DkArgs da;
    memset(&da, 0, sizeof(da));
    if (dK && B > 0) {
        da.x = x;
        da.dy = dy;
        da.K = K;
        da.partial = partial;
        da.gld = gld;
        da.img = img;
        da.C = C;
        da.H = H;
        da.W = W;
        da.oh = oh;
        da.ow = ow;
        da.N = C * k * k;
        da.B = B;
        da.nt = cdiv(C, 16);
        const int groups = cdiv(k * k, dk_taps(k)), most = dk_parts(B, C, H, W, k);
        dk_bands(da, B, H, W, k, big, da.nt * da.nt * groups, most);
        da.nbi = cdiv(H, da.RB) * da.bx;
        da.nb = cdiv(B, da.ni) * da.nbi;
        da.bpp = cdiv(da.nb, most);
        parts = cdiv(da.nb, da.bpp);
        da.dK = parts == 1 ? dK : nullptr;
        const int wlast = W - (da.bx - 1) * da.WB;
        da.d_nbi = make_div(da.nbi);
        da.d_bx = make_div(da.bx);
        da.d_nt = make_div(da.nt);
        da.d_w = make_div(da.WB);
        da.d_wl = make_div(wlast);
        da.d_xw = make_div(da.WB + da.pc);
        da.d_xwl = make_div(wlast + da.pc);
        da.parts = parts;
        da.d_nt2 = make_div(da.nt * da.nt);
        da.d_parts = make_div(parts);
        da.d_yr = make_div(da.RB);
        da.d_xr = make_div(da.RB + da.pr);
        da.blocks = da.nt * da.nt * parts * groups;
    }
    // one launch for both, but for images of 2 GB or more
    const DkArgs none = {};
    const DkArgs &beside = big ? none : da;
    int rc = FINC_OK;
    if (dx && B > 0) {
        rc = layer_grads(dy, dx, K, B, C, H, W, k, corner, img, beside, stream);
        if (rc == FINC_EUNSUPPORTED) {
            ConvArgs ca = conv_args(dy, img, dx, img, K, nullptr, nullptr, 0, B, C, C, H, W, k);
            ca.ph = k - 1 - oh;
            ca.pw = k - 1 - ow;
            ca.flip = 1;
            ca.fself = oh * k + ow;
            for_k(k, [&](auto kc) { launch_gemm_grad<decltype(kc)::value>(ca, beside, stream); });
            rc = conv_launched();
        }
    }
    if (rc == FINC_OK && da.blocks > 0 && (big || !dx)) {
        for_k(k, [&](auto kc) {
            constexpr int KC = decltype(kc)::value;
            auto *kernel = big                   ? dk_kernel<KC, kDkOne, true>
                           : da.form == kDkCrop  ? dk_kernel<KC, kDkCrop, false>
                           : da.form == kDkMulti ? dk_kernel<KC, kDkMulti, false>
                                                 : dk_kernel<KC, kDkOne, false>;
            hipLaunchKernelGGL(kernel, dim3(da.blocks), dim3(256), 0, stream, da);
        });
        rc = conv_launched();
    }
    if (rc != FINC_OK || !dK || parts == 1)
        return rc;
    hipLaunchKernelGGL(dk_reduce_kernel, dim3((n + 31) / 32), dim3(256), 0, stream, partial, parts,
                       K, dK, gld, C, k, H, W, oh, ow);
    return conv_launched();
}



// ---- actnorm backward -----------------------------------------------------
// y = s x + b per channel: dx = s dy; ds[c] = sum dy x + gld H W / s[c];
// db[c] = sum dy.  Block (c, part) covers images [part bpp, (part+1) bpp) of
// channel c: it writes dx there and its two sums (fp64, each thread's
// elements in order, then a fixed tree) to partial[(c parts + part) 2 + .];
// actnorm_reduce_kernel adds the parts in order.
// The parts are few (their sums are in the caller's workspace), so a block is
// wide and a thread has four 16-byte loads of x and of dy in flight where the
// planes allow them: latency bound otherwise (64 x 24 x 16 x 16: 28.9 us with
// 24 blocks of 256 threads, one value a load).
constexpr int kAnThreads = 1024;
constexpr int kAnU = 4;

template <typename V>   // float4 (planes of a multiple of 4 values, 16-byte aligned) or float
__global__ __launch_bounds__(kAnThreads) void actnorm_bwd_kernel(const float *x, const float *dy,
                                                                 const float *s, float *dx,
                                                                 double *partial, int B, int C,
                                                                 int HW, int bpp, int parts,
                                                                 Div d_hv) {
    constexpr int N = sizeof(V) / sizeof(float);
    __shared__ double red[2][kAnThreads / 64];
    const int c = blockIdx.x, part = blockIdx.y, tid = threadIdx.x;
    const int b0 = part * bpp, b1 = min(b0 + bpp, B);
    const int hv = HW / N, n = (b1 - b0) * hv;   // (fewer than 2^31 values in all)
    const float sc = s[c];
    double sx = 0.0, sy = 0.0;
    for (unsigned base = tid; base < (unsigned)n; base += kAnU * kAnThreads) {
        V g[kAnU], v[kAnU];
        long long at[kAnU];
#pragma unroll
        for (int u = 0; u < kAnU; ++u) {
            const int i = (int)min(base + u * kAnThreads, (unsigned)n - 1);
            const int b = divi(i, d_hv), p = i - b * hv;
            at[u] = ((long long)(b0 + b) * C + c) * hv + p;
            g[u] = reinterpret_cast<const V *>(dy)[at[u]];
            v[u] = reinterpret_cast<const V *>(x)[at[u]];
        }
#pragma unroll
        for (int u = 0; u < kAnU; ++u) {
            if (base + u * kAnThreads >= (unsigned)n)
                break;
            float *gv = reinterpret_cast<float *>(&g[u]);
            const float *xv = reinterpret_cast<const float *>(&v[u]);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                sx += (double)gv[e] * (double)xv[e];
                sy += (double)gv[e];
                gv[e] *= sc;
            }
            if (dx)
                reinterpret_cast<V *>(dx)[at[u]] = g[u];
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        sx += __shfl_xor(sx, off);
        sy += __shfl_xor(sy, off);
    }
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = sx;
        red[1][tid >> 6] = sy;
    }
    __syncthreads();
    if (tid < 2) {
        double v = 0.0;
        for (int w = 0; w < kAnThreads / 64; ++w)
            v += red[tid][w];
        partial[((long long)c * parts + part) * 2 + tid] = v;
    }
}

__global__ __launch_bounds__(64) void actnorm_reduce_kernel(const double *partial, int parts,
                                                            const float *s, float *ds, float *db,
                                                            double gld, int C, int HW) {
    const int c = blockIdx.x * 64 + threadIdx.x;
    if (c >= C)
        return;
    double sx = 0.0, sy = 0.0;
    for (int z = 0; z < parts; ++z) {
        sx += partial[((long long)c * parts + z) * 2];
        sy += partial[((long long)c * parts + z) * 2 + 1];
    }
    if (ds)
        ds[c] = (float)(sx + gld * (double)HW / (double)s[c]);
    if (db)
        db[c] = (float)sy;
}

// Parts of the batch per channel: about 512 blocks over the chip, at least
// 16 K values per block.
int actnorm_parts(int B, int C, int HW) {
    long long parts = 512 / C;
    const long long per = (16384 + HW - 1) / HW;   // images per block at minimum
    if (parts > (B + per - 1) / per)
        parts = (B + per - 1) / per;
    return (int)(parts < 1 ? 1 : parts);
}

// ---- negative log-likelihood ----------------------------------------------
// One block per image: each latent's values in a fixed order (thread t takes
// t, t + 256, ...; fp64), a fixed tree over the threads, the latents in order.
constexpr int kNllMaxL = 16;
struct NllArgs {
    const float *z[kNllMaxL];
    long long n[kNllMaxL];
    int L;
    long long D;
    const double *logdet;
    double *nll, *bpd;
};

__global__ __launch_bounds__(256) void gauss_nll_kernel(NllArgs a) {
    __shared__ double red[256];
    const int b = blockIdx.x, tid = threadIdx.x;
    double total = 0.0;
    for (int l = 0; l < a.L; ++l) {
        const float *zb = a.z[l] + (long long)b * a.n[l];
        double q = 0.0;
        for (long long e = tid; e < a.n[l]; e += 256) {
            const double v = zb[e];
            q += v * v;
        }
        red[tid] = q;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (tid < h)
                red[tid] += red[tid + h];
            __syncthreads();
        }
        total += red[0];
        __syncthreads();
    }
    if (tid == 0) {
        const double log2pi = 1.8378770664093454836;   // log(2 pi)
        const double nll = 0.5 * (total + (double)a.D * log2pi) - a.logdet[b];
        a.nll[b] = nll;
        if (a.bpd)
            a.bpd[b] = nll / ((double)a.D * 0.69314718055994530942);   // / (D log 2)
    }
}


// ---- the multi-scale stack's training direction ----------------------------
// (B C H W < 2^31 values: int indices)

// y = s[c] x + b[c] (actnorm forward).
__global__ __launch_bounds__(256) void affine_kernel(const float *x, float *y, const float *s,
                                                     const float *b, int n, Div d_HW, Div d_C,
                                                     int C) {
    for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) {
        const int pl = divi(e, d_HW), c = pl - divi(pl, d_C) * C;
        y[e] = s[c] * x[e] + b[c];
    }
}

// Split and squeeze of a level's output h (B, C, H, W): channels [C/2, C)
// go to the latent z (B, C/2, H, W); channel c < C/2 at (2 i + dy, 2 j + dx)
// goes to channel 4 c + 2 dy + dx of the next level's input (B, 2C, H/2, W/2).
__global__ __launch_bounds__(256) void split_squeeze_kernel(const float *h, float *nxt, float *z,
                                                            int n, int C, int H, int W, Div d_HW,
                                                            Div d_C, Div d_W) {
    const int HW = H * W, Ch = C / 2;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) {
        const int pl = divi(e, d_HW), p = e - pl * HW;
        const int b = divi(pl, d_C), c = pl - b * C;
        if (c >= Ch) {
            z[(b * Ch + c - Ch) * HW + p] = h[e];
        } else {
            const int i = divi(p, d_W), j = p - i * W;
            const int co = 4 * c + 2 * (i & 1) + (j & 1);
            nxt[((b * 2 * C + co) * (H / 2) + (i >> 1)) * (W / 2) + (j >> 1)] = h[e];
        }
    }
}

// Its adjoint: the gradient of a level's output, g (B, C, H, W), from the
// gradient of the next level's input gn (B, 2C, H/2, W/2) -- unsqueezed,
// first half -- and the latent's gradient dz (B, C/2, H, W), second half.
__global__ __launch_bounds__(256) void unsqueeze_concat_kernel(const float *gn, const float *dz,
                                                               float *g, int n, int C, int H,
                                                               int W, Div d_HW, Div d_C,
                                                               Div d_W) {
    const int HW = H * W, Ch = C / 2;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) {
        const int pl = divi(e, d_HW), p = e - pl * HW;
        const int b = divi(pl, d_C), c = pl - b * C;
        if (c >= Ch) {
            g[e] = dz[(b * Ch + c - Ch) * HW + p];
        } else {
            const int i = divi(p, d_W), j = p - i * W;
            const int co = 4 * c + 2 * (i & 1) + (j & 1);
            g[e] = gn[((b * 2 * C + co) * (H / 2) + (i >> 1)) * (W / 2) + (j >> 1)];
        }
    }
}

// The stack's log|det| for one image -- every block's H W sum_c
// log|K[c][c][self]| and every actnorm's H W sum_c log|s_c| -- in fp64, each
// thread's terms in order and a fixed tree; written for every image.
__global__ __launch_bounds__(256) void stack_logdet_kernel(const float *K, const float *scale,
                                                           int L, int U, int C1, int H1, int W1,
                                                           int k, double *logdet, int B) {
    __shared__ double red[256];
    const int tid = threadIdx.x;
    double acc = 0.0;
    long long koff = 0, soff = 0;
    for (int l = 0; l < L; ++l) {
        const int C = C1 << l;
        const double hw = (double)(H1 >> l) * (double)(W1 >> l);
        const long long ksz = (long long)C * C * k * k;
        // per unit: 4 C diagonal entries, then C scales
        for (int t = tid; t < U * 5 * C; t += 256) {
            const int u = t / (5 * C), r = t - u * 5 * C;
            if (r < 4 * C) {
                const int q = r / C, c = r - q * C;
                const int oh = (q == 0 || q == 1) ? k - 1 : 0, ow = (q == 0 || q == 2) ? k - 1 : 0;
                const float d = K[koff + (4ll * u + q) * ksz + ((long long)(c * C + c) * k + oh) * k + ow];
                acc += hw * log(fabs((double)d));
            } else {
                acc += hw * log(fabs((double)scale[soff + (long long)u * C + (r - 4 * C)]));
            }
        }
        koff += 4ll * U * ksz;
        soff += (long long)U * C;
    }
    red[tid] = acc;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h)
            red[tid] += red[tid + h];
        __syncthreads();
    }
    for (int b = tid; b < B; b += 256)
        logdet[b] = red[0];
}

int ew_blocks(long long n) { return (int)(n / 256 + 1 < 4096 ? n / 256 + 1 : 4096); }

struct StackShape {
    int B, L, U, C1, H1, W1, k;
    long long n0;   // values of a level-0 activation
    int C(int l) const { return C1 << l; }
    int H(int l) const { return H1 >> l; }
    int W(int l) const { return W1 >> l; }
    long long n(int l) const { return n0 >> l; }   // (C doubles, H W quarters)
    long long koff(int l) const {
        long long o = 0;
        for (int m = 0; m < l; ++m)
            o += 4ll * U * C(m) * C(m) * k * k;
        return o;
    }
    long long soff(int l) const {
        long long o = 0;
        for (int m = 0; m < l; ++m)
            o += (long long)U * C(m);
        return o;
    }
    long long kfloats() const { return koff(L); }
    long long sfloats() const { return soff(L); }
};

bool stack_shape_ok(const StackShape &s) {
    if (s.B < 0 || s.L < 1 || s.L > 8 || s.U < 0 || s.C1 < 1 || s.H1 < 1 || s.W1 < 1 || s.k < 1 ||
        s.k > FINC_MAX_K)
        return false;
    if (s.L > 1 && ((s.C1 & 1) || ((s.H1 | s.W1) & ((1 << (s.L - 1)) - 1))))
        return false;
    return (s.C1 << (s.L - 1)) <= FINC_MAX_C && s.n0 < (1ll << 31);
}

// Workspace of the stack's training calls: per level its 2 U + 1 activations
// (unit inputs, unit outputs, the level's output), three level-0 gradient
// buffers, and the unit and actnorm backward workspaces of the largest level.
struct StackWs {
    size_t acts, grads, unit_ws, an_ws, total;
};
StackWs stack_ws(const StackShape &s) {
    StackWs w;
    long long na = 0;
    for (int l = 0; l < s.L; ++l)
        na += (2ll * s.U + 1) * s.n(l);
    w.acts = up256b((size_t)na * sizeof(float));
    w.grads = 3 * up256b((size_t)s.n0 * sizeof(float));
    w.unit_ws = 0;
    w.an_ws = 0;
    for (int l = 0; l < s.L; ++l) {
        w.unit_ws = imax_sz(w.unit_ws, finc_unit_backward_workspace_bytes(s.B, s.C(l), s.H(l), s.W(l), s.k));
        w.an_ws = imax_sz(w.an_ws, finc_actnorm_backward_workspace_bytes(s.B, s.C(l), s.H(l), s.W(l)));
    }
    w.unit_ws = up256b(w.unit_ws);
    w.an_ws = up256b(w.an_ws);
    w.total = w.acts + w.grads + w.unit_ws + w.an_ws;
    return w;
}

// The forward direction, keeping every level's activations in acts (level l
// at acts + aoff[l]: h_0 = the level's input, t_0, h_1, t_1, ..., h_U = its
// output; t_u = unit(h_u), h_{u+1} = actnorm(t_u)); level 0's h_0 is x
// itself and the top level's h_U is written to its latent z[L-1] directly.
inline const float *stack_h(const float *x, const float *acts, const long long *aoff,
                            const StackShape &s, int l, int u) {
    return (l == 0 && u == 0) ? x : acts + aoff[l] + 2ll * u * s.n(l);
}

int stack_forward_keep(const float *x, float *const *z, const float *K, const float *scale,
                       const float *bias, const StackShape &s, float *acts, long long *aoff,
                       hipStream_t st) {
    long long o = 0;
    for (int l = 0; l < s.L; ++l) {
        const int C = s.C(l), H = s.H(l), W = s.W(l);
        const long long n = s.n(l), ksz = (long long)C * C * s.k * s.k;
        aoff[l] = o;
        o += (2ll * s.U + 1) * n;
        const bool top = l == s.L - 1;
        for (int u = 0; u < s.U; ++u) {
            const float *hu = stack_h(x, acts, aoff, s, l, u);
            float *tu = acts + aoff[l] + (2ll * u + 1) * n;
            float *nx = (top && u == s.U - 1) ? z[l] : tu + n;
            int rc = finc_unit_forward(hu, tu, K + s.koff(l) + 4ll * u * ksz, nullptr, nullptr,
                                       s.B, C, H, W, s.k, st);
            if (rc != FINC_OK)
                return rc;
            if (s.B > 0) {
                hipLaunchKernelGGL(affine_kernel, dim3(ew_blocks(n)), dim3(256), 0, st, tu, nx,
                                   scale + s.soff(l) + (long long)u * C,
                                   bias + s.soff(l) + (long long)u * C, (int)n, make_div(H * W),
                                   make_div(C), C);
                rc = conv_launched();
                if (rc != FINC_OK)
                    return rc;
            }
        }
        if (s.B == 0)
            continue;
        const float *hout = stack_h(x, acts, aoff, s, l, s.U);
        if (top) {
            if (s.U == 0 && hipMemcpyAsync(z[l], hout, (size_t)n * sizeof(float),
                                           hipMemcpyDeviceToDevice, st) != hipSuccess)
                return FINC_EHIP;
        } else {
            hipLaunchKernelGGL(split_squeeze_kernel, dim3(ew_blocks(n)), dim3(256), 0, st, hout,
                               acts + o, z[l], (int)n, C, H, W, make_div(H * W), make_div(C),
                               make_div(W));
            const int rc = conv_launched();
            if (rc != FINC_OK)
                return rc;
        }
    }
    return FINC_OK;
}

}  // namespace

extern "C" {

size_t finc_backward_workspace_bytes(int B, int C, int H, int W, int k) {
    if (!valid_bwd_shape(B, C, H, W, k))
        return 0;
    const int parts = dk_parts(B, C, H, W, k);
    return up256b((size_t)parts * C * C * k * k * sizeof(float));
}

int finc_backward(const float *x, const float *dy, const float *K, float *dx, float *dK,
                  double gld, int B, int C, int H, int W, int k, int corner, void *workspace,
                  hipStream_t stream) {
    if (!valid_bwd_shape(B, C, H, W, k) || corner < FINC_TL || corner > FINC_BR ||
        (B > 0 && (!x || !dy)) || !K || !workspace || ((uintptr_t)workspace & 255u))
        return FINC_EINVAL;
    const size_t act = (size_t)B * C * H * W * sizeof(float);
    const size_t wts = (size_t)C * C * k * k * sizeof(float);
    const size_t wsb = finc_backward_workspace_bytes(B, C, H, W, k);
    if (dx && (overlapb(dx, act, x, act) || overlapb(dx, act, dy, act) ||
               overlapb(dx, act, K, wts) || (dK && overlapb(dx, act, dK, wts)) ||
               overlapb(dx, act, workspace, wsb)))
        return FINC_EINVAL;
    if (dK && (overlapb(dK, wts, x, act) || overlapb(dK, wts, dy, act) ||
               overlapb(dK, wts, K, wts) || overlapb(dK, wts, workspace, wsb)))
        return FINC_EINVAL;
    if (overlapb(workspace, wsb, x, act) || overlapb(workspace, wsb, dy, act) ||
        overlapb(workspace, wsb, K, wts))
        return FINC_EINVAL;
    return launch_layer_backward(x, dy, K, dx, dK, gld, B, C, H, W, k, corner,
                                 (long long)C * H * W, (float *)workspace, stream);
}


// ---- backward of the FInC units ---------------------------------------------

size_t finc_unit_backward_workspace_bytes(int B, int C, int H, int W, int k) {
    if (!valid_bwd_shape(B, C, H, W, k))
        return 0;
    return 4 * up256b((size_t)B * C * H * W * sizeof(float)) +
           finc_backward_workspace_bytes(B, C, H, W, k);
}

int finc_unit_backward(const float *x, const float *dy, const float *K4, float *dx, float *dK4,
                       double gld, int B, int C, int H, int W, int k, void *workspace,
                       hipStream_t stream) {
    if (!valid_bwd_shape(B, C, H, W, k) || (B > 0 && (!x || !dy)) || !K4 || !workspace ||
        ((uintptr_t)workspace & 255u))
        return FINC_EINVAL;
    const size_t act = (size_t)B * C * H * W * sizeof(float);
    const size_t wts = 4 * (size_t)C * C * k * k * sizeof(float);
    const size_t wsb = finc_unit_backward_workspace_bytes(B, C, H, W, k);
    const void *ins[3] = {x, dy, K4};
    const size_t insz[3] = {act, act, wts};
    for (int i = 0; i < 3; ++i)
        if (overlapb(workspace, wsb, ins[i], insz[i]) || (dx && overlapb(dx, act, ins[i], insz[i])) ||
            (dK4 && overlapb(dK4, wts, ins[i], insz[i])))
            return FINC_EINVAL;
    if ((dx && (overlapb(dx, act, workspace, wsb) || (dK4 && overlapb(dx, act, dK4, wts)))) ||
        (dK4 && overlapb(dK4, wts, workspace, wsb)))
        return FINC_EINVAL;
    const size_t ksz = (size_t)C * C * k * k;
    char *w = (char *)workspace;
    const size_t slot = up256b(act);
    float *h[4] = {(float *)x, (float *)w, (float *)(w + slot), (float *)(w + 2 * slot)};
    float *g = (float *)(w + 3 * slot);
    float *partial = (float *)(w + 4 * slot);
    // the inputs of blocks TR, BL, BR, recomputed: h[q + 1] = block q (h[q])
    for (int q = 0; q < 3 && B > 0; ++q) {
        const int rc = finc_forward(h[q], h[q + 1], K4 + q * ksz, nullptr, nullptr, B, C, H, W,
                                    k, q, stream);
        if (rc != FINC_OK)
            return rc;
    }
    // blocks in reverse; the gradient alternates between g and the freed slots
    const float *gin = dy;
    float *gout[4] = {dx, g, h[3], g};   // block q writes its input gradient to gout[q]
    for (int q = 3; q >= 0; --q) {
        const int rc = launch_layer_backward(h[q], gin, K4 + q * ksz, gout[q],
                                             dK4 ? dK4 + q * ksz : nullptr, gld, B, C, H, W, k,
                                             q, (long long)C * H * W, partial, stream);
        if (rc != FINC_OK)
            return rc;
        gin = gout[q];
    }
    return FINC_OK;
}

size_t finc_split_backward_workspace_bytes(int B, int C, int H, int W, int k) {
    if (C % 4 != 0 || !valid_bwd_shape(B, C / 4, H, W, k))
        return 0;
    return finc_backward_workspace_bytes(B, C / 4, H, W, k);
}

int finc_split_backward(const float *x, const float *dy, const float *Kq4, float *dx,
                        float *dKq4, double gld, int B, int C, int H, int W, int k,
                        void *workspace, hipStream_t stream) {
    if (C % 4 != 0 || !valid_bwd_shape(B, C / 4, H, W, k) || (B > 0 && (!x || !dy)) || !Kq4 ||
        !workspace || ((uintptr_t)workspace & 255u))
        return FINC_EINVAL;
    const int q = C / 4;
    const size_t act = (size_t)B * C * H * W * sizeof(float);
    const size_t wts = 4 * (size_t)q * q * k * k * sizeof(float);
    const size_t wsb = finc_split_backward_workspace_bytes(B, C, H, W, k);
    const void *ins[3] = {x, dy, Kq4};
    const size_t insz[3] = {act, act, wts};
    for (int i = 0; i < 3; ++i)
        if (overlapb(workspace, wsb, ins[i], insz[i]) || (dx && overlapb(dx, act, ins[i], insz[i])) ||
            (dKq4 && overlapb(dKq4, wts, ins[i], insz[i])))
            return FINC_EINVAL;
    if ((dx && (overlapb(dx, act, workspace, wsb) || (dKq4 && overlapb(dx, act, dKq4, wts)))) ||
        (dKq4 && overlapb(dKq4, wts, workspace, wsb)))
        return FINC_EINVAL;
    const long long img = (long long)C * H * W, plane = (long long)q * H * W;
    const size_t ksz = (size_t)q * q * k * k;
    for (int g = 0; g < 4; ++g) {   // quarter g: corner g on channels [g q, (g+1) q)
        const int rc = launch_layer_backward(
            B > 0 ? x + g * plane : x, B > 0 ? dy + g * plane : dy, Kq4 + g * ksz,
            dx && B > 0 ? dx + g * plane : nullptr, dKq4 ? dKq4 + g * ksz : nullptr, gld, B, q,
            H, W, k, g, img, (float *)workspace, stream);
        if (rc != FINC_OK)
            return rc;
    }
    return FINC_OK;
}

// ---- actnorm backward and the negative log-likelihood -----------------------

size_t finc_actnorm_backward_workspace_bytes(int B, int C, int H, int W) {
    if (B < 0 || C < 1 || H < 1 || W < 1 || (long long)B * C * H * W >= (1ll << 31))
        return 0;
    return up256b((size_t)2 * C * actnorm_parts(B, C, H * W) * sizeof(double));
}

int finc_actnorm_backward(const float *x, const float *dy, const float *s, float *dx, float *ds,
                          float *db, double gld, int B, int C, int H, int W, void *workspace,
                          hipStream_t stream) {
    const size_t wsb = finc_actnorm_backward_workspace_bytes(B, C, H, W);
    if (wsb == 0 || (B > 0 && (!x || !dy)) || !s || !workspace || ((uintptr_t)workspace & 255u))
        return FINC_EINVAL;
    const size_t act = (size_t)B * C * H * W * sizeof(float), vec = (size_t)C * sizeof(float);
    const void *ins[3] = {x, dy, s};
    const size_t insz[3] = {act, act, vec};
    void *outs[4] = {dx, ds, db, workspace};
    const size_t outsz[4] = {act, vec, vec, wsb};
    for (int o = 0; o < 4; ++o) {
        if (!outs[o])
            continue;
        for (int i = 0; i < 3; ++i)
            if (overlapb(outs[o], outsz[o], ins[i], insz[i]))
                return FINC_EINVAL;
        for (int o2 = o + 1; o2 < 4; ++o2)
            if (outs[o2] && overlapb(outs[o], outsz[o], outs[o2], outsz[o2]))
                return FINC_EINVAL;
    }
    const int HW = H * W, parts = actnorm_parts(B, C, HW);
    const int bpp = B > 0 ? cdiv(B, parts) : 0;
    double *partial = (double *)workspace;
    const int np = B > 0 ? cdiv(B, bpp) : 0;   // parts that hold images
    if (np > 0) {
        const bool v4 = HW % 4 == 0 &&
                        (((uintptr_t)x | (uintptr_t)dy | (uintptr_t)dx) & 15u) == 0;
        if (v4)
            hipLaunchKernelGGL(actnorm_bwd_kernel<float4>, dim3(C, np), dim3(kAnThreads), 0, stream,
                               x, dy, s, dx, partial, B, C, HW, bpp, np, make_div(HW / 4));
        else
            hipLaunchKernelGGL(actnorm_bwd_kernel<float>, dim3(C, np), dim3(kAnThreads), 0, stream,
                               x, dy, s, dx, partial, B, C, HW, bpp, np, make_div(HW));
        const int rc = conv_launched();
        if (rc != FINC_OK)
            return rc;
    }
    if (!ds && !db)
        return FINC_OK;
    hipLaunchKernelGGL(actnorm_reduce_kernel, dim3((C + 63) / 64), dim3(64), 0, stream, partial,
                       np, s, ds, db, gld, C, HW);
    return conv_launched();
}

int finc_gauss_nll(const float *const *z, const long long *n, int L, int B, const double *logdet,
                   double *nll, double *bpd, hipStream_t stream) {
    if (L < 1 || L > kNllMaxL || B < 0 || !z || !n || !logdet || !nll)
        return FINC_EINVAL;
    NllArgs a;
    memset(&a, 0, sizeof(a));
    a.L = L;
    for (int l = 0; l < L; ++l) {
        if (n[l] < 1 || (B > 0 && !z[l]))
            return FINC_EINVAL;
        a.z[l] = z[l];
        a.n[l] = n[l];
        a.D += n[l];
    }
    const size_t per = (size_t)B * sizeof(double);
    if (overlapb(nll, per, logdet, per) || (bpd && (overlapb(bpd, per, logdet, per) ||
                                                    overlapb(bpd, per, nll, per))))
        return FINC_EINVAL;
    for (int l = 0; l < L; ++l) {
        const size_t zb = (size_t)B * n[l] * sizeof(float);
        if (overlapb(nll, per, z[l], zb) || (bpd && overlapb(bpd, per, z[l], zb)))
            return FINC_EINVAL;
    }
    a.logdet = logdet;
    a.nll = nll;
    a.bpd = bpd;
    if (B == 0)
        return FINC_OK;
    hipLaunchKernelGGL(gauss_nll_kernel, dim3(B), dim3(256), 0, stream, a);
    return conv_launched();
}


// ---- the multi-scale stack's training direction ------------------------------

size_t finc_stack_train_workspace_bytes(int B, int L, int U, int C1, int H1, int W1, int k) {
    StackShape s{B, L, U, C1, H1, W1, k, (long long)B * C1 * H1 * W1};
    if (!stack_shape_ok(s))
        return 0;
    return stack_ws(s).total;
}

static bool stack_buffers_ok(const StackShape &s, const float *x, const float *const *z,
                             const float *K, const float *scale, const float *bias,
                             void *workspace, const void *const *outs, const size_t *outsz,
                             int nouts) {
    if ((s.B > 0 && !x) || !z || !K || !scale || !bias || !workspace ||
        ((uintptr_t)workspace & 255u))
        return false;
    const size_t wsb = stack_ws(s).total;
    const size_t xb = (size_t)s.n0 * sizeof(float);
    const void *ins[4] = {x, K, scale, bias};
    const size_t insz[4] = {xb, (size_t)s.kfloats() * sizeof(float),
                            (size_t)s.sfloats() * sizeof(float),
                            (size_t)s.sfloats() * sizeof(float)};
    for (int l = 0; l < s.L; ++l)
        if (s.B > 0 && !z[l])
            return false;
    for (int i = 0; i < 4; ++i)
        if (overlapb(workspace, wsb, ins[i], insz[i]))
            return false;
    for (int o = 0; o < nouts; ++o) {
        if (!outs[o])
            continue;
        if (overlapb(outs[o], outsz[o], workspace, wsb))
            return false;
        for (int i = 0; i < 4; ++i)
            if (overlapb(outs[o], outsz[o], ins[i], insz[i]))
                return false;
        for (int o2 = o + 1; o2 < nouts; ++o2)
            if (outs[o2] && overlapb(outs[o], outsz[o], outs[o2], outsz[o2]))
                return false;
    }
    return true;
}

int finc_stack_forward(const float *x, float *const *z, double *logdet, const float *K,
                       const float *scale, const float *bias, int B, int L, int U, int C1,
                       int H1, int W1, int k, void *workspace, hipStream_t stream) {
    StackShape s{B, L, U, C1, H1, W1, k, (long long)B * C1 * H1 * W1};
    if (!stack_shape_ok(s) || !z)
        return FINC_EINVAL;
    const void *outs[10];
    size_t outsz[10];
    int no = 0;
    for (int l = 0; l < L; ++l) {
        outs[no] = z[l];
        outsz[no++] = (size_t)(l == L - 1 ? s.n(l) : s.n(l) / 2) * sizeof(float);
    }
    outs[no] = logdet;
    outsz[no++] = (size_t)B * sizeof(double);
    if (!stack_buffers_ok(s, x, (const float *const *)z, K, scale, bias, workspace, outs, outsz,
                          no))
        return FINC_EINVAL;
    long long aoff[8];
    int rc = stack_forward_keep(x, z, K, scale, bias, s, (float *)workspace, aoff, stream);
    if (rc != FINC_OK || !logdet || B == 0)
        return rc;
    hipLaunchKernelGGL(stack_logdet_kernel, dim3(1), dim3(256), 0, stream, K, scale, L, U, C1,
                       H1, W1, k, logdet, B);
    return conv_launched();
}

int finc_stack_backward(const float *x, const float *const *dz, const float *K,
                        const float *scale, const float *bias, float *dx, float *dK,
                        float *dscale, float *dbias, double gld, int B, int L, int U, int C1,
                        int H1, int W1, int k, void *workspace, hipStream_t stream) {
    StackShape s{B, L, U, C1, H1, W1, k, (long long)B * C1 * H1 * W1};
    if (!stack_shape_ok(s) || !dz)
        return FINC_EINVAL;
    const void *outs[4] = {dx, dK, dscale, dbias};
    const size_t outsz[4] = {(size_t)s.n0 * sizeof(float), (size_t)s.kfloats() * sizeof(float),
                             (size_t)s.sfloats() * sizeof(float),
                             (size_t)s.sfloats() * sizeof(float)};
    if (!stack_buffers_ok(s, x, dz, K, scale, bias, workspace, outs, outsz, 4))
        return FINC_EINVAL;
    for (int l = 0; l < L; ++l) {   // the latents' gradients are inputs too
        const size_t zb = (size_t)(l == L - 1 ? s.n(l) : s.n(l) / 2) * sizeof(float);
        for (int o = 0; o < 4; ++o)
            if (outs[o] && overlapb(outs[o], outsz[o], dz[l], zb))
                return FINC_EINVAL;
        if (overlapb(workspace, stack_ws(s).total, dz[l], zb))
            return FINC_EINVAL;
    }
    const StackWs w = stack_ws(s);
    char *base = (char *)workspace;
    float *acts = (float *)base;
    float *gbuf[3];
    for (int i = 0; i < 3; ++i)
        gbuf[i] = (float *)(base + w.acts + i * up256b((size_t)s.n0 * sizeof(float)));
    void *unit_ws = base + w.acts + w.grads, *an_ws = base + w.acts + w.grads + w.unit_ws;
    // the forward again, keeping its activations (the latents it writes go to
    // a gradient buffer, unused until the forward is done)
    float *zscratch[8];
    for (int l = 0; l < L; ++l)
        zscratch[l] = gbuf[2];
    long long aoff[8];
    int rc = stack_forward_keep(x, zscratch, K, scale, bias, s, acts, aoff, stream);
    if (rc != FINC_OK)
        return rc;
    // gin: the gradient of the activation reached so far (the top latent's
    // gradient first); results alternate between two buffers, the input's
    // gradient goes to dx
    float *buf[2] = {gbuf[0], gbuf[2]}, *gt = gbuf[1];
    int cur = 0;
    const float *gin = dz[L - 1];
    for (int l = L - 1; l >= 0; --l) {
        const int C = s.C(l), H = s.H(l), W = s.W(l);
        const long long n = s.n(l), ksz = (long long)C * C * k * k;
        if (l < L - 1 && B > 0) {   // gin: the next level's input gradient
            float *o = buf[cur];
            cur ^= 1;
            hipLaunchKernelGGL(unsqueeze_concat_kernel, dim3(ew_blocks(n)), dim3(256), 0, stream,
                               gin, dz[l], o, (int)n, C, H, W, make_div(H * W), make_div(C),
                               make_div(W));
            rc = conv_launched();
            if (rc != FINC_OK)
                return rc;
            gin = o;
        }
        for (int u = U - 1; u >= 0; --u) {
            const float *hu = stack_h(x, acts, aoff, s, l, u);
            const float *tu = acts + aoff[l] + (2ll * u + 1) * n;
            const long long so = s.soff(l) + (long long)u * C;
            rc = finc_actnorm_backward(tu, gin, scale + so, gt, dscale ? dscale + so : nullptr,
                                       dbias ? dbias + so : nullptr, gld, B, C, H, W, an_ws,
                                       stream);
            if (rc != FINC_OK)
                return rc;
            const bool last = l == 0 && u == 0;
            float *o = last ? dx : buf[cur];
            if (!last)
                cur ^= 1;
            rc = finc_unit_backward(hu, gt, K + s.koff(l) + 4ll * u * ksz, o,
                                    dK ? dK + s.koff(l) + 4ll * u * ksz : nullptr, gld, B, C, H,
                                    W, k, unit_ws, stream);
            if (rc != FINC_OK)
                return rc;
            gin = o;
        }
    }
    // (no unit at level 0: the input's gradient is the level's)
    if (dx && U == 0 && B > 0 &&
        hipMemcpyAsync(dx, gin, (size_t)s.n0 * sizeof(float), hipMemcpyDeviceToDevice, stream) !=
            hipSuccess)
        return FINC_EHIP;
    return FINC_OK;
}

}  // extern "C"
