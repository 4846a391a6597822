// conv_gemm.h -- an R x R convolution with per-axis offsets as an fp32 MFMA
// implicit GEMM on gfx950 (v_mfma_f32_16x16x4_f32), shared by the full flow (the
// narrow convolutions: fewer than 64 output channels) and the backward of the
// masked layer (its input gradient, a convolution of the output gradient, where
// it does not run as the forward), and the shifted sum of the taps' products
// that the wide ones (split_gemm.h, coupling_net.h) end with.
//
//   y[b][co][i][j] = act(bias[co] + sum_{ci,a,c} Wt[co][ci][a][c] *
//                        x[b][ci][i + a - ph][j + c - pw]) * oscale[co]
//
// zeros outside the image; act = ReLU or identity; oscale = exp(3 ls[co]) or
// 1; bias may be null (0).  Weights are OIHW, so W[co][k] with
// k = ci R^2 + a R + c is contiguous in k.  Pixels are flattened over the
// batch (q = b H W + p), so a block's tile may span images.
//
// Block: 256 threads, 4 waves arranged WCO (along c_out) x 4 / WCO (along
// pixels); each wave computes 16 c_out x 16 NS pixels.  K is staged conv_kc
// values at a time (32 or 64): A[co][k] (weights) and B[px][k] (the gathered
// input window, im2col on the fly), rows padded by four floats, the next chunk's
// global loads in flight during the current chunk's MFMAs.  Within one 16-wide
// slice of k, lane group kq takes k = 4 kq .. 4 kq + 3 as the four MFMAs' k (one
// float4 LDS read each for A and B).  A long K may be split into parts
// (blockIdx.z) whose raw sums a second kernel adds in order.  Every summation
// order is fixed: results are bitwise deterministic.
#ifndef FINC_CONV_GEMM_H
#define FINC_CONV_GEMM_H

#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include "device_common.h"
#include "finc.h"

using namespace finc_detail;

namespace {

inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

typedef FastDiv Div;
inline Div make_div(int d) { return make_fastdiv(d); }
__device__ inline int divi(int x, const Div &f) { return fdiv(x, f); }

struct ConvArgs {
    const float *x;
    float *y;
    const float *Wt;     // (Co, Ci, R, R)
    const float *bias;   // (Co) or null
    const float *ls;     // (Co) or null
    int relu;
    int B, Ci, Co, H, W, K;   // K = Ci R^2
    int ph, pw;               // input row / column offset: i + a - ph, j + c - pw
    long long xs, ys;         // floats from one image to the next
    Div d_HW, d_W;
    // split over K (blockIdx.z = part): part z sums chunks [z cps, (z+1) cps)
    // and writes its raw sums to partial + z Co Q (c_out-major)
    float *partial;
    int cps;
    // flip: Wt is a (Co, Co, R, R) kernel M read transposed over channels and
    // flipped in space, W[co][ci][a][c] = M[ci][co][R-1-a][R-1-c], with the
    // entries at M's tap fself zeroed where M's input channel exceeds its
    // output channel (co > ci here): the input gradient's weights of a
    // masked convolution with kernel M.
    int flip, fself;
};

constexpr int kConvThreads = 256;

// k values staged at a time (KC): 32 for the 64 c_out x 64 px tile (half the
// LDS of 64, so twice the blocks a compute unit holds), 64 for the narrow
// tiles (a block's 16 weight rows are staged by 256 threads a quad each).
template <int WCO>
constexpr int conv_kc() {
    return WCO == 4 ? 32 : 64;
}

// LDS floats of one block of the <WCO, NS> configuration (rows of conv_kc + 4
// floats).
template <int WCO, int NS>
constexpr int conv_lds_floats() {
    return (16 * WCO + 16 * NS * (4 / WCO)) * (conv_kc<WCO>() + 4);
}

// One output tile (bx along pixels, by along c_out, bz the part of K) with
// the block's LDS at lds (conv_lds_floats<WCO, NS>() floats, 16-byte aligned).
// ACC: accumulators of a sum, 1, or 4 (k mod 4, joined pairwise: a quarter of
// the rounding chain, as the forward's sums).
template <int R, int WCO, int NS, int ACC = 1>
__device__ __forceinline__ void conv_tile(const ConvArgs &a, int bx, int by, int bz, float *lds) {
    constexpr int BM = 16 * WCO, BN = 16 * NS * (4 / WCO), KC = conv_kc<WCO>();
    constexpr int SK = KC + 4, KQ = KC / 4;   // row stride, quads per chunk row
    constexpr int TPP = kConvThreads / BN;   // threads per staged pixel
    constexpr int QPT = KQ / TPP;            // k quads per thread (B)
    constexpr int AQ = BM * KQ / kConvThreads;   // weight quads per thread
    static_assert(QPT >= 1 && AQ >= 1, "every thread stages whole quads");
    float *As = lds, *Bs = lds + BM * SK;
    const int tid = threadIdx.x, lane = tid & 63, kq = lane >> 4, li = lane & 15;
    const int wave = tid >> 6, wco = wave % WCO, wpx = wave / WCO;
    const int co0 = by * BM;
    const int n0 = bx * BN;
    const int HW = a.H * a.W, Q = a.B * HW;

    // this thread's staged pixel and its window's validity per tap
    const int spx = tid % BN, sk0 = tid / BN;   // pixel slot; first k quad
    const int q = n0 + spx;
    const bool qok = q < Q;
    const int qb = qok ? divi(q, a.d_HW) : 0, qp = qok ? q - qb * HW : 0;
    const int qi = divi(qp, a.d_W), qj = qp - qi * a.W;
    unsigned long long tapok = 0;
#pragma unroll
    for (int t = 0; t < R * R; ++t) {
        const int ii = qi + t / R - a.ph, jj = qj + t % R - a.pw;
        if (qok && ii >= 0 && ii < a.H && jj >= 0 && jj < a.W)
            tapok |= 1ull << t;
    }
    const float *xq = a.x + (long long)qb * a.xs + qp;

    float ra[AQ][4], rb[QPT][4];
    auto load_chunk = [&](int k0) {
#pragma unroll
        for (int u = 0; u < AQ; ++u) {
            const int idx = tid + u * kConvThreads;
            const int col = idx / KQ, kk = k0 + 4 * (idx % KQ);
            const int co = co0 + col;
            const float *w = a.Wt + (long long)(co < a.Co ? co : 0) * a.K;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bool ok = co < a.Co && kk + e < a.K;
                long long off = kk + e;
                if (a.flip) {   // M[ci][co][R^2 - 1 - t], t = a R + c
                    const int ci = (int)((unsigned)(kk + e) / (R * R));
                    const int t = R * R - 1 - (kk + e - ci * R * R);
                    off = ((long long)ci * a.Co + co) * (R * R) + t;
                    ok = ok && !(t == a.fself && co > ci);
                }
                const float v = (a.flip ? a.Wt : w)[ok ? off : 0];
                ra[u][e] = ok ? v : 0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < QPT; ++u) {
            const int kk = k0 + 4 * (sk0 + u * TPP);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = kk + e;
                const int ci = (int)((unsigned)k / (R * R));
                const int t = k - ci * R * R;
                const int ta = t / R, tb = t - ta * R;
                const bool ok = k < a.K && ((tapok >> t) & 1ull);
                const long long off = (long long)ci * HW + (ta - a.ph) * a.W + (tb - a.pw);
                const float v = xq[ok ? off : 0];
                rb[u][e] = ok ? v : 0.0f;
            }
        }
    };
    auto store_chunk = [&] {
#pragma unroll
        for (int u = 0; u < AQ; ++u) {
            const int idx = tid + u * kConvThreads;
            *reinterpret_cast<float4 *>(&As[(idx / KQ) * SK + 4 * (idx % KQ)]) =
                make_float4(ra[u][0], ra[u][1], ra[u][2], ra[u][3]);
        }
#pragma unroll
        for (int u = 0; u < QPT; ++u)
            *reinterpret_cast<float4 *>(&Bs[spx * SK + 4 * (sk0 + u * TPP)]) =
                make_float4(rb[u][0], rb[u][1], rb[u][2], rb[u][3]);
    };

    f32x4 sum[ACC][NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int v = 0; v < ACC; ++v)
            sum[v][s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int nall = (a.K + KC - 1) / KC;
    const int cbeg = a.partial ? bz * a.cps : 0;
    const int nchunk = a.partial ? min(a.cps, nall - cbeg) : nall;
    load_chunk(cbeg * KC);
    store_chunk();
    __syncthreads();
    const float *arow = &As[(wco * 16 + li) * SK + 4 * kq];
    const float *brow = &Bs[(wpx * 16 * NS + li) * SK + 4 * kq];
    for (int c = 0; c < nchunk; ++c) {
        if (c + 1 < nchunk)
            load_chunk((cbeg + c + 1) * KC);   // in flight during the MFMAs
#pragma unroll
        for (int blk = 0; blk < KC / 16; ++blk) {
            const float4 w4 = *reinterpret_cast<const float4 *>(arow + 16 * blk);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const float4 b4 = *reinterpret_cast<const float4 *>(brow + 16 * s * SK + 16 * blk);
                sum[0][s] = mfma4(w4.x, b4.x, sum[0][s]);
                sum[1 % ACC][s] = mfma4(w4.y, b4.y, sum[1 % ACC][s]);
                sum[2 % ACC][s] = mfma4(w4.z, b4.z, sum[2 % ACC][s]);
                sum[3 % ACC][s] = mfma4(w4.w, b4.w, sum[3 % ACC][s]);
            }
        }
        if (c + 1 < nchunk) {
            __syncthreads();
            store_chunk();
            __syncthreads();
        }
    }
    f32x4 acc[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
        acc[s] = ACC == 4 ? (sum[0][s] + sum[1 % ACC][s]) + (sum[2 % ACC][s] + sum[3 % ACC][s])
                          : sum[0][s];
    if (a.partial) {   // raw sums of this part of K
        float *pz = a.partial + (long long)bz * a.Co * Q;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int qo = n0 + wpx * 16 * NS + 16 * s + li;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int co = co0 + wco * 16 + 4 * kq + rr;
                if (qo < Q && co < a.Co)
                    pz[(long long)co * Q + qo] = acc[s][rr];
            }
        }
        return;
    }
    // epilogue: lane (kq, li) holds c_out 4 kq + rr of pixel li of each slot
    float bv[4], sv[4];
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        const int co = co0 + wco * 16 + 4 * kq + rr;
        const int cc = co < a.Co ? co : 0;
        bv[rr] = a.bias ? a.bias[cc] : 0.0f;
        sv[rr] = a.ls ? expf(3.0f * a.ls[cc]) : 1.0f;
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int qo = n0 + wpx * 16 * NS + 16 * s + li;
        if (qo >= Q)
            continue;
        const int b = divi(qo, a.d_HW), p = qo - b * HW;
        float *yq = a.y + (long long)b * a.ys + p;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int co = co0 + wco * 16 + 4 * kq + rr;
            if (co < a.Co) {
                float v = acc[s][rr] + bv[rr];
                if (a.relu)
                    v = fmaxf(v, 0.0f);
                yq[(long long)co * HW] = v * sv[rr];
            }
        }
    }
}

template <int R, int WCO, int NS>
__global__ __launch_bounds__(kConvThreads) void conv_kernel(ConvArgs a) {
    __shared__ __attribute__((aligned(16))) float lds[conv_lds_floats<WCO, NS>()];
    conv_tile<R, WCO, NS>(a, blockIdx.x, blockIdx.y, blockIdx.z, lds);
}

// The parts of a K-split convolution added in order (part 0 first), then
// bias, ReLU and the output scale, as the unsplit kernel's epilogue does.
__global__ __launch_bounds__(256) void conv_reduce_kernel(ConvArgs a, int parts) {
    const int Q = a.B * a.H * a.W, HW = a.H * a.W;
    const long long n = (long long)a.Co * Q;
    for (long long e = blockIdx.x * 256ll + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const int co = (int)(e / Q), q = (int)(e - (long long)co * Q);
        float v = 0.0f;
        for (int z = 0; z < parts; ++z)
            v += a.partial[(long long)z * n + e];
        v += a.bias ? a.bias[co] : 0.0f;
        if (a.relu)
            v = fmaxf(v, 0.0f);
        if (a.ls)
            v *= expf(3.0f * a.ls[co]);
        const int b = divi(q, a.d_HW), p = q - b * HW;
        a.y[(long long)b * a.ys + (long long)co * HW + p] = v;
    }
}

int conv_launched() { return hipGetLastError() == hipSuccess ? FINC_OK : FINC_EHIP; }

// Parts a narrow convolution's K is split into (at most; their partial sums
// take kMaxParts Co B H W floats).
constexpr int kMaxParts = 8;

// The shifted sum of the nine tap rows of each channel of a tap-rows GEMM
// Z (B, 9 C, H, W): y[b][c][i][j] = (bias[c] + sum over taps t = 3 a + d, in
// order, of Z[b][9 c + t][i + a - 1][j + d - 1], zero outside) * exp(3 ls[c]).
__global__ __launch_bounds__(256) void shift_add_kernel(const float *Z, float *y, long long ys,
                                                        const float *bias, const float *ls,
                                                        int B, int C, int H, int W, Div d_HW,
                                                        Div d_W, Div d_C) {
    const int HW = H * W, n = B * C * HW;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256) {
        const int pl = divi(e, d_HW), p = e - pl * HW;
        const int b = divi(pl, d_C), c = pl - b * C;
        const int i = divi(p, d_W), j = p - i * W;
        const float *zb = Z + (long long)b * 9 * C * HW;
        float v = 0.0f;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int ii = i + t / 3 - 1, jj = j + t % 3 - 1;
            if (ii >= 0 && ii < H && jj >= 0 && jj < W)
                v += zb[(long long)(9 * c + t) * HW + ii * W + jj];
        }
        v += bias ? bias[c] : 0.0f;
        if (ls)
            v *= expf(3.0f * ls[c]);
        y[(long long)b * ys + (long long)c * HW + p] = v;
    }
}

// Arguments of an R x R "same" convolution.
inline ConvArgs conv_args(const float *x, long long xs, float *y, long long ys, const float *Wt,
                          const float *bias, const float *ls, int relu, int B, int Ci, int Co,
                          int H, int W, int R) {
    ConvArgs a;
    memset(&a, 0, sizeof(a));
    a.x = x;
    a.y = y;
    a.Wt = Wt;
    a.bias = bias;
    a.ls = ls;
    a.relu = relu;
    a.B = B;
    a.Ci = Ci;
    a.Co = Co;
    a.H = H;
    a.W = W;
    a.K = Ci * R * R;
    a.ph = a.pw = (R - 1) / 2;
    a.xs = xs;
    a.ys = ys;
    a.d_HW = make_div(H * W);
    a.d_W = make_div(W);
    return a;
}

// A narrow R x R "same" convolution (C_out < 64, compile-time instances of
// R).  A long K is split into parts of at least 8 chunks, so that the grid
// covers the chip: the number of parts depends on K only (not on the batch)
// and the parts are added in order, so results stay deterministic and
// independent of B.  partial: kMaxParts Co B H W floats, or null (no split).
template <int R>
int launch_conv_r(ConvArgs a, hipStream_t st, float *partial) {
    const long long Q = (long long)a.B * a.H * a.W;
    const int nchunk = cdiv(a.K, conv_kc<1>());
    int parts = 1;
    if (partial)
        while (parts < kMaxParts && nchunk >= 16 * parts)
            parts *= 2;
    a.cps = cdiv(nchunk, parts);
    parts = cdiv(nchunk, a.cps);
    a.partial = parts > 1 ? partial : nullptr;
    const dim3 grid(cdiv(Q, 128), cdiv(a.Co, 16), parts);
    hipLaunchKernelGGL((conv_kernel<R, 1, 2>), grid, dim3(kConvThreads), 0, st, a);
    if (parts > 1) {
        const int rc = conv_launched();
        if (rc != FINC_OK)
            return rc;
        const long long n = (long long)a.Co * Q;
        hipLaunchKernelGGL(conv_reduce_kernel, dim3((unsigned)(n / 256 + 1 < 8192 ? n / 256 + 1 : 8192)),
                           dim3(256), 0, st, a, parts);
    }
    return conv_launched();
}

}  // namespace

#endif  // FINC_CONV_GEMM_H
