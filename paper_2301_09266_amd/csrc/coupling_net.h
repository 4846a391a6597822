// coupling_net.h -- the coupling network of a Step in one launch, up to the
// tap products of its last convolution:
//
//   h1 = ReLU(W1 * va + b1)   3x3 "same", C/2 -> hid
//   h2 = ReLU(W2 h1 + b2)     1x1, hid -> hid
//   Z[9 c + t] = W3[c][.][t] h2   (nine 1x1 products per output channel; the
//                              shifted sum of conv_gemm.h makes the 3x3 of it)
//
// at fp32 precision on the bf16 matrix cores (the split of split_gemm.h: six
// products of three bf16 parts a value, the large one and the five small ones
// in accumulators of their own).
//
// Block: 512 threads, 32 pixels, every channel.  h1 and then h2 stay in LDS as
// bf16 parts, [plane][octet of channels][pixel][8] (96 KB at hid = 512), so
// nothing of the network but Z passes through memory.  A wave owns fragments
// of 32 output channels x 32 pixels (two of them at hid = 512); the weights go
// straight from L2 to its registers (no other wave needs them); no barrier
// inside a layer.  A kernel of its own first splits the weights and lays them
// out in the order the lanes read them, for as many Steps as the scratch holds
// (read in place, a load of a wave meets 32 rows, and tap rows no two
// neighbouring values).
//
// Why 32 pixels: all of hid = 512 channels of h1 must fit LDS, and the small
// levels of a flow have few pixels (1,600 at 4 x 4, batch 100).
//
// What bounds it: a tile reads all weights from L2 (2.4 MB with its input at C =
// 12, 98% of it hits: 78 GB/s a compute unit, 32 bytes a cycle, in each of the four
// rounds of 800 tiles on 256 compute units, the last of 32), with the matrix cores
// at 45% of their rate meanwhile; the small levels have fewer tiles than the chip
// compute units.  hid = 512, batch 100, against three fp32 GEMM launches:
// 12 x 16 x 16 304 -> 122 us, 24 x 8 x 8 132 -> 38 us, 48 x 4 x 4 87 -> 46 us.
//
// Sums that are not finite (infinite inputs, an overflow; the split parts of
// infinities meet opposite infinities and zeros) are computed again with the
// fp32 matrix instruction, as split_gemm.h does: the three layers launched one
// by one there give the same bits, order of sums included.
#ifndef FINC_COUPLING_NET_H
#define FINC_COUPLING_NET_H

#include "split_gemm.h"

namespace {

constexpr int kNetMaxHid = 512;   // h in LDS
constexpr int kNetThreads = 512, kNetWaves = 8, kNetPx = 32;
constexpr int kNetOct = kNetPx * 16;   // bytes of an octet of one plane

struct NetArgs {
    const float *v;   // level tensor, its first Ch channels are the input
    long long vs;     // floats from one image to the next
    const float *W1, *b1, *W2, *b2, *W3;
    const float *pk;  // the packed weights of W1, W2, W3
    float *Z;         // (B, 9 C, H, W)
    int B, Ch, C, hid, H, W;
    int n1, nh, nz;   // 32-value steps of conv1's K, fragments of hid and of 9 C
    Div d_HW, d_W;
};

// (the sums of up to four fragments change waves over the input window)
inline int net_x_bytes(int n1) { return 3 * kNetOct * 4 * n1 > 16384 ? 3 * kNetOct * 4 * n1 : 16384; }
inline size_t net_lds_bytes(const NetArgs &a) {
    return (size_t)3 * kNetOct * 4 * a.nh + net_x_bytes(a.n1) + 256 * a.nh;
}

// Packed weights of a layer with nf fragments of 32 rows and n steps of 32
// values of K: [fragment][step][half s][part][lane][8] in bf16, lane (lh, l32)
// holding row 32 f + l32, values 32 step + 16 s + 8 lh .. + 7 (zero where the
// row or value does not exist).  The three layers in turn.
constexpr int kNetStep = 1536;   // floats' worth of a fragment's step
inline long long net_pack_floats(int n1, int nh, int nz) {
    return (long long)kNetStep * (nh * n1 + nh * nh + nz * nh);
}

struct PackArgs {
    const float *W1, *W2, *W3;   // of the first Step
    long long ps, os;            // floats from one Step to the next: weights, packed
    float *out;
    int K1, C, hid, n1, nh, nz;
};

// blockIdx.y: the Step; a thread writes the three parts of eight values
__global__ __launch_bounds__(256) void net_pack_kernel(PackArgs a) {
    const int n = 128 * (a.nh * a.n1 + a.nh * a.nh + a.nz * a.nh);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n)
        return;
    int g = i >> 7, layer = 0;   // (fragment, step) of the layer
    if (g >= a.nh * a.n1) {
        g -= a.nh * a.n1;
        layer = 1;
        if (g >= a.nh * a.nh) {
            g -= a.nh * a.nh;
            layer = 2;
        }
    }
    const int ns = layer == 0 ? a.n1 : a.nh, f = g / ns, it = g - f * ns;
    const int l = i & 63, row = 32 * f + (l & 31), s = (i >> 6) & 1;
    const int k = 32 * it + s * 16 + (l >> 5) * 8;
    const int K = layer == 0 ? a.K1 : a.hid, rows = layer == 2 ? 9 * a.C : a.hid;
    const float *w = (layer == 0 ? a.W1 : layer == 1 ? a.W2 : a.W3) + blockIdx.y * a.ps;
    const int st = layer == 2 ? 9 : 1;
    w += layer == 2 ? (long long)(row / 9) * K * 9 + row % 9 : (long long)row * K;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        v[e] = row < rows && k + e < K ? w[(k + e) * st] : 0.0f;
    unsigned p[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        split2<false>(v[2 * j], v[2 * j + 1], p[j]);
    u32x4 *o = reinterpret_cast<u32x4 *>(a.out + blockIdx.y * a.os) + (i >> 6) * 192 + l;
#pragma unroll
    for (int t = 0; t < 3; ++t)
        o[64 * t] = u32x4{p[0][t], p[1][t], p[2][t], p[3][t]};
}

// This lane's weights of a 32-value step.
template <int NF>
__device__ __forceinline__ void net_load(const float *const (&wp)[NF], int it,
                                         u32x4 (&w)[NF][2][3]) {
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int t = 0; t < 3; ++t)
                w[f][s][t] = *reinterpret_cast<const u32x4 *>(wp[f] + it * kNetStep + s * 768 + t * 256);
}

// acc[f] = sum over 32-value steps it0 .. it1 - 1 of the packed weights wp[f]
// (of this lane; step it0's already in wa) times the LDS columns at b (planes
// PL bytes apart).  A step's loads of the next one's weights are spread over
// its products, one after each pair: in one group they would hold the wave (a
// 16-byte load of a wave takes the address unit 16 cycles, eight waves share
// it) and with it its products.  The LDS reads run half a step ahead.
template <int NF>
__device__ __forceinline__ void net_gemm(const float *const (&wp)[NF], int it0, int it1,
                                         u32x4 (&wa)[NF][2][3], const char *b, int PL,
                                         f32x16 (&hi)[NF]) {
    f32x16 lo[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            hi[f][r] = lo[f][r] = 0.0f;
    u32x4 wb[NF][2][3];
    bf16x8 fb[2][3];
    auto read = [&](int half, bf16x8 (&f)[3]) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 3; ++t)
            f[t] = *reinterpret_cast<const bf16x8 *>(b + half * 2 * kNetOct + t * PL);
    };
    // step it with weights w; loads step nx's into wn
    auto mul = [&](int it, const u32x4 (&w)[NF][2][3], int nx, u32x4 (&wn)[NF][2][3])
                   __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            read(s == 0 ? 2 * it + 1 : 2 * nx, fb[1 - s]);
            constexpr int ta[6] = {2, 0, 1, 1, 0, 0}, tb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int t = 0; t < 6; ++t) {
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const bf16x8 fa = __builtin_bit_cast(bf16x8, w[f][s][ta[t]]);
                    if (t < 5)
                        lo[f] = mfma_bf16(fa, fb[s][tb[t]], lo[f]);
                    else
                        hi[f] = mfma_bf16(fa, fb[s][tb[t]], hi[f]);
                }
                if (t < 3)
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        wn[f][s][t] = *reinterpret_cast<const u32x4 *>(
                            wp[f] + nx * kNetStep + s * 768 + t * 256);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    read(2 * it0, fb[0]);
    // (past the end: the last step's weights again, unused)
    int it = it0;
    for (; it + 2 <= it1; it += 2) {
        mul(it, wa, it + 1, wb);
        mul(it + 1, wb, min(it + 2, it1 - 1), wa);
    }
    if (it < it1)
        mul(it, wa, it, wb);
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            hi[f][r] += lo[f][r];
}

// Sums of fragment f of a layer (0, 1, 2: conv1, conv2, the tap rows) that are
// not finite, again with the fp32 matrix instruction: lane (lh, l32) feeds row
// / pixel l32 with k = 2 step + lh, the input read from memory (qi, qj: the
// pixel) or put together from its parts in LDS.
__device__ __forceinline__ void net_repair(const NetArgs &a, int layer, int f, f32x16 &acc,
                                           const float *xq, int qi, int qj, const char *Hs) {
    float nonfinite = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        nonfinite = fmaf(acc[r], 0.0f, nonfinite);
    if (!__any(nonfinite != 0.0f))
        return;
    const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5, co = 32 * f + l32;
    const int K = layer == 0 ? 9 * a.Ch : a.hid, rows = layer == 2 ? 9 * a.C : a.hid;
    const int PH = 4 * a.nh * kNetOct, HW = a.H * a.W, st = layer == 2 ? 9 : 1;
    const float *w = layer == 0   ? a.W1 + (long long)co * K
                     : layer == 1 ? a.W2 + (long long)co * K
                                  : a.W3 + (long long)(co / 9) * K * 9 + co % 9;
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        s[r] = 0.0f;
    for (int k0 = 0; k0 < K; k0 += 2) {
        const int k = k0 + lh;
        float wv = 0.0f, x = 0.0f;
        if (k < K) {
            if (co < rows)
                wv = w[k * st];
            if (layer == 0) {
                const int ci = k / 9, t = k - 9 * ci, di = t / 3 - 1, dj = t % 3 - 1;
                if ((unsigned)(qi + di) < (unsigned)a.H && (unsigned)(qj + dj) < (unsigned)a.W)
                    x = xq[(long long)ci * HW + di * a.W + dj];
            } else {
                const char *h = Hs + (k >> 3) * kNetOct + l32 * 16 + (k & 7) * 2;
                float p[3];
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    p[t] = __uint_as_float((unsigned)*reinterpret_cast<const uint16_t *>(h + t * PH) << 16);
                x = p[1] < INFINITY ? (p[0] + p[1]) + p[2] : p[1];   // (h >= 0: never NaN)
            }
        }
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, x, s, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
        if (!(fabsf(acc[r]) < INFINITY))
            acc[r] = s[r];
}

__global__ __launch_bounds__(kNetThreads, 2) void coupling_net_kernel(NetArgs a) {
    extern __shared__ __attribute__((aligned(16))) char nlds[];
    const int PH = 4 * a.nh * kNetOct, PX = 4 * a.n1 * kNetOct;
    char *Hs = nlds, *Xs = nlds + 3 * PH;
    // b1, b2, padded with zeros
    float *bs = reinterpret_cast<float *>(Xs + (3 * PX > 16384 ? 3 * PX : 16384));
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HW = a.H * a.W, Q = a.B * HW, n0 = blockIdx.x * kNetPx;
    const int K1 = 9 * a.Ch;
    const int q = min(n0 + l32, Q - 1), qb = divi(q, a.d_HW), qp = q - qb * HW;
    const int qi = divi(qp, a.d_W), qj = qp - qi * a.W;
    const float *xq = a.v + (long long)qb * a.vs + qp;
    const float *pk = a.pk + 4 * lane;   // packed weights of this lane
    // conv1's input window of the tile's pixels (thread: pixel l32), the biases
    auto stage = [&]() __attribute__((always_inline)) {
        for (int i = tid; i < 64 * a.nh; i += kNetThreads) {
            const int co = i < 32 * a.nh ? i : i - 32 * a.nh;
            const float v = (i < 32 * a.nh ? a.b1 : a.b2)[min(co, a.hid - 1)];
            bs[i] = co < a.hid ? v : 0.0f;
        }
        for (int o = tid >> 5; o < 4 * a.n1; o += kNetThreads / 32) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = 8 * o + e, ke = k < K1 ? k : 0, ci = ke / 9, t = ke - 9 * ci;
                const int di = t / 3 - 1, dj = t % 3 - 1;
                const bool ok = k < K1 && (unsigned)(qi + di) < (unsigned)a.H &&
                                (unsigned)(qj + dj) < (unsigned)a.W;
                const float v = xq[ok ? (long long)ci * HW + di * a.W + dj : 0];
                x[e] = ok ? v : 0.0f;
            }
            unsigned w[4][3];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                split2<false>(x[2 * i], x[2 * i + 1], w[i]);
#pragma unroll
            for (int t = 0; t < 3; ++t)
                *reinterpret_cast<u32x4 *>(Xs + t * PX + o * kNetOct + l32 * 16) =
                    u32x4{w[0][t], w[1][t], w[2][t], w[3][t]};
        }
    };
    // h = ReLU(acc + bias) of fragment f into LDS, register r of lane (lh,
    // l32) being channel 32 f + 8 (r / 4) + 4 lh + r % 4 of pixel l32
    auto put_h = [&](int f, const f32x16 &acc, const float *bias) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 b4 = *reinterpret_cast<const float4 *>(bias + 32 * f + 8 * g + 4 * lh);
            const float b[4] = {b4.x, b4.y, b4.z, b4.w};
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = fmaxf(acc[4 * g + e] + b[e], 0.0f);
            }
            unsigned p[2][3];
            split2<true>(v[0], v[1], p[0]);
            split2<true>(v[2], v[3], p[1]);
#pragma unroll
            for (int t = 0; t < 3; ++t)
                *reinterpret_cast<uint2 *>(Hs + t * PH + (4 * f + g) * kNetOct + l32 * 16 + lh * 8) =
                    make_uint2(p[0][t], p[1][t]);
        }
    };
    const char *xb = Xs + lh * kNetOct + l32 * 16, *hb = Hs + lh * kNetOct + l32 * 16;
    const float *pk2 = pk + a.nh * a.n1 * kNetStep, *pk3 = pk2 + a.nh * a.nh * kNetStep;
    // the wave's NF fragments of h1 and of h2 (a wave without one: NF = 1,
    // own = false)
    auto layers = [&](auto nf, bool own) __attribute__((always_inline)) {
        constexpr int NF = decltype(nf)::value;
        const float *wp1[NF], *wp2[NF];
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int f = own ? wave + kNetWaves * i : 0;
            wp1[i] = pk + f * a.n1 * kNetStep;
            wp2[i] = pk2 + f * a.nh * kNetStep;
        }
        u32x4 w[NF][2][3];
        f32x16 h[NF];
        net_load(wp1, 0, w);
        stage();
        __syncthreads();
        if (own) {
            net_gemm(wp1, 0, a.n1, w, xb, PX, h);
#pragma unroll
            for (int i = 0; i < NF; ++i)
                net_repair(a, 0, wave + kNetWaves * i, h[i], xq, qi, qj, Hs);
        }
        net_load(wp2, 0, w);
        if (own)
#pragma unroll
            for (int i = 0; i < NF; ++i)
                put_h(wave + kNetWaves * i, h[i], bs);
        __syncthreads();
        if (own) {
            net_gemm(wp2, 0, a.nh, w, hb, PH, h);
#pragma unroll
            for (int i = 0; i < NF; ++i)
                net_repair(a, 1, wave + kNetWaves * i, h[i], xq, qi, qj, Hs);
        }
        __syncthreads();   // every wave has read h1
        if (own)
#pragma unroll
            for (int i = 0; i < NF; ++i)
                put_h(wave + kNetWaves * i, h[i], bs + 32 * a.nh);
    };
    if (wave + kNetWaves < a.nh)
        layers(std::integral_constant<int, 2>{}, true);
    else
        layers(std::integral_constant<int, 1>{}, wave < a.nh);
    {   // tap rows 9 c + t
        const int rows3 = 9 * a.C;
        float *zq = a.Z + (long long)qb * rows3 * HW + qp;
        auto put_z = [&](int f, f32x16 &acc) __attribute__((always_inline)) {
            net_repair(a, 2, f, acc, xq, qi, qj, Hs);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 32 * f + 8 * (r / 4) + 4 * lh + r % 4;
                if (row < rows3 && n0 + l32 < Q)
                    zq[(long long)row * HW] = acc[r];
            }
        };
        // few fragments: waves w and w + 4 take half of K each, the second
        // half's sums through LDS
        const bool halves = a.nz <= kNetWaves / 2;
        const int part = halves ? wave >> 2 : 0, mid = (a.nh + 1) / 2;
        const int it0 = part * mid, it1 = halves && !part ? mid : a.nh;
        int f = halves ? wave & 3 : wave;
        if (f + kNetWaves < a.nz) {
            const float *const wp[2] = {pk3 + f * a.nh * kNetStep, pk3 + (f + kNetWaves) * a.nh * kNetStep};
            u32x4 w[2][2][3];
            f32x16 z[2];
            net_load(wp, 0, w);
            __syncthreads();
            net_gemm(wp, 0, a.nh, w, hb, PH, z);
            put_z(f, z[0]);
            put_z(f + kNetWaves, z[1]);
            f += 2 * kNetWaves;
        } else {
            __syncthreads();
        }
        f32x16 z[1];
        if (f < a.nz && it0 < it1) {
            const float *const wp[1] = {pk3 + f * a.nh * kNetStep};
            u32x4 w[1][2][3];
            net_load(wp, it0, w);
            net_gemm(wp, it0, it1, w, hb, PH, z);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                z[0][r] = 0.0f;
        }
        if (halves) {
            float4 *xs = reinterpret_cast<float4 *>(Xs) + f * 256 + lane;
            if (f < a.nz && part)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    xs[64 * g] = make_float4(z[0][4 * g], z[0][4 * g + 1], z[0][4 * g + 2],
                                             z[0][4 * g + 3]);
            __syncthreads();
            if (f < a.nz && !part)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 x = xs[64 * g];
                    z[0][4 * g] += x.x;
                    z[0][4 * g + 1] += x.y;
                    z[0][4 * g + 2] += x.z;
                    z[0][4 * g + 3] += x.w;
                }
        }
        if (f < a.nz && !part)
            put_z(f, z[0]);
    }
}

}  // namespace

#endif  // FINC_COUPLING_NET_H
