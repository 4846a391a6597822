// split_gemm.h -- the flow's wide convolutions (64 output channels and more)
// as GEMMs on the bf16 matrix cores, at fp32 precision.
//
//   y[b][co][p] = act(bias[co] + sum_k W[co][k] X[k][b, p])
//
// for a 1x1 convolution (k = c_in), a 3x3 "same" convolution (X gathered) and
// the tap rows of conv_gemm.h.  Each fp32 operand is split exactly into three
// bf16 values, v = v0 + v1 + v2, each what is left rounded to nearest (the split
// of G. Henry, P. T. P. Tang and A. Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019), so that
// |v1| <= 2^-8 and |v2| <= 2^-17 of v's power of two, and the product keeps the
// six terms down to 2^-16 of v0 w0: the two of the three dropped that matter, v1
// w2 and v2 w1, are together at most 2^-24 of it, as one rounding to fp32, and of
// either sign (with v0 cut off instead of rounded 2^-22, and of one sign for some
// operands: 2.4e-7 whatever the sum's length).  v0 w0 goes to one fp32
// accumulator, the five smaller terms to another: the matrix core's adds
// truncate, and small terms added to the large sum would lose bits there.
// Error of the network against fp64 (12 x 8 x 8, batch 64, normal data), this and
// the fp32 matrix instruction: hid = 1 7.4e-8, 1.3e-7, 32 9.6e-8, 2.7e-7, 512
// 1.3e-7, 3.9e-7; all operands 1.0077972, hid = 16 5.9e-9, 7.1e-8.  Of a value below
// 2^-110 only the bits from 2^-133 on are kept (bf16 has no smaller ones).
// Infinities, NaNs and sums that overflow would meet zeros and opposite
// infinities of the split: sums that are not finite are computed again with the
// fp32 matrix instruction.
//
// What bounds it: six 32x32x16 bf16 instructions (32 cycles each) do the work
// of eight 32x32x2 fp32 ones (64 cycles each), 2.7 times the fp32 rate; the
// splits' vector work and one barrier a chunk leave half of that.  520 -> 520
// 1x1 on 25,600 pixels: 106 us (131 TFLOP/s; the fp32 instruction's rate 70).
//
// Block: 256 threads, BM output channels x BN pixels, 2 x 2 waves of (BM / 2)
// x (BN / 2), in 32 x 32 fragments.  K in chunks of NO octets (8 values): while
// a chunk's products run, the next chunk's values are split in registers and
// written to the other LDS buffer, and the loads of the one after are in
// flight; one barrier a chunk.  LDS holds [plane][octet][row][8], so every
// 16-byte access of a wave is contiguous over the rows.
#ifndef FINC_SPLIT_GEMM_H
#define FINC_SPLIT_GEMM_H

#include <type_traits>

#include "conv_gemm.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Two floats into their three bf16 parts (the first in the low half), each part
// what is left rounded to nearest.  KEPT: the first one does not round to
// infinity, so that the parts' sum is the value again (coupling_net.h holds h1 and
// h2 as parts alone, and the same products are taken here); else a sum with such
// a value is not finite and computed again from memory.
template <bool KEPT>
__device__ __forceinline__ void split2(float x, float y, unsigned (&w)[3]) {
    constexpr float kMax = 0x1.fefffep127f;   // the largest that rounds to a finite bf16
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const bool cap = KEPT && t == 0;
        const f32x2 v = {cap ? __builtin_amdgcn_fmed3f(x, -kMax, kMax) : x,
                         cap ? __builtin_amdgcn_fmed3f(y, -kMax, kMax) : y};
        w[t] = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
        if (t < 2) {
            x -= __uint_as_float(w[t] << 16);
            y -= __uint_as_float(w[t] & 0xffff0000u);
        }
    }
}

__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Bytes between the octets of a plane: the rows' 16 bytes each, and 32 more
// so that the weights' writes (neighbouring lanes hold octets of one row)
// fall in different banks.
template <int ROWS>
constexpr int split_oct() {
    return ROWS * 16 + 32;
}

template <int R, int BM, int BN, int NO, bool TROWS>
__global__ __launch_bounds__(256, 2) void split_gemm_kernel(ConvArgs a, int nco) {
    static_assert(R == 1 || !TROWS, "tap rows are 1x1 products");
    constexpr int FM = BM / 64, FN = BN / 64;             // 32 x 32 fragments of a wave
    constexpr int OA = split_oct<BM>(), OB = split_oct<BN>(), PA = NO * OA, PB = NO * OB;
    constexpr int UA = BM * NO / 256, UB = BN * NO / 256;   // octets a thread stages
    static_assert(UA >= 1 && UB >= 1, "every thread stages whole octets");
    constexpr int kBuf = 3 * (PA + PB);
    __shared__ __attribute__((aligned(16))) char lds[2 * kBuf];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;
    // blocks go to the eight XCDs in turn: the output-channel tiles of a
    // pixel tile are neighbours on one XCD, whose L2 then holds the pixels
    const int slot = (int)blockIdx.x >> 3, tn = ((int)blockIdx.x & 7) + 8 * (slot / nco);
    const int co0 = (slot % nco) * BM, n0 = tn * BN;
    const int HW = a.H * a.W, Q = a.B * HW;
    if (n0 >= Q)
        return;
    // whole chunks (R = 3: all of them, its gather zeroes what is past K), and
    // R = 1's last one when K is not a multiple of it
    const int nfull = R == 3 ? (a.K + 8 * NO - 1) / (8 * NO) : a.K / (8 * NO);

    // this thread's pixel (B) and weight rows (A); octets bo + (256 / BN) u of
    // a chunk are the same for a whole wave
    const int bpx = tid % BN, bo = __builtin_amdgcn_readfirstlane(tid / BN);
    const int q = min(n0 + bpx, Q - 1), qb = divi(q, a.d_HW), qp = q - qb * HW;
    const float *xq = a.x + (long long)qb * a.xs + qp;
    unsigned tapok = 0;   // (R = 3) taps of the pixel inside the image
    if constexpr (R == 3) {
        const int qi = divi(qp, a.d_W), qj = qp - qi * a.W;
#pragma unroll
        for (int t = 0; t < 9; ++t)
            if ((unsigned)(qi + t / 3 - 1) < (unsigned)a.H &&
                (unsigned)(qj + t % 3 - 1) < (unsigned)a.W)
                tapok |= 1u << t;
    }
    // weights W[row][k]: rows of K values, a thread's octets side by side with
    // its neighbours'; tap rows W[9 c + t][k] = M[c][k][t]: neighbouring
    // threads take neighbouring rows, whose values are side by side.  Raw
    // buffer loads: rows that do not exist, and values past the last row, read
    // 0; past the end of another row they meet zeros of B.
    const int ao = TROWS ? tid / BM : tid % NO, arow = TROWS ? tid % BM : tid / NO;
    const int wend = a.Co * a.K * 4;   // bytes (at most 4096 x 9 x 4096 floats)
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.Wt), (short)0, wend, 0x00020000);
    constexpr int kStep = TROWS ? 36 : 4;   // bytes from k to k + 1
    int wrow[UA];
#pragma unroll
    for (int u = 0; u < UA; ++u) {
        const int co = co0 + arow + (TROWS ? 0 : u * (256 / NO));
        const int k0 = 8 * (ao + (TROWS ? u * (256 / BM) : 0));
        wrow[u] = co < a.Co ? (TROWS ? (co / 9 * a.K * 9 + co % 9) * 4 : co * a.K * 4) + k0 * kStep
                            : wend;
    }
    auto load_a = [&](int c, float (&v)[UA][8]) __attribute__((always_inline)) {
        const int at = c * 8 * NO * kStep;
#pragma unroll
        for (int u = 0; u < UA; ++u) {
            if constexpr (TROWS) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[u][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                            rw, wrow[u] + e * kStep, at, 0));
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h) {   // (a buffer load needs 4-byte alignment only)
                    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rw, wrow[u] + 16 * h, at, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[u][4 * h + e] = __uint_as_float(w[e]);
                }
            }
        }
    };
    auto load_b = [&](int c, float (&v)[UB][8], auto whole) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            const int k = 8 * (NO * c + bo + (256 / BN) * u);   // wave-uniform
            if constexpr (R == 1) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const bool ok = decltype(whole)::value || k + e < a.K;
                    const float x = xq[(long long)(ok ? k + e : 0) * HW];
                    v[u][e] = ok ? x : 0.0f;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int ke = min(k + e, a.K - 1), ci = ke / 9, t = ke - 9 * ci;
                    const bool ok = (tapok >> t & (k + e < a.K ? 1u : 0u)) != 0;
                    const long long off = (long long)ci * HW + (t / 3 - 1) * a.W + t % 3 - 1;
                    const float x = xq[ok ? off : 0];
                    v[u][e] = ok ? x : 0.0f;
                }
            }
        }
    };
    auto put = [&](const float (&v)[8], char *dst, int plane, auto kept) __attribute__((always_inline)) {
        unsigned w[4][3];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            split2<decltype(kept)::value>(v[2 * i], v[2 * i + 1], w[i]);
#pragma unroll
        for (int t = 0; t < 3; ++t)
            *reinterpret_cast<u32x4 *>(dst + t * plane) = u32x4{w[0][t], w[1][t], w[2][t], w[3][t]};
    };
    auto store = [&](int c, const float (&va)[UA][8], const float (&vb)[UB][8])
                     __attribute__((always_inline)) {
        char *As = lds + (c & 1) * kBuf, *Bs = As + 3 * PA;
#pragma unroll
        for (int u = 0; u < UA; ++u)
            put(va[u], TROWS ? As + (ao + u * (256 / BM)) * OA + arow * 16
                             : As + ao * OA + (arow + u * (256 / NO)) * 16, PA,
                std::false_type{});
#pragma unroll
        for (int u = 0; u < UB; ++u)
            put(vb[u], Bs + (bo + (256 / BN) * u) * OB + bpx * 16, PB, std::integral_constant<bool, R == 1>{});
    };

    f32x16 hi[FM][FN], lo[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                hi[i][j][r] = lo[i][j][r] = 0.0f;
    const char *ar = lds + lh * OA + (wm * (BM / 2) + l32) * 16;
    const char *br = lds + 3 * PA + lh * OB + (wn * (BN / 2) + l32) * 16;
    // Up to 128 tap rows are summed in two halves of K (of whole 32-value
    // steps), as coupling_net.h does with them: the same bits from either.
    const int mid = TROWS && a.Co <= 128 ? ((a.K + 31) / 32 + 1) / 2 * 32 : 0;
    f32x16 first[FM][FN];
    auto half = [&](int k) __attribute__((always_inline)) {   // k: values summed so far
        if constexpr (TROWS && FM * FN == 1) {
            if (k == mid) {   // (mid = 0: before anything)
                first[0][0] = hi[0][0] + lo[0][0];
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    hi[0][0][r] = lo[0][0][r] = 0.0f;
            }
        }
    };
    // the products of a chunk in LDS buffer c & 1
    auto products = [&](int c) __attribute__((always_inline)) {
        const int buf = (c & 1) * kBuf;
#pragma unroll
        for (int s = 0; s < NO / 2; ++s) {   // 16 values of k each
            bf16x8 fa[FM][3], fb[FN][3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    fa[i][t] =
                        *reinterpret_cast<const bf16x8 *>(ar + buf + 2 * s * OA + t * PA + i * 512);
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    fb[j][t] =
                        *reinterpret_cast<const bf16x8 *>(br + buf + 2 * s * OB + t * PB + j * 512);
            }
            constexpr int ta[5] = {2, 0, 1, 1, 0}, tb[5] = {0, 2, 1, 0, 1};
#pragma unroll
            for (int t = 0; t < 5; ++t)
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        lo[i][j] = mfma_bf16(fa[i][ta[t]], fb[j][tb[t]], lo[i][j]);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    hi[i][j] = mfma_bf16(fa[i][0], fb[j][0], hi[i][j]);
        }
    };
    if (nfull > 0) {
        float ra[2][UA][8], rb[2][UB][8];
        const int last = nfull - 1;
        load_a(0, ra[0]);
        load_b(0, rb[0], std::true_type{});
        load_a(min(1, last), ra[1]);
        load_b(min(1, last), rb[1], std::true_type{});
        store(0, ra[0], rb[0]);
        __syncthreads();
        // chunk c: its products, chunk c + 1 (in registers ca, cb) into LDS,
        // the loads of chunk c + 2 into na, nb.  (No branch: after the last
        // chunk its own values are loaded and stored again, unread.)
        auto step = [&](int c, float (&ca)[UA][8], float (&cb)[UB][8], float (&na)[UA][8],
                        float (&nb)[UB][8]) __attribute__((always_inline)) {
            load_a(min(c + 2, last), na);
            load_b(min(c + 2, last), nb, std::true_type{});
            half(8 * NO * c);
            products(c);
            store(c + 1, ca, cb);
            __syncthreads();
        };
        int c = 0;
        for (; c + 2 <= nfull; c += 2) {
            step(c, ra[1], rb[1], ra[0], rb[0]);
            step(c + 1, ra[0], rb[0], ra[1], rb[1]);
        }
        if (c < nfull)
            step(c, ra[1], rb[1], ra[0], rb[0]);
    }
    if (R == 1 && nfull * 8 * NO < a.K) {   // the rest of K
        float va[UA][8], vb[UB][8];
        load_a(nfull, va);
        load_b(nfull, vb, std::false_type{});
        store(nfull, va, vb);
        __syncthreads();
        half(8 * NO * nfull);
        products(nfull);
    }
    float nonfinite = 0.0f;   // NaN as soon as one sum is not finite
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                hi[i][j][r] += lo[i][j][r];
                if (TROWS && FM * FN == 1 && mid > 0 && mid < a.K)
                    hi[i][j][r] = first[i][j][r] + hi[i][j][r];
                nonfinite = fmaf(hi[i][j][r], 0.0f, nonfinite);
            }
    const int cow = co0 + wm * (BM / 2), nw = n0 + wn * (BN / 2);
    if (__any(nonfinite != 0.0f)) {
        // the fp32 matrix instruction, straight from memory: lane (lh, l32)
        // feeds row / pixel l32 of a fragment with k = 2 step + lh
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int co = cow + 32 * i + l32, qq = min(nw + 32 * j + l32, Q - 1);
                const int b = divi(qq, a.d_HW), p = qq - b * HW, pi = divi(p, a.d_W), pj = p - pi * a.W;
                const float *xp = a.x + (long long)b * a.xs + p;
                const float *wp = TROWS ? a.Wt + (long long)(co / 9) * a.K * 9 + co % 9
                                        : a.Wt + (long long)co * a.K;
                f32x16 acc;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[r] = 0.0f;
                for (int k0 = 0; k0 < a.K; k0 += 2) {
                    const int k = k0 + lh;
                    float w = 0.0f, x = 0.0f;
                    if (k < a.K) {
                        if (co < a.Co)
                            w = wp[TROWS ? k * 9 : k];
                        const int ci = R == 1 ? k : k / 9, t = R == 1 ? 4 : k - 9 * ci;
                        const int di = t / 3 - 1, dj = t % 3 - 1;
                        if ((unsigned)(pi + di) < (unsigned)a.H && (unsigned)(pj + dj) < (unsigned)a.W)
                            x = xp[(long long)ci * HW + di * a.W + dj];
                    }
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w, x, acc, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (!(fabsf(hi[i][j][r]) < INFINITY))
                        hi[i][j][r] = acc[r];
            }
    }
    // register r of lane (lh, l32): channel 8 (r / 4) + 4 lh + r % 4, pixel l32
    auto out = [&](auto whole) {   // whole: every channel of the tile exists
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int cb = cow + 32 * i + 4 * lh;
            float bv[16], sv[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int co = cb + 8 * (r / 4) + r % 4;
                const bool ok = decltype(whole)::value || co < a.Co;
                bv[r] = a.bias && ok ? a.bias[co] : 0.0f;
                sv[r] = a.ls && ok ? expf(3.0f * a.ls[co]) : 1.0f;
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int qo = nw + 32 * j + l32;
                if (qo < Q) {
                    const int b = divi(qo, a.d_HW), p = qo - b * HW;
                    float *yq = a.y + (long long)b * a.ys + p + (long long)cb * HW;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        float v = hi[i][j][r] + bv[r];
                        if (a.relu)
                            v = fmaxf(v, 0.0f);
                        if (decltype(whole)::value || cb + 8 * (r / 4) + r % 4 < a.Co)
                            yq[(long long)(8 * (r / 4) + r % 4) * HW] = v * sv[r];
                    }
                }
            }
        }
    };
    if (co0 + BM <= a.Co)
        out(std::true_type{});
    else
        out(std::false_type{});
}

constexpr long long kWideSmallGrid = 256;   // blocks: one per compute unit

template <int R, int BM, int BN, int NO, bool TROWS>
void launch_split_tile(const ConvArgs &a, hipStream_t st) {
    const int nco = cdiv(a.Co, BM), npx = cdiv((long long)a.B * a.H * a.W, BN);
    hipLaunchKernelGGL((split_gemm_kernel<R, BM, BN, NO, TROWS>), dim3((npx + 7) / 8 * 8 * nco),
                       dim3(256), 0, st, a, nco);
}

template <int R, bool TROWS>
void launch_split(const ConvArgs &a, hipStream_t st) {
    const long long Q = (long long)a.B * a.H * a.W;
    // (up to 128 tap rows: the tile that sums in halves)
    if (!(TROWS && a.Co <= 128) && (long long)cdiv(a.Co, 128) * cdiv(Q, 128) >= kWideSmallGrid)
        launch_split_tile<R, 128, 128, 2, TROWS>(a, st);
    else
        launch_split_tile<R, 64, 64, 4, TROWS>(a, st);
}

}  // namespace

#endif  // FINC_SPLIT_GEMM_H
