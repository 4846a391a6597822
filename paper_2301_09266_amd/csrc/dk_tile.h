// dk_tile.h -- the weight gradient of a masked k x k layer, by blocks of 256
// threads, for the kernels that launch them alone or beside the input gradient.
#ifndef FINC_DK_TILE_H
#define FINC_DK_TILE_H

#include <type_traits>

#include "device_common.h"

namespace finc_detail {

// dK as a GEMM over positions, tap by tap: D_t[co][ci] = sum over positions of
// dy[co][pos] x[ci][pos + tap t].  A block takes one tile of 16 c_out x 16 c_in
// with up to nine taps over a part of the positions, in bands of up to 256
// positions of an image, or of several whole small images, one below the other
// (a band costs its latencies however few positions it has).  dy and x, with the
// k - 1 halo rows and columns its corner reads, are staged in LDS as
// [channel quad][pixel][4], so a tap is an LDS offset.  A step is four positions: one A read, then a B read and a
// v_mfma_f32_16x16x4_f32 a tap; the four waves take the steps in turn and their
// sums meet in order.  Part z covers bands [z bpp, (z+1) bpp) and writes its sums
// to partial + z C (C k^2); a single part writes dK itself.
//
// What bounds it: a few memory latencies and two barriers a band, and the matrix
// instructions (32 cycles a tap and four positions).  With the sum of the parts,
// 12 x 32 x 32, batch 64: 13.3 us, 48 x 8 x 8, batch 256: 26.9 us; staged column
// by column, with k^2 gathers and their index arithmetic an input value, 23.6 and
// 49.6 us; a band's reads a step ahead with running indices instead of the
// divisions 14.8 us (more registers, no less time).
struct DkArgs {
    const float *x, *dy, *K;
    float *partial, *dK;   // (dK: written in place of the sums of one part)
    double gld;
    long long img;   // floats from one image to the next (x and dy)
    int C, H, W, oh, ow, N;
    int B, ni;             // images; images of a band (more than one: whole images)
    int pr, pc;            // halo rows and columns of a band of x
    int form;              // of the bands, FORM below
    int RB, WB, nb, bpp;   // rows and columns of a band's image, bands, bands of a part
    int nbi, bx, nt;       // bands of an image, bands across it, channel tiles
    int parts, blocks;     // parts; blocks in all
    // divisions: nbi, bx, nt, nt^2, parts; the columns of a full and of the last
    // band across, and the same with the halo; rows of an image in a band of dy and x
    FastDiv d_nbi, d_bx, d_nt, d_nt2, d_parts, d_w, d_wl, d_xw, d_xwl, d_yr, d_xr;
};

// Forms of the bands (dk_tile).
enum { kDkOne = 0, kDkMulti = 1, kDkCrop = 2 };

// LDS pixels of a band of dy and of x with the halo, the quads' planes 16 floats apart modulo 64 (the reads of a
// step then fall in different banks).
constexpr int kDkPos = 256;
constexpr int dk_x(int k, bool multi) {
    return multi ? (k <= 3 ? 576 : 704) : (32 + k - 1) * (8 + k - 1);
}
constexpr int dk_plane(int n) { return (n + 11) / 16 * 16 + 4; }

// Entry (co, ci, t) of dK from its sum v over the positions: 0 where masked,
// the log|det| term on the self diagonal (in fp64).
__device__ inline float dk_entry(float v, int co, int ci, int t, const float *K, double gld, int C,
                                 int k, int H, int W, int oh, int ow) {
    if (t != oh * k + ow || ci < co)
        return v;
    if (ci > co)
        return 0.0f;
    return (float)((double)v +
                   gld * (double)H * (double)W / (double)K[(co * C + co) * k * k + t]);
}

// Taps of a block: all of k^2 <= 4, else nine.
constexpr int dk_taps(int k) { return k <= 2 ? k * k : 9; }

template <int K, int FORM>
constexpr int dk_lds_floats() {
    constexpr int st = 16 * (dk_plane(dk_x(K, FORM != kDkOne)) + dk_plane(kDkPos)), red = 4 * (dk_taps(K) + (FORM == kDkCrop)) * 16 * 17;
    return st > red ? st : red;
}

// Block blk of nt^2 parts groups, 256 threads, dk_lds_floats<K, FORM>() floats of LDS.
// FORM: kDkOne, or kDkMulti, bands that may hold several images, or kDkCrop,
// besides, images of fewer rows or columns than K, with only the halo that a tap
// can reach in one.  (Instances of their own: the image of a pixel costs the
// registers of a wave a SIMD, the taps outside the image 10 to 20%.)  BIG: images
// of 2 GB or more (no 32-bit offsets; kDkOne).
template <int K, int FORM, bool BIG>
__device__ __forceinline__ void dk_tile(const DkArgs &a, int blk, float *lds) {
    constexpr bool MULTI = FORM >= kDkMulti, CROP = FORM == kDkCrop;
    constexpr int G = dk_taps(K), K2 = K * K, P = K - 1;
    constexpr int XP = dk_plane(dk_x(K, MULTI)), YP = dk_plane(kDkPos);
    float *Xs = lds, *Ys = lds + 16 * XP;
    const int tid = threadIdx.x, lane = tid & 63, kq = lane >> 4, li = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pg = fdiv(blk, a.d_nt2), tile = blk - pg * a.nt * a.nt;
    const int tg = fdiv(pg, a.d_parts), part = pg - tg * a.parts, t0 = tg * G;
    const int cit = fdiv(tile, a.d_nt), cot = tile - cit * a.nt;
    const int HW = a.H * a.W;
    const int PR = CROP ? a.pr : P, PC = CROP ? a.pc : P;
    const int oh = CROP ? min(a.oh, PR) : a.oh, ow = CROP ? min(a.ow, PC) : a.ow;
    // (CROP: a tap that is outside the image wherever it is reads the positions
    // themselves, and takes its sums, of dy times zeros, from one of their own)
    constexpr int GA = CROP ? G + 1 : G;
    f32x4 acc[GA];
#pragma unroll
    for (int t = 0; t < GA; ++t)
        acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto inside = [&](int tt, int &ta, int &tb) __attribute__((always_inline)) {
        ta = tt / K - (CROP ? a.oh - oh : 0);
        tb = tt % K - (CROP ? a.ow - ow : 0);
        return !CROP || ((unsigned)ta <= (unsigned)PR && (unsigned)tb <= (unsigned)PC);
    };
    const int lq = li >> 2, le = li & 3;
    // n pixels of a region `cols` wide at (r0, c0) of each of nim images (`rows`
    // rows each), channels ch0 .. + 15, into dst: a thread takes a channel quad
    // of a pixel, U of them a round; zeros outside the image and past the
    // channels (raw buffer loads, which read 0 past the end: no branch, a round's
    // loads in flight together)
    auto stage = [&](auto uc, const float *src, float *dst, int plane, int n, int cols, const FastDiv &dc,
                     int rows, const FastDiv &dr, int nim, int r0, int c0, int ch0)
                     __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value;
        const unsigned nb = BIG ? 0u : (unsigned)((MULTI ? (nim - 1) * (int)a.img : 0) + a.C * HW) * 4u;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(src), (short)0, (int)nb, 0x00020000);
        for (int base = tid; base < 4 * n; base += 256 * U) {
            float v[U][4];
            int to[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = base + 256 * u, px = i >> 2, q = i & 3;
                const int pr = fdiv(px, dc), pc = px - pr * cols, im = MULTI ? fdiv(pr, dr) : 0;
                const int ii = r0 + pr - im * rows, jj = c0 + pc;
                const bool in = i < 4 * n && (unsigned)ii < (unsigned)a.H && (unsigned)jj < (unsigned)a.W;
                to[u] = i < 4 * n ? (q * plane + px) * 4 : -1;
                const int c0q = ch0 + 4 * q;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool ok = in && c0q + e < a.C;
                    if constexpr (BIG)
                        v[u][e] = ok ? src[(long long)(c0q + e) * HW + (long long)ii * a.W + jj] : 0.0f;
                    else
                        v[u][e] = __builtin_bit_cast(
                            float, __builtin_amdgcn_raw_buffer_load_b32(
                                       rs,
                                       (int)(ok ? (unsigned)((MULTI ? im * (int)a.img : 0) + (c0q + e) * HW +
                                                         ii * a.W + jj) * 4u
                                                : nb),
                                       0, 0));
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (to[u] >= 0)
                    *reinterpret_cast<float4 *>(dst + to[u]) =
                        make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
        }
    };
    const int band1 = min((part + 1) * a.bpp, a.nb);
    for (int band = part * a.bpp; band < band1; ++band) {
        const int ng = fdiv(band, a.d_nbi), r = band - ng * a.nbi, n = MULTI ? ng * a.ni : ng;
        const int br = fdiv(r, a.d_bx), bc = r - br * a.bx;
        const int r0 = br * a.RB, c0 = bc * a.WB, nim = MULTI ? min(a.ni, a.B - n) : 1;
        const int rb = min(a.RB, a.H - r0), wb = min(a.WB, a.W - c0), wx = wb + PC;
        const FastDiv dw = wb == a.WB ? a.d_w : a.d_wl, dxw = wb == a.WB ? a.d_xw : a.d_xwl;
        const int np = nim * rb * wb, steps = (np + 3) / 4;
        __syncthreads();   // the band before has been read
        stage(std::integral_constant<int, 3>{}, a.x + n * a.img, Xs, XP, nim * (rb + PR) * wx, wx, dxw,
              a.RB + PR, a.d_xr, nim, r0 - oh, c0 - ow, 16 * cit);
        stage(std::integral_constant<int, 4>{}, a.dy + n * a.img, Ys, YP, np, wb, dw, a.RB, a.d_yr, nim,
              r0, c0, 16 * cot);
        if (tid < 16 && np + (tid & 3) < 4 * steps)   // positions past the band's end
            *reinterpret_cast<float4 *>(Ys + ((tid >> 2) * YP + np + (tid & 3)) * 4) =
                make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        int off[G];   // of the taps (past the last one: the first again, unused)
#pragma unroll
        for (int t = 0; t < G; ++t) {
            const int tt = K2 > G ? (t0 + t < K2 ? t0 + t : 0) : t;
            int ta, tb;
            off[t] = inside(tt, ta, tb) ? (ta * wx + tb) * 4 : 0;
        }
        __syncthreads();
        auto step = [&](int s, auto end) __attribute__((always_inline)) {
            const int pos = 4 * s + kq, pp = min(pos, np - 1);
            int i = fdiv(pp, dw);
            const int j = pp - i * wb;
            if (MULTI)   // (the halo rows of the images above)
                i += fdiv(i, a.d_yr) * PR;
            const float av = Ys[(lq * YP + pos) * 4 + le];
            const float *xp = Xs + (lq * XP + i * wx + j) * 4 + le;
            float bv[G];
#pragma unroll
            for (int t = 0; t < G; ++t)
                bv[t] = xp[off[t]];
            if constexpr (decltype(end)::value) {
#pragma unroll
                for (int t = 0; t < G; ++t)
                    bv[t] = pos < np ? bv[t] : 0.0f;
            }
#pragma unroll
            for (int t = 0; t < G; ++t)
                acc[t] = mfma4(av, bv[t], acc[t]);
            if constexpr (CROP)
                acc[G] = mfma4(av, 0.0f, acc[G]);
        };
        // (a last step's positions past the band's end: dy = 0 times an infinite x
        // would be NaN)
        const int full = np >> 2;
        for (int s = wave; s < full; s += 4)
            step(s, std::false_type{});
        if (full < steps && (full & 3) == wave)
            step(full, std::true_type{});
    }
    // lane (kq, li) of a wave holds D_t[co 4 kq + rr][ci li]; the waves' sums in order
    __syncthreads();
#pragma unroll
    for (int t = 0; t < GA; ++t)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
            lds[((wave * GA + t) * 16 + 4 * kq + rr) * 17 + li] = acc[t][rr];
    __syncthreads();
    const int g = min(G, K2 - t0);
    float *pz = a.partial + (long long)part * a.C * a.N;
    const int row = tid >> 4, col = tid & 15, co = 16 * cot + row, ci = 16 * cit + col;
    if (co >= a.C || ci >= a.C)
        return;
    const long long o = (long long)co * a.N + ci * K2 + t0;
#pragma unroll
    for (int t = 0; t < G; ++t) {
        int from = t, ta, tb;
        if (CROP && !inside(t0 + t, ta, tb))
            from = G;
        auto at = [&](int w) { return lds[((w * GA + from) * 16 + row) * 17 + col]; };
        const float v = ((at(0) + at(1)) + at(2)) + at(3);
        if (t >= g)
            break;
        if (a.dK)
            a.dK[o + t] = dk_entry(v, co, ci, t0 + t, a.K, a.gld, a.C, K, a.H, a.W, a.oh, a.ow);
        else
            pz[o + t] = v;
    }
}

}  // namespace finc_detail

#endif  // FINC_DK_TILE_H
