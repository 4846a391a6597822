// device_common.h -- what the kernels of several translation units share.
#ifndef FINC_DEVICE_COMMON_H
#define FINC_DEVICE_COMMON_H

#include <hip/hip_runtime.h>

namespace finc_detail {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Division of a non-negative int by a divisor fixed on the host, as a
// multiply-high and two shifts (Granlund and Montgomery's round-up method:
// l = ceil(log2 d), m = floor(2^32 (2^l - d) / d) + 1; exact for every
// 32-bit dividend).
struct FastDiv {
    unsigned m;
    int s1, s2;
};
inline FastDiv make_fastdiv(int d) {
    int l = 0;
    while ((1ull << l) < (unsigned long long)d)
        ++l;
    FastDiv f;
    f.m = (unsigned)((((1ull << l) - (unsigned long long)d) << 32) / (unsigned long long)d + 1);
    f.s1 = l < 1 ? l : 1;
    f.s2 = l > 1 ? l - 1 : 0;
    return f;
}
__device__ inline int fdiv(int x, const FastDiv &f) {
    const unsigned t = __umulhi(f.m, (unsigned)x);
    return (int)((t + (((unsigned)x - t) >> f.s1)) >> f.s2);
}

}  // namespace finc_detail

#endif  // FINC_DEVICE_COMMON_H
