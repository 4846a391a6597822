// finc_detail.h -- calls between the library's translation units that are not
// part of its ABI.
#ifndef FINC_DETAIL_H
#define FINC_DETAIL_H

#include <hip/hip_runtime_api.h>

namespace finc_detail {

struct DkArgs;

// dx = J^T dy of one layer (arguments checked by the caller), images img floats
// apart in dy and dx, and in the same launch dk.blocks blocks of dk_tile.h;
// FINC_EUNSUPPORTED, with nothing launched, where the forward's plan is and where
// the caller's implicit GEMM is the better one.
__attribute__((visibility("hidden"))) int layer_grads(const float *dy, float *dx, const float *K,
                                                      int B, int C, int H, int W, int k,
                                                      int corner, long long img, const DkArgs &dk,
                                                      hipStream_t stream);

}  // namespace finc_detail

#endif  // FINC_DETAIL_H
