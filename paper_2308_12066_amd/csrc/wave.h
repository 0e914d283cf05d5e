// Device code on the 64 lanes of one wavefront.
#ifndef PGMOE_WAVE_H
#define PGMOE_WAVE_H
#include <hip/hip_runtime.h>

namespace pgmoe {

// Inclusive prefix sum over the 64 lanes of a wavefront (all of them active) with data-parallel
// primitives: four shifts inside each row of 16 lanes, then lane 15 of row 0 / 2 into row 1 / 3
// and lane 31 into rows 2 and 3.  Six VALU operations instead of six trips through the LDS crossbar.
template <int CTRL, int ROW_MASK>
__device__ inline int dpp_or_zero(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);  // lanes without a source get 0
}
__device__ inline int wave_incl_scan(int v) {
    v += dpp_or_zero<0x111, 0xf>(v);  // row_shr:1
    v += dpp_or_zero<0x112, 0xf>(v);  // row_shr:2
    v += dpp_or_zero<0x114, 0xf>(v);  // row_shr:4
    v += dpp_or_zero<0x118, 0xf>(v);  // row_shr:8
    v += dpp_or_zero<0x142, 0xa>(v);  // row_bcast:15 -> rows 1 and 3
    v += dpp_or_zero<0x143, 0xc>(v);  // row_bcast:31 -> rows 2 and 3
    return v;
}

}  // namespace pgmoe
#endif  // PGMOE_WAVE_H
