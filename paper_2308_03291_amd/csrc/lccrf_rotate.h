// A vector-matrix product by ONE wave, lane = tag: the source values come by DPP row rotation, sixteen at a time, the blocks of sixteen
// tags by the gfx950 permlane swaps, and a lane's matrix entries stand in the order its rotations consume them.  (lccrf_lane.hip, lccrf_semi.hip)
#pragma once

#include "lccrf_device.h"

namespace lccrf {

// acc[0] + .. + acc[3] += sum over n of (a of the lane n places to the left in its row of sixteen) * e[n]
// (four accumulators: a lone wave sees the full latency of every dependent instruction).
#define LCCRF_FM(N, ACC, E) "v_fmac_f32_dpp %" #ACC ", %4, %" #E " row_ror:" #N " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ void fmac_rotations(float (&acc)[4], float a, const float (&e)[16]) {
    asm volatile("s_nop 1\n\t"  // a vector result needs two wait states before a DPP read
        "v_fmac_f32_e32 %0, %4, %5\n\t"
        LCCRF_FM(1, 1, 6) LCCRF_FM(2, 2, 7) LCCRF_FM(3, 3, 8) LCCRF_FM(4, 0, 9) LCCRF_FM(5, 1, 10) LCCRF_FM(6, 2, 11)
        LCCRF_FM(7, 3, 12) LCCRF_FM(8, 0, 13) LCCRF_FM(9, 1, 14) LCCRF_FM(10, 2, 15) LCCRF_FM(11, 3, 16)
        LCCRF_FM(12, 0, 17) LCCRF_FM(13, 1, 18) LCCRF_FM(14, 2, 19) LCCRF_FM(15, 3, 20)
        : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3])
        : "v"(a), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(e[4]), "v"(e[5]), "v"(e[6]), "v"(e[7]), "v"(e[8]),
          "v"(e[9]), "v"(e[10]), "v"(e[11]), "v"(e[12]), "v"(e[13]), "v"(e[14]), "v"(e[15]));
}
#undef LCCRF_FM
// The same with the accumulators' first terms as plain products: nothing has to be cleared.
#define LCCRF_FM(N, ACC, E) "v_fmac_f32_dpp %" #ACC ", %4, %" #E " row_ror:" #N " row_mask:0xf bank_mask:0xf\n\t"
#define LCCRF_ML(N, ACC, E) "v_mul_f32_dpp %" #ACC ", %4, %" #E " row_ror:" #N " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ void mul_rotations(float (&acc)[4], float a, const float (&e)[16]) {
    asm volatile("s_nop 1\n\t"
        "v_mul_f32_e32 %0, %4, %5\n\t"
        LCCRF_ML(1, 1, 6) LCCRF_ML(2, 2, 7) LCCRF_ML(3, 3, 8) LCCRF_FM(4, 0, 9) LCCRF_FM(5, 1, 10) LCCRF_FM(6, 2, 11)
        LCCRF_FM(7, 3, 12) LCCRF_FM(8, 0, 13) LCCRF_FM(9, 1, 14) LCCRF_FM(10, 2, 15) LCCRF_FM(11, 3, 16)
        LCCRF_FM(12, 0, 17) LCCRF_FM(13, 1, 18) LCCRF_FM(14, 2, 19) LCCRF_FM(15, 3, 20)
        : "=&v"(acc[0]), "=&v"(acc[1]), "=&v"(acc[2]), "=&v"(acc[3])
        : "v"(a), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(e[4]), "v"(e[5]), "v"(e[6]), "v"(e[7]), "v"(e[8]),
          "v"(e[9]), "v"(e[10]), "v"(e[11]), "v"(e[12]), "v"(e[13]), "v"(e[14]), "v"(e[15]));
}
#undef LCCRF_FM
#undef LCCRF_ML

// The blocks of sixteen tags of a vector, each in every row of sixteen lanes that meets it.  NBLK 1: 16 tags; 2: 32 tags, held twice, copy
// `copy` of the lane meeting one block; 3 and 4: 48 and 64 tags.
template <int NBLK>
__device__ __forceinline__ void rotation_blocks(float x, int copy, float (&Ab)[4]) {
    if constexpr (NBLK == 1) {
        Ab[0] = x;
    } else {
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
        if constexpr (NBLK == 2) {
            Ab[0] = copy == 0 ? __int_as_float(p[0]) : __int_as_float(p[1]);  // block `copy` in both rows of the copy
        } else {
            const auto y = __builtin_amdgcn_permlane32_swap(p[0], p[0], false, false);
            const auto w = __builtin_amdgcn_permlane32_swap(p[1], p[1], false, false);
            Ab[0] = __int_as_float(y[0]); Ab[2] = __int_as_float(y[1]);
            Ab[1] = __int_as_float(w[0]); Ab[3] = __int_as_float(w[1]);
        }
    }
}

}  // namespace lccrf
