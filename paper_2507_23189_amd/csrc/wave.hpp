// Reductions over a wave's rows of 16 lanes, without LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace mcmie {

// v with its lanes permuted within rows of 16 (a DPP control).
template <int CTRL>
__device__ __forceinline__ double row_move(double v)
{
    const int2 x = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, int2{__builtin_amdgcn_mov_dpp(x.x, CTRL, 0xF, 0xF, true),
                                           __builtin_amdgcn_mov_dpp(x.y, CTRL, 0xF, 0xF, true)});
}
// op over each row of 16 lanes, in every lane: exchanges between neighbours,
// pairs, the halves of 8 and of 16 (quad_perm 1032 and 2301, row_half_mirror,
// row_mirror).
template <class Op>
__device__ __forceinline__ double row_reduce(double v, Op op)
{
    v = op(v, row_move<0xB1>(v));
    v = op(v, row_move<0x4E>(v));
    v = op(v, row_move<0x141>(v));
    return op(v, row_move<0x140>(v));
}

}  // namespace mcmie
