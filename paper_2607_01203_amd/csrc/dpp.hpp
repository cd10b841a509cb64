// dpp.hpp -- sums over neighbouring lanes by data-parallel-primitive moves.
#pragma once
#include <hip/hip_runtime.h>

namespace leb {

// x + x of the partner lane of a data-parallel-primitive pattern (no LDS):
// 0xB1, 0x4E: lanes 1, 2 away within four; 0x141, 0x140: mirrored within eight, sixteen
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
    union { double d; int w[2]; } u;
    u.d = x;
    u.w[0] = __builtin_amdgcn_mov_dpp(u.w[0], CTRL, 0xf, 0xf, true);
    u.w[1] = __builtin_amdgcn_mov_dpp(u.w[1], CTRL, 0xf, 0xf, true);
    return x + u.d;
}
__device__ __forceinline__ double sum4(double x) { return dpp_add<0x4E>(dpp_add<0xB1>(x)); }
__device__ __forceinline__ double sum8(double x) { return dpp_add<0x141>(sum4(x)); }
__device__ __forceinline__ double sum16(double x) { return dpp_add<0x140>(sum8(x)); }

}  // namespace leb
