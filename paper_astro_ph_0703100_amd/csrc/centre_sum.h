// The FP64 sums of the centre (mean position) inside single waves (device code), for few
// particles: bitwise what the two launches of the general path add, a first stage of one
// 256-particle block per 256 threads (tree over the threads, distances 128, 64, ... 1) and
// a second stage over the blocks' sums (the same tree).
#pragma once

#include "nbody_internal.h"

namespace nbody {
namespace centre {

// v + (value of lane + W, for the lanes below W), the tree step of distance W inside a wave.
template <int W>
__device__ __forceinline__ double tree_step(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = (int)b, hi = (int)(b >> 32);
    auto join = [](int l, int h) {
        return __longlong_as_double((long long)(((unsigned long long)(unsigned)h << 32) | (unsigned)l));
    };
    if constexpr (W == 32) {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        return join(l[0], h[0]) + join(l[1], h[1]);
    } else if constexpr (W == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return join(l[0], h[0]) + join(l[1], h[1]);
    } else {
        constexpr int kCtrl = W == 8 ? 0x128 :  // row_ror 8
                              W == 4 ? 0x12C :  // row_ror 12: lane l receives lane l + 4
                              W == 2 ? 0x4E :   // quad_perm [2, 3, 0, 1]
                                       0xB1;    // quad_perm [1, 0, 3, 2]
        return v + join(__builtin_amdgcn_mov_dpp(lo, kCtrl, 0xF, 0xF, false),
                        __builtin_amdgcn_mov_dpp(hi, kCtrl, 0xF, 0xF, false));
    }
}

// First stage: the tree sum of a block whose threads l, l + 64, l + 128 and l + 192 hold
// lane l's four values; lane 0 returns it.
__device__ __forceinline__ double wave_sum(const double (&v)[4]) {
    double s = (v[0] + v[2]) + (v[1] + v[3]);  // distances 128 and 64
    s = tree_step<32>(s);
    s = tree_step<16>(s);
    s = tree_step<8>(s);
    s = tree_step<4>(s);
    s = tree_step<2>(s);
    return tree_step<1>(s);
}

// Second stage over sh[0 .. chunks), chunks <= 32 (the other blocks hold zeros: the tree's
// distances above 16 add nothing); every lane returns it.
__device__ __forceinline__ double second_stage(const double *sh, int chunks, int lane) {
    double s = lane < chunks ? sh[lane & 31] : 0.0;
    s = tree_step<16>(s);
    s = tree_step<8>(s);
    s = tree_step<4>(s);
    s = tree_step<2>(s);
    s = tree_step<1>(s);
    return __shfl(s, 0);
}

}  // namespace centre
}  // namespace nbody
