// The FP64 sums of the centre (mean position) inside single waves (device code), for few
// particles: bitwise what the two launches of the general path add, a first stage of one
// 256-particle block per 256 threads (tree over the threads, distances 128, 64, ... 1) and
// a second stage over the blocks' sums (the same tree).
#pragma once

#include "nbody_internal.h"

namespace nbody {
namespace centre {

struct Plus {
    __device__ double operator()(double a, double b) const { return a + b; }
};

// op(v, value of lane + W), for the lanes below W: the tree step of distance W inside a wave.
template <int W, class Op = Plus>
__device__ __forceinline__ double tree_step(double v, Op op = Op()) {
    const long long b = __double_as_longlong(v);
    const int lo = (int)b, hi = (int)(b >> 32);
    auto join = [](int l, int h) {
        return __longlong_as_double((long long)(((unsigned long long)(unsigned)h << 32) | (unsigned)l));
    };
    if constexpr (W == 32) {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        return op(join(l[0], h[0]), join(l[1], h[1]));
    } else if constexpr (W == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return op(join(l[0], h[0]), join(l[1], h[1]));
    } else {
        constexpr int kCtrl = W == 8 ? 0x128 :  // row_ror 8
                              W == 4 ? 0x12C :  // row_ror 12: lane l receives lane l + 4
                              W == 2 ? 0x4E :   // quad_perm [2, 3, 0, 1]
                                       0xB1;    // quad_perm [1, 0, 3, 2]
        return op(v, join(__builtin_amdgcn_mov_dpp(lo, kCtrl, 0xF, 0xF, false),
                          __builtin_amdgcn_mov_dpp(hi, kCtrl, 0xF, 0xF, false)));
    }
}

// The tree over 256 values, lane l holding those of threads l, l + 64, l + 128 and l + 192;
// lane 0 returns the result.
template <class Op>
__device__ __forceinline__ double wave_tree(const double (&v)[4], Op op) {
    double s = op(op(v[0], v[2]), op(v[1], v[3]));  // distances 128 and 64
    s = tree_step<32>(s, op);
    s = tree_step<16>(s, op);
    s = tree_step<8>(s, op);
    s = tree_step<4>(s, op);
    s = tree_step<2>(s, op);
    return tree_step<1>(s, op);
}

// First stage: the tree sum of a block; lane 0 returns it.
__device__ __forceinline__ double wave_sum(const double (&v)[4]) { return wave_tree(v, Plus()); }

// The tree sums of a block's 256 threads, NC values each (all threads must call it): wave c
// adds value c and returns the sum in its lane 0.  One barrier instead of one per distance,
// and the second stage without any: 8 Hermite steps of 4099 particles (a finalize with two
// first stages and a conversion with the second, each) 211 -> 202 us, a force from 10007 FP64
// positions 43.1 -> 42.4 us.
template <int NC>
__device__ __forceinline__ double block_sum(const double (&s)[NC], double (&sh)[NC][256]) {
    static_assert(NC <= 4, "a wave per value");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int c = 0; c < NC; ++c) sh[c][threadIdx.x] = s[c];
    __syncthreads();
    if (wave >= NC) return 0.0;
    double v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = sh[wave][k * 64 + lane];
    return wave_sum(v);
}

// Second stage over the kCentreBlocks partials [block][3] of the first, component c; every
// lane of the wave returns it.
__device__ __forceinline__ double partials_sum(const double *part, int c) {
    static_assert(kCentreBlocks == 256, "four partials per lane");
    const int lane = threadIdx.x & 63;
    double v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = part[(k * 64 + lane) * 3 + c];
    return __shfl(wave_sum(v), 0);
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
