// Force-jerk-potential pipelines (device code, included by the .hip files that launch
// them): force, jerk and potential in one pass, as in the pipeline of the
// paper's Appendix A (the interaction of a fourth-order Hermite integrator, Sec. 4.1).
// With d = x_j - x_i, w = v_j - v_i and s^2 = |d|^2 + eps^2:
//   a_i    +=  m_j d / s^3
//   jerk_i +=  m_j (w - 3 (d.w / s^2) d) / s^3
//   phi_i  -=  m_j / s
// j-records are 8 floats (x, y, z, m, vx, vy, vz, 0: two LDS reads per j); i-records
// hold position and velocity.  27 FP32 VALU operations and one v_rsq_f32 per pair.
// Three pipelines: FP32 inputs (GravityJerk), FP64 state relative to per-i-tile centres
// (GravityJerkTile), and separate i- and j-sets (GravityJerkIJ).
#pragma once

#include "tile_engine.h"

namespace nbody {
namespace {

// One pair term, instruction by instruction, in the order and with the s_nop that gfx950 runs
// fastest (see gravity_pair_timed): d, s^2 as an FMA chain and w; d.w; 1/s from the hardware
// reciprocal square root; m/s, m/s^3 and 3 d.w/s^2; w - (3 d.w/s^2) d; the sums.  The engine
// hands the j == i pair a massless record (null_j): with d and w exactly zero and m = 0 it
// adds exactly zero to a, the jerk and phi.
#define NBODY_JERK_PAIR(POT_INSTR)                                                            \
    asm("v_sub_f32 %[dx], %[jx], %[xi]\n\t"                                                   \
        "v_sub_f32 %[dy], %[jy], %[yi]\n\t"                                                   \
        "v_sub_f32 %[dz], %[jz], %[zi]\n\t"                                                   \
        "v_fma_f32 %[t], %[dx], %[dx], %[e2]\n\t"                                             \
        "v_fmac_f32 %[t], %[dy], %[dy]\n\t"                                                   \
        "v_fmac_f32 %[t], %[dz], %[dz]\n\t"                                                   \
        "v_sub_f32 %[wx], %[jvx], %[vxi]\n\t"                                                 \
        "v_sub_f32 %[wy], %[jvy], %[vyi]\n\t"                                                 \
        "v_sub_f32 %[wz], %[jvz], %[vzi]\n\t"                                                 \
        "v_mul_f32 %[q], %[dx], %[wx]\n\t"                                                    \
        "v_fmac_f32 %[q], %[dy], %[wy]\n\t"                                                   \
        "v_fmac_f32 %[q], %[dz], %[wz]\n\t"                                                   \
        "s_nop 0\n\t"                                                                         \
        "v_rsq_f32 %[t], %[t]\n\t"                                                            \
        "s_nop 0\n\t"                                                                         \
        "v_mul_f32 %[u], %[t], %[t]\n\t"                                                      \
        "v_mul_f32 %[t], %[jm], %[t]\n\t"                                                     \
        "v_mul_f32 %[q], %[q], %[u]\n\t"                                                      \
        "v_mul_f32 %[u], %[t], %[u]\n\t"                                                      \
        "v_mul_f32 %[q], 0x40400000, %[q]\n\t"                                                \
        "v_fma_f32 %[wx], -%[q], %[dx], %[wx]\n\t"                                            \
        "v_fma_f32 %[wy], -%[q], %[dy], %[wy]\n\t"                                            \
        "v_fma_f32 %[wz], -%[q], %[dz], %[wz]\n\t"                                            \
        "v_fmac_f32 %[ax], %[u], %[dx]\n\t"                                                   \
        "v_fmac_f32 %[ay], %[u], %[dy]\n\t"                                                   \
        "v_fmac_f32 %[az], %[u], %[dz]\n\t"                                                   \
        "v_fmac_f32 %[bx], %[u], %[wx]\n\t"                                                   \
        "v_fmac_f32 %[by], %[u], %[wy]\n\t"                                                   \
        "v_fmac_f32 %[bz], %[u], %[wz]\n\t" POT_INSTR                                         \
        : [ax] "+&v"(acc[0]), [ay] "+&v"(acc[1]), [az] "+&v"(acc[2]), [bx] "+&v"(acc[3]),     \
          [by] "+&v"(acc[4]), [bz] "+&v"(acc[5]), [ph] "+&v"(acc[6]), [dx] "=&v"(dx),         \
          [dy] "=&v"(dy), [dz] "=&v"(dz), [wx] "=&v"(wx), [wy] "=&v"(wy), [wz] "=&v"(wz),     \
          [t] "=&v"(t), [u] "=&v"(u), [q] "=&v"(q)                                            \
        : [jx] "v"(j[0]), [jy] "v"(j[1]), [jz] "v"(j[2]), [jm] "v"(j[3]), [jvx] "v"(j[4]),    \
          [jvy] "v"(j[5]), [jvz] "v"(j[6]), [xi] "v"(xi), [yi] "v"(yi), [zi] "v"(zi),         \
          [vxi] "v"(vxi), [vyi] "v"(vyi), [vzi] "v"(vzi), [e2] "s"(eps2))

template <bool POT>
__device__ __forceinline__ void jerk_pair_timed(const float *j, float xi, float yi, float zi,
                                                float vxi, float vyi, float vzi, float eps2,
                                                float (&acc)[7]) {
    float dx, dy, dz, wx, wy, wz, t, u, q;
    if constexpr (POT)
        NBODY_JERK_PAIR("v_sub_f32 %[ph], %[ph], %[t]\n\t");
    else
        NBODY_JERK_PAIR("");
}
#undef NBODY_JERK_PAIR

struct GravityJerk {
    static constexpr int kJWords = 8;
    static constexpr int kOut = 7;  // ax, ay, az, jx, jy, jz, phi
    // 14 two-sum operations per block of 128 pairs (64 before: 1.6 % slower, and at
    // 256-j tiles the four unrolled blocks took 85 VGPRs, 5 waves per SIMD).
    static constexpr int kBlockJ = nbody::kBlockJ;
    static constexpr int kMaxIpl = 2;
    static constexpr bool kLone = false;
    using Args = JerkArgs;
    struct IState {
        float x, y, z, vx, vy, vz;
    };
    struct Ctx {};
    static __device__ __forceinline__ int n_i(const Args &a) { return a.n; }
    static __device__ __forceinline__ int n_j(const Args &a) { return a.n; }
    static __device__ __forceinline__ Ctx make_ctx(const Args &, int) { return {}; }
    static __device__ __forceinline__ IState load_i(const Args &a, const Ctx &, int i) {
        return {a.x[i], a.y[i], a.z[i], a.vx[i], a.vy[i], a.vz[i]};
    }
    static __device__ __forceinline__ void load_j(const Args &a, const Ctx &, int b, unsigned j, float (&r)[8]) {
        r[0] = (a.x + b)[j];
        r[1] = (a.y + b)[j];
        r[2] = (a.z + b)[j];
        r[3] = (a.m + b)[j];
        r[4] = (a.vx + b)[j];
        r[5] = (a.vy + b)[j];
        r[6] = (a.vz + b)[j];
        r[7] = 0.0f;
    }
    // A massless particle at rest at the origin: every term carries m = 0.
    static __device__ __forceinline__ void pad_j(float (&r)[8]) {
#pragma unroll
        for (int c = 0; c < 8; ++c) r[c] = 0.0f;
    }
    // The j == i pair: same position and velocity, no mass.
    static constexpr bool kSelf = true;
    static __device__ __forceinline__ void null_j(float (&r)[8]) { r[3] = 0.0f; }
    template <bool POT, bool MANY>
    static __device__ __forceinline__ void pair_timed(const float *j, const IState &i, float eps2,
                                                      float (&acc)[kOut]) {
        jerk_pair_timed<POT>(j, i.x, i.y, i.z, i.vx, i.vy, i.vz, eps2, acc);
    }
};

// FP64 state relative to the block's i-tile centres (mean position and mean velocity):
// the i-records and every staged j-record are converted as fp32(x - c_I), fp32(v - w_I),
// so the pair arithmetic sees the tile's own scale.  For j == i both conversions are the
// same operation and d = w = 0 exactly.
struct GravityJerkTile {
    static constexpr int kJWords = 8;
    static constexpr int kOut = 7;
    static constexpr int kBlockJ = GravityJerk::kBlockJ;
    static constexpr int kMaxIpl = 2;
    static constexpr bool kLone = false;
    using Args = JerkTileArgs;
    using IState = GravityJerk::IState;
    struct Ctx {
        double cx, cy, cz, wx, wy, wz;
    };
    static __device__ __forceinline__ int n_i(const Args &a) { return a.n; }
    static __device__ __forceinline__ int n_j(const Args &a) { return a.n; }
    static __device__ __forceinline__ Ctx make_ctx(const Args &a, int i0) {
        const size_t t = 3 * (size_t)(i0 / a.itile);
        return {a.cx[t], a.cx[t + 1], a.cx[t + 2], a.cv[t], a.cv[t + 1], a.cv[t + 2]};
    }
    static __device__ __forceinline__ IState load_i(const Args &a, const Ctx &c, int i) {
        return {(float)(a.x[i] - c.cx),  (float)(a.y[i] - c.cy),  (float)(a.z[i] - c.cz),
                (float)(a.vx[i] - c.wx), (float)(a.vy[i] - c.wy), (float)(a.vz[i] - c.wz)};
    }
    static __device__ __forceinline__ void load_j(const Args &a, const Ctx &c, int b, unsigned j, float (&r)[8]) {
        r[0] = (float)((a.x + b)[j] - c.cx);
        r[1] = (float)((a.y + b)[j] - c.cy);
        r[2] = (float)((a.z + b)[j] - c.cz);
        r[3] = (a.m + b)[j];
        r[4] = (float)((a.vx + b)[j] - c.wx);
        r[5] = (float)((a.vy + b)[j] - c.wy);
        r[6] = (float)((a.vz + b)[j] - c.wz);
        r[7] = 0.0f;
    }
    static __device__ __forceinline__ void pad_j(float (&r)[8]) { GravityJerk::pad_j(r); }
    static constexpr bool kSelf = true;
    static __device__ __forceinline__ void null_j(float (&r)[8]) { GravityJerk::null_j(r); }
    template <bool POT, bool MANY>
    static __device__ __forceinline__ void pair_timed(const float *j, const IState &i, float eps2,
                                                      float (&acc)[kOut]) {
        jerk_pair_timed<POT>(j, i.x, i.y, i.z, i.vx, i.vy, i.vz, eps2, acc);
    }
};

// Separate i- and j-sets (an active subset of a system against all of it, or two
// systems): every (i, j) pair is summed, with one softening for all.  Padding
// j-records are massless and far away (1e18), so their terms are exactly zero even
// with eps = 0 (s^2 stays a finite normal float and every product with m = 0 is 0).
struct GravityJerkIJ {
    static constexpr int kJWords = 8;
    static constexpr int kOut = 7;
    static constexpr int kBlockJ = GravityJerk::kBlockJ;
    static constexpr int kMaxIpl = 2;
    static constexpr bool kLone = false;
    using Args = JerkIJArgs;
    using IState = GravityJerk::IState;
    struct Ctx {};
    static __device__ __forceinline__ int n_i(const Args &a) { return a.ni; }
    static __device__ __forceinline__ int n_j(const Args &a) { return a.nj; }
    static __device__ __forceinline__ Ctx make_ctx(const Args &, int) { return {}; }
    static __device__ __forceinline__ IState load_i(const Args &a, const Ctx &, int i) {
        return {a.xi[i], a.yi[i], a.zi[i], a.vxi[i], a.vyi[i], a.vzi[i]};
    }
    static __device__ __forceinline__ void load_j(const Args &a, const Ctx &, int b, unsigned j, float (&r)[8]) {
        r[0] = (a.x + b)[j];
        r[1] = (a.y + b)[j];
        r[2] = (a.z + b)[j];
        r[3] = (a.m + b)[j];
        r[4] = (a.vx + b)[j];
        r[5] = (a.vy + b)[j];
        r[6] = (a.vz + b)[j];
        r[7] = 0.0f;
    }
    static __device__ __forceinline__ void pad_j(float (&r)[8]) {
        r[0] = r[1] = r[2] = 1e18f;
#pragma unroll
        for (int c = 3; c < 8; ++c) r[c] = 0.0f;
    }
    static constexpr bool kSelf = false;  // separate sets: every pair is summed
    template <bool POT, bool MANY>
    static __device__ __forceinline__ void pair_timed(const float *j, const IState &i, float eps2,
                                                      float (&acc)[kOut]) {
        jerk_pair_timed<POT>(j, i.x, i.y, i.z, i.vx, i.vy, i.vz, eps2, acc);
    }
};

}  // namespace
}  // namespace nbody
