// Force engine for systems whose j-records all fit in the LDS of a compute unit (device code,
// header-only): the shapes of the split engine with Q = 32 or 64 lanes per i-particle, IPL 1
// and n <= 8192.  The FP32 sums are the split engine's (lane q of an i-particle takes the
// records q, q + Q, ... of each tile of jt records, one FP32 block per tile); around them:
//
//   * one block per compute unit (256 in all) stages every record once and synchronises
//     once (the split engine: tiles, for every 4 to 8 i's); its waves then hold 1 or 2 of
//     the block's i's each and no barrier follows.  Spreading the i's over whole compute
//     units evens out the SIMDs: N = 4500 and 6500 take 4.4 and 6.3 i's per SIMD here,
//     where 4-wave blocks of the split engine fill them in steps of 2;
//   * records past the end are not visited, but for the rest of a group of 4 (the split
//     engine runs whole tiles);
//   * with Q = 32 a wave's halves take different tiles of the same i's, so that each record
//     read from LDS serves 2 i's (PLAIN, where the tiles of an i-particle are one chain,
//     and the tiles left over: the same tile for different i's);
//   * FP64 positions are staged as fp32(x - c) by the block itself, which first adds the
//     FP64 centre c in the order of the centre launches: no centre and conversion launch.
//
// Bound by VALU issue, 55 to 60 clocks per pair and SIMD (37 where many launches' worth of
// waves follow each other), over about 3 us of launch, staging and first loads.  us per
// call against the split engine (N = 2049 / 3500 / 4096 / 4500 / 5000 / 7000 / 8191): FP32
// positions 6.0 / 9.3 / 9.7 / 12.7 / 13.5 / 20.8 / 27.6, before 7.1 / 10.8 / 10.2 / 15.5 /
// 15.6 / 25.4 / 29.0; FP64 positions 7.5 / 11.1 / 11.5 / 14.7 / 15.5 / 23.5 / 30.8 with the
// centre and conversion, which took 2.4 to 3 us and a launch of their own.
#pragma once

#include "centre_sum.h"
#include "gravity.h"
#include "split_engine.h"

namespace nbody {
namespace set {

// Blocks of a launch: one per compute unit, at least as many i's as waves.  Waves per block:
// up to 1024 and 2048 particles one i-particle per wave; above, 12 do better than 8 and 16
// (N = 3000: 7.5, 8.5 and 8.6 us; 4096: 9.8, 11.3 and 10.3; 5000: 13.3 and 14.7 with 12 and
// 16) as long as 2 i's per wave are enough.
constexpr int kBlocks = 256;
constexpr int kMaxWaves = 16;
constexpr int kChunks = 2;  // 256-particle chunks a wave stages at most
inline int waves_for(int64_t n, bool pairs) {
    if (pairs) return kMaxWaves;
    return n <= 4 * kBlocks ? 4 : n <= 8 * kBlocks ? 8 : n <= 24 * kBlocks ? 12 : kMaxWaves;
}

inline size_t lds_bytes(int64_t n) {
    return ((size_t)n + 255) / 256 * 256 * sizeof(float4) + 3 * 32 * sizeof(double);
}

// All records into tile[0 .. n rounded up to 256) (padding: massless, at the origin).
template <bool F64>
__device__ __forceinline__ void stage(const SetArgs &a, float4 *tile) {
    const int n = a.n;
    const int chunks = (n + 255) / 256;
    const int threads = blockDim.x;
    if constexpr (!F64) {
        for (int i = threadIdx.x; i < chunks * 256; i += threads)
            tile[i] = i < n ? make_float4(a.pos[i], a.pos[n + i], a.pos[2 * n + i], a.m[i])
                            : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
        // A wave holds whole 256-particle chunks, at most kChunks.
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int waves = threads >> 6;
        double *sh = reinterpret_cast<double *>(tile + chunks * 256);  // [3][32]
        double v[kChunks][3][4];
        float m[kChunks][4];
#pragma unroll
        for (int d = 0; d < kChunks; ++d)
            if (wave + d * waves < chunks)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int i = (wave + d * waves) * 256 + k * 64 + lane;
                    const bool ok = i < n;
                    v[d][0][k] = ok ? a.pos64[i] : 0.0;
                    v[d][1][k] = ok ? a.pos64[n + i] : 0.0;
                    v[d][2][k] = ok ? a.pos64[2 * n + i] : 0.0;
                    m[d][k] = ok ? a.m[i] : 0.0f;
                }
        double c[3] = {0.0, 0.0, 0.0};
        if (a.centred) {
#pragma unroll
            for (int d = 0; d < kChunks; ++d)
                if (wave + d * waves < chunks)
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const double s = centre::wave_sum(v[d][q]);
                        if (lane == 0) sh[q * 32 + wave + d * waves] = s;
                    }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 3; ++q) c[q] = centre::second_stage(sh + q * 32, chunks, lane) / (double)n;
        }
#pragma unroll
        for (int d = 0; d < kChunks; ++d)
            if (wave + d * waves < chunks)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int i = (wave + d * waves) * 256 + k * 64 + lane;
                    tile[i] = i < n ? make_float4((float)(v[d][0][k] - c[0]), (float)(v[d][1][k] - c[1]),
                                                  (float)(v[d][2][k] - c[2]), m[d][k])
                                    : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
    }
    __syncthreads();
}

// `rows` records tl[0], tl[Q], ... against the lane's C i-records, added into acc.  With
// SELF, own[k] is the offset of the lane's k-th own particle from tl.
template <int C, int Q, bool FULL, bool SELF>
__device__ __forceinline__ void rows_pass(const float4 *tl, int rows, const Gravity::IState *is,
                                          const int *own, float eps2, float (*acc)[Gravity::kOut]) {
    constexpr int A = 4;
    auto read = [&](float(&jr)[A][4], int r) {
#pragma unroll
        for (int p = 0; p < A; ++p) {
            const float4 v = tl[(r + p) * Q];
            jr[p][0] = v.x;
            jr[p][1] = v.y;
            jr[p][2] = v.z;
            jr[p][3] = v.w;
        }
    };
#pragma unroll 1
    for (int r = 0; r < rows; r += A) {
        float jr[A][4];
        read(jr, r);
#pragma unroll
        for (int p = 0; p < A; ++p)
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const float m = SELF && (r + p) * Q == own[k] ? 0.0f : jr[p][3];
                const float z[4] = {jr[p][0], jr[p][1], jr[p][2], m};
                if constexpr (C > 1)
                    Gravity::pair_timed<FULL, true>(z, is[k], eps2, acc[k]);
                else
                    Gravity::pair<FULL>(z, is[k], eps2, acc[k]);
            }
    }
}

// Adds one FP32 block to a lane's sums of one particle.
template <int MODE>
__device__ __forceinline__ void add_block(float (&h)[4], float (&l)[4], double (&d)[4],
                                          const float (&b)[4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if constexpr (MODE == NBODY_COMP)
            engine::two_sum(h[c], l[c], b[c]);
        else if constexpr (MODE == NBODY_FP64RED)
            d[c] += (double)b[c];
        else
            h[c] = b[c];
    }
}

// One wave's C particles from i0 against all records.
template <class Sink, int C, int Q, int MODE, bool FULL>
__device__ __forceinline__ void wave_set(const SetArgs &a, const typename Sink::Args &f,
                                         const float4 *tile, int i0) {
    constexpr int H = 64 / Q;             // halves of a wave with tiles (or i's) of their own
    constexpr int CH = (C + H - 1) / H;   // i's of a lane where the halves take different i's
    const int lane = threadIdx.x & 63;
    const int q = lane % Q, h = lane / Q;
    const int n = a.n, jt = a.jt;
    float hs[C][4], ls[C][4];
    double ds[C][4];
    Gravity::IState is[C];
    int own[C];
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const float4 r = tile[i0 + k];
        is[k] = {r.x, r.y, r.z};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            hs[k][c] = ls[k][c] = 0.0f;
            ds[k][c] = 0.0;
        }
    }
    // FP32 blocks of tile t (its records from `base`, `rows` of them a lane) for NC i's.
    auto block = [&](auto nc, int base, int rows, const Gravity::IState *im, int im0,
                     float(*bs)[4]) {
        constexpr int NC = decltype(nc)::value;
        const float4 *tl = tile + base + q;
        // Uniform: does any of the wave's tiles hold one of its particles?
        const int lo = __builtin_amdgcn_readfirstlane(base);
        const int hi = lo + (NC == C ? H : 1) * jt;
        if (lo < i0 + C && i0 < hi) {
#pragma unroll
            for (int k = 0; k < NC; ++k) own[k] = im0 + k - base - q;
            rows_pass<NC, Q, FULL, true>(tl, rows, im, own, a.eps2, bs);
        } else {
            rows_pass<NC, Q, FULL, false>(tl, rows, im, own, a.eps2, bs);
        }
    };
    int t = 0;
    if constexpr (MODE != NBODY_PLAIN || H == 1) {
        // Every lane holds all C i's; the halves take different tiles.
        const int whole = H == 1 ? (n + jt - 1) / jt : n / jt / H * H;
#pragma unroll 1
        for (; t < whole; t += H) {
            // The tiles left decide a wave's priority: left to themselves the oldest waves
            // finish first and the last one runs alone, at half the rate (N = 8191: 29.4
            // instead of 27.6 us).
            if (4 * t < whole)
                __builtin_amdgcn_s_setprio(3);
            else if (2 * t < whole)
                __builtin_amdgcn_s_setprio(2);
            else if (4 * t < 3 * whole)
                __builtin_amdgcn_s_setprio(1);
            else
                __builtin_amdgcn_s_setprio(0);
            const int base = (t + h) * jt;
            const int rows = H == 1 ? min(jt, n - t * jt + Q - 1) / Q : jt / Q;
            float bs[C][4];
#pragma unroll
            for (int k = 0; k < C; ++k)
#pragma unroll
                for (int c = 0; c < 4; ++c) bs[k][c] = MODE == NBODY_PLAIN ? hs[k][c] : -0.0f;
            block(std::integral_constant<int, C>{}, base, rows, is, i0, bs);
#pragma unroll
            for (int k = 0; k < C; ++k) add_block<MODE>(hs[k], ls[k], ds[k], bs[k]);
        }
    }
    if constexpr (H == 2) {
        // Every lane takes the same tiles; the halves hold different i's.
        Gravity::IState im[CH];
#pragma unroll
        for (int k = 0; k < CH; ++k) {
            const int b = CH + k < C ? CH + k : C - 1;
            im[k] = {h ? is[b].x : is[k].x, h ? is[b].y : is[k].y, h ? is[b].z : is[k].z};
        }
#pragma unroll 1
        for (; t * jt < n; ++t) {
            const int rows = min(jt, n - t * jt + Q - 1) / Q;
            float bs[CH][4];
#pragma unroll
            for (int k = 0; k < CH; ++k)
#pragma unroll
                for (int c = 0; c < 4; ++c) bs[k][c] = MODE == NBODY_PLAIN ? hs[k][c] : -0.0f;
            block(std::integral_constant<int, CH>{}, t * jt, rows, im, i0 + h * CH, bs);
            if constexpr (MODE == NBODY_PLAIN) {
#pragma unroll
                for (int k = 0; k < CH; ++k) add_block<MODE>(hs[k], ls[k], ds[k], bs[k]);
            } else {
#pragma unroll
                for (int k = 0; k < C; ++k)
                    if (h == k / CH) add_block<MODE>(hs[k], ls[k], ds[k], bs[k % CH]);
            }
        }
    }
    // Lane 4 k + c stores slot c of particle k.
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < C; ++k)
#pragma unroll
        for (int c = 0; c < Sink::stores(FULL); ++c) {
            double r;
            if constexpr (MODE == NBODY_FP64RED) {
                r = split::group_sum<64>(ds[k][c]);
            } else if constexpr (MODE == NBODY_COMP) {
                r = split::group_sum<64>((double)hs[k][c] + (double)ls[k][c]);
            } else if constexpr (H == 1) {
                r = (double)split::group_sum<64>(hs[k][c]);
            } else {
                const float s = split::group_sum<Q>(hs[k % CH][c]);
                r = (double)__shfl(s, k / CH * Q);
            }
            v = lane == 4 * k + c ? r : v;
        }
    if (lane < 4 * C && (lane & 3) < Sink::stores(FULL))
        Sink::put(f, i0 + lane / 4, lane & 3, [&](int) { return v; });
}

// Grid: kBlocks blocks (fewer if there are fewer i's than that many blocks of waves) of
// waves_for(n) waves, lds_bytes(n) of LDS.
template <class Sink, int Q, int MODE, bool FULL, bool F64>
__global__ __launch_bounds__(64 * kMaxWaves) void set_kernel(SetArgs a, typename Sink::Args f) {
    extern __shared__ float4 tile[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int b0 = (int)((long long)a.n * blockIdx.x / gridDim.x);
    const int nb = (int)((long long)a.n * (blockIdx.x + 1) / gridDim.x) - b0;
    stage<F64>(a, tile);
    // The i's of the wave: pairs (PLAIN with two halves), or evenly, the larger shares first
    // (waves w, w + 4, w + 8, ... share a SIMD).
    const bool pairs = Q == 32 && MODE == NBODY_PLAIN;
    const int per = nb / waves, rem = nb % waves;
    const int i0 = b0 + (pairs ? 2 * wave : wave * per + min(wave, rem));
    const int cnt = pairs ? min(nb - 2 * wave, 2) : per + (wave < rem);
    if (cnt == 1)
        wave_set<Sink, 1, Q, MODE, FULL>(a, f, tile, i0);
    else if (cnt == 2)
        wave_set<Sink, 2, Q, MODE, FULL>(a, f, tile, i0);
}

}  // namespace set
}  // namespace nbody
