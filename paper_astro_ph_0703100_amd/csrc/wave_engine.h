// Pair engine for gfx950 in which every wavefront works on its own (device code,
// header-only).  Same pipelines (Op) as described in tile_engine.h.
//
//   * a wave holds 64 * IPL i-particles (IPL i-records per lane, lane-strided); the W
//     waves of a block hold the same i's and share out the FP32 blocks of BJ j's of
//     the block's j-segment in contiguous runs;
//   * a wave stages 64 j-records at a time (kLongStage: 256) in its own LDS slice (one record
//     per lane, the next 64 already on their way to registers) and reads each one back with
//     broadcast 16-byte reads, one record ahead of the pairs.  Nothing but the wave
//     itself touches the slice, so there is no barrier in the loop;
//   * accumulation (PLAIN: one FP32 sum per segment; FP64RED:
//     FP32 blocks of BJ j's added in FP64; COMP: FP32 blocks added into an FP32 (hi, lo)
//     pair by a two-sum).  A PLAIN segment is one chain of additions, so there each wave
//     takes a segment of its own;
//   * at the end the waves' sums of each i-particle are added in FP64 through LDS, in
//     wave order.  With one segment they are the result, stored through the Sink (what
//     the FP64 finalize would store); otherwise they are the segment's partial sums.
// Every sum has a fixed order: results are bitwise reproducible per launch shape.
#pragma once

#include "tile_engine.h"

namespace nbody {
namespace wave {

// j-records a wave stages at a time: one per lane; four in PLAIN launches of few waves, where
// nothing hides the way through LDS (separate sets, 1024 i's x 8192 j's: 12.7 us, with one 13.1;
// N = 16384 in one segment: 539 and 562 us; with 1 to 5 waves per SIMD it costs, N = 8192: 29.1
// and 25.9 us).
constexpr int kStage = 64, kLongStage = 256;
// Above kLoneWaves and up to this many (5 per SIMD, all there at once, with chains of 128 to 512
// pairs), the waves of a launch should end together (kEven, one record per lane).  N = 4099 /
// 5000 / 8192 / 9000 / 10007, with the finalize: force-jerk 22.7 / 27.5 / 47.4 / 54.0 / 69.3
// -> 21.7 / 26.0 / 42.8 / 51.3 / 67.9 us, adjoint 26.3 / 31.2 / 52.2 / 63.0 / 81.3 -> 25.0 /
// 29.4 / 48.8 / 58.9 / 78.8 us; force, N = 8192 / 9000, 26.9 / 32.0 -> 24.4 / 29.6 us; PLAIN,
// N = 6000 / 8000 / 9000, force-jerk 37.3 / 48.8 / 57.7 -> 34.8 / 44.6 / 54.3 us.  With 6 per
// SIMD nothing is gained (N = 7000: 41.2 -> 41.0) or lost (N = 12000: 92 -> 96 us), under one
// it costs 2 % (N = 2100), and where waves follow each other priorities only disturb their
// order (PLAIN force, N = 20011: 124 -> 132 us).
constexpr int64_t kEvenWaves = 5120;
enum Run { kMany, kLone, kEven };
constexpr int stage_of(int mode, Run run) {
    return mode == NBODY_PLAIN && run == kLone ? kLongStage : kStage;
}

// Bytes of LDS of a block of `waves` waves: staging, then the cross-wave sums.
template <class Op>
constexpr size_t lds_bytes(int waves, int records = kStage) {
    const size_t stage = (size_t)records * Op::kJWords * 4;
    const size_t sums = (size_t)64 * Op::kOut * 8;
    return waves * (stage > sums ? stage : sums);
}

// The records [0, cnt) of the wave's slice against the lane's IPL i-records, added into
// acc.  With SELF, slot self[k] holds the lane's k-th own particle.
template <class Op, int IPL, int ST, bool FULL, bool SELF>
__device__ __forceinline__ void stage_pass(const float4 *tl, int cnt,
                                           const typename Op::IState (&is)[IPL], float eps2,
                                           float (&acc)[IPL][Op::kOut], int lane, int d0) {
    constexpr int W = Op::kJWords;
    constexpr int V = W / 4;
    constexpr int U = wave_unroll(IPL);  // (padding adds zero)
    static_assert(ST % U == 0, "whole iterations per stage");
    float4 cur[V], nxt[V];
#pragma unroll
    for (int v = 0; v < V; ++v) cur[v] = tl[v];
#pragma unroll 1
    for (int j0 = 0; j0 < cnt; j0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // The next record is read while this one's pairs run (past the last record of
            // the slice: the first one again, unused).
            const int jn = u + 1 < U ? j0 + u + 1 : (j0 + U) & (ST - 1);
#pragma unroll
            for (int v = 0; v < V; ++v) nxt[v] = tl[jn * V + v];
            // Keeps the reads one record ahead: free to move, the scheduler hoists every
            // read of the unrolled loop and runs out of registers.
            __builtin_amdgcn_sched_barrier(0);
            float jr[W];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                jr[4 * v] = cur[v].x;
                jr[4 * v + 1] = cur[v].y;
                jr[4 * v + 2] = cur[v].z;
                jr[4 * v + 3] = cur[v].w;
            }
#pragma unroll
            for (int k = 0; k < IPL; ++k) {
                if constexpr (SELF) {
                    float z[W];
#pragma unroll
                    for (int w = 0; w < W; ++w) z[w] = jr[w];
                    Op::null_j(z);
                    const bool own = j0 + u == d0 + k * 64 + lane;
#pragma unroll
                    for (int w = 0; w < W; ++w) z[w] = own ? z[w] : jr[w];
                    Op::template pair_timed<FULL, (IPL > 1)>(z, is[k], eps2, acc[k]);
                } else {
                    Op::template pair_timed<FULL, (IPL > 1)>(jr, is[k], eps2, acc[k]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < V; ++v) cur[v] = nxt[v];
        }
    }
}

// The same with one record per lane and few waves on the chip: a lone wave issues an
// instruction every 4.7 clocks whatever it depends on, so what counts is their number.  A
// records are read ahead of their pairs and the compiler interleaves the A pair bodies, which
// leaves no s_nop (a lone wave: 73 clocks per gravity pair instead of 86).  A = 8 for PLAIN
// sums (N = 16384 in one segment: 565 us, with A = 4 612, then 539 in long stages), whose waves
// are alone on their SIMD.
// The other modes take 4: of blocks of 5 to 8 waves two share a SIMD (N = 600 / 1000: 8.5 / 10.1
// us, with A = 8 8.9 / 10.1; in blocks of 4, N = 1500 / 2500, 10.0 / 10.7 and 9.5 / 10.2).
template <class Op, int A, int ST, bool FULL, bool SELF>
__device__ __forceinline__ void lone_pass(const float4 *tl, int cnt,
                                          const typename Op::IState (&is)[1], float eps2,
                                          float (&acc)[1][Op::kOut], int lane, int d0) {
    constexpr int W = Op::kJWords;
    constexpr int V = W / 4;
    static_assert(ST % (2 * A) == 0, "whole groups per stage");
    float jr[2][A][W];
    auto read = [&](int h, int j0) {
#pragma unroll
        for (int p = 0; p < A; ++p)
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const float4 q = tl[(j0 + p) * V + v];
                jr[h][p][4 * v] = q.x;
                jr[h][p][4 * v + 1] = q.y;
                jr[h][p][4 * v + 2] = q.z;
                jr[h][p][4 * v + 3] = q.w;
            }
    };
    auto pairs = [&](int h, int j0) {
#pragma unroll
        for (int p = 0; p < A; ++p)
            engine::pair_k<Op, FULL, SELF>(jr[h][p], j0 + p, d0 + lane, is[0], eps2, acc[0]);
    };
    read(0, 0);
#pragma unroll 1
    for (int j0 = 0; j0 < cnt; j0 += 2 * A) {
        read(1, j0 + A);
        __builtin_amdgcn_sched_barrier(0);
        pairs(0, j0);
        __builtin_amdgcn_sched_barrier(0);
        read(0, (j0 + 2 * A) & (ST - 1));
        __builtin_amdgcn_sched_barrier(0);
        pairs(1, j0 + A);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The less of a wave's work is done, the higher its priority.  Left to themselves the oldest
// waves of a SIMD finish first and the last one runs alone, at half the rate; that counts
// where no others take their places.
__device__ __forceinline__ void priority_by_rest(int t, int all) {
    if (4 * t < all)
        __builtin_amdgcn_s_setprio(3);
    else if (2 * t < all)
        __builtin_amdgcn_s_setprio(2);
    else if (4 * t < 3 * all)
        __builtin_amdgcn_s_setprio(1);
    else
        __builtin_amdgcn_s_setprio(0);
}

// One wave's work: its 64 * IPL i-particles from i0 (ni of them exist) against the
// j-range [j0, j0 + nj), in FP32 blocks of BJ from j0 on.  All arguments are uniform.
// Sums: FP64RED ds, COMP hs and ls, PLAIN hs.
template <class Op, int IPL, int BJ, int MODE, bool FULL, Run RUN = kMany>
__device__ __forceinline__ void wave_work(const typename Op::Args &a, float4 *tl, int i0, int ni,
                                          int j0, int nj, float eps2,
                                          float (&hs)[IPL][Op::kOut], float (&ls)[IPL][Op::kOut],
                                          double (&ds)[IPL][Op::kOut]) {
    constexpr int W = Op::kJWords;
    constexpr int V = W / 4;
    constexpr int NO = Op::kOut;
    constexpr int ST = stage_of(MODE, RUN);
    constexpr int RPL = ST / 64;  // records per lane and stage
    constexpr int PER = MODE == NBODY_PLAIN ? 1 : BJ / ST;  // stages per FP32 block
    static_assert(MODE == NBODY_PLAIN || BJ % ST == 0, "whole stages per FP32 block");
    const int lane = threadIdx.x & 63;
    const typename Op::Ctx ctx = Op::make_ctx(a, i0);

    typename Op::IState is[IPL];
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        const int q = k * 64 + lane;
        is[k] = Op::load_i(a, ctx, i0 + (q < ni ? q : ni - 1));
    }
#pragma unroll
    for (int k = 0; k < IPL; ++k)
#pragma unroll
        for (int c = 0; c < NO; ++c) {
            hs[k][c] = 0.0f;
            ls[k][c] = 0.0f;
            ds[k][c] = 0.0;
        }

    float rec[RPL][W];
    auto fetch64 = [&](int b, float(&q)[W]) {
        if (b + 64 <= nj) {
            Op::load_j(a, ctx, j0 + b, (unsigned)lane, q);
        } else {
            Op::pad_j(q);
            if (b + lane < nj) Op::load_j(a, ctx, j0 + b, (unsigned)lane, q);
        }
    };
    // The first record is no part of the loop: in a loop of one the branches around the adjoint's
    // loads were kept apart (PLAIN, N = 20484 / 31381: 305 / 733 us, 299 / 724 as it is here).
    auto fetch = [&](int t) {
        fetch64(t * ST, rec[0]);
#pragma unroll
        for (int r = 1; r < RPL; ++r) fetch64(t * ST + r * 64, rec[r]);
    };
    const int stages = (nj + ST - 1) / ST;
    if (stages > 0) fetch(0);
    for (int t0 = 0; t0 < stages; t0 += PER) {
        float bs[IPL][NO];
        if constexpr (MODE != NBODY_PLAIN)
#pragma unroll
            for (int k = 0; k < IPL; ++k)
#pragma unroll
                for (int c = 0; c < NO; ++c) bs[k][c] = -0.0f;
        const int t1 = min(t0 + PER, stages);
#pragma unroll 1
        for (int t = t0; t < t1; ++t) {
            if constexpr (RUN == kEven) priority_by_rest(t, stages);
            // LDS serves a wave's accesses in order, so the slice can be rewritten as soon
            // as its last reads are issued; the fences keep the compiler to that order.
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int r = 0; r < RPL; ++r)
#pragma unroll
                for (int v = 0; v < V; ++v)
                    tl[(r * 64 + lane) * V + v] = make_float4(rec[r][4 * v], rec[r][4 * v + 1],
                                                              rec[r][4 * v + 2], rec[r][4 * v + 3]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (t + 1 < stages) fetch(t + 1);
            const int jt0 = j0 + t * ST;
            const int cnt = min(ST, nj - t * ST);
            const int d0 = i0 - jt0;
            auto pass = [&](auto self) {
                constexpr bool SELF = decltype(self)::value;
                auto run = [&](float(&acc)[IPL][NO]) {
                    if constexpr (RUN == kLone)
                        lone_pass<Op, MODE == NBODY_PLAIN ? 8 : 4, ST, FULL, SELF>(
                            tl, cnt, is, eps2, acc, lane, d0);
                    else
                        stage_pass<Op, IPL, ST, FULL, SELF>(tl, cnt, is, eps2, acc, lane, d0);
                };
                if constexpr (MODE == NBODY_PLAIN)
                    run(hs);
                else
                    run(bs);
            };
            if constexpr (Op::kSelf) {
                // Does this stage hold any of the wave's own i's?
                if (jt0 < i0 + 64 * IPL && i0 < jt0 + ST)
                    pass(std::true_type{});
                else
                    pass(std::false_type{});
            } else {
                pass(std::false_type{});
            }
        }
        if constexpr (MODE != NBODY_PLAIN)
#pragma unroll
            for (int k = 0; k < IPL; ++k)
#pragma unroll
                for (int c = 0; c < NO; ++c) {
                    if constexpr (MODE == NBODY_COMP)
                        engine::two_sum(hs[k][c], ls[k][c], bs[k][c]);
                    else
                        ds[k][c] += (double)bs[k][c];
                }
    }
}

// Wave `wave`'s contiguous run of the FP32 blocks of a segment of snj j's.
struct Range {
    int j0, nj;
};
template <int BJ>
__device__ __forceinline__ Range block_run(int snj, int wave, int waves) {
    const int nb = (snj + BJ - 1) / BJ;
    const int b0 = nb * wave / waves * BJ;
    return {b0, max(0, min(nb * (wave + 1) / waves * BJ, snj) - b0)};
}

// A wave's PLAIN sums of the particles i0 + k 64 + lane (those below `end` exist): the
// outputs (whole), or column col of the segment's partial planes.
template <class Sink, int IPL, bool FULL, int NO>
__device__ __forceinline__ void store_plain(const typename Sink::Args &f, int i0, int end,
                                            const float (&hs)[IPL][NO], bool whole, float *part,
                                            size_t plane, size_t col) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        const int i = i0 + k * 64 + lane;
        if (whole) {
            if (i < end)
#pragma unroll
                for (int c = 0; c < Sink::stores(FULL); ++c)
                    Sink::put(f, i, c, [&](int o) { return (double)hs[k][o]; });
        } else {
#pragma unroll
            for (int c = 0; c < NO; ++c) part[c * plane + col + k * 64 + lane] = hs[k][c];
        }
    }
}

// Cross-wave sums of the block's particles i0 + k 64 + lane, one IPL slot at a time:
// [wave][output][lane] in LDS, then wave w adds the outputs (store slots) w, w + waves, ...
// of the slot's 64 particles in wave order and stores them: outputs (whole), or column col
// of the segment's partial planes.  All waves of the block must call it.
template <class Sink, int IPL, int MODE, bool FULL, int NO>
__device__ __forceinline__ void store_sums(const typename Sink::Args &f, double *sums, int wave,
                                           int waves, int i0, int end, const float (&hs)[IPL][NO],
                                           const float (&ls)[IPL][NO], const double (&ds)[IPL][NO],
                                           bool whole, float *part, size_t plane, size_t col) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NO; ++c)
            if (FULL || c < NO - 1)
                sums[(wave * NO + c) * 64 + lane] =
                    MODE == NBODY_COMP ? (double)hs[k][c] + (double)ls[k][c] : ds[k][c];
        __syncthreads();
        const int i = i0 + k * 64 + lane;
        auto total = [&](int o) {
            double v = sums[o * 64 + lane];
            for (int w = 1; w < waves; ++w) v += sums[(w * NO + o) * 64 + lane];
            return v;
        };
        if (whole) {
            if (i < end)
                for (int c = wave; c < Sink::stores(FULL); c += waves) Sink::put(f, i, c, total);
        } else {
            for (int c = wave; c < (FULL ? NO : NO - 1); c += waves) {
                const double v = total(c);
                const size_t q = col + k * 64 + lane;
                if constexpr (MODE == NBODY_FP64RED) {
                    reinterpret_cast<double *>(part)[c * plane + q] = v;
                } else {
                    const float hi = (float)v;
                    part[c * plane + q] = hi;
                    part[(NO + c) * plane + q] = (float)(v - (double)hi);
                }
            }
        }
    }
}

// Grid launch: blockIdx.x = group of 64 * IPL i's, blockIdx.y = j-segment of a.seg_len
// j's (PLAIN: one segment per wave, blockDim.x / 64 of them per block).  Partial planes
// [segment][word][npad], or, with `whole` (nseg = 1), the outputs through the Sink.  RUN: for
// launches of so many waves.
template <class Op, class Sink, int IPL, int BJ, int MODE, bool FULL, Run RUN>
__global__ __launch_bounds__(1024) void wave_kernel(typename Op::Args a, typename Sink::Args f,
                                                    int nseg, bool whole) {
    constexpr int NO = Op::kOut;
    constexpr int V = Op::kJWords / 4;
    constexpr int WO = NO * engine::words_per_out<MODE>();
    static_assert(Sink::kOutputs == NO, "the output stage reads the pipeline's outputs");
    extern __shared__ float4 lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int n = Op::n_i(a);
    const int i0 = blockIdx.x * (64 * IPL);
    const int ni = min(64 * IPL, n - i0);
    const int s = MODE == NBODY_PLAIN ? blockIdx.y * waves + wave : blockIdx.y;
    if (s >= nseg) return;  // PLAIN only: whole waves, and no barrier follows there
    const int j0 = s * a.seg_len;
    const int nj = max(0, min(a.seg_len, Op::n_j(a) - j0));
    const size_t plane = (size_t)a.npad;
    float *part = static_cast<float *>(a.part) + (size_t)s * WO * plane;
    float4 *tl = lds + wave * stage_of(MODE, RUN) * V;
    float hs[IPL][NO], ls[IPL][NO];
    double ds[IPL][NO];
    if constexpr (MODE == NBODY_PLAIN) {
        wave_work<Op, IPL, BJ, MODE, FULL, RUN>(a, tl, i0, ni, j0, nj, a.eps2, hs, ls, ds);
        store_plain<Sink, IPL, FULL>(f, i0, n, hs, whole, part, plane, (size_t)i0);
    } else {
        const Range r = block_run<BJ>(nj, wave, waves);
        wave_work<Op, IPL, BJ, MODE, FULL, RUN>(a, tl, i0, ni, j0 + r.j0, r.nj, a.eps2, hs, ls, ds);
        store_sums<Sink, IPL, MODE, FULL>(f, reinterpret_cast<double *>(lds), wave, waves, i0, n,
                                          hs, ls, ds, whole, part, plane, (size_t)i0);
    }
}

// Launch-shape dispatch: IPL up to Op::kMaxIpl, FP32 blocks of 64 or 128 j's (PLAIN sums
// have no blocks).
template <class Op, class Sink>
using WaveFn = void (*)(typename Op::Args, typename Sink::Args, int, bool);

template <class Op, class Sink, int IPL, Run RUN>
WaveFn<Op, Sink> pick_mode(int bj, int mode, bool full) {
    switch (mode) {
        case NBODY_PLAIN:
            return full ? wave_kernel<Op, Sink, IPL, 64, NBODY_PLAIN, true, RUN>
                        : wave_kernel<Op, Sink, IPL, 64, NBODY_PLAIN, false, RUN>;
        case NBODY_FP64RED:
            if (bj == 64)
                return full ? wave_kernel<Op, Sink, IPL, 64, NBODY_FP64RED, true, RUN>
                            : wave_kernel<Op, Sink, IPL, 64, NBODY_FP64RED, false, RUN>;
            return full ? wave_kernel<Op, Sink, IPL, 128, NBODY_FP64RED, true, RUN>
                        : wave_kernel<Op, Sink, IPL, 128, NBODY_FP64RED, false, RUN>;
        case NBODY_COMP:
            if (bj == 64)
                return full ? wave_kernel<Op, Sink, IPL, 64, NBODY_COMP, true, RUN>
                            : wave_kernel<Op, Sink, IPL, 64, NBODY_COMP, false, RUN>;
            return full ? wave_kernel<Op, Sink, IPL, 128, NBODY_COMP, true, RUN>
                        : wave_kernel<Op, Sink, IPL, 128, NBODY_COMP, false, RUN>;
    }
    return nullptr;
}

template <class Op, class Sink>
WaveFn<Op, Sink> pick_wave(int ipl, int bj, int mode, bool full, Run run) {
    static_assert(Op::kBlockJ == 128, "FP32 blocks of 64 or 128 j's");
    switch (ipl) {
        case 1:
            if constexpr (Op::kLone)
                if (run == kLone) return pick_mode<Op, Sink, 1, kLone>(bj, mode, full);
            return run == kEven ? pick_mode<Op, Sink, 1, kEven>(bj, mode, full)
                                : pick_mode<Op, Sink, 1, kMany>(bj, mode, full);
        case 2: return pick_mode<Op, Sink, 2, kMany>(bj, mode, full);
        case 4:
            if constexpr (Op::kMaxIpl >= 4) return pick_mode<Op, Sink, 4, kMany>(bj, mode, full);
    }
    return nullptr;
}

// One launch of cfg's wave shape; ni i-particles.  With cfg.direct the outputs are
// stored by the launch itself (f), otherwise its partial sums await the finalize.
template <class Op, class Sink>
nbody_status launch(const TileCfg &cfg, int precision, bool full, int64_t ni,
                    const typename Op::Args &a, const typename Sink::Args &f, hipStream_t s) {
    const int64_t groups = (ni + 64 * cfg.wi - 1) / (64 * cfg.wi);
    int wpb = cfg.wpb;
    while (groups * 64 * wpb > kMaxThreads) wpb /= 2;  // from 2^28 i's on
    const int64_t waves = groups * cfg.nseg * (precision == NBODY_PLAIN ? 1 : wpb);
    const Run run = cfg.wi > 1                             ? kMany
                    : waves <= kLoneWaves                  ? (Op::kLone ? kLone : kMany)
                    : waves <= kEvenWaves                  ? kEven
                                                           : kMany;
    auto fn = pick_wave<Op, Sink>(cfg.wi, cfg.bj, precision, full, run);
    if (!fn) return set_error(NBODY_EUNSUPPORTED, "no pair kernel for this ipl/jtile/precision");
    if (ni <= 0 || cfg.nseg <= 0) return NBODY_OK;
    const int per_block = precision == NBODY_PLAIN ? wpb : 1;  // segments per block
    const dim3 grid((unsigned)groups,
                    (unsigned)((cfg.nseg + per_block - 1) / per_block));
    hipLaunchKernelGGL(fn, grid, dim3(64 * wpb), lds_bytes<Op>(wpb, stage_of(precision, run)), s,
                       a, f, cfg.nseg, cfg.direct);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

}  // namespace wave
}  // namespace nbody
