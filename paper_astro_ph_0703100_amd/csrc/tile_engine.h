// What the pair engines for gfx950 share (device code, header-only): the pipeline interface,
// the two-sum, the pass over an LDS tile and the sums of segment partials.  The grid engine
// itself is in wave_engine.h; the split, whole-set and symmetric engines have headers of
// their own.
//
// The paper's library evaluates arbitrary pair interactions from a user-written pipeline
// description that reads an i-record and a j-record and accumulates outputs
// (Sec. 4.5, Appendix A).  This engine is that idea on CDNA4: a pipeline type `Op`
// supplies the records and the pair body; the engine supplies the blocking.
//
//   * each lane keeps IPL i-records in VGPRs (lane-strided so global loads and stores
//     coalesce); j-records pass through LDS, the J-BAG / J-PACKING of Sec. 2.2, and are
//     read back with broadcast 16-byte reads;
//   * the j == i pair is left out of every sum (eq. (1) sums over the other
//     particles): in the few stretches of j's that hold some of a wave's own i's (i- and
//     j-sets the same, Op::kSelf), each lane swaps the record of its own particle
//     for Op::null_j of it (same position, nothing that adds), by a compare and a
//     select per pair; all others run the plain pass;
//   * accumulation (Sec. 2.2.2, eq. (2); Sec. 3.4):
//       PLAIN   - one FP32 accumulator per output and (i, segment);
//       FP64RED - FP32 partial over each block of min(Op::kBlockJ, JT) j's, added into FP64;
//       COMP    - FP32 partial over each block, added into an FP32 (hi, lo) pair by an
//                 error-free two-sum;
//   * partial sums go to scratch planes [segment][word][npad]; a finalize kernel adds
//     the segments in a fixed order in FP64 (PLAIN: FP32).
// No atomics: every result is a fixed-order sum, bitwise reproducible per launch shape.
//
// An Op provides:
//   static constexpr int kJWords;            // floats per j-record (multiple of 4)
//   static constexpr int kOut;               // outputs per i
//   static constexpr int kBlockJ;            // j's per FP32 block before compensation
//   struct Args;                             // kernel arguments (seg_len, eps2, part, npad, ...)
//   static int n_i(const Args&), n_j(const Args&);  // i- and j-counts of a grid launch
//   struct IState;                           // per-i registers
//   struct Ctx;                              // per-block context (e.g. a reference centre)
//   static Ctx make_ctx(const Args&, int i0);
//   static IState load_i(const Args&, const Ctx&, int i);
//   static void load_j(const Args&, const Ctx&, int b, unsigned j, float (&r)[kJWords]);
//                                            // record b + j (b uniform over the wave)
//   static void pad_j(float (&r)[kJWords]);  // a record that adds exactly zero
//   static constexpr bool kSelf;             // i- and j-sets are one set (j == i exists)
//   static void null_j(float (&r)[kJWords]); // (kSelf only) turns a j-record into one at
//                                            // the same place that adds nothing: the
//                                            // j == i pair then adds exactly zero
//   template <bool FULL> static void pair(const float *jr, const IState&, float eps2,
//                                         float (&acc)[kOut]);
//   (FULL = false may skip the last output.)  For the engines that let the compiler order the
//   pairs: split, symmetric, whole-set, and the wave engine where kLone.
// For the wave engine:
//   static constexpr int kMaxIpl;            // most i-records per lane
//   static constexpr bool kLone;             // has a variant for launches of few waves
//   template <bool FULL, bool MANY> static void pair_timed(...as pair...);
//                                            // the pair in a fixed instruction order; MANY:
//                                            // several i-records per lane
#pragma once

#include <type_traits>

#include "nbody_internal.h"

namespace nbody {
namespace engine {

// s_waitcnt vmcnt(0) (expcnt and lgkmcnt left at their maxima, 7 and 15, in the gfx9
// encoding): wait for every outstanding vector-memory load of the wave.  Issued once
// after the first j-tile is staged, it tells the compiler that the i-record loads have
// completed; otherwise it waits on them inside the tile loop, where the in-order load
// counter also holds back the prefetch of the next tile (its latency then shows at
// every tile).
constexpr int kWaitVmem = 0x0F70;

// Knuth's error-free sum: hi + lo += b with hi = fl(hi + b) and the rounding error of
// that addition added to lo.
__device__ __forceinline__ void two_sum(float &hi, float &lo, float b) {
    const float s = hi + b;
    const float bb = s - hi;
    const float err = (hi - (s - bb)) + (b - bb);
    hi = s;
    lo = lo + err;
}

// One pair of the lane's k-th i-record with j-record jr; with SELF, the record of the
// lane's own particle (tile slot jj == self[k]) is replaced by Op::null_j of it.
template <class Op, bool FULL, bool SELF>
__device__ __forceinline__ void pair_k(const float *jr, int jj, int self_k,
                                       const typename Op::IState &is, float eps2,
                                       float (&acc)[Op::kOut]) {
    if constexpr (SELF) {
        float r[Op::kJWords];
        float z[Op::kJWords];
#pragma unroll
        for (int w = 0; w < Op::kJWords; ++w) r[w] = z[w] = jr[w];
        Op::null_j(z);
        const bool own = jj == self_k;
#pragma unroll
        for (int w = 0; w < Op::kJWords; ++w) r[w] = own ? z[w] : r[w];
        Op::template pair<FULL>(r, is, eps2, acc);
    } else {
        Op::template pair<FULL>(jr, is, eps2, acc);
    }
}

// One LDS tile: all JT j-records against the lane's IPL i-records.  With SELF, self[k]
// is the tile slot of the lane's k-th own particle (outside [0, JT) if not in it).
template <class Op, int IPL, int JT, int MODE, bool FULL, bool SELF = false>
__device__ __forceinline__ void tile_pass(const float4 *tl, const typename Op::IState (&is)[IPL],
                                          float eps2, float (&hs)[IPL][Op::kOut],
                                          float (&ls)[IPL][Op::kOut],
                                          double (&ds)[IPL][Op::kOut],
                                          const int (&self)[IPL]) {
    constexpr int W = Op::kJWords;
    constexpr int NO = Op::kOut;
    auto read = [&](int jj, float (&jr)[W]) {
#pragma unroll
        for (int v = 0; v < W / 4; ++v) {
            const float4 q4 = tl[jj * (W / 4) + v];
            jr[4 * v] = q4.x;
            jr[4 * v + 1] = q4.y;
            jr[4 * v + 2] = q4.z;
            jr[4 * v + 3] = q4.w;
        }
    };
    // The pass with the self test runs on a few tiles only: a shorter unroll keeps its
    // code small.
    constexpr int kUnrollPlain = SELF ? 4 : 8;
    if constexpr (MODE == NBODY_PLAIN) {
#pragma unroll kUnrollPlain
        for (int jj = 0; jj < JT; ++jj) {
            float jr[W];
            read(jj, jr);
#pragma unroll
            for (int k = 0; k < IPL; ++k)
                pair_k<Op, FULL, SELF>(jr, jj, self[k], is[k], eps2, hs[k]);
        }
    } else {
        constexpr int BJ = JT < Op::kBlockJ ? JT : Op::kBlockJ;
        static_assert(JT % BJ == 0, "blocks tile the j-tile");
        for (int jb = 0; jb < JT; jb += BJ) {
            float bs[IPL][NO];
#pragma unroll
            for (int k = 0; k < IPL; ++k)
#pragma unroll
                for (int c = 0; c < NO; ++c) bs[k][c] = -0.0f;
            // Unrolled 32 pairs deep: longer blocks loop over that body (a scalar
            // branch per 32 pairs) instead of growing the code and the build time.
            constexpr int kUnroll = SELF ? 8 : 32;
#pragma unroll kUnroll
            for (int jj = 0; jj < BJ; ++jj) {
                float jr[W];
                read(jb + jj, jr);
#pragma unroll
                for (int k = 0; k < IPL; ++k)
                    pair_k<Op, FULL, SELF>(jr, jb + jj, self[k], is[k], eps2, bs[k]);
            }
#pragma unroll
            for (int k = 0; k < IPL; ++k)
#pragma unroll
                for (int c = 0; c < NO; ++c) {
                    if constexpr (MODE == NBODY_COMP)
                        two_sum(hs[k][c], ls[k][c], bs[k][c]);
                    else
                        ds[k][c] += (double)bs[k][c];
                }
        }
    }
}

// Words (4 bytes) of partial sums per output, i-particle and segment.
template <int MODE>
constexpr int words_per_out() {
    return MODE == NBODY_PLAIN ? 1 : 2;
}

// Fixed-order sums of the segment partials.  Segment s holds, per output c, the words
// [s][c][plane] (PLAIN: FP32; FP64RED: FP64) or [s][c][plane] = hi and [s][NO + c][plane]
// = lo (COMP: FP32), summed as r += hi; r += lo.  The loads run a batch of segments
// ahead of the additions, which stay strictly sequential in s: with few particles the
// finalize has few waves and is bound by load latency, not bandwidth.
template <int NO, int MODE>
struct PartialLayout {
    using T = typename std::conditional<MODE == NBODY_FP64RED, double, float>::type;
    static constexpr int kWords = MODE == NBODY_COMP ? 2 : 1;  // hi (, lo) per output
    static constexpr int kStride = kWords * NO;                 // words per segment and column
};

// Segments whose loads a finalize thread issues ahead of its additions: 8 when the
// finalize has under 4 waves per SIMD (bound by load latency: at N = 16384 the force
// finalize went from 18 to 6 us), 1 otherwise (bound by bandwidth; a deeper batch only
// scatters the DRAM accesses: at N = 131072 it went from 26 to 39 us).
inline int finalize_batch(int64_t n, int outputs) {
    return n * outputs < (int64_t)4 * 1024 * 64 ? 8 : 1;
}

// One output c of particle i (FP64 for FP64RED/COMP, FP32 for PLAIN, returned widened).
template <int NO, int MODE, int BATCH>
__device__ __forceinline__ double sum_partial_output(const void *part, int nseg, size_t plane,
                                                     int i, int c) {
    using L = PartialLayout<NO, MODE>;
    using T = typename L::T;
    const T *p = static_cast<const T *>(part) + i + (size_t)c * plane;
    const size_t step = (size_t)L::kStride * plane;
    const size_t lo = (size_t)NO * plane;  // COMP: offset of the lo word
    using Acc = typename std::conditional<MODE == NBODY_PLAIN, float, double>::type;
    Acc r = 0;
    int s = 0;
    for (; s + BATCH <= nseg; s += BATCH) {
        T v[BATCH][L::kWords];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            v[b][0] = p[(size_t)(s + b) * step];
            if constexpr (L::kWords == 2) v[b][L::kWords - 1] = p[(size_t)(s + b) * step + lo];
        }
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
#pragma unroll
            for (int w = 0; w < L::kWords; ++w) r = r + (Acc)v[b][w];
    }
    for (; s < nseg; ++s) {
        r = r + (Acc)p[(size_t)s * step];
        if constexpr (L::kWords == 2) r = r + (Acc)p[(size_t)s * step + lo];
    }
    return (double)r;
}

// All NO outputs of particle i in r[0 .. NO), each with the rounding of the
// corresponding sum_partial_output.
template <int NO, int MODE, int BATCH>
__device__ __forceinline__ void sum_partials(const void *part, int nseg, size_t plane, int i,
                                             double (&r)[NO]) {
    using L = PartialLayout<NO, MODE>;
    using T = typename L::T;
    const T *p = static_cast<const T *>(part) + i;
    const size_t step = (size_t)L::kStride * plane;
    const size_t lo = (size_t)NO * plane;
    using Acc = typename std::conditional<MODE == NBODY_PLAIN, float, double>::type;
    Acc acc[NO];
#pragma unroll
    for (int c = 0; c < NO; ++c) acc[c] = 0;
    int s = 0;
    for (; s + BATCH <= nseg; s += BATCH) {
        T v[BATCH][NO][L::kWords];
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
#pragma unroll
            for (int c = 0; c < NO; ++c) {
                v[b][c][0] = p[(size_t)(s + b) * step + (size_t)c * plane];
                if constexpr (L::kWords == 2)
                    v[b][c][L::kWords - 1] = p[(size_t)(s + b) * step + (size_t)c * plane + lo];
            }
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
#pragma unroll
            for (int c = 0; c < NO; ++c)
#pragma unroll
                for (int w = 0; w < L::kWords; ++w) acc[c] = acc[c] + (Acc)v[b][c][w];
    }
    for (; s < nseg; ++s)
#pragma unroll
        for (int c = 0; c < NO; ++c) {
            acc[c] = acc[c] + (Acc)p[(size_t)s * step + (size_t)c * plane];
            if constexpr (L::kWords == 2)
                acc[c] = acc[c] + (Acc)p[(size_t)s * step + (size_t)c * plane + lo];
        }
#pragma unroll
    for (int c = 0; c < NO; ++c) r[c] = (double)acc[c];
}

}  // namespace engine
}  // namespace nbody
