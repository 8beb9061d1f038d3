// Morton (Z-order) permutation of FP64 positions, so that consecutive particles - and
// therefore the i-tiles of the pair kernels - are spatially compact.  That is what
// makes per-i-tile reference centres (NBODY_CENTRE_TILE) pay off.
//
// Every particle gets a 64-bit word: the interleaved quantised coordinates in its high
// bits and its index in the low bits; the index bits of the sorted words are the
// permutation.  Ties in the key are broken by index, so the order is unique.
//
//   * up to kSmall particles: one block does it all in LDS (bounding box, words, bitonic
//     network or radix passes), one launch;
//   * above: a stable radix sort of the key bits alone, from the least significant digit
//     (the words start in index order, so ties stay in it).  Each pass is three launches:
//     digit counts of every tile, prefix sums of the counts over the tiles (one block per
//     digit), and the scatter, which ranks a tile's words by digit with wave ballots,
//     puts them in that order in LDS and writes each digit's run contiguously.
//
// Bound: 16 bytes read and written per word and pass, 6 passes of 7 bits at 2^20
// particles, but at that size each launch takes longer to start and to fill than its traffic.
// 2^20 particles: 112 us in 19 launches, 779 us in the 210 launches of a bitonic network in
// global memory.  Prefix sums and the final box run inside waves and the counts are plain
// additions: with 8 and 9 block-wide steps for the former and ballots for the latter 139 us.
#include <algorithm>
#include <utility>

#include "centre_sum.h"
#include "nbody_internal.h"

namespace nbody {
namespace {

constexpr int kBoxBlocks = 256;  // one slot of the final reduction each
constexpr int kBoxThreads = 512;
// One block sorts up to kSmall words in LDS (64 KB), up to kBitonic by a bitonic network
// (N = 1000: 17.1 us, by radix passes 20.4; 2048: 24.6 and 23.8; 4096: 43.9 and 37.0; 8192:
// 85.4 and 64.5 us; 8193, in 19 launches: 84.2 us).
constexpr int kBitonic = 1024;
constexpr int kSmall = 8192;
constexpr int kSmallThreads = 1024;
constexpr int kTile = 4096;        // words per block of the radix passes
constexpr int kTileThreads = 512;  // 8 waves, 8 rows of 64 words each
constexpr int kRows = kTile / kTileThreads;
constexpr int kWaves = kTileThreads / 64;
constexpr int kMaxDigits = 256;

// Lowest and highest coordinates in lo/hi [3][threads] reduced to slot 0 of each.
template <int THREADS>
__device__ __forceinline__ void reduce_box(double (*lo)[THREADS], double (*hi)[THREADS]) {
    __syncthreads();
    for (int w = THREADS / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lo[c][threadIdx.x] = fmin(lo[c][threadIdx.x], lo[c][threadIdx.x + w]);
                hi[c][threadIdx.x] = fmax(hi[c][threadIdx.x], hi[c][threadIdx.x + w]);
            }
        __syncthreads();
    }
}

// This thread's box of the particles first, first + stride, ...
template <int THREADS, int AHEAD = 1>
__device__ __forceinline__ void thread_box(int64_t n, const double *pos, int64_t first,
                                           int64_t stride, double (*lo)[THREADS],
                                           double (*hi)[THREADS]) {
    double l[3] = {INFINITY, INFINITY, INFINITY}, h[3] = {-INFINITY, -INFINITY, -INFINITY};
#pragma unroll AHEAD
    for (int64_t i = first; i < n; i += stride)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double v = pos[c * n + i];
            l[c] = fmin(l[c], v);
            h[c] = fmax(h[c], v);
        }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        lo[c][threadIdx.x] = l[c];
        hi[c][threadIdx.x] = h[c];
    }
}

struct Lowest {
    __device__ double operator()(double a, double b) const { return fmin(a, b); }
};
struct Highest {
    __device__ double operator()(double a, double b) const { return fmax(a, b); }
};

// Six values of each of 256 slots, v[6 slot + c], reduced by one wave: lowest for c < 3,
// highest above; lane 0 returns them.
__device__ __forceinline__ void wave_box(const double *v, double (&l)[3], double (&h)[3]) {
    const int lane = threadIdx.x & 63;
    double x[6][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < 6; ++c) x[c][k] = v[6 * (k * 64 + lane) + c];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        l[c] = centre::wave_tree(x[c], Lowest());
        h[c] = centre::wave_tree(x[c + 3], Highest());
    }
}

__global__ __launch_bounds__(kBoxThreads) void box_partial_kernel(int64_t n, const double *pos,
                                                                 double *part) {
    __shared__ double lo[3][kBoxThreads], hi[3][kBoxThreads];
    thread_box<kBoxThreads, 4>(n, pos, (int64_t)blockIdx.x * kBoxThreads + threadIdx.x,
                            (int64_t)gridDim.x * kBoxThreads, lo, hi);
    reduce_box<kBoxThreads>(lo, hi);
    if (threadIdx.x < 3) {
        part[6 * blockIdx.x + threadIdx.x] = lo[threadIdx.x][0];
        part[6 * blockIdx.x + 3 + threadIdx.x] = hi[threadIdx.x][0];
    }
}

// Moves bit b of the low 21 bits of v to bit 3b, by doubling the gaps between groups of
// bits (v has at most 21 significant bits; higher ones are dropped).
__device__ __forceinline__ uint64_t spread3(uint64_t v) {
    v &= 0x1fffffull;
    v = (v | (v << 32)) & 0x001f00000000ffffull;
    v = (v | (v << 16)) & 0x001f0000ff0000ffull;
    v = (v | (v << 8)) & 0x100f00f00f00f00full;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

// Word of particle i: coordinates quantised to qbits in the box, interleaved, then the
// index in ibits.
__device__ __forceinline__ uint64_t particle_word(int64_t i, const double (&x)[3],
                                                  const double (&lo)[3], const double (&hi)[3],
                                                  int qbits, int ibits) {
    const uint64_t low = (1ull << qbits) - 1;
    const double top = (double)low;
    uint64_t key = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double span = hi[c] - lo[c];
        double q = span > 0.0 ? (x[c] - lo[c]) / span * top : 0.0;
        q = q < 0.0 ? 0.0 : (q > top ? top : q);
        key |= spread3((uint64_t)q & low) << (2 - c);
    }
    return (key << ibits) | (uint64_t)i;
}

// Up to kBitonic particles in one block: npow (a power of two >= n) words in LDS.
__global__ __launch_bounds__(kSmallThreads) void small_kernel(int n, int npow, const double *pos,
                                                             int qbits, int ibits, int32_t *perm) {
    extern __shared__ uint64_t words[];
    // The box reduction comes first, in the same memory.
    double(*lo)[kSmallThreads] = reinterpret_cast<double(*)[kSmallThreads]>(words);
    double(*hi)[kSmallThreads] = lo + 3;
    const int t = threadIdx.x;
    thread_box<kSmallThreads>(n, pos, t, kSmallThreads, lo, hi);
    reduce_box<kSmallThreads>(lo, hi);
    double l[3], h[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        l[c] = lo[c][0];
        h[c] = hi[c][0];
    }
    __syncthreads();
    for (int i = t; i < npow; i += kSmallThreads) {
        uint64_t w = ~0ull;
        if (i < n) {
            const double x[3] = {pos[i], pos[n + i], pos[2 * n + i]};
            w = particle_word(i, x, l, h, qbits, ibits);
        }
        words[i] = w;
    }
    __syncthreads();
    for (int k = 2; k <= npow; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int p = t; p < npow / 2; p += kSmallThreads) {
                const int i = 2 * p - (p & (j - 1));  // p with a zero inserted at bit log2 j
                const uint64_t x = words[i], y = words[i + j];
                if ((x > y) == ((i & k) == 0)) {
                    words[i] = y;
                    words[i + j] = x;
                }
            }
            __syncthreads();
        }
    const uint64_t mask = (1ull << ibits) - 1;
    for (int i = t; i < n; i += kSmallThreads) perm[i] = (int32_t)(words[i] & mask);
}

// Lanes of the wave that hold a word (valid) with this lane's digit.
__device__ __forceinline__ unsigned long long peers(unsigned d, int bits, bool valid) {
    unsigned long long m = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
        const bool one = (d >> b) & 1u;
        const unsigned long long v = __ballot(one);
        m &= one ? v : ~v;
    }
    return m;
}

// Inclusive prefix sum over the wave's lanes.
__device__ __forceinline__ unsigned wave_prefix(unsigned v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned o = __shfl_up(v, d);
        v += lane >= d ? o : 0;
    }
    return v;
}

// Up to ROWS * kSmallThreads particles in one block: the radix passes below with every word in
// registers between them and in LDS during them.  A wave holds ROWS consecutive rows of 64.
template <int ROWS>
__global__ __launch_bounds__(kSmallThreads) void small_radix_kernel(int n, const double *pos,
                                                                   int qbits, int ibits, int bits,
                                                                   int passes, int32_t *perm) {
    constexpr int W = kSmallThreads / 64;
    __shared__ unsigned hist[W][kMaxDigits];  // per wave, then the wave's first slot
    __shared__ unsigned scan[kMaxDigits / 64];
    extern __shared__ uint64_t words[];
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = t >> 6;
    // The box first, in the words' memory.
    double(*lo)[kSmallThreads] = reinterpret_cast<double(*)[kSmallThreads]>(words);
    double(*hi)[kSmallThreads] = lo + 3;
    thread_box<kSmallThreads>(n, pos, t, kSmallThreads, lo, hi);
    reduce_box<kSmallThreads>(lo, hi);
    double l[3], h[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        l[c] = lo[c][0];
        h[c] = hi[c][0];
    }
    uint64_t w[ROWS];
    bool valid[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int i = (wave * ROWS + r) * 64 + lane;
        valid[r] = i < n;
        w[r] = 0;
        if (valid[r]) {
            const double x[3] = {pos[i], pos[n + i], pos[2 * n + i]};
            w[r] = particle_word(i, x, l, h, qbits, ibits);
        }
    }
    const unsigned digits = 1u << bits;
    for (int p = 0; p < passes; ++p) {
        const int shift = ibits + p * bits;
        __syncthreads();
        for (int q = t; q < W * kMaxDigits; q += kSmallThreads) (&hist[0][0])[q] = 0;
        __syncthreads();
        unsigned slot[ROWS];
        volatile unsigned *mine = hist[wave];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const unsigned d = (unsigned)(w[r] >> shift) & (digits - 1);
            const unsigned long long m = peers(d, bits, valid[r]);
            const unsigned before = mine[d];
            slot[r] = before + (unsigned)__popcll(m & ((1ull << lane) - 1));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (valid[r] && lane == __ffsll((long long)m) - 1) mine[d] = before + (unsigned)__popcll(m);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        __syncthreads();
        // Digit t: exclusive prefix sums of its counts over the digits, then over the waves.
        unsigned own = 0;
        if (t < kMaxDigits)
            for (int v = 0; v < W; ++v) own += hist[v][t];
        unsigned to = wave_prefix(own);
        if (wave < kMaxDigits / 64 && lane == 63) scan[wave] = to;
        __syncthreads();
        if (t < kMaxDigits) {
#pragma unroll
            for (int v = 0; v < kMaxDigits / 64; ++v) to += v < wave ? scan[v] : 0;
            unsigned first = to - own;
            for (int v = 0; v < W; ++v) {
                const unsigned c = hist[v][t];
                hist[v][t] = first;
                first += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (valid[r]) words[hist[wave][(unsigned)(w[r] >> shift) & (digits - 1)] + slot[r]] = w[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
            if (valid[r]) w[r] = words[(wave * ROWS + r) * 64 + lane];
    }
    const uint64_t mask = (1ull << ibits) - 1;
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (valid[r]) perm[(wave * ROWS + r) * 64 + lane] = (int32_t)(w[r] & mask);
}

// The tile's digit counts into counts[digit][tile].  Lanes add one by one to one of kCopies sets
// of counts each, so that few of a wave's additions meet where many words share a digit, as
// the high digits of clustered particles do (2^20 particles of a Plummer sphere: with one set
// 127 us, with eight 112 us; uniform ones 112 us with either).
constexpr int kCopies = 8;
constexpr int kCopyStride = kMaxDigits + 8;  // the copies of a digit in different banks
__device__ __forceinline__ void tile_counts(const uint64_t (&w)[kRows], const bool (&valid)[kRows],
                                            int shift, int bits,
                                            unsigned (&sh)[kCopies * kCopyStride],
                                            unsigned *counts, int tiles) {
    const unsigned digits = 1u << bits;
    for (int q = threadIdx.x; q < kCopies * kCopyStride; q += kTileThreads) sh[q] = 0;
    __syncthreads();
    unsigned *mine = sh + (threadIdx.x % kCopies) * kCopyStride;
#pragma unroll
    for (int r = 0; r < kRows; ++r)
        if (valid[r]) atomicAdd(&mine[(unsigned)(w[r] >> shift) & (digits - 1)], 1u);
    __syncthreads();
    for (unsigned d = threadIdx.x; d < digits; d += kTileThreads) {
        unsigned sum = 0;
#pragma unroll
        for (int k = 0; k < kCopies; ++k) sum += sh[k * kCopyStride + d];
        counts[(size_t)d * tiles + blockIdx.x] = sum;
    }
}

// Index of row r's word of this lane: a wave holds kRows consecutive rows of 64.
__device__ __forceinline__ int64_t word_index(int r) {
    return (int64_t)blockIdx.x * kTile + (threadIdx.x >> 6) * (kRows * 64) + r * 64 + (threadIdx.x & 63);
}

// Final reduction of the box (by every wave), the words of the block's
// tile, and the first digit's counts.
__global__ __launch_bounds__(kTileThreads) void word_kernel(int64_t n, const double *pos,
                                                           const double *part, int qbits, int ibits,
                                                           int bits, uint64_t *words,
                                                           unsigned *counts, int tiles) {
    __shared__ unsigned sh[kCopies * kCopyStride];
    double x[kRows][3];
    bool valid[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const int64_t i = word_index(r);
        valid[r] = i < n;
#pragma unroll
        for (int c = 0; c < 3; ++c) x[r][c] = valid[r] ? pos[c * n + i] : 0.0;
    }
    double l[3], h[3];
    wave_box(part, l, h);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        l[c] = __shfl(l[c], 0);
        h[c] = __shfl(h[c], 0);
    }
    uint64_t w[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const int64_t i = word_index(r);
        w[r] = 0;
        if (valid[r]) {
            w[r] = particle_word(i, x[r], l, h, qbits, ibits);
            words[i] = w[r];
        }
    }
    tile_counts(w, valid, ibits, bits, sh, counts, tiles);
}

__global__ __launch_bounds__(kTileThreads) void count_kernel(int64_t n, const uint64_t *words,
                                                            int shift, int bits, unsigned *counts,
                                                            int tiles) {
    __shared__ unsigned sh[kCopies * kCopyStride];
    uint64_t w[kRows];
    bool valid[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const int64_t i = word_index(r);
        valid[r] = i < n;
        w[r] = valid[r] ? words[i] : 0;
    }
    tile_counts(w, valid, shift, bits, sh, counts, tiles);
}

// Exclusive prefix sum of v over the block's threads (256); total in `sum`.
__device__ __forceinline__ unsigned block_prefix(unsigned v, unsigned (&sh)[4], unsigned *sum) {
    const int wave = threadIdx.x >> 6;
    const unsigned incl = wave_prefix(v);
    __syncthreads();
    if (threadIdx.x % 64 == 63) sh[wave] = incl;
    __syncthreads();
    unsigned before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        before += w < wave ? sh[w] : 0;
        all += sh[w];
    }
    *sum = all;
    return before + incl - v;
}

// Block d: counts[d][0 .. tiles) to exclusive prefix sums, and the digit's total.
__global__ __launch_bounds__(256) void scan_kernel(unsigned *counts, unsigned *totals, int tiles) {
    __shared__ unsigned sh[4];
    unsigned *row = counts + (size_t)blockIdx.x * tiles;
    unsigned run = 0;
    for (int b = 0; b < tiles; b += 256) {
        const int q = b + threadIdx.x;
        const unsigned v = q < tiles ? row[q] : 0;
        unsigned sum;
        const unsigned pre = block_prefix(v, sh, &sum);
        if (q < tiles) row[q] = run + pre;
        run += sum;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = run;
}

// Stable scatter of the tile by the digit; the last pass writes the permutation instead.
template <bool LAST>
__global__ __launch_bounds__(kTileThreads) void scatter_kernel(int64_t n, const uint64_t *in,
                                                              int shift, int bits,
                                                              const unsigned *counts,
                                                              const unsigned *totals, int tiles,
                                                              uint64_t *out, int32_t *perm,
                                                              uint64_t mask) {
    __shared__ uint64_t sorted[kTile];
    __shared__ unsigned hist[kWaves][kMaxDigits];  // per wave, then the wave's first local slot
    __shared__ unsigned scan[2][kMaxDigits / 64];  // per wave
    __shared__ unsigned dest[kMaxDigits];          // output slot - local slot of each digit's
                                                   // words (modulo 2^32)
    const unsigned digits = 1u << bits;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = t >> 6;
    for (int v = 0; v < kWaves; ++v)
        for (int q = t; q < kMaxDigits; q += kTileThreads) hist[v][q] = 0;

    uint64_t w[kRows];
    bool valid[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const int64_t i = word_index(r);
        valid[r] = i < n;
        w[r] = valid[r] ? in[i] : 0;
    }
    unsigned total = 0, before_tile = 0;  // digit t's, needed after the ranks
    if (t < (int)digits) {
        total = totals[t];
        before_tile = counts[(size_t)t * tiles + blockIdx.x];
    }
    __syncthreads();
    // Rank of each word among the wave's words of the same digit, row by row.
    unsigned dg[kRows], rank[kRows];
    volatile unsigned *mine = hist[wave];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        dg[r] = (unsigned)(w[r] >> shift) & (digits - 1);
        const unsigned long long m = peers(dg[r], bits, valid[r]);
        const unsigned before = mine[dg[r]];
        rank[r] = before + (unsigned)__popcll(m & ((1ull << lane) - 1));
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (valid[r] && lane == __ffsll((long long)m) - 1) mine[dg[r]] = before + (unsigned)__popcll(m);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    // Digit t: its count in the tile, and exclusive prefix sums over the digits of the
    // tile's counts (local slots) and of the totals (output slots).
    unsigned own = 0;
    if (t < (int)digits)
        for (int v = 0; v < kWaves; ++v) own += hist[v][t];
    unsigned own_to = wave_prefix(own), total_to = wave_prefix(total);
    if (wave < kMaxDigits / 64 && lane == 63) {
        scan[0][wave] = own_to;
        scan[1][wave] = total_to;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kMaxDigits / 64; ++v)
        if (v < wave) {
            own_to += scan[0][v];
            total_to += scan[1][v];
        }
    if (t < (int)digits) {
        unsigned slot = own_to - own;
        dest[t] = total_to - total + before_tile - slot;
        for (int v = 0; v < kWaves; ++v) {
            const unsigned c = hist[v][t];
            hist[v][t] = slot;
            slot += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRows; ++r)
        if (valid[r]) sorted[hist[wave][dg[r]] + rank[r]] = w[r];
    __syncthreads();
    const int64_t left = n - (int64_t)blockIdx.x * kTile;
    const int cnt = left < kTile ? (int)left : kTile;
    for (int q = t; q < cnt; q += kTileThreads) {
        const uint64_t v = sorted[q];
        const unsigned o = dest[(unsigned)(v >> shift) & (digits - 1)] + (unsigned)q;
        if constexpr (LAST)
            perm[o] = (int32_t)(v & mask);
        else
            out[o] = v;
    }
}

int tiles_of(int64_t n) { return (int)((n + kTile - 1) / kTile); }

}  // namespace

size_t morton_scratch_bytes(int64_t n) {
    if (n <= kSmall) return 256;
    return 2 * sizeof(uint64_t) * (size_t)n + sizeof(double) * 6 * kBoxBlocks +
           sizeof(unsigned) * kMaxDigits * ((size_t)tiles_of(n) + 1);
}

nbody_status launch_morton_order(int64_t n, const double *pos64, int32_t *perm, void *scratch,
                                 hipStream_t s) {
    if (n <= 0) return NBODY_OK;
    int ibits = 0;
    while ((int64_t(1) << ibits) < n) ++ibits;
    const int qbits = (64 - ibits) / 3;
    const int key_bits = 3 * qbits;
    const int passes = (key_bits + 7) / 8;
    const int bits = (key_bits + passes - 1) / passes;  // digits of 6 to 8 bits
    if (n <= kBitonic) {
        int npow = 1;
        while (npow < n) npow <<= 1;
        // At least the box reduction's six doubles per thread.
        size_t lds = sizeof(uint64_t) * (size_t)npow;
        if (lds < sizeof(double) * 6 * kSmallThreads) lds = sizeof(double) * 6 * kSmallThreads;
        hipLaunchKernelGGL(small_kernel, dim3(1), dim3(kSmallThreads), lds, s, (int)n, npow, pos64,
                           qbits, ibits, perm);
        NBODY_HIP_CHECK(hipGetLastError());
        return NBODY_OK;
    }
    if (n <= kSmall) {
        auto fn = n <= 2 * kSmallThreads   ? small_radix_kernel<2>
                  : n <= 4 * kSmallThreads ? small_radix_kernel<4>
                                           : small_radix_kernel<8>;
        const size_t lds = std::max(sizeof(uint64_t) * (size_t)n, sizeof(double) * 6 * kSmallThreads);
        hipLaunchKernelGGL(fn, dim3(1), dim3(kSmallThreads), lds, s, (int)n, pos64, qbits, ibits, bits,
                           passes, perm);
        NBODY_HIP_CHECK(hipGetLastError());
        return NBODY_OK;
    }
    uint64_t *words = static_cast<uint64_t *>(scratch);
    uint64_t *other = words + n;
    double *part = reinterpret_cast<double *>(other + n);
    unsigned *totals = reinterpret_cast<unsigned *>(part + 6 * kBoxBlocks);
    unsigned *counts = totals + kMaxDigits;
    const int tiles = tiles_of(n);
    const uint64_t mask = (1ull << ibits) - 1;
    const dim3 grid((unsigned)tiles), block(kTileThreads);
    hipLaunchKernelGGL(box_partial_kernel, dim3(kBoxBlocks), dim3(kBoxThreads), 0, s, n, pos64, part);
    hipLaunchKernelGGL(word_kernel, grid, block, 0, s, n, pos64, (const double *)part, qbits, ibits,
                       bits, words, counts, tiles);
    for (int p = 0; p < passes; ++p) {
        const int shift = ibits + p * bits;
        if (p)
            hipLaunchKernelGGL(count_kernel, grid, block, 0, s, n, (const uint64_t *)words, shift,
                               bits, counts, tiles);
        hipLaunchKernelGGL(scan_kernel, dim3(1u << bits), dim3(256), 0, s, counts, totals, tiles);
        if (p + 1 == passes)
            hipLaunchKernelGGL(scatter_kernel<true>, grid, block, 0, s, n, (const uint64_t *)words,
                               shift, bits, (const unsigned *)counts, (const unsigned *)totals,
                               tiles, other, perm, mask);
        else
            hipLaunchKernelGGL(scatter_kernel<false>, grid, block, 0, s, n, (const uint64_t *)words,
                               shift, bits, (const unsigned *)counts, (const unsigned *)totals,
                               tiles, other, perm, mask);
        std::swap(words, other);
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

}  // namespace nbody
