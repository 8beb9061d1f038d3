// Force evaluation of one system: the gravity pipeline on the wave engine (grid
// launch), the FP64 finalize, and the FP64-position pre-pass (centre, conversion).
#include "centre_sum.h"
#include "gravity.h"
#include "outputs.h"
#include "wave_engine.h"

namespace nbody {
namespace {

// Fixed-order sum of the segment partials (PLAIN in FP32, the other modes in FP64),
// one thread per (particle, output) so that few particles with many segments still
// fill the chip.  The partials hold no j == i term (the pair kernel left it out); with
// include_self the potential gets -m_i / eps, formed in FP64.
// With kick_v set, the velocity kick of a leapfrog step follows in FP64.
// Grid: (ceil(n / 256), 4 outputs, or 3 without potentials).
template <int MODE, int BATCH>
__global__ __launch_bounds__(256) void finalize_kernel(FinalizeArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (i >= a.n) return;
    ForceOut::put(a, i, c, [&](int o) {
        return engine::sum_partial_output<kForceOutputs, MODE, BATCH>(a.part, a.nseg,
                                                                      (size_t)a.npad, i, o);
    });
}

// The same between two leapfrog steps: block (b, c) holds component c of the particles
// [256 b, 256 b + 256), so after the drift it also sums its part of the centre's first stage.
// Grid: (kCentreBlocks, 3).
template <int MODE, int BATCH>
__global__ __launch_bounds__(256) void finalize_step_kernel(FinalizeArgs a, double *centre_part) {
    __shared__ double sh[1][256];
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int c = blockIdx.y;
    double x = 0.0;
    if (i < a.n)
        x = ForceOut::store(a, (size_t)c * a.n + i,
                            engine::sum_partial_output<kForceOutputs, MODE, BATCH>(
                                a.part, a.nseg, (size_t)a.npad, i, c));
    const double sum = centre::block_sum<1>({x}, sh);
    if (threadIdx.x == 0) centre_part[3 * blockIdx.x + c] = sum;
}

// Two-stage fixed-order FP64 mean of the positions [3][n]: kCentreBlocks partial
// sums, then their fixed-order sum.  Deterministic for a given n.

__global__ __launch_bounds__(256) void centre_partial_kernel(int64_t n, const double *pos,
                                                            double *part) {
    __shared__ double sh[3][256];
    double s[3] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] += pos[c * n + i];
    const double sum = centre::block_sum(s, sh);
    const int c = threadIdx.x >> 6;
    if (c < 3 && threadIdx.x % 64 == 0) part[blockIdx.x * 3 + c] = sum;
}

// The second stage fused with the conversion to FP32: every wave adds the kCentreBlocks
// partials in the same fixed tree order, so all use the identical centre c = sum / n, then
// converts its 64 particles to fp32(x - c).
__device__ __forceinline__ void convert_centred(int64_t n, const double *pos, const double *part,
                                                float *out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double x[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) x[c] = i < n ? pos[c * n + i] : 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double mean = centre::partials_sum(part, c) / (double)n;
        if (i < n) out[c * n + i] = (float)(x[c] - mean);
    }
}

__global__ __launch_bounds__(256) void centred_convert_kernel(int64_t n, const double *pos,
                                                             const double *part, float *out) {
    convert_centred(n, pos, part, out);
}

// The second stage and conversion of two arrays (blockIdx.y).
__global__ __launch_bounds__(256) void centred_convert2_kernel(int64_t n, const double *a,
                                                              const double *a_part, float *a_out,
                                                              const double *b,
                                                              const double *b_part, float *b_out) {
    const double *pos = blockIdx.y ? b : a;
    const double *part = blockIdx.y ? b_part : a_part;
    float *out = blockIdx.y ? b_out : a_out;
    convert_centred(n, pos, part, out);
}

// Centre and conversion in one launch, for few particles (kSelfCentre): each block adds the
// whole centre in the order of the two stages, a wave taking 256 particles (one first-stage
// block) at a time with its lanes holding what would be four threads, two at a time in flight
// (the latency of the loads is most of the launch; blocks of 16 waves, which need fewer
// rounds of them, take longer to start: 16 steps of 2048 particles 180 instead of 172 us).
// Reading every position per block costs less than the launch of a separate first stage.
__global__ __launch_bounds__(256) void self_centred_convert_kernel(int64_t n, const double *a,
                                                                  float *a_out, const double *b,
                                                                  float *b_out) {
    __shared__ double sh[3][32];
    const double *pos = blockIdx.y ? b : a;
    float *out = blockIdx.y ? b_out : a_out;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunks = (int)((n + 255) / 256);  // at most 32
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double mine[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) mine[c] = i < n ? pos[c * n + i] : 0.0;
    for (int q0 = wave; q0 < chunks; q0 += 8) {
        double v[2][3][4];
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int64_t p = (q0 + 4 * d) * 256 + k * 64 + lane;
                    v[d][c][k] = p < n ? pos[c * n + p] : 0.0;
                }
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double s = centre::wave_sum(v[d][c]);
                if (lane == 0 && q0 + 4 * d < chunks) sh[c][q0 + 4 * d] = s;
            }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double mean = centre::second_stage(sh[c], chunks, lane) / (double)n;
        if (i < n) out[c * n + i] = (float)(mine[c] - mean);
    }
}

__global__ __launch_bounds__(256) void convert_kernel(int64_t n, const double *pos,
                                                     const double *centre, float *out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
#pragma unroll
    for (int c = 0; c < 3; ++c) out[c * n + i] = (float)(pos[c * n + i] - (centre ? centre[c] : 0.0));
}

// Mean position of each i-tile of `itile` consecutive particles, FP64, one block per
// tile, fixed-order tree: the reference centres of NBODY_CENTRE_TILE.
__global__ __launch_bounds__(256) void tile_centre_kernel(int64_t n, int itile, const double *pos,
                                                         double *centres) {
    __shared__ double sh[3][256];
    const int64_t b = (int64_t)blockIdx.x * itile;
    const int64_t e = b + itile < n ? b + itile : n;
    double s[3] = {0.0, 0.0, 0.0};
    for (int64_t p = b + threadIdx.x; p < e; p += 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] += pos[c * n + p];
    const double sum = centre::block_sum(s, sh);
    const int c = threadIdx.x >> 6;
    if (c < 3 && threadIdx.x % 64 == 0) centres[3 * blockIdx.x + c] = sum / (double)(e - b);
}

}  // namespace

nbody_status launch_tile_centres(int64_t n, int itile, const double *pos64, double *centres,
                                 hipStream_t s) {
    if (n <= 0) return NBODY_OK;
    const int64_t tiles = (n + itile - 1) / itile;
    hipLaunchKernelGGL(tile_centre_kernel, dim3((unsigned)tiles), dim3(256), 0, s, n, itile, pos64,
                       centres);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_pair_tile(const TileCfg &cfg, int precision, bool with_pot,
                              const TilePairArgs &a, const FinalizeArgs &f, hipStream_t s) {
    return wave::launch<GravityTile, ForceOut>(cfg, precision, with_pot, a.n, a, f, s);
}

nbody_status launch_pair(const TileCfg &cfg, int precision, bool with_pot, const PairArgs &a,
                         const FinalizeArgs &f, hipStream_t s) {
    return wave::launch<Gravity, ForceOut>(cfg, precision, with_pot, a.n, a, f, s);
}

template <int MODE>
void launch_finalize_mode(dim3 grid, bool deep, const FinalizeArgs &a, hipStream_t s) {
    if (deep)
        hipLaunchKernelGGL((finalize_kernel<MODE, 8>), grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((finalize_kernel<MODE, 1>), grid, dim3(256), 0, s, a);
}

nbody_status launch_finalize(int precision, const FinalizeArgs &a, hipStream_t s) {
    if (a.n <= 0) return NBODY_OK;
    const int outputs = a.pot ? 4 : 3;
    const dim3 grid((a.n + 255) / 256, outputs);
    const bool deep = engine::finalize_batch(a.n, outputs) > 1;
    switch (precision) {
        case NBODY_PLAIN: launch_finalize_mode<NBODY_PLAIN>(grid, deep, a, s); break;
        case NBODY_FP64RED: launch_finalize_mode<NBODY_FP64RED>(grid, deep, a, s); break;
        case NBODY_COMP: launch_finalize_mode<NBODY_COMP>(grid, deep, a, s); break;
        default: return set_error(NBODY_EINVAL, "unknown precision mode");
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

template <int MODE>
void launch_finalize_step_mode(bool deep, const FinalizeArgs &a, double *centre_part,
                               hipStream_t s) {
    const dim3 grid(kCentreBlocks, 3);
    if (deep)
        hipLaunchKernelGGL((finalize_step_kernel<MODE, 8>), grid, dim3(256), 0, s, a, centre_part);
    else
        hipLaunchKernelGGL((finalize_step_kernel<MODE, 1>), grid, dim3(256), 0, s, a, centre_part);
}

nbody_status launch_finalize_step(int precision, const FinalizeArgs &a, double *centre_part,
                                  hipStream_t s) {
    if (a.n <= 0) return NBODY_OK;
    const bool deep = engine::finalize_batch(a.n, 3) > 1;
    switch (precision) {
        case NBODY_PLAIN: launch_finalize_step_mode<NBODY_PLAIN>(deep, a, centre_part, s); break;
        case NBODY_FP64RED: launch_finalize_step_mode<NBODY_FP64RED>(deep, a, centre_part, s); break;
        case NBODY_COMP: launch_finalize_step_mode<NBODY_COMP>(deep, a, centre_part, s); break;
        default: return set_error(NBODY_EINVAL, "unknown precision mode");
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

size_t centre_scratch_bytes() { return sizeof(double) * 3 * kCentreBlocks; }

nbody_status launch_centred_convert(int64_t n, const double *pos64, double *scratch,
                                    float *pos32, hipStream_t s) {
    if (n <= 0) return NBODY_OK;
    if (n <= kSelfCentreOne) return launch_self_centred_convert(n, pos64, pos32, nullptr, nullptr, s);
    hipLaunchKernelGGL(centre_partial_kernel, dim3(kCentreBlocks), dim3(256), 0, s, n, pos64, scratch);
    NBODY_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(centred_convert_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       n, pos64, (const double *)scratch, pos32);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_centred_convert_ready(int64_t n, const double *pos64, const double *scratch,
                                          float *pos32, hipStream_t s) {
    if (n <= 0) return NBODY_OK;
    hipLaunchKernelGGL(centred_convert_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       n, pos64, scratch, pos32);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_centred_convert_ready2(int64_t n, const double *a64, const double *a_part,
                                           float *a32, const double *b64, const double *b_part,
                                           float *b32, hipStream_t s) {
    if (n <= 0) return NBODY_OK;
    hipLaunchKernelGGL(centred_convert2_kernel, dim3((unsigned)((n + 255) / 256), 2), dim3(256), 0, s,
                       n, a64, a_part, a32, b64, b_part, b32);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_self_centred_convert(int64_t n, const double *a64, float *a32, const double *b64,
                                         float *b32, hipStream_t s) {
    if (n <= 0) return NBODY_OK;
    if (n > kSelfCentre) return set_error(NBODY_EINVAL, "too many particles for a one-launch centre");
    hipLaunchKernelGGL(self_centred_convert_kernel,
                       dim3((unsigned)((n + 255) / 256), b64 ? 2 : 1), dim3(256), 0, s, n, a64, a32,
                       b64, b32);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_convert(int64_t n, const double *pos64, const double *centre, float *pos32,
                            hipStream_t s) {
    if (n <= 0) return NBODY_OK;
    hipLaunchKernelGGL(convert_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, pos64,
                       centre, pos32);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

}  // namespace nbody
