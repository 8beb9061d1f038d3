// Kernels of the ragged batched path: many independent systems stored back to back
// (system k owns the global indices [offsets[k], offsets[k+1])).
//
//   * pair work: one block per work item of the plan (some i's x one j-range of one
//     system), in decreasing order of cost, on the wave engine; a system whose j-range is
//     not split gets its outputs (and the fused leapfrog kick) stored right there;
//   * finalize: per particle of the other systems, the fixed-order FP64 sum of the
//     segment partials (no j == i term: the pair kernel left it out) and the kick;
//   * per-system FP64 centres (one block per system, fixed-order reduction) and the
//     conversion of FP64 positions to FP32 relative to them.
#include <algorithm>

#include "centre_sum.h"
#include "gravity.h"
#include "outputs.h"
#include "wave_engine.h"

namespace nbody {
namespace {

// One block per work item, the dispatcher taking them in order: the expensive items start
// first and the small ones fill the tail.
template <int IPL, int BJ, int MODE, bool FULL>
__global__ __launch_bounds__(1024) void batched_pair_kernel(PairArgs a, FinalizeArgs f,
                                                            BatchSched sc) {
    constexpr int V = Gravity::kJWords / 4;
    extern __shared__ float4 lds[];
    const BatchItem it = sc.items[blockIdx.x];
    const float e = sc.eps[it.sys];
    const float eps2 = e * e;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    float4 *tl = lds + wave * wave::kStage * V;
    float hs[IPL][4], ls[IPL][4];
    double ds[IPL][4];
    float *part = static_cast<float *>(sc.part) + it.part;
    if constexpr (MODE == NBODY_PLAIN) {
        wave::wave_work<Gravity, IPL, BJ, MODE, FULL>(a, tl, it.i0, it.ni, it.j0, it.nj, eps2, hs,
                                                      ls, ds);
        wave::store_plain<ForceOut, IPL, FULL>(f, it.i0, it.i0 + it.ni, hs, it.whole, part,
                                               (size_t)it.npad, (size_t)it.col0);
    } else {
        const wave::Range r = wave::block_run<BJ>(it.nj, wave, waves);
        wave::wave_work<Gravity, IPL, BJ, MODE, FULL>(a, tl, it.i0, it.ni, it.j0 + r.j0, r.nj, eps2,
                                                      hs, ls, ds);
        wave::store_sums<ForceOut, IPL, MODE, FULL>(f, reinterpret_cast<double *>(lds), wave,
                                                    waves, it.i0, it.i0 + it.ni, hs, ls, ds, it.whole,
                                                    part, (size_t)it.npad, (size_t)it.col0);
    }
}

template <int MODE>
__global__ __launch_bounds__(256) void batched_finalize_kernel(BatchFinalizeArgs a) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= a.total) return;
    const int k = a.sys_of[p];
    const int64_t col = p - a.offsets[k];
    if (a.nseg[k] <= 1) return;  // stored by the pair launch
    const int npad = a.npad[k];
    const void *base = static_cast<const float *>(a.part) + a.part_base[k];
    double r[4];
    engine::sum_partials<4, MODE, 1>(base, a.nseg[k], (size_t)npad, (int)col, r);
    const size_t n = (size_t)a.total;
    a.acc[p] = r[0];
    a.acc[n + p] = r[1];
    a.acc[2 * n + p] = r[2];
    if (a.pot) a.pot[p] = r[3];
    if (a.kick_v) {
#pragma unroll
        for (int c = 0; c < 3; ++c) a.kick_v[c * n + p] += a.kick_h * r[c];
    }
}

// Mean position of each system in FP64: block k sums its particles with a fixed
// stride pattern and tree, so the result is reproducible.
__global__ __launch_bounds__(256) void system_centre_kernel(const int64_t *offsets, int64_t total,
                                                           const double *pos, double *centre) {
    __shared__ double sh[3][256];
    const int k = blockIdx.x;
    const int64_t b = offsets[k], e = offsets[k + 1];
    double s[3] = {0.0, 0.0, 0.0};
    for (int64_t p = b + threadIdx.x; p < e; p += 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] += pos[c * total + p];
    const double sum = centre::block_sum(s, sh);
    const int c = threadIdx.x >> 6;
    if (c < 3 && threadIdx.x % 64 == 0) centre[3 * k + c] = e > b ? sum / (double)(e - b) : 0.0;
}

// One block per system: the leapfrog's first kick and drift (v not null), the FP64 centre in
// the order of system_centre_kernel, and the conversion relative to it.
__global__ __launch_bounds__(256) void system_step_kernel(const int64_t *offsets, int64_t total,
                                                         double *x, double *v, const double *a,
                                                         double h, double dt, float *out) {
    __shared__ double sh[3][256];
    const int64_t b = offsets[blockIdx.x], e = offsets[blockIdx.x + 1];
    double s[3] = {0.0, 0.0, 0.0};
    for (int64_t p = b + threadIdx.x; p < e; p += 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int64_t q = c * total + p;
            double xx = x[q];
            if (v) {
                const double vv = v[q] + h * a[q];
                v[q] = vv;
                xx = xx + dt * vv;
                x[q] = xx;
            }
            s[c] += xx;
        }
    const double sum = centre::block_sum(s, sh);
    const int wave = threadIdx.x >> 6;
    if (wave < 3 && threadIdx.x % 64 == 0) sh[wave][0] = sum;  // wave c alone reads sh[c] before
    __syncthreads();
    for (int64_t p = b + threadIdx.x; p < e; p += 256)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int64_t q = c * total + p;
            out[q] = (float)(x[q] - sh[c][0] / (double)(e - b));
        }
}

__global__ __launch_bounds__(256) void batched_convert_kernel(int64_t total, const double *pos,
                                                             const int32_t *sys_of,
                                                             const double *centre, float *out) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= total) return;
    const int k = sys_of[p];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        out[c * total + p] = (float)(pos[c * total + p] - (centre ? centre[3 * k + c] : 0.0));
}

}  // namespace

namespace {

using BatchFn = void (*)(PairArgs, FinalizeArgs, BatchSched);

template <int IPL>
BatchFn pick_batched(int jt, int mode, bool full) {
    switch (mode) {
        case NBODY_PLAIN:
            return full ? batched_pair_kernel<IPL, 64, NBODY_PLAIN, true>
                        : batched_pair_kernel<IPL, 64, NBODY_PLAIN, false>;
        case NBODY_FP64RED:
            if (jt == 64)
                return full ? batched_pair_kernel<IPL, 64, NBODY_FP64RED, true>
                            : batched_pair_kernel<IPL, 64, NBODY_FP64RED, false>;
            return full ? batched_pair_kernel<IPL, 128, NBODY_FP64RED, true>
                        : batched_pair_kernel<IPL, 128, NBODY_FP64RED, false>;
        case NBODY_COMP:
            if (jt == 64)
                return full ? batched_pair_kernel<IPL, 64, NBODY_COMP, true>
                            : batched_pair_kernel<IPL, 64, NBODY_COMP, false>;
            return full ? batched_pair_kernel<IPL, 128, NBODY_COMP, true>
                        : batched_pair_kernel<IPL, 128, NBODY_COMP, false>;
    }
    return nullptr;
}

}  // namespace

nbody_status launch_batched_pair(int ipl, int jt, int waves, int precision, bool with_pot,
                                 const PairArgs &a, const FinalizeArgs &f, const BatchSched &sc,
                                 hipStream_t s) {
    const BatchFn fn = ipl == 1   ? pick_batched<1>(jt, precision, with_pot)
                       : ipl == 2 ? pick_batched<2>(jt, precision, with_pot)
                       : ipl == 4 ? pick_batched<4>(jt, precision, with_pot)
                                  : nullptr;
    if (!fn) return set_error(NBODY_EUNSUPPORTED, "no batched kernel for this shape");
    // One launch unless the items are more than its threads allow (2^24 items of 4 waves).
    const int64_t most = kMaxThreads / (64 * waves);
    for (int64_t first = 0; first < sc.nitems; first += most) {
        const int64_t count = std::min<int64_t>(most, sc.nitems - first);
        const BatchSched part{sc.items + first, (int)count, sc.eps, sc.part};
        hipLaunchKernelGGL(fn, dim3((unsigned)count), dim3(64 * waves),
                           wave::lds_bytes<Gravity>(waves), s, a, f, part);
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_batched_finalize(int precision, const BatchFinalizeArgs &a, hipStream_t s) {
    if (a.total <= 0) return NBODY_OK;
    const dim3 grid((unsigned)((a.total + 255) / 256));
    switch (precision) {
        case NBODY_PLAIN: hipLaunchKernelGGL(batched_finalize_kernel<NBODY_PLAIN>, grid, dim3(256), 0, s, a); break;
        case NBODY_FP64RED: hipLaunchKernelGGL(batched_finalize_kernel<NBODY_FP64RED>, grid, dim3(256), 0, s, a); break;
        case NBODY_COMP: hipLaunchKernelGGL(batched_finalize_kernel<NBODY_COMP>, grid, dim3(256), 0, s, a); break;
        default: return set_error(NBODY_EINVAL, "unknown precision mode");
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_system_centres(int nsys, const int64_t *offsets, int64_t total,
                                   const double *pos64, double *centre, hipStream_t s) {
    if (nsys <= 0) return NBODY_OK;
    hipLaunchKernelGGL(system_centre_kernel, dim3(nsys), dim3(256), 0, s, offsets, total, pos64, centre);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_system_step(int nsys, const int64_t *offsets, int64_t total, double *x, double *v,
                                const double *a, double h, double dt, float *pos32,
                                hipStream_t s) {
    if (nsys <= 0) return NBODY_OK;
    hipLaunchKernelGGL(system_step_kernel, dim3(nsys), dim3(256), 0, s, offsets, total, x, v, a, h,
                       dt, pos32);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_batched_convert(int64_t total, const double *pos64, const int32_t *sys_of,
                                    const double *centre, float *pos32, hipStream_t s) {
    if (total <= 0) return NBODY_OK;
    hipLaunchKernelGGL(batched_convert_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                       total, pos64, sys_of, centre, pos32);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

}  // namespace nbody
