// Launch of the adjoint pipeline on FP32 positions and the FP64 finalize of its
// partial sums.
#include "adjoint_pipeline.h"
#include "centre_sum.h"
#include "outputs.h"
#include "wave_engine.h"

namespace nbody {
namespace {

// One thread per (particle, store slot), as in the force finalize: fixed-order sums of
// the segment partials (which hold no j == k term), then dL/dx_k (slots 0-2, from the
// slot's own sum and the sum B_k) or dL/dm_k (slot 3, the negated mass sum).  Grid:
// (ceil(n / 256), 4 slots, or 3 without dL/dm).
template <int MODE, int BATCH>
__global__ __launch_bounds__(256) void vjp_finalize_kernel(VjpFinalizeArgs a) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (k >= a.n) return;
    VjpOut::put(a, k, c, [&](int o) {
        return engine::sum_partial_output<kVjpOutputs, MODE, BATCH>(a.part, a.nseg,
                                                                    (size_t)a.npad, k, o);
    });
}

// The same between two reverse leapfrog steps: slots 0-2 also update vbar and abar and sum
// their part of the centre's first stage over `next`.  Grid: (kCentreBlocks, 4 slots, or 3).
template <int MODE, int BATCH>
__global__ __launch_bounds__(256) void vjp_finalize_step_kernel(VjpFinalizeArgs a,
                                                               const double *next,
                                                               double *centre_part) {
    __shared__ double sh[1][256];
    const int k = blockIdx.x * 256 + threadIdx.x;
    const int c = blockIdx.y;
    if (k < a.n)
        VjpOut::put(a, k, c, [&](int o) {
            return engine::sum_partial_output<kVjpOutputs, MODE, BATCH>(a.part, a.nseg,
                                                                        (size_t)a.npad, k, o);
        });
    if (c < 3) {
        const double sum = centre::block_sum<1>({k < a.n ? next[(size_t)c * a.n + k] : 0.0}, sh);
        if (threadIdx.x == 0) centre_part[3 * blockIdx.x + c] = sum;
    }
}

}  // namespace

nbody_status launch_vjp(const TileCfg &cfg, int precision, const VjpArgs &a, bool with_mass,
                        const VjpFinalizeArgs &f, hipStream_t s) {
    return wave::launch<Adjoint, VjpOut>(cfg, precision, with_mass, a.n, a, f, s);
}

template <int MODE>
void launch_vjp_finalize_mode(dim3 grid, bool deep, const VjpFinalizeArgs &a, hipStream_t s) {
    if (deep)
        hipLaunchKernelGGL((vjp_finalize_kernel<MODE, 8>), grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((vjp_finalize_kernel<MODE, 1>), grid, dim3(256), 0, s, a);
}

template <int MODE>
void launch_vjp_finalize_step_mode(dim3 grid, bool deep, const VjpFinalizeArgs &a,
                                   const double *next, double *centre_part, hipStream_t s) {
    if (deep)
        hipLaunchKernelGGL((vjp_finalize_step_kernel<MODE, 8>), grid, dim3(256), 0, s, a, next, centre_part);
    else
        hipLaunchKernelGGL((vjp_finalize_step_kernel<MODE, 1>), grid, dim3(256), 0, s, a, next, centre_part);
}

nbody_status launch_vjp_finalize_step(int precision, const VjpFinalizeArgs &a, const double *next,
                                      double *centre_part, hipStream_t s) {
    if (a.n <= 0) return NBODY_OK;
    const int outputs = a.grad_mass ? 4 : 3;
    const dim3 grid(kCentreBlocks, outputs);
    const bool deep = engine::finalize_batch(a.n, outputs) > 1;
    switch (precision) {
        case NBODY_PLAIN:
            launch_vjp_finalize_step_mode<NBODY_PLAIN>(grid, deep, a, next, centre_part, s);
            break;
        case NBODY_FP64RED:
            launch_vjp_finalize_step_mode<NBODY_FP64RED>(grid, deep, a, next, centre_part, s);
            break;
        case NBODY_COMP:
            launch_vjp_finalize_step_mode<NBODY_COMP>(grid, deep, a, next, centre_part, s);
            break;
        default: return set_error(NBODY_EINVAL, "unknown precision mode");
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_vjp_finalize(int precision, const VjpFinalizeArgs &a, hipStream_t s) {
    if (a.n <= 0) return NBODY_OK;
    const int outputs = a.grad_mass ? 4 : 3;
    const dim3 grid((a.n + 255) / 256, outputs);
    const bool deep = engine::finalize_batch(a.n, outputs) > 1;
    switch (precision) {
        case NBODY_PLAIN: launch_vjp_finalize_mode<NBODY_PLAIN>(grid, deep, a, s); break;
        case NBODY_FP64RED: launch_vjp_finalize_mode<NBODY_FP64RED>(grid, deep, a, s); break;
        case NBODY_COMP: launch_vjp_finalize_mode<NBODY_COMP>(grid, deep, a, s); break;
        default: return set_error(NBODY_EINVAL, "unknown precision mode");
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

}  // namespace nbody
