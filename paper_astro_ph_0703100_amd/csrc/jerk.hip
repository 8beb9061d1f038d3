// Launch of the force-jerk-potential pipeline on FP32 inputs and the FP64 finalize of
// its partial sums (shared by every force-jerk path).
#include "centre_sum.h"
#include "jerk_pipeline.h"
#include "outputs.h"
#include "wave_engine.h"

namespace nbody {
namespace {

// One thread per (particle, output): fixed-order sums as in the force finalize (the
// partials hold no j == i term).  Grid: (ceil(n / 256), 7 outputs, or 6 without potentials).
template <int MODE, int BATCH>
__global__ __launch_bounds__(256) void jerk_finalize_kernel(JerkFinalizeArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (i >= a.n) return;
    JerkOut::put(a, i, c, [&](int o) {
        return engine::sum_partial_output<kJerkOutputs, MODE, BATCH>(a.part, a.nseg,
                                                                     (size_t)a.npad, i, o);
    });
}

// The same at the end of a Hermite step: thread (i, component c) adds the acceleration and the
// jerk, corrects, predicts the next state, and sums its part of the centres' first stages over
// that (x_part null: no next step).  Grid: (kCentreBlocks, 3).
template <int MODE, int BATCH>
__global__ __launch_bounds__(256) void jerk_finalize_step_kernel(JerkFinalizeArgs a, double *x_part,
                                                                double *v_part) {
    __shared__ double sh[2][256];
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int c = blockIdx.y;
    double2 p = make_double2(0.0, 0.0);
    if (i < a.n) {
        auto sum = [&](int o) {
            return engine::sum_partial_output<kJerkOutputs, MODE, BATCH>(a.part, a.nseg,
                                                                         (size_t)a.npad, i, o);
        };
        p = JerkOut::step(a, (size_t)c * a.n + i, sum(c), sum(c + 3));
    }
    if (!x_part) return;
    const double sum = centre::block_sum<2>({p.x, p.y}, sh);
    if (threadIdx.x == 0) x_part[3 * blockIdx.x + c] = sum;
    if (threadIdx.x == 64) v_part[3 * blockIdx.x + c] = sum;
}

}  // namespace

nbody_status launch_jerk(const TileCfg &cfg, int precision, bool with_pot, const JerkArgs &a,
                         const JerkFinalizeArgs &f, hipStream_t s) {
    return wave::launch<GravityJerk, JerkOut>(cfg, precision, with_pot, a.n, a, f, s);
}

template <int MODE>
void launch_jerk_finalize_mode(dim3 grid, bool deep, const JerkFinalizeArgs &a, hipStream_t s) {
    if (deep)
        hipLaunchKernelGGL((jerk_finalize_kernel<MODE, 8>), grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((jerk_finalize_kernel<MODE, 1>), grid, dim3(256), 0, s, a);
}


template <int MODE>
void launch_jerk_finalize_step_mode(bool deep, const JerkFinalizeArgs &a, double *x_part,
                                    double *v_part, hipStream_t s) {
    const dim3 grid(kCentreBlocks, 3);
    if (deep)
        hipLaunchKernelGGL((jerk_finalize_step_kernel<MODE, 8>), grid, dim3(256), 0, s, a, x_part, v_part);
    else
        hipLaunchKernelGGL((jerk_finalize_step_kernel<MODE, 1>), grid, dim3(256), 0, s, a, x_part, v_part);
}

nbody_status launch_jerk_finalize_step(int precision, const JerkFinalizeArgs &a, double *x_part,
                                       double *v_part, hipStream_t s) {
    if (a.n <= 0) return NBODY_OK;
    const bool deep = engine::finalize_batch(a.n, 3) > 1;
    switch (precision) {
        case NBODY_PLAIN: launch_jerk_finalize_step_mode<NBODY_PLAIN>(deep, a, x_part, v_part, s); break;
        case NBODY_FP64RED: launch_jerk_finalize_step_mode<NBODY_FP64RED>(deep, a, x_part, v_part, s); break;
        case NBODY_COMP: launch_jerk_finalize_step_mode<NBODY_COMP>(deep, a, x_part, v_part, s); break;
        default: return set_error(NBODY_EINVAL, "unknown precision mode");
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

nbody_status launch_jerk_finalize(int precision, const JerkFinalizeArgs &a, hipStream_t s) {
    if (a.n <= 0) return NBODY_OK;
    const int outputs = a.pot ? 7 : 6;
    const dim3 grid((a.n + 255) / 256, outputs);
    const bool deep = engine::finalize_batch(a.n, outputs) > 1;
    switch (precision) {
        case NBODY_PLAIN: launch_jerk_finalize_mode<NBODY_PLAIN>(grid, deep, a, s); break;
        case NBODY_FP64RED: launch_jerk_finalize_mode<NBODY_FP64RED>(grid, deep, a, s); break;
        case NBODY_COMP: launch_jerk_finalize_mode<NBODY_COMP>(grid, deep, a, s); break;
        default: return set_error(NBODY_EINVAL, "unknown precision mode");
    }
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

}  // namespace nbody
