// Force evaluation of one system of at most kSetMax particles with every record in LDS: pairs,
// cross-lane sums and outputs in one launch, from FP32 positions, or from FP64 positions with
// their centre.
#include <algorithm>

#include "outputs.h"
#include "set_engine.h"

namespace nbody {
namespace {

using SetFn = void (*)(SetArgs, FinalizeArgs);

template <int Q, int MODE, bool FULL>
SetFn pick_source(bool f64) {
    return f64 ? set::set_kernel<ForceOut, Q, MODE, FULL, true>
               : set::set_kernel<ForceOut, Q, MODE, FULL, false>;
}

template <int Q>
SetFn pick_set(int mode, bool full, bool f64) {
    switch (mode) {
        case NBODY_PLAIN:
            return full ? pick_source<Q, NBODY_PLAIN, true>(f64) : pick_source<Q, NBODY_PLAIN, false>(f64);
        case NBODY_FP64RED:
            return full ? pick_source<Q, NBODY_FP64RED, true>(f64)
                        : pick_source<Q, NBODY_FP64RED, false>(f64);
        case NBODY_COMP:
            return full ? pick_source<Q, NBODY_COMP, true>(f64) : pick_source<Q, NBODY_COMP, false>(f64);
    }
    return nullptr;
}

}  // namespace

nbody_status launch_pair_set(const TileCfg &cfg, int precision, bool with_pot, const SetArgs &a,
                             const FinalizeArgs &f, hipStream_t s) {
    if (a.n <= 0) return NBODY_OK;
    if (!set_shape(cfg, a.n) || !(a.pos || a.pos64))
        return set_error(NBODY_EUNSUPPORTED, "no whole-set force kernel for this shape");
    auto fn = cfg.jl == 64 ? pick_set<64>(precision, with_pot, a.pos64 != nullptr)
                           : pick_set<32>(precision, with_pot, a.pos64 != nullptr);
    if (!fn) return set_error(NBODY_EINVAL, "unknown precision mode");
    const bool pairs = cfg.jl == 32 && precision == NBODY_PLAIN;
    const int waves = set::waves_for(a.n, pairs);
    const int blocks = std::min(set::kBlocks, (a.n + waves - 1) / waves);
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(64 * waves), set::lds_bytes(a.n), s, a, f);
    NBODY_HIP_CHECK(hipGetLastError());
    return NBODY_OK;
}

}  // namespace nbody
