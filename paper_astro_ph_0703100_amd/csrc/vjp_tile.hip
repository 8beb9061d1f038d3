// Launch of the adjoint pipeline on FP64 positions relative to per-i-tile centres (its
// own translation unit, so the two sets of kernel instantiations compile in parallel).
#include "adjoint_pipeline.h"
#include "outputs.h"
#include "wave_engine.h"

namespace nbody {

nbody_status launch_vjp_tile(const TileCfg &cfg, int precision, const VjpTileArgs &a,
                             bool with_mass, const VjpFinalizeArgs &f, hipStream_t s) {
    return wave::launch<AdjointTile, VjpOut>(cfg, precision, with_mass, a.n, a, f, s);
}

}  // namespace nbody
