// Launch of the force-jerk-potential pipeline with separate i- and j-sets (its own
// translation unit, so the kernel sets compile in parallel).
#include "jerk_pipeline.h"
#include "outputs.h"
#include "wave_engine.h"

namespace nbody {

nbody_status launch_jerk_ij(const TileCfg &cfg, int precision, bool with_pot, const JerkIJArgs &a,
                            const JerkFinalizeArgs &f, hipStream_t s) {
    return wave::launch<GravityJerkIJ, JerkOut>(cfg, precision, with_pot, a.ni, a, f, s);
}

}  // namespace nbody
