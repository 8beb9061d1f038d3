// Launch of the force-jerk-potential pipeline on FP64 state relative to per-i-tile
// centres (its own translation unit, so the kernel sets compile in parallel).
#include "jerk_pipeline.h"
#include "outputs.h"
#include "wave_engine.h"

namespace nbody {

nbody_status launch_jerk_tile(const TileCfg &cfg, int precision, bool with_pot,
                              const JerkTileArgs &a, const JerkFinalizeArgs &f, hipStream_t s) {
    return wave::launch<GravityJerkTile, JerkOut>(cfg, precision, with_pot, a.n, a, f, s);
}

}  // namespace nbody
