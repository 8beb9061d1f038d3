// Pair kernel with separate i- and j-sets (the paper's library interface, Sec. 3.1):
// the GravityIJ pipeline on the wave engine.  The FP64 reduction is the single-set
// finalize without the self term.
#include "gravity.h"
#include "outputs.h"
#include "wave_engine.h"

namespace nbody {

nbody_status launch_pair_ij(const TileCfg &cfg, int precision, bool with_pot, const IJPairArgs &a,
                            const FinalizeArgs &f, hipStream_t s) {
    return wave::launch<GravityIJ, ForceOut>(cfg, precision, with_pot, a.ni, a, f, s);
}

}  // namespace nbody
