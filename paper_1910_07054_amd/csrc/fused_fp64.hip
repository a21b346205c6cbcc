// Instances of the generic fused y pass: double precision, field.
#include "fused_generic.hpp"

namespace hfd {
hipError_t fused_fp64(HFD_FUSED_ARGS)
{
    return fused_ly<double, false>(LY, nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
}
}  // namespace hfd
