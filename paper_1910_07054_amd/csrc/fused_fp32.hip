// Instances of the generic fused y pass: single precision, field.
#include "fused_generic.hpp"

namespace hfd {
hipError_t fused_fp32(HFD_FUSED_ARGS)
{
    return fused_ly<float, false>(LY, nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
}
}  // namespace hfd
