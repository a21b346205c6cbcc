// Instances of the generic fused y pass: single precision, transpose.
#include "fused_generic.hpp"

namespace hfd {
hipError_t fused_fp32_adj(HFD_FUSED_ARGS)
{
    return fused_ly<float, true>(LY, nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
}
}  // namespace hfd
