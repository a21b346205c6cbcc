// Choice of the fused y-pass kernel (y-DFT, z-mixing, inverse y-DFT in LDS): the
// generic one (layer count up to NZMAX at run time, fused_generic.hpp); single-precision
// 256- and 512-point columns of up to 10 layers and 1024-point columns of up
// to 4 go to the exact-layer-count kernels (fused_exact_*.hip).
#include "fused_generic.hpp"

namespace hfd {

bool fused_supported(bool fp64, int LY, int nz, size_t* lds_bytes)
{
    const size_t lds = (fp64 ? 16 : 8) * 3 * (size_t)nz * fft_region(LY);
    if (lds_bytes) *lds_bytes = lds;
    if (LY < 8 || LY > 1024) return false;
    if ((fp64 ? nzmax_for<double>(nz, LY) : nzmax_for<float>(nz, LY)) == 0) return false;
    return lds <= kMaxFusedLds;
}

hipError_t launch_fused(bool fp64, int LY, int nz, void* X, int ny, int M, int B, const void* Q,
                        long long qcs, const int* qslot, int QX, int QY, const void* lp, int bpg,
                        int adjoint, const void* twy, hipStream_t s, bool generic)
{
    (void)QX;
    if (!fused_supported(fp64, LY, nz, nullptr)) return hipErrorInvalidValue;
    if (bpg < 1 || B % bpg != 0) return hipErrorInvalidValue;
    const int G = B / bpg;
    if (!generic && fused_exact_supported(fp64, LY, nz))
        return launch_fused_exact(LY, nz, adjoint, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, twy, s);
    auto run = fp64 ? (adjoint ? fused_fp64_adj : fused_fp64) : (adjoint ? fused_fp32_adj : fused_fp32);
    return run(LY, nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, twy, s);
}

}  // namespace hfd
