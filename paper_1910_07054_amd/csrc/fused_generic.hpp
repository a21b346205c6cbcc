// Launch of the generic fused y-pass kernel (layer count up to NZMAX at run time),
// instantiated per precision and direction in files of their own (compile time).
#pragma once
#include "field_kernels.hpp"
#include "launch.hpp"

namespace hfd {

constexpr size_t kMaxFusedLds = 163840;  // 160 KB of LDS per CU on gfx950

// register budget: 1024-point columns run 16 waves per block (128 VGPRs),
// which holds the accumulators of at most 4 layers
template <typename R>
int nzmax_for(int nz, int LY)
{
    if (sizeof(R) == 8 || LY >= 1024) return nz <= 4 ? 4 : 0;
    return nz <= 4 ? 4 : (nz <= 8 ? 8 : (nz <= 12 ? 12 : 0));
}

inline hipError_t set_lds(const void* kernel, size_t lds)
{
    // the limit is raised once to the largest possible size
    return lds > 65536 ? ensure_lds_limit(kernel, (int)kMaxFusedLds) : hipSuccess;
}

template <typename R, int LY, int NZMAX, bool ADJ, int NT>
hipError_t fused_n(int nz, void* X, int ny, int M, int bpg, int G, const void* Q, long long qcs, const int* qslot,
                   int QY, const void* lp, const void* tw, hipStream_t s)
{
    const size_t lds = sizeof(cpx<R>) * 3 * (size_t)nz * fft_region(LY);
    hipError_t e = set_lds((const void*)k_ymix_fused<R, LY, NZMAX, ADJ, NT>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_ymix_fused<R, LY, NZMAX, ADJ, NT>), dim3(M, bpg, G), dim3(NT), lds, s, (cpx<R>*)X, ny, nz,
                       M, (const R*)Q, qcs, qslot, QY, (const R*)lp, bpg, (const cpx<R>*)tw);
    return hipGetLastError();
}

// Threads per block: as many as run the column's transforms in one round while the
// launch stays within 512 threads per CU (256 CUs), the least beyond, where threads
// without a frequency to mix only hold registers that another block could use.
// Fused stage with 512 threads, with `most` and with `least`:
//   30 x 30 x 12, 32 states (64-point columns)           92, 91, 28 us
//   30 x 30 x 4, 64 states, FP64                          55, 20, 15
//   64 x 64 x 3, 16 states, FP64 (128-point columns)      28, 18, 14
//   1000 x 60 x 5 (128-point columns, 1024 blocks)        32, 32, 13
//   128 x 128 x 3, 16 states, FP64 (256-point columns)    63, 63, 43
//   64 x 64 x 3, FP64 (64 blocks)                        7.7, 7.4, 8.4
//   64 x 64 x 6, 4 states (256 blocks)                  11.5, 11.5, 13.0
//   512 x 64 x 3, FP64 (512 blocks, 256 threads at most) 13.4, 9.0, 9.8
template <typename R, int LY, int NZMAX, bool ADJ>
hipError_t fused_a(int nz, void* X, int ny, int M, int bpg, int G, const void* Q, long long qcs, const int* qslot,
                   int QY, const void* lp, const void* tw, hipStream_t s)
{
    constexpr int most = FusedShape<LY, NZMAX>::most(), least = FusedShape<LY, NZMAX>::least;
    if constexpr (most > least) {
        if ((long long)M * bpg * G * most <= 512 * 256)
            return fused_n<R, LY, NZMAX, ADJ, most>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    }
    return fused_n<R, LY, NZMAX, ADJ, least>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
}

template <typename R, int LY, bool ADJ>
hipError_t fused_nz(int nz, void* X, int ny, int M, int bpg, int G, const void* Q, long long qcs, const int* qslot,
                    int QY, const void* lp, const void* tw, hipStream_t s)
{
    switch (nzmax_for<R>(nz, LY)) {
    case 4: return fused_a<R, LY, 4, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    case 8:
        if constexpr (sizeof(R) == 4 && LY < 1024)
            return fused_a<R, LY, 8, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
        return hipErrorInvalidValue;
    case 12:
        if constexpr (sizeof(R) == 4 && LY < 1024)
            return fused_a<R, LY, 12, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

template <typename R, bool ADJ>
hipError_t fused_ly(int LY, int nz, void* X, int ny, int M, int bpg, int G, const void* Q,
                    long long qcs, const int* qslot, int QY, const void* lp, const void* tw,
                    hipStream_t s)
{
    switch (LY) {
    case 8: return fused_nz<R, 8, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    case 16: return fused_nz<R, 16, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    case 32: return fused_nz<R, 32, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    case 64: return fused_nz<R, 64, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    case 128: return fused_nz<R, 128, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    case 256: return fused_nz<R, 256, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    case 512: return fused_nz<R, 512, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    case 1024: return fused_nz<R, 1024, ADJ>(nz, X, ny, M, bpg, G, Q, qcs, qslot, QY, lp, tw, s);
    default: return hipErrorInvalidValue;
    }
}

// arguments as fused_ly
#define HFD_FUSED_ARGS                                                                                     \
    int LY, int nz, void *X, int ny, int M, int bpg, int G, const void *Q, long long qcs, const int *qslot, \
        int QY, const void *lp, const void *tw, hipStream_t s
hipError_t fused_fp32(HFD_FUSED_ARGS);
hipError_t fused_fp32_adj(HFD_FUSED_ARGS);
hipError_t fused_fp64(HFD_FUSED_ARGS);
hipError_t fused_fp64_adj(HFD_FUSED_ARGS);

}  // namespace hfd
