// Instances of the y-pass column kernels and of the five-pass z-mixing kernel.
#include "field_kernels.hpp"
#include "launch.hpp"

namespace hfd {

// Blocks of a column pass.  Columns per group pay for its twiddles, but the chip
// wants 4 blocks per CU to start from and 8 where there are enough columns: 1024
// blocks against 2048 took 9.4 and 10.6 us at 256 x 256 x 8, 44 and 48 us at
// 1024 x 1024 x 3, 139 and 134 us at 16 states of 256 x 256 x 10.
template <typename R, int LY>
static unsigned y_blocks(long long ncols, bool walk)
{
    const long long need = (ncols + YPassShape<R, LY>::NG - 1) / YPassShape<R, LY>::NG;
    const long long some = need / 2 < 1024 ? 1024 : need / 2 > 2048 ? 2048 : need / 2;
    return (unsigned)(!walk || need < some ? need : some);
}

template <typename R, int LY>
static hipError_t yfwd_t(const void* in, void* out, int n, long long ncols, const void* tw,
                         hipStream_t s)
{
    if (2 * n > LY || ncols < 1) return ncols < 1 ? hipSuccess : hipErrorInvalidValue;
    const bool walk = YPassShape<R, LY>::WALK_FWD;
    if (!walk && ncols > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_yfwd<R, LY>), dim3(y_blocks<R, LY>(ncols, walk)), dim3(YPassShape<R, LY>::NT), 0, s,
                       (const cpx<R>*)in, (cpx<R>*)out, n, ncols, (const cpx<R>*)tw);
    return hipGetLastError();
}

template <typename R, int LY>
static hipError_t yinv_t(const void* in, void* out, int n, long long ncols, const void* tw,
                         hipStream_t s)
{
    if (2 * n > LY || ncols < 1) return ncols < 1 ? hipSuccess : hipErrorInvalidValue;
    hipLaunchKernelGGL((k_yinv<R, LY>), dim3(y_blocks<R, LY>(ncols, true)), dim3(YPassShape<R, LY>::NT), 0, s,
                       (const cpx<R>*)in, (cpx<R>*)out, n, ncols, (const cpx<R>*)tw);
    return hipGetLastError();
}

#define HFD_Y_CASES(F, R, ...)                         \
    switch (LY) {                                      \
    case 8: return F<R, 8>(__VA_ARGS__);               \
    case 16: return F<R, 16>(__VA_ARGS__);             \
    case 32: return F<R, 32>(__VA_ARGS__);             \
    case 64: return F<R, 64>(__VA_ARGS__);             \
    case 128: return F<R, 128>(__VA_ARGS__);           \
    case 256: return F<R, 256>(__VA_ARGS__);           \
    case 512: return F<R, 512>(__VA_ARGS__);           \
    case 1024: return F<R, 1024>(__VA_ARGS__);         \
    case 2048: return F<R, 2048>(__VA_ARGS__);         \
    case 4096: return F<R, 4096>(__VA_ARGS__);         \
    default: return hipErrorInvalidValue;              \
    }

hipError_t launch_yfwd(bool fp64, int LY, const void* in, void* out, int n_in, long long ncols,
                       const void* twy, hipStream_t s)
{
    if (fp64) { HFD_Y_CASES(yfwd_t, double, in, out, n_in, ncols, twy, s) }
    HFD_Y_CASES(yfwd_t, float, in, out, n_in, ncols, twy, s)
}

hipError_t launch_yinv(bool fp64, int LY, const void* in, void* out, int n_out, long long ncols,
                       const void* twy, hipStream_t s)
{
    if (fp64) { HFD_Y_CASES(yinv_t, double, in, out, n_out, ncols, twy, s) }
    HFD_Y_CASES(yinv_t, float, in, out, n_out, ncols, twy, s)
}

// Blocks that share a tile of the mixing kernel: more than one where the tiles
// alone leave the chip short of blocks (below 512, two per CU; 64 x 64 x 60 in
// FP64, 128 tiles: 425 us with one block of 15 waves each, 136 with 4 of 8) or
// where a block of NT threads does not hold all target groups.
static int mix_parts(int ngrp, int max_waves, long long tiles)
{
    int parts = 1;
    while ((ngrp + parts - 1) / parts > max_waves || (tiles * parts < 512 && ngrp > 2 * parts)) ++parts;
    const int waves = (ngrp + parts - 1) / parts;
    return (ngrp + waves - 1) / waves;
}

// Two target layers per wave in blocks of up to 8 waves; above 32 layers in
// FP32 four in blocks of up to 16, which reads the tile once (64 layers: 979
// against 1106 us; 32 layers: 265 against 259).
static bool mix_wide(bool fp64, int nz) { return !fp64 && nz > 32; }

static long long mix_tiles(int LY, int nkx, int B) { return (long long)((LY / 2 + 31) / 32) * nkx * B; }

bool mix_generic_in_place(bool fp64, int nz, int M, int LY, int B)
{
    const bool wide = mix_wide(fp64, nz);
    const int ib = wide ? 4 : 2;
    return mix_parts((nz + ib - 1) / ib, wide ? 16 : 8, mix_tiles(LY, M, B)) == 1;
}

template <typename R, int IB, int NT>
static hipError_t mix_tile_t(const void* Mh, void* Hh, int nz, int M, int LY, int B, const void* Q,
                             long long qcs, const int* qslot, int QY, const void* lp, int bpg, int adjoint,
                             int kx0, int nkx, hipStream_t s)
{
    const long long tiles = mix_tiles(LY, nkx, B);
    const int ngrp = (nz + IB - 1) / IB, parts = mix_parts(ngrp, NT / 64, tiles);
    const int waves = (ngrp + parts - 1) / parts;
    const long long nblk = (tiles * parts + 7) / 8 * 8;
    if (nblk > 0x7fffffffLL || (parts > 1 && Mh == Hh)) return hipErrorInvalidValue;
    // up to 96 KB of staged spectra (64 layers in FP32, 32 in FP64); more in chunks
    const int per = 3 * 64 * (int)sizeof(cpx<R>), chunks = (nz * per + 98303) / 98304;
    const int jc = (nz + chunks - 1) / chunks;
    const size_t lds = (size_t)jc * per;
    const hipError_t e = ensure_lds_limit((const void*)k_mix_tile<R, IB, NT>, lds > 65536 ? 98304 : 0);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_mix_tile<R, IB, NT>), dim3((unsigned)nblk), dim3(64 * waves), lds, s,
                       (const cpx<R>*)Mh, (cpx<R>*)Hh, nz, M, LY, (const R*)Q, qcs, qslot, QY, (const R*)lp,
                       bpg, adjoint, kx0, (int)tiles, B, jc, parts);
    return hipGetLastError();
}

hipError_t launch_mix_generic(bool fp64, const void* Mh, void* Hh, int nz, int M, int LY, int B,
                              const void* Q, long long qcs, const int* qslot, int QY, const void* lp,
                              int bpg, int adjoint, int kx0, int nkx, hipStream_t s)
{
    if (nkx <= 0) return hipSuccess;
    if (fp64)
        return mix_tile_t<double, 2, 512>(Mh, Hh, nz, M, LY, B, Q, qcs, qslot, QY, lp, bpg, adjoint, kx0, nkx, s);
    if (mix_wide(fp64, nz))
        return mix_tile_t<float, 4, 1024>(Mh, Hh, nz, M, LY, B, Q, qcs, qslot, QY, lp, bpg, adjoint, kx0, nkx, s);
    return mix_tile_t<float, 2, 512>(Mh, Hh, nz, M, LY, B, Q, qcs, qslot, QY, lp, bpg, adjoint, kx0, nkx, s);
}

}  // namespace hfd
