// Equidistant layers: the convolution theorem along z as well (eq. FFT_3D of
// Sec. 3.1, the equidistant case the paper compares against in Sec. 3.2).
//
// With equal thickness t and a uniform pitch p (z_i = z_0 + i p) the tensor of
// layers i, j depends on the offset d = i - j only, so the layer sum
// h_i = -sum_j N(d = i - j) * m_j is a convolution along z.  After the x and y
// transforms it is done per lateral frequency by a length-Lz transform along
// the layer axis (zero padded, Lz >= 2 nz), a 3x3 product with the 3-D Fourier
// tensor, and the inverse transform: O(nz log nz) per frequency instead of the
// O(nz^2) explicit sum.
//
// 3-D Fourier tensor: the 2D spectra of N(d) for d in [-(nz-1), nz-1] are real
// (xx, yy, zz, xy) or imaginary (xz, yz) by lateral parity; xz and yz are odd
// in d, the others even, so their transforms along z are real as well:
//   T(kz) = sum_d Q(d) cos(2 pi kz d / Lz)   (xx, yy, zz, xy)
//   T(kz) = sum_d Q(d) sin(2 pi kz d / Lz)   (xz, yz; Q = imaginary part)
// stored on kx in [0, Lx/2], kz in [0, Lz/2], ky in [0, Ly/2]; xy is odd in ky,
// xz odd in kz, yz odd in ky and kz.
#include "field_kernels.hpp"
#include "launch.hpp"

namespace hfd {

// T3[kx][kz][c][ky] = (1/Lz) sum_d Q2[d][c][kx][ky] (cos | sin)(2 pi kz d / Lz)
// Q2: FP64 [2nz-1][6][QX][QY] (offset d at index d + nz - 1).
template <typename R>
__global__ __launch_bounds__(256) void k_zdft3(const double* __restrict__ Q2, R* __restrict__ T3,
                                               int nz, int LZ, int QX, int QY)
{
    const int LZH = LZ / 2 + 1;
    const long long n = (long long)QX * LZH * 6 * QY;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    const int ky = (int)(idx % QY);
    const int c = (int)((idx / QY) % 6);
    const int kz = (int)((idx / ((long long)QY * 6)) % LZH);
    const int kx = (int)(idx / ((long long)QY * 6 * LZH));
    const bool odd = c == 4 || c == 5;
    const long long dstride = 6LL * QX * QY;
    const double* q = Q2 + ((long long)c * QX + kx) * QY + ky;
    double acc = 0.0;
    for (int d = -(nz - 1); d <= nz - 1; ++d) {
        double sn, cs;
        sincospi(2.0 * (double)kz * (double)d / (double)LZ, &sn, &cs);
        acc += q[(long long)(d + nz - 1) * dstride] * (odd ? sn : cs);
    }
    T3[idx] = (R)(acc / (double)LZ);
}

// A wave takes NQ transforms of one component, lane = g NQ + q with q the
// transform (consecutive ky) and g the lane's place in it: a load or store
// moves NQ consecutive ky of each of the GT layers.  16 values per lane from 64
// points on, so that NQ = 16 ky are one 128-byte line (8 at 128 points).
template <typename R, int LZ>
struct ZPassShape {
    static constexpr int V = LZ <= 32 ? fft_vals(LZ) : 16;
    static constexpr int GT = LZ / V, NQ = 64 / GT;
    static constexpr int PB = NQ >= 16 ? 1 : 16 / NQ;   // waves per component
    static constexpr int TP = NQ * PB;                  // ky points per block
    static constexpr int NT = 3 * 64 * PB;
    // LDS slots per transform: odd, so that lanes on consecutive ky take
    // different banks
    static constexpr int RS = fft_region(LZ) | 1;
    static constexpr int LZH = LZ / 2 + 1;
};

// z pass: block = TP consecutive ky of one kx column of one state.  The 3 nz
// spectra go from memory into the first radix pass of their transforms along z
// (zero padded to LZ), are multiplied by the real symmetric 3x3 tensor, a thread
// taking kz and LZ - kz, which share its entries, and leave from the last pass of
// the inverse transforms, first nz layers only.
// Column 0 holds Z = A + iB, A and B the y spectra of the real columns kx = 0 and
// kx = Lx/2: its blocks run A(ky) = (Z(ky) + conj Z(-ky)) / 2 and then
// B(ky) = (Z(ky) - conj Z(-ky)) / (2i) through the same steps and store A' + iB'.
// Bound by the Infinity Cache and HBM: 256 x 256 x 32 (101 MB each way, 52 MB of tensor
// read twice) 115 -> 72 us with the unpacking and repacking of column 0 (two launches
// before), 256 x 256 x 16 in FP64 86 -> 58.  Staging the zero-padded spectra in LDS with
// 8 lanes per transform on consecutive layers moved 64-byte pieces and kept the
// product's lanes on one LDS bank.  Registers for 3 waves per SIMD: 4 spill the 64-point
// transform in FP32 (72 -> 158 us).
template <typename R, int LZ>
__global__ __launch_bounds__((ZPassShape<R, LZ>::NT), (sizeof(R) == 4 ? 3 : 2)) void k_zpass3(
    const cpx<R>* __restrict__ Mh, cpx<R>* __restrict__ Hh, int nz, int M, int LY, const R* __restrict__ T3,
    int QY, const cpx<R>* __restrict__ twz)
{
    using SH = ZPassShape<R, LZ>;
    constexpr int TP = SH::TP, NT = SH::NT, RS = SH::RS, LZH = SH::LZH, V = SH::V, NQ = SH::NQ;
    __shared__ cpx<R> sh[3 * TP * RS];
    const int kx = blockIdx.y, b = blockIdx.z, ky0 = blockIdx.x * TP;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = w / SH::PB, pt = (w % SH::PB) * NQ + lane % NQ, g = lane / NQ;
    const int tr = c * TP + pt, ky = ky0 + pt;
    const bool live = ky < LY;
    const long long sst = (long long)M * LY;
    const long long base = ((long long)b * 3 * nz + c * nz) * sst + (long long)kx * LY;
    const cpx<R>* src = Mh + base + (live ? ky : 0);
    const cpx<R>* srn = Mh + base + (live ? (LY - ky) & (LY - 1) : 0);
    cpx<R>* dst = Hh + base + ky;
    cpx<R>* reg = sh + tr * RS;
    Twiddles<R, LZ, V> tw;
    tw.load(g, twz, 1);

    cpx<R> keep[V / 2 > 0 ? V / 2 : 1];  // A' of the packed column
    for (int part = 0; part < (kx == 0 ? 2 : 1); ++part) {
        cpx<R> v[V];
        if (kx != 0) {
            fft_first_loads<R, LZ, true>(v, g, [&](int l) -> cpx<R> {
                return l < nz ? src[l * sst] : cpx<R>{R(0), R(0)};
            });
        } else {
            fft_first_loads<R, LZ, true>(v, g, [&](int l) -> cpx<R> {
                if (l >= nz) return {R(0), R(0)};
                const cpx<R> z = src[l * sst], n = srn[l * sst];
                return part == 0 ? cpx<R>{R(0.5) * (z.x + n.x), R(0.5) * (z.y - n.y)}
                                 : cpx<R>{R(0.5) * (z.y + n.y), R(0.5) * (n.x - z.x)};
            });
            if (part > 0) __syncthreads();
        }
        wave_fft_pre<R, LZ, false, true>(reg, g, tw, v, [&](int pos, cpx<R> z) { reg[pos] = z; });
        __syncthreads();
        // 3x3 product per (point, +-kz)
        const R* Tk = T3 + (long long)(part == 0 ? kx : M) * LZH * 6 * QY;
        for (int idx = tid; idx < TP * LZH; idx += NT) {
            const int p = idx % TP, kz = idx / TP, k1 = ky0 + p;
            if (k1 >= LY) continue;
            const R sy = k1 <= LY / 2 ? R(1) : R(-1);
            const R* t = Tk + (long long)kz * 6 * QY + (k1 <= LY / 2 ? k1 : LY - k1);
            const R xx = t[0], yy = t[QY], zz = t[2 * QY], xy = sy * t[3 * QY];
            R xz = t[4 * QY], yz = sy * t[5 * QY];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && (kz == 0 || 2 * kz == LZ)) break;
                cpx<R>* w = sh + p * RS + (h == 0 ? kz : LZ - kz);
                const cpx<R> X = w[0], Y = w[TP * RS], Z = w[2 * TP * RS];
                w[0] = {xx * X.x + xy * Y.x + xz * Z.x, xx * X.y + xy * Y.y + xz * Z.y};
                w[TP * RS] = {xy * X.x + yy * Y.x + yz * Z.x, xy * X.y + yy * Y.y + yz * Z.y};
                w[2 * TP * RS] = {xz * X.x + yz * Y.x + zz * Z.x, xz * X.y + yz * Y.y + zz * Z.y};
                xz = -xz;  // odd in kz
                yz = -yz;
            }
        }
        __syncthreads();
        int i = 0;
        wave_fft<R, LZ, true, false, true>(
            reg, g, tw, [&](int pos) -> cpx<R> { return reg[pos]; },
            [&](int l, cpx<R> z) {
                cpx<R>& k = keep[i++];
                if (kx == 0) z = part == 0 ? z : cpx<R>{k.x - z.y, k.y + z.x};
                k = z;
                if (live && l < nz && (kx != 0 || part == 1)) dst[l * sst] = z;
            });
    }
}

namespace {

template <typename R>
hipError_t zpass_r(int LZ, const void* Mh, void* Hh, int nz, int M, int LY, int B, const void* T3, int QY,
                   const void* twz, hipStream_t s)
{
#define HFD_ZPASS_CASE(L)                                                                          \
    case L: {                                                                                      \
        dim3 grid((LY + ZPassShape<R, L>::TP - 1) / ZPassShape<R, L>::TP, M, B);                   \
        hipLaunchKernelGGL((k_zpass3<R, L>), grid, dim3(ZPassShape<R, L>::NT), 0, s,               \
                           (const cpx<R>*)Mh, (cpx<R>*)Hh, nz, M, LY, (const R*)T3, QY,            \
                           (const cpx<R>*)twz);                                                    \
        return hipGetLastError();                                                                  \
    }
    switch (LZ) {
        HFD_ZPASS_CASE(2)
        HFD_ZPASS_CASE(4)
        HFD_ZPASS_CASE(8)
        HFD_ZPASS_CASE(16)
        HFD_ZPASS_CASE(32)
        HFD_ZPASS_CASE(64)
        HFD_ZPASS_CASE(128)
    default: return hipErrorInvalidValue;
    }
#undef HFD_ZPASS_CASE
}

}  // namespace

hipError_t launch_zdft3(bool out_fp64, const double* Q2, void* T3, int nz, int LZ, int QX, int QY,
                        hipStream_t s)
{
    const long long n = (long long)QX * (LZ / 2 + 1) * 6 * QY;
    const long long nb = (n + 255) / 256;
    if (nb > 0x7fffffffLL) return hipErrorInvalidValue;
    if (out_fp64)
        hipLaunchKernelGGL(k_zdft3<double>, dim3((unsigned)nb), dim3(256), 0, s, Q2, (double*)T3, nz,
                           LZ, QX, QY);
    else
        hipLaunchKernelGGL(k_zdft3<float>, dim3((unsigned)nb), dim3(256), 0, s, Q2, (float*)T3, nz,
                           LZ, QX, QY);
    return hipGetLastError();
}

hipError_t launch_eq3d_mix(bool fp64, int LZ, const void* Mh, void* Hh, int nz, int M, int LY, int B,
                           const void* T3, int QY, const void* twz, hipStream_t s)
{
    if (!Mh || !Hh || Mh == Hh || !T3 || !twz || B > 65535 || 2 * nz > (LZ < 2 ? 0 : LZ)) return hipErrorInvalidValue;
    if (fp64) return zpass_r<double>(LZ, Mh, Hh, nz, M, LY, B, T3, QY, twz, s);
    return zpass_r<float>(LZ, Mh, Hh, nz, M, LY, B, T3, QY, twz, s);
}

}  // namespace hfd
