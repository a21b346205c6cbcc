// Field-path kernels: h = -N * m by the hybrid scheme of Sec. 3.1 --
// 2D DFT along x and y (zero padded to Lx x Ly), an explicit sum over layers
// per lateral frequency, inverse 2D DFT, crop.
//
// Data layout (per state b, signal s = c * nz + l for component c, layer l):
//   m, h   [B][S][ny][nx]           real, x fastest
//   X1     [B][S][M][ny]            complex, M = Lx/2 columns of the x
//                                   half-spectrum, y fastest; column 0 packs
//                                   the two real columns kx = 0 and kx = Lx/2
//                                   as X(0) + i X(Lx/2)
//   Mh, Hh [B][S][M][Ly]            full y spectra (five-pass path only)
//   Q      [G][Lx/2+1][P][5][Ly/2+1] Fourier tensor on the quadrant kx in
//                                   [0, Lx/2], ky in [0, Ly/2] (contiguous per
//                                   kx column), unique pairs i <= j, components
//                                   xx, yy, xy, xz, yz of
//                                   t_i * (-DFT2(N^{ij}) / (Lx Ly)); real part
//                                   for xx, yy, xy, imaginary part for xz, yz
//   lp     [G][2][nz]               1 / t_l and -t_l / (Lx Ly) (trace of the
//                                   self-pair block, which fixes zz)
#pragma once
#include <type_traits>

#include "hfd_device.hpp"

namespace hfd {

// Values per lane of the x passes' transforms, one choice per length, precision and call:
// the order of a transform's roundings follows from it, and a state's results depend
// neither on the batch it is in nor on which of its gradients are asked for.  256 points
// (rows of 129 to 256 cells) take 16: two radix-16 passes with one exchange instead of
// 8 8 4 with two, and half the threads per row.  At equal tile heights, 8 and 16 values:
// 256 x 256 x 8 (24 rows) forward 6.8, 6.3 us, inverse 6.1, 5.4, FP64 (8 rows) 9.7, 8.9 and
// 8.2, 7.1; 32 layers (32 rows) 18.6, 16.7 and 19.4, 18.2; 16 states of 10 layers (32 rows)
// 94, 91 and 78, 79.  The FP32 forward passes of a gradient call all stay at 8: the
// thickness gradient is an FP64 result, and keeps its values (16 are as accurate and
// move its seventh digit) at 0.5 % of the call.  At 128 points 16 values are slower below
// 8192 rows (128 x 128 x 8: 3.3 + 3.2 us against 3.7 + 3.5) and a little faster above
// (8 states: 9.5 + 8.3 against 8.7 + 8.3), so 8 for all.
template <typename R>
__host__ __device__ constexpr int x_vals(int M, bool gradient = false)
{
    return M == 256 && !(gradient && sizeof(R) == 4) ? 16 : fft_vals(M);
}

// Rows are numbered flat over all signals (row r = signal r / ny, y = r % ny)
// and a block takes TY consecutive rows, one wave or part of a wave per row,
// RPG rows one after the other where TY rows would need more than 512 threads.
// The transposed side of a pass moves TY consecutive y of one kx: TY = 16 rows
// (8 in FP64) are one 128-byte line.  TYO = 0 picks that, or one wave of rows
// if that is more, halved until the tile fits in 80 KB of LDS.
template <typename R, int LX, int TYO, int XV>
struct XPassShape {
    static constexpr int M = LX / 2;
    static constexpr int V = XV;
    static constexpr int GT = M / V;
    // odd LDS row stride: the transposed accesses take 16 rows of one kx from
    // 16 different slots
    static constexpr int RS = fft_region(M) | 1;
    static constexpr int pick_ty()
    {
        if (TYO > 0) return TYO;
        int ty = sizeof(R) == 4 ? 16 : 8;
        if (GT * ty < 64) ty = 64 / GT;
        while (ty > 1 && sizeof(cpx<R>) * (size_t)ty * RS > 81920) ty /= 2;
        return ty;
    }
    static constexpr int TY = pick_ty();
    static constexpr int RPG = GT * TY > 512 ? 2 : 1;   // rows per group (GT TY <= 1024)
    static constexpr int NG = TY / RPG;
    static constexpr int NT = GT * NG;
    static constexpr size_t LDS = sizeof(cpx<R>) * TY * RS;
    // waves per SIMD the register budget is cut for: 128 VGPRs hold an FP32
    // transform of up to 16 values per lane with its twiddles, 168 an FP64 one
    // of 8; longer ones would spill at that
    static constexpr int WPE =
        sizeof(R) == 4 ? (V <= 16 ? 4 : 2) : (V <= 8 ? 3 : (V <= 16 ? 2 : 1));
    // kx pairs (k, M - k) per thread of the transposed side, 0 <= k < M/2
    // (pair 0 is k = 0 and k = M/2, each its own mirror)
    static constexpr int KI = V * RPG / 2, KS = NT / TY;
    static_assert(TY % RPG == 0 && NT % TY == 0 && KI * KS == M / 2, "x pass tile");
};

// n / d for n < 2^32 by a multiplication (d >= 1; make(d) on the host), the unsigned
// form of T. Granlund and P. L. Montgomery, "Division by invariant integers using
// multiplication", PLDI 1994:
// q = (t + (n - t) / 2) >> (l - 1), t = mulhi(n, m), m = 2^32 (2^l - d) / d + 1,
// l = ceil(log2 d)
struct FastDiv {
    unsigned m, s1, s2;
    static FastDiv make(unsigned d)
    {
        unsigned l = 0;
        while ((1ull << l) < d) ++l;
        return {(unsigned)((((1ull << l) - d) << 32) / d + 1), l < 1 ? l : 1u, l < 1 ? 0u : l - 1};
    }
    __device__ __forceinline__ unsigned div(unsigned n) const
    {
        const unsigned t = __umulhi(n, m);
        return (t + ((n - t) >> s1)) >> s2;
    }
};

// Split of the packed real transform on one pair (k, M - k): the complex
// spectrum Z of z[n] = x[2n] + i x[2n+1] against the half spectrum X of x,
// with X[0] and X[M] packed as X[0] + i X[M]; w = exp(-2 pi i k / LX).
// pair0: a = entry 0, b = entry M/2.
template <typename R>
__device__ __forceinline__ void real_split_fwd(cpx<R>& a, cpx<R>& b, cpx<R> w, bool pair0)
{
    const cpx<R> E = {R(0.5) * (a.x + b.x), R(0.5) * (a.y - b.y)};
    const cpx<R> O = {R(0.5) * (a.y + b.y), R(0.5) * (b.x - a.x)};
    const cpx<R> wO = cmul(w, O);
    const cpx<R> p = cadd(E, wO), q = cconj(csub(E, wO));
    const cpx<R> p0 = {a.x + a.y, a.x - a.y}, q0 = cconj(b);
    a = pair0 ? p0 : p;
    b = pair0 ? q0 : q;
}
// packed half spectrum -> spectrum of z (unnormalized, twice the forward's input)
template <typename R>
__device__ __forceinline__ void real_split_inv(cpx<R>& a, cpx<R>& b, cpx<R> w, bool pair0)
{
    const cpx<R> P = {a.x + b.x, a.y - b.y};   // a + conj(b)
    const cpx<R> Qd = {a.x - b.x, a.y + b.y};  // a - conj(b)
    const cpx<R> T = cmul(cconj(w), Qd);
    const cpx<R> p = {P.x - T.y, P.y + T.x}, q = {P.x + T.y, T.x - P.y};
    const cpx<R> p0 = {a.x + a.y, a.x - a.y}, q0 = {R(2) * b.x, R(-2) * b.y};
    a = pair0 ? p0 : p;
    b = pair0 ? q0 : q;
}

// ---------------------------------------------------------------------------
// x pass, forward: each row of nx <= LX/2 reals (zero padded to LX) -> packed
// half spectrum of LX/2 complex values, written transposed (y fastest).
// A length-LX real transform is one complex transform of length LX/2 on
// z[n] = x[2n] + i x[2n+1] followed by the even/odd split; z[n] is zero for
// n >= LX/4, which the first radix pass skips.  The rows' spectra meet in LDS
// once: the split runs on the transposed side, where a thread takes the pairs
// (k, M - k) of one row and consecutive threads consecutive rows, straight
// into the stores.
// Bound by the latency of its one round trip at small row counts and by HBM at
// large ones.  All global accesses of a thread are requested together, and
// the indices are divided out once per thread; with the split in the rows (one
// more LDS round trip) and an index division per element the two passes of
// 64 states of 512 x 512 x 4 took 932 + 1360 us, now 630 + 565 (2.4 GB each at
// 3.8 and 4.3 TB/s; a copy runs at 4.9), those of one 256 x 256 x 8 state 9.1 + 8.7,
// now 6.3 + 5.4.  (With the exchange layout of FP64, pos + pos/8, in FP32 too that
// forward pass takes 573 us and no other size gains: it waits for its stores, which
// meet differently.)
// ---------------------------------------------------------------------------
template <typename R, int LX, int TYO = 0, int XV = x_vals<R>(LX / 2)>
__global__ __launch_bounds__((XPassShape<R, LX, TYO, XV>::NT), (XPassShape<R, LX, TYO, XV>::WPE)) void k_xfwd(
    const R* __restrict__ in, cpx<R>* __restrict__ out, int nx, int ny, int nrows, FastDiv dny,
    const cpx<R>* __restrict__ twx)
{
    using S = XPassShape<R, LX, TYO, XV>;
    constexpr int M = S::M, V = S::V, GT = S::GT, NG = S::NG, TY = S::TY, RS = S::RS, RPG = S::RPG;
    constexpr int KI = S::KI, KS = S::KS;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<R>* sh = reinterpret_cast<cpx<R>*>(smem_raw);
    const int r0 = blockIdx.x * TY;
    const int tid = threadIdx.x, grp = tid / GT, g = tid % GT;

    cpx<R> v[RPG][V];
#pragma unroll
    for (int q = 0; q < RPG; ++q) {
        const int fr = r0 + grp + q * NG;
        // rows are contiguous, so row fr starts at fr nx
        const R* src = in + (long long)fr * nx;
        const int lim = fr < nrows ? nx : 0;
        if ((nx & 1) == 0) {
            // even rows: (x[2n], x[2n+1]) is one aligned 2-element load
            const cpx<R>* src2 = reinterpret_cast<const cpx<R>*>(src);
            const int nh = lim >> 1;
            fft_first_loads<R, M, true>(v[q], g, [&](int pos) -> cpx<R> {
                return pos < nh ? src2[pos] : cpx<R>{R(0), R(0)};
            });
        } else {
            fft_first_loads<R, M, true>(v[q], g, [&](int pos) -> cpx<R> {
                const int n0 = 2 * pos;
                return {n0 < lim ? src[n0] : R(0), n0 + 1 < lim ? src[n0 + 1] : R(0)};
            });
        }
    }
    Twiddles<R, M, S::V> tw;
    tw.load(g, twx, 2);
    const int rb = tid % TY, kb = tid / TY;
    cpx<R> ws[KI];
#pragma unroll
    for (int i = 0; i < KI; ++i) ws[i] = twx[kb + i * KS];
#pragma unroll
    for (int q = 0; q < RPG; ++q) {
        cpx<R>* row = sh + (grp + q * NG) * RS;
        wave_fft_pre<R, M, false, true>(row, g, tw, v[q], [&](int pos, cpx<R> z) { row[pos] = z; });
    }
    __syncthreads();
    const int fr = r0 + rb;
    if (fr >= nrows) return;
    const int sig = (int)dny.div((unsigned)fr), y = fr - sig * ny;
    cpx<R>* dst = out + (long long)sig * M * ny + y;
    const cpx<R>* row = sh + rb * RS;
#pragma unroll
    for (int i = 0; i < KI; ++i) {
        const int k = kb + i * KS;
        const int kn = k == 0 ? M / 2 : M - k;
        cpx<R> a = row[k], b = row[kn];
        real_split_fwd(a, b, ws[i], k == 0);
        dst[(long long)k * ny] = a;
        dst[(long long)kn * ny] = b;
    }
}

// ---------------------------------------------------------------------------
// x pass, inverse: packed half spectrum (transposed) -> nx <= LX/2 reals per
// row (only that half of the transform is kept).  Unnormalized; the 1/(Lx Ly)
// is folded into the tensor.  The mirror image of k_xfwd: a thread requests
// all its pairs (k, M - k) of one row, splits them in registers and puts them
// into LDS, where the row's group finds its first radix pass.
// ---------------------------------------------------------------------------
template <typename R, int LX, int TYO = 0, int XV = x_vals<R>(LX / 2)>
__global__ __launch_bounds__((XPassShape<R, LX, TYO, XV>::NT), (XPassShape<R, LX, TYO, XV>::WPE)) void k_xinv(
    const cpx<R>* __restrict__ in, R* __restrict__ out, int nx, int ny, int nrows, FastDiv dny,
    const cpx<R>* __restrict__ twx)
{
    using S = XPassShape<R, LX, TYO, XV>;
    constexpr int M = S::M, GT = S::GT, NG = S::NG, TY = S::TY, RS = S::RS, RPG = S::RPG;
    constexpr int KI = S::KI, KS = S::KS;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<R>* sh = reinterpret_cast<cpx<R>*>(smem_raw);
    const int r0 = blockIdx.x * TY;
    const int tid = threadIdx.x, grp = tid / GT, g = tid % GT;
    {
        const int rb = tid % TY, kb = tid / TY;
        // (rows past the end read the last one; their group returns below)
        const int fr = r0 + rb < nrows ? r0 + rb : nrows - 1;
        const int sig = (int)dny.div((unsigned)fr), y = fr - sig * ny;
        const cpx<R>* src = in + (long long)sig * M * ny + y;
        cpx<R>* row = sh + rb * RS;
        cpx<R> a[KI], b[KI];
#pragma unroll
        for (int i = 0; i < KI; ++i) {
            const int k = kb + i * KS;
            a[i] = src[(long long)k * ny];
            b[i] = src[(long long)(k == 0 ? M / 2 : M - k) * ny];
        }
#pragma unroll
        for (int i = 0; i < KI; ++i) {
            const int k = kb + i * KS;
            real_split_inv(a[i], b[i], twx[k], k == 0);
            row[k] = a[i];
            row[k == 0 ? M / 2 : M - k] = b[i];
        }
    }
    // (in FP64 the twiddles would not fit beside the pairs)
    Twiddles<R, M, S::V> tw;
    if constexpr (sizeof(R) == 4) tw.load(g, twx, 2);
    __syncthreads();
    if constexpr (sizeof(R) == 8) tw.load(g, twx, 2);
#pragma unroll
    for (int q = 0; q < RPG; ++q) {
        const int fr = r0 + grp + q * NG;
        if (fr >= nrows) break;
        cpx<R>* row = sh + (grp + q * NG) * RS;
        R* dst = out + (long long)fr * nx;
        auto ld = [&](int pos) -> cpx<R> { return row[pos]; };
        if ((nx & 1) == 0) {
            cpx<R>* dst2 = reinterpret_cast<cpx<R>*>(dst);
            const int nh = nx >> 1;
            wave_fft<R, M, true, false, true>(row, g, tw, ld, [&](int pos, cpx<R> v) {
                if (pos < nh) dst2[pos] = v;
            });
        } else {
            wave_fft<R, M, true, false, true>(row, g, tw, ld, [&](int pos, cpx<R> v) {
                const int n0 = 2 * pos;
                if (n0 < nx) dst[n0] = v.x;
                if (n0 + 1 < nx) dst[n0 + 1] = v.y;
            });
        }
    }
}

// ---------------------------------------------------------------------------
// x pass of the tensor tables from their quadrants: row y < ny of array sig
// holds W(p, y), p < nx, of component sig % 6 (order xx yy zz xy xz yz); the
// full periodic row of length LX is W(p) at p and sx W(p) at LX - p (sx = -1
// for the x-odd components xy and xz), zero between.  Its transform is real
// for an x-even row and imaginary for an x-odd one; that part is stored
// transposed, out[sig][kx][y] for kx in [0, LX/2] (columns of ny reals; the
// rows kx = 0 and LX/2 of x-odd components are exactly zero).
// ---------------------------------------------------------------------------
template <int LX, int TYO = 0>
using XTabShape = XPassShape<double, LX, TYO, fft_vals(LX / 2)>;

template <int LX, int TYO = 0>
__global__ __launch_bounds__((XTabShape<LX, TYO>::NT), (XTabShape<LX, TYO>::WPE)) void k_xtab(
    const double* __restrict__ in, double* __restrict__ out, int nx, int ny, int nrows,
    const cpx<double>* __restrict__ twx)
{
    using R = double;
    using S = XTabShape<LX, TYO>;
    constexpr int M = S::M, GT = S::GT, NG = S::NG, TY = S::TY, RS = S::RS;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<R>* sh = reinterpret_cast<cpx<R>*>(smem_raw);
    const int r0 = blockIdx.x * TY;
    const int tid = threadIdx.x, grp = tid / GT, g = tid % GT;
    Twiddles<R, M, S::V> tw;
    tw.load(g, twx, 2);
    for (int r = grp; r < TY; r += NG) {
        const int fr = r0 + r;
        if (fr >= nrows) break;
        const int sig = fr / ny, y = fr - sig * ny;
        const int c6 = sig % 6;
        const R sx = (c6 == 3 || c6 == 4) ? R(-1) : R(1);
        const R* src = in + ((long long)sig * ny + y) * nx;
        auto xv = [&](int x) -> R {
            if (x < nx) return src[x];
            const int m = LX - x;
            return m < nx ? sx * src[m] : R(0);
        };
        cpx<R>* row = sh + r * RS;
        wave_fft<R, M, false>(
            row, g, tw, [&](int pos) -> cpx<R> { return {xv(2 * pos), xv(2 * pos + 1)}; },
            [&](int pos, cpx<R> v) { row[pos] = v; });
    }
    __syncthreads();
    const int fr = r0 + tid % TY;
    if (fr >= nrows) return;
    const int sig = fr / ny, y = fr - sig * ny;
    const int c6 = sig % 6;
    const bool xodd = (c6 == 3 || c6 == 4);
    double* dst = out + (long long)sig * (M + 1) * ny + y;
    const cpx<R>* row = sh + (tid % TY) * RS;
#pragma unroll
    for (int i = 0; i < S::KI; ++i) {
        const int k = tid / TY + i * S::KS;
        const int kn = k == 0 ? M / 2 : M - k;
        cpx<R> a = row[k], b = row[kn];
        real_split_fwd(a, b, twx[k], k == 0);
        // entry 0 holds X[0] + i X[M] (both real for an x-even row)
        dst[(long long)k * ny] = xodd ? (k == 0 ? R(0) : a.y) : a.x;
        dst[(long long)kn * ny] = xodd ? b.y : b.x;
        if (k == 0) dst[(long long)M * ny] = xodd ? R(0) : a.y;
    }
}

// ---------------------------------------------------------------------------
// z-mixing of one frequency pair.  For the unique layer pairs i <= j the
// stored block S^{ij} = t_i T^{ij} (T = -DFT2(N)/(Lx Ly)) is applied both
// ways: H_i += S^{ij} M_j and H_j += conj(S^{ij}) M_i (reciprocity
// t_j T^{ji} = conj(t_i T^{ij})).  Real components: xx, yy, zz, xy; imaginary
// components: xz, yz.  zz follows from the trace: sum of the diagonal of
// S^{ij} is dg_i on the self pair and 0 otherwise (the trace of N is the
// overlap volume over the target volume).  Point b carries the sign sb of the
// components that are odd in ky (xy, yz).
// Arrays are indexed [c * NZMAX + layer].
// ---------------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void block_apply(cpx<R>& hx, cpx<R>& hy, cpx<R>& hz, cpx<R> X, cpx<R> Y,
                                            cpx<R> Z, R xx, R yy, R zz, R xy, R xz, R yz)
{
    // real parts (xx, yy, zz, xy) multiply, imaginary parts (i xz, i yz) rotate
    hx.x = fma(xx, X.x, hx.x); hx.x = fma(xy, Y.x, hx.x); hx.x = fma(-xz, Z.y, hx.x);
    hx.y = fma(xx, X.y, hx.y); hx.y = fma(xy, Y.y, hx.y); hx.y = fma(xz, Z.x, hx.y);
    hy.x = fma(xy, X.x, hy.x); hy.x = fma(yy, Y.x, hy.x); hy.x = fma(-yz, Z.y, hy.x);
    hy.y = fma(xy, X.y, hy.y); hy.y = fma(yy, Y.y, hy.y); hy.y = fma(yz, Z.x, hy.y);
    hz.x = fma(-xz, X.y, hz.x); hz.x = fma(-yz, Y.y, hz.x); hz.x = fma(zz, Z.x, hz.x);
    hz.y = fma(xz, X.x, hz.y); hz.y = fma(yz, Y.x, hz.y); hz.y = fma(zz, Z.y, hz.y);
}

// On the kx = 0 and kx = Lx/2 rows of the tensor xy and xz vanish (both are
// odd in x, lateral parity); EDGE = 1 drops them.
template <int EDGE, typename R>
__device__ __forceinline__ void block_apply_e(cpx<R>& hx, cpx<R>& hy, cpx<R>& hz, cpx<R> X, cpx<R> Y,
                                              cpx<R> Z, R xx, R yy, R zz, R xy, R xz, R yz)
{
    if constexpr (EDGE == 0) {
        block_apply(hx, hy, hz, X, Y, Z, xx, yy, zz, xy, xz, yz);
    } else {
        hx.x = fma(xx, X.x, hx.x); hx.y = fma(xx, X.y, hx.y);
        hy.x = fma(yy, Y.x, hy.x); hy.x = fma(-yz, Z.y, hy.x);
        hy.y = fma(yy, Y.y, hy.y); hy.y = fma(yz, Z.x, hy.y);
        hz.x = fma(-yz, Y.y, hz.x); hz.x = fma(zz, Z.x, hz.x);
        hz.y = fma(yz, Y.x, hz.y); hz.y = fma(zz, Z.y, hz.y);
    }
}

// Tensor values of one target row i (pairs (i, j), j >= i), 5 components each;
// sl maps the stack's pair u to its slot of the tensor table.
template <typename R, int NZMAX>
struct TensorRow {
    R v[NZMAX][5];
    // row i starts at pair index u = i nz - i (i - 1) / 2
    template <int EDGE = 0>
    __device__ __forceinline__ void load(const UniformBuf<R>& qcol, unsigned kq, int QY, int nz, int i,
                                         const int* __restrict__ sl)
    {
        const int u = i * nz - i * (i - 1) / 2;
#pragma unroll
        for (int j = 0; j < NZMAX; ++j)
            if (j >= i && j < nz) {
                const int slot = sl[u + j - i];
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    const bool need = EDGE == 0 || c < 2 || c == 4;
                    v[j][c] = need ? qcol.ld(kq, (unsigned)((slot * 5 + c) * QY)) : R(0);
                }
            }
    }
};

// One frequency point: H_i += S^{ij} M_j and, for i < j, H_j += conj(S^{ij}) M_i.
// qcol views the tensor table from a wave-uniform base (one kx row); kq is the
// lane's element offset (the quadrant ky, plus the row for the packed column);
// pair u, component c sits at (sl[u] * 5 + c) * QY + kq.
// sg is the sign of the ky-odd components (xy, yz).
// Row i + 1 of the tensor is loaded while row i is applied; `first` holds
// row 0, loaded by the caller ahead of time.
template <typename R, int NZMAX, int EDGE = 0, class In>
__device__ __forceinline__ void mix1(int nz, In in, cpx<R>* H, const UniformBuf<R>& qcol,
                                     unsigned kq, int QY, const int* __restrict__ sl, R sg,
                                     const R* dg, const TensorRow<R, NZMAX>& first)
{
#pragma unroll
    for (int k = 0; k < 3 * NZMAX; ++k) H[k] = {R(0), R(0)};
    // double buffering needs two rows of registers; above 8 layers the rows
    // are loaded one at a time
    constexpr bool DB = NZMAX <= 8;
    TensorRow<R, NZMAX> cur = first, nxt;
#pragma unroll
    for (int i = 0; i < NZMAX; ++i) {
        if (i < nz) {
            if constexpr (DB) {
                if (i + 1 < NZMAX && i + 1 < nz) nxt.template load<EDGE>(qcol, kq, QY, nz, i + 1, sl);
            } else if (i > 0) {
                cur.template load<EDGE>(qcol, kq, QY, nz, i, sl);
            }
            const cpx<R> ix = in(0, i), iy = in(1, i), iz = in(2, i);
#pragma unroll
            for (int j = i; j < NZMAX; ++j) {
                if (j < nz) {
                    const R xx = cur.v[j][0], yy = cur.v[j][1], xy = sg * cur.v[j][2],
                            xz = cur.v[j][3], yz = sg * cur.v[j][4];
                    R zz = -(xx + yy);
                    if (i == j) zz += dg[i];
                    if (i == j) {
                        block_apply_e<EDGE>(H[i], H[NZMAX + i], H[2 * NZMAX + i], ix, iy, iz, xx, yy,
                                            zz, xy, xz, yz);
                    } else {
                        const cpx<R> jx = in(0, j), jy = in(1, j), jz = in(2, j);
                        block_apply_e<EDGE>(H[i], H[NZMAX + i], H[2 * NZMAX + i], jx, jy, jz, xx, yy,
                                            zz, xy, xz, yz);
                        block_apply_e<EDGE>(H[j], H[NZMAX + j], H[2 * NZMAX + j], ix, iy, iz, xx, yy,
                                            zz, xy, -xz, -yz);
                    }
                }
            }
            if constexpr (DB) {
                if (i + 1 < NZMAX) cur = nxt;
            }
        }
    }
}

template <typename R, int NZMAX, int EDGE = 0, class In>
__device__ __forceinline__ void mix1(int nz, In in, cpx<R>* H, const UniformBuf<R>& qcol,
                                     unsigned kq, int QY, const int* __restrict__ sl, R sg,
                                     const R* dg)
{
    TensorRow<R, NZMAX> first;
    first.template load<EDGE>(qcol, kq, QY, nz, 0, sl);
    mix1<R, NZMAX, EDGE>(nz, in, H, qcol, kq, QY, sl, sg, dg, first);
}

// The two points of the packed column that are their own mirror (ky = 0 and
// LY/2) need four real mixings: A = Re Z with the kx = 0 row and B = Im Z with
// the kx = M row, at both points.  With LY lanes for LY + 2 mixings they are
// spread over the lanes of one wave: lane e takes one (point, part, target
// layer i) and sums over the source layers.  All blocks there are diagonal
// and real (xy, xz and yz vanish on those rows and columns).  Q is the tensor
// table, whose rows kx = 0 and kx = M come first (Q and Q + qcs), sl the
// stack's slot map; lpg holds 1/t and the trace terms.  The
// points are read by prep() and written by finish(), and no other lane touches
// them.  prep() requests the operands (called before the lane's own mixing, so that
// their latency overlaps it); finish() sums and writes the results.
template <typename R, int LY, int NZMAX, bool ADJ>
struct MirrorPoints {
    R xx[NZMAX], yy[NZMAX], v[3][NZMAX];
    int i, part, kp;
    bool act;

    __device__ __forceinline__ void prep(const cpx<R>* sh, int nz, int e, const R* __restrict__ Q,
                                         long long qcs, const int* __restrict__ sl, int QY,
                                         const R* lpg)
    {
        i = e % NZMAX;
        part = (e / NZMAX) & 1;
        const int pt = e / (2 * NZMAX);
        act = pt < 2 && i < nz;
        const int ii = i < nz ? i : nz - 1;
        kp = pt == 1 ? LY / 2 : 0;
        const UniformBuf<R> qb0(Q, (unsigned)(2 * qcs * sizeof(R)));
        const unsigned off = (unsigned)(kp + (part ? qcs : 0LL));
#pragma unroll
        for (int j = 0; j < NZMAX; ++j) {
            const int jj = j < nz ? j : ii;
            const int a = ii < jj ? ii : jj, b = ii < jj ? jj : ii;
            // the row and the slot differ between lanes, so they go into the
            // lane offset (the second offset of a buffer load must be wave-uniform)
            const unsigned o = off + (unsigned)(sl[a * nz - a * (a - 1) / 2 + (b - a)] * 5 * QY);
            xx[j] = qb0.ld(o, 0u);
            yy[j] = qb0.ld(o + QY, 0u);
        }
#pragma unroll
        for (int j = 0; j < NZMAX; ++j) {
            const int jj = j < nz ? j : 0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const cpx<R> z = sh[(c * nz + jj) * fft_region(LY) + kp];
                R x = part ? z.y : z.x;
                if constexpr (ADJ) x *= lpg[jj];
                v[c][j] = (act && j < nz) ? x : R(0);
            }
        }
    }

    __device__ __forceinline__ void finish(cpx<R>* sh, int nz, const R* lpg)
    {
        wave_sync();  // the whole wave has read its operands
        const int ii = i < nz ? i : nz - 1;
        const R dgi = lpg[nz + ii];
        R acc[3] = {R(0), R(0), R(0)};
#pragma unroll
        for (int j = 0; j < NZMAX; ++j) {
            const R zz = (j == ii ? dgi : R(0)) - (xx[j] + yy[j]);
            acc[0] = fma(xx[j], v[0][j], acc[0]);
            acc[1] = fma(yy[j], v[1][j], acc[1]);
            acc[2] = fma(zz, v[2][j], acc[2]);
        }
        if (act) {
            const R sc = ADJ ? R(1) : lpg[i];
#pragma unroll
            for (int c = 0; c < 3; ++c)
                reinterpret_cast<R*>(&sh[(c * nz + i) * fft_region(LY) + kp])[part] = acc[c] * sc;
        }
    }
};

// Threads of a fused block: at least one per frequency (and a wave), at most as many
// as run the column's 3 nz transforms in one round (8 values each), within 512 below
// 1024 points.
template <int LY, int NZMAX>
struct FusedShape {
    static constexpr int least = LY < 64 ? 64 : LY;
    static constexpr int most()
    {
        int n = least;
        while (n < 512 && n < 3 * NZMAX * LY / 8) n *= 2;
        return n;
    }
};

// ---------------------------------------------------------------------------
// Fused y pass for one kx column of one state: forward y-DFT of the 3 nz
// signals (input zero padded from ny to LY), z-mixing per ky, inverse y-DFT
// cropped to ny.  All 3 nz spectra stay in LDS.  Lanes 2t and 2t+1 mix the ky
// pair (t, LY - t) (t = 0: ky = 0 and LY/2), which share one quadrant tensor
// entry, so the two lanes read the same addresses.
// Column 0 carries kx = 0 and kx = Lx/2 packed as A + iB; they are separated
// with the Hermitian symmetry in ky, mixed with their own tensor rows and
// packed again.  adjoint != 0 applies the transpose (inputs scaled by 1/t
// instead of the outputs).
// ---------------------------------------------------------------------------
// Body of the fused y pass for column kx of state b (stack geom); the
// kernels below launch it on a grid (M, states per stack, stacks).
template <typename R, int LY, int NZMAX, bool ADJ, int NT>
__device__ __forceinline__ void ymix_column(int kx, int b, int geom, cpx<R>* __restrict__ X,
                                            int ny, int nz, int M, const R* __restrict__ Q,
                                            long long qcs, const int* __restrict__ qslot, int QY,
                                            const R* __restrict__ lp,
                                            const cpx<R>* __restrict__ twy)
{
    constexpr int V = fft_vals(LY), GT = LY / V, NG = NT / GT;
    constexpr int LYP = fft_region(LY);  // LDS slots per signal
    static_assert(NT >= LY, "one thread per frequency");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<R>* sh = reinterpret_cast<cpx<R>*>(smem_raw);
    const int S = 3 * nz;
    const long long sstride = (long long)M * ny;
    cpx<R>* col = X + ((long long)b * S * M + kx) * ny;
    const int tid = threadIdx.x, grp = tid / GT, g = tid % GT;
    Twiddles<R, LY> tw;
    tw.load(g, twy, 1);

    // lane -> frequency point of the mixing phase (see below); the first tensor
    // row of an ordinary column is requested now so that its latency overlaps
    // the forward transforms
    const int t = tid >> 1, p = tid & 1;
    const int ky = p == 0 ? t : (t == 0 ? LY / 2 : LY - t);   // this lane's point
    const int kq = p == 0 ? t : (t == 0 ? LY / 2 : t);        // its quadrant column
    const int P = nz * (nz + 1) / 2;
    const int* sl = qslot + (long long)geom * P;              // the stack's pair slots
    const UniformBuf<R> qb(Q + tab_row(kx, M) * qcs, (unsigned)(qcs * sizeof(R)));
    // packed column: rows kx = 0 and kx = M (adjacent in the table) from one
    // uniform base, the row in the lane offset
    const UniformBuf<R> qb0(Q, (unsigned)(2 * qcs * sizeof(R)));
    const unsigned off0 = (unsigned)(t + (p == 0 ? 0LL : qcs));
    // (above 8 layers, or with 1024 threads per block, the registers do not
    // hold a prefetched row)
    constexpr bool EARLY_ROW = NZMAX <= 8 && NT <= 512;
    TensorRow<R, NZMAX> row0;
    if constexpr (EARLY_ROW) {
        if (kx != 0) {
            if (t < LY / 2) row0.load(qb, (unsigned)kq, QY, nz, 0, sl);
        } else if (t != 0 && t < LY / 2) {
            row0.template load<1>(qb0, off0, QY, nz, 0, sl);
        }
    }

    // forward transforms: the inputs of all of this group's signals are
    // requested first, then transformed one after the other
    constexpr int NR = (3 * NZMAX + NG - 1) / NG;   // signals per group, at most
    cpx<R> xin[NR][V];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int s = grp + r * NG;
        if (s < S) {
            const cpx<R>* src = col + s * sstride;
            fft_first_loads<R, LY, true>(xin[r], g, [&](int pos) -> cpx<R> {
                return pos < ny ? src[pos] : cpx<R>{R(0), R(0)};
            });
        }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int s = grp + r * NG;
        if (s < S) {
            cpx<R>* reg = sh + s * LYP;
            wave_fft_pre<R, LY, false, true>(reg, g, tw, xin[r], [&](int pos, cpx<R> v) { reg[pos] = v; });
        }
    }
    __syncthreads();

    // ky = 0 and LY/2 of the packed column are mixed by the first wave; its
    // operands are requested before the wave's own mixing where the register
    // budget allows (up to 512 threads per block)
    constexpr bool mirror_early = NT <= 512;
    MirrorPoints<R, LY, NZMAX, ADJ> mirror;
    const bool mirror_wave = kx == 0 && tid < 64;
    if (mirror_early && mirror_wave)
        mirror.prep(sh, nz, tid, Q, qcs, sl, QY, lp + (long long)geom * 2 * nz);

    if (t < LY / 2) {
        const R* lpg = lp + (long long)geom * 2 * nz;
        R invt[NZMAX], dg[NZMAX];
#pragma unroll
        for (int i = 0; i < NZMAX; ++i) {
            invt[i] = i < nz ? lpg[i] : R(0);
            dg[i] = i < nz ? lpg[nz + i] : R(0);
        }
        // sources scaled by 1/t for the transpose (T A T^-1), targets otherwise
        auto isc = [&](int l) -> R { return invt[l]; };
        cpx<R> H[3 * NZMAX];
        auto store = [&](int ky) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int l = 0; l < NZMAX; ++l)
                    if (l < nz) {
                        cpx<R> v = H[c * NZMAX + l];
                        if constexpr (!ADJ) v = cscale(v, invt[l]);
                        sh[(c * nz + l) * LYP + ky] = v;
                    }
        };
        auto ld = [&](int c, int l, int k) -> cpx<R> {
            cpx<R> v = sh[(c * nz + l) * LYP + k];
            if constexpr (ADJ) v = cscale(v, isc(l));
            return v;
        };
        const R sg = (p == 1 && t != 0) ? R(-1) : R(1);
        if (kx != 0) {
            auto in = [&](int c, int l) -> cpx<R> { return ld(c, l, ky); };
            if constexpr (EARLY_ROW) mix1<R, NZMAX>(nz, in, H, qb, (unsigned)kq, QY, sl, sg, dg, row0);
            else mix1<R, NZMAX>(nz, in, H, qb, (unsigned)kq, QY, sl, sg, dg);
            store(ky);
        } else if (t != 0) {
            // column 0 holds Z = A + iB with A the kx = 0 and B the kx = Lx/2
            // column: A(ky) = (Z(ky) + conj Z(-ky))/2, B(ky) = (Z(ky) - conj Z(-ky))/(2i).
            // Lane p = 0 mixes A(t) with row 0, lane p = 1 mixes B(t) with row M;
            // W(t) = HA + i HB, W(-t) = conj(HA) + i conj(HB).
            const int k1 = t, k2 = LY - t;
            auto in = [&](int c, int l) -> cpx<R> {
                const cpx<R> z1 = ld(c, l, k1), z2 = ld(c, l, k2);
                return p == 0 ? cpx<R>{R(0.5) * (z1.x + z2.x), R(0.5) * (z1.y - z2.y)}
                              : cpx<R>{R(0.5) * (z1.y + z2.y), R(0.5) * (z2.x - z1.x)};
            };
            // on the rows kx = 0 and kx = M only xx, yy, zz and yz are non-zero
            if constexpr (EARLY_ROW) mix1<R, NZMAX, 1>(nz, in, H, qb0, off0, QY, sl, R(1), dg, row0);
            else mix1<R, NZMAX, 1>(nz, in, H, qb0, off0, QY, sl, R(1), dg);
#pragma unroll
            for (int k = 0; k < 3 * NZMAX; ++k) {
                const cpx<R> o = {__shfl_xor(H[k].x, 1), __shfl_xor(H[k].y, 1)};
                const cpx<R> A = p == 0 ? H[k] : o, Bv = p == 0 ? o : H[k];
                H[k] = p == 0 ? cpx<R>{A.x - Bv.y, A.y + Bv.x} : cpx<R>{A.x + Bv.y, Bv.x - A.y};
            }
            store(p == 0 ? k1 : k2);
        }
    }
    if (mirror_wave) {
        if constexpr (!mirror_early)
            mirror.prep(sh, nz, tid, Q, qcs, sl, QY, lp + (long long)geom * 2 * nz);
        mirror.finish(sh, nz, lp + (long long)geom * 2 * nz);
    }
    __syncthreads();

    for (int s = grp; s < S; s += NG) {
        cpx<R>* dst = col + s * sstride;
        cpx<R>* reg = sh + s * LYP;
        wave_fft<R, LY, true, false, true>(
            reg, g, tw, [&](int pos) -> cpx<R> { return reg[pos]; },
            [&](int pos, cpx<R> v) {
                if (pos < ny) dst[pos] = v;
            });
    }
}

// Grid (M, states per stack, stacks): the stack index is blockIdx.z, so no
// integer division is needed (on gfx950 it runs on the vector unit, and a
// buffer descriptor built from its result is treated as a per-lane value).
template <typename R, int LY, int NZMAX, bool ADJ, int NT>
__global__ __launch_bounds__(NT) void k_ymix_fused(
    cpx<R>* __restrict__ X, int ny, int nz, int M, const R* __restrict__ Q, long long qcs,
    const int* __restrict__ qslot, int QY, const R* __restrict__ lp, int bpg,
    const cpx<R>* __restrict__ twy)
{
    const int geom = blockIdx.z;
    ymix_column<R, LY, NZMAX, ADJ, NT>(blockIdx.x, geom * bpg + blockIdx.y, geom, X, ny, nz, M, Q, qcs, qslot, QY, lp,
                                       twy);
}

// ---------------------------------------------------------------------------
// Fused y pass for a stack of exactly NZ layers (single precision, 256-, 512-
// or 1024-point columns): the same three phases as ymix_column, with every loop
// over layers and layer pairs unrolled.  A lane's 3 NZ input values sit in
// registers for the whole mixing, which walks the NZ (NZ + 1) / 2 stored pairs
// in order (i, j >= i) and applies each block both ways; the tensor entries
// are plain loads that the compiler schedules ahead of their use.  The column
// spectra are read and written through buffer descriptors whose size is the
// column's ny values: the zero padding of the forward transform and the crop
// of the inverse come from the descriptor's range check.  Column 0 (the packed
// kx = 0 and Lx/2 columns) runs ymix_column (up to 512-point columns) or a
// separate k_ymix_fused launch (1024-point columns).
// NT = 512, 8 waves of up to 256 VGPRs; 256 for short columns in many blocks
// (see fused_exact_a).
// ---------------------------------------------------------------------------
template <typename R, int LY, int NZ, bool ADJ, int NT>
__global__ __launch_bounds__(NT) void k_ymix_fused_nz(
    cpx<R>* __restrict__ X, int ny, int M, const R* __restrict__ Q, long long qcs,
    const int* __restrict__ qslot, int QY, const R* __restrict__ lp, int bpg,
    const cpx<R>* __restrict__ twy)
{
    constexpr int V = fft_vals(LY), GT = LY / V, NG = NT / GT;
    constexpr int S = 3 * NZ, P = NZ * (NZ + 1) / 2;
    constexpr int LYP = fft_region(LY);    // LDS slots per signal
    constexpr int NR = (S + NG - 1) / NG;  // signals per wave, at most
    // one transform per wavefront (512- and 1024-point columns), or two
    // (256-point columns: each half-wave transforms its own signal, so the
    // column reads and writes use per-lane addresses instead of descriptors)
    static_assert(sizeof(R) == 4 && (GT == 64 || GT == 32), "single precision, 256 to 1024 points");
    constexpr bool WHOLE_WAVE = GT == 64;
    // 512-point columns: block 0 runs the packed column 0 with the generic
    // body (one thread per frequency, as here); longer columns leave column 0
    // to a separate launch of k_ymix_fused and start at kx = 1
    constexpr bool OWN_COL0 = LY <= 512;
    const int kx = blockIdx.x + (OWN_COL0 ? 0 : 1), geom = blockIdx.z, b = geom * bpg + blockIdx.y;
    if constexpr (OWN_COL0) {
        if (kx == 0) {
            ymix_column<R, LY, NZ, ADJ, NT>(0, b, geom, X, ny, NZ, M, Q, qcs, qslot, QY, lp, twy);
            return;
        }
    }
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<R>* sh = reinterpret_cast<cpx<R>*>(smem_raw);
    const long long sstride = (long long)M * ny;
    cpx<R>* col = X + ((long long)b * S * M + kx) * ny;
    const int tid = threadIdx.x, grp = tid / GT, g = tid % GT;
    const int cbytes = ny * (int)sizeof(cpx<R>);
    const int p = tid & 1;
    const int* sl = qslot + geom * P;  // the stack's pair slots (scalar loads)
    const UniformBuf<R> qb(Q + (long long)tab_row(kx, M) * qcs, (unsigned)(qcs * sizeof(R)));

    // forward transforms: the inputs of all of this wave's signals are
    // requested first, then transformed one after the other
    {
        Twiddles<R, LY> tw;
        tw.load(g, twy, 1);
        cpx<R> xin[NR][V];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if constexpr (WHOLE_WAVE) {
                const int s = __builtin_amdgcn_readfirstlane(grp + r * NG);
                if (s < S) {
                    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
                        (void*)(col + s * sstride), (short)0, cbytes, 0x00020000);
                    fft_first_loads<R, LY, true>(xin[r], g, [&](int pos) -> cpx<R> {
                        return __builtin_bit_cast(cpx<R>, __builtin_amdgcn_raw_buffer_load_b64(
                                                              src, pos * (int)sizeof(cpx<R>), 0, 0));
                    });
                }
            } else {
                const int s = grp + r * NG;
                if (s < S) {
                    const cpx<R>* src = col + s * sstride;
                    fft_first_loads<R, LY, true>(xin[r], g, [&](int pos) -> cpx<R> {
                        return pos < ny ? src[pos] : cpx<R>{R(0), R(0)};
                    });
                }
            }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int s = grp + r * NG;
            if (s < S) {
                cpx<R>* reg = sh + s * LYP;
                wave_fft_pre<R, LY, false, true>(reg, g, tw, xin[r],
                                           [&](int pos, cpx<R> v) { reg[pos] = v; });
            }
        }
    }
    __syncthreads();

    // mixing: lanes 2t and 2t+1 take ky = t and LY - t (t = 0: 0 and LY/2),
    // which share the quadrant tensor entry t; t steps by NT / 2
    const R* lpg = lp + (long long)geom * 2 * NZ;
    for (int t = tid >> 1; t < LY / 2; t += NT / 2) {
        const int ky = p == 0 ? t : (t == 0 ? LY / 2 : LY - t);
        const int kq = p == 0 ? t : (t == 0 ? LY / 2 : t);
        const R sg = (p == 1 && t != 0) ? R(-1) : R(1);
        {
            cpx<R> in[3][NZ], H[3][NZ];
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int l = 0; l < NZ; ++l) {
                    cpx<R> v = sh[(c * NZ + l) * LYP + ky];
                    if constexpr (ADJ) v = cscale(v, lpg[l]);  // T A T^-1: sources scaled by 1/t
                    in[c][l] = v;
                    H[c][l] = {R(0), R(0)};
                }
#pragma unroll
            for (int i = 0; i < NZ; ++i)
#pragma unroll
                for (int j = i; j < NZ; ++j) {
                    const int u = i * NZ - i * (i - 1) / 2 + (j - i);
                    auto q = [&](int c) -> R { return qb.ld((unsigned)kq, (unsigned)((sl[u] * 5 + c) * QY)); };
                    const R xx = q(0), yy = q(1), xy = sg * q(2), xz = q(3), yz = sg * q(4);
                    R zz = -(xx + yy);
                    if (i == j) {
                        zz += lpg[NZ + i];
                        block_apply(H[0][i], H[1][i], H[2][i], in[0][i], in[1][i], in[2][i], xx, yy,
                                    zz, xy, xz, yz);
                    } else {
                        block_apply(H[0][i], H[1][i], H[2][i], in[0][j], in[1][j], in[2][j], xx, yy,
                                    zz, xy, xz, yz);
                        block_apply(H[0][j], H[1][j], H[2][j], in[0][i], in[1][i], in[2][i], xx, yy,
                                    zz, xy, -xz, -yz);
                    }
                }
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int l = 0; l < NZ; ++l) {
                    cpx<R> v = H[c][l];
                    if constexpr (!ADJ) v = cscale(v, lpg[l]);  // targets scaled by 1/t
                    sh[(c * NZ + l) * LYP + ky] = v;
                }
        }
    }
    __syncthreads();

    // inverse transforms; stores beyond the column's ny values are dropped
    {
        Twiddles<R, LY> tw;
        tw.load(g, twy, 1);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if constexpr (WHOLE_WAVE) {
                const int s = __builtin_amdgcn_readfirstlane(grp + r * NG);
                if (s < S) {
                    const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(
                        (void*)(col + s * sstride), (short)0, cbytes, 0x00020000);
                    cpx<R>* reg = sh + s * LYP;
                    wave_fft<R, LY, true, false, true>(
                        reg, g, tw, [&](int pos) -> cpx<R> { return reg[pos]; },
                        [&](int pos, cpx<R> v) {
                            __builtin_amdgcn_raw_buffer_store_b64(
                                __builtin_bit_cast(__attribute__((__vector_size__(8))) unsigned, v),
                                dst, pos * (int)sizeof(cpx<R>), 0, 0);
                        });
                }
            } else {
                const int s = grp + r * NG;
                if (s < S) {
                    cpx<R>* dst = col + s * sstride;
                    cpx<R>* reg = sh + s * LYP;
                    wave_fft<R, LY, true, false, true>(
                        reg, g, tw, [&](int pos) -> cpx<R> { return reg[pos]; },
                        [&](int pos, cpx<R> v) {
                            if (pos < ny) dst[pos] = v;
                        });
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Five-pass path: y transforms and mixing as separate kernels (any nz).
// ---------------------------------------------------------------------------
template <typename R, int LY>
struct YPassShape {
    static constexpr int V = fft_vals(LY);
    static constexpr int GT = LY / V;
    static constexpr int NG0 = 256 / GT;
    static constexpr int NGL = (int)(65536 / (sizeof(cpx<R>) * fft_region(LY)));
    static constexpr int NG = NG0 < NGL ? NG0 : (NGL < 1 ? 1 : NGL);
    static constexpr int NT = NG * GT;
    // whether the groups of k_yfwd walk over columns: not in FP64 from 2048 points on,
    // where kept twiddles leave no registers for the next column (4096 points: 172
    // registers spilled instead of 106) and a block is one group, so that two columns each
    // make a long last round.  Walking, 2304 columns of 2048 cells took 139 us instead of 117,
    // 6144 of 1025 283 instead of 278, 2304 of 1000 (2048 points) 35.7 instead of 32.3.
    // k_yinv, which stores half of a transform, gains with many columns: 275 us
    // instead of 354 for the 6144.
    static constexpr bool WALK_FWD = sizeof(R) == 4 || LY < 2048;
};

// Columns of n_in <= LY/2 complex values (zero padded to LY: the first radix pass
// skips the zero half) -> LY spectrum values.  Bound by the Infinity Cache and
// HBM.  A group keeps its twiddles and walks over columns (y_blocks): they are 14
// loads per lane of a 512-point transform, whose data are 4 loads and 8 stores.
// 480 layer components of 256 x 512 points (16 states of 256 x 256 x 10; 757 MB):
// 168 -> 144 us forward, 155 -> 148 us back (5.2 TB/s); 96 of 256 x 512 (151 MB): 31 -> 26 and
// 33 -> 26 us; 9 of 1024 x 2048: 55 -> 47 and 51 -> 46 us.
// Requesting the next column's values before the current one's transform gained
// nothing more.
template <typename R, int LY>
__global__ __launch_bounds__((YPassShape<R, LY>::NT)) void k_yfwd(const cpx<R>* __restrict__ in,
                                                                cpx<R>* __restrict__ out, int n_in,
                                                                long long ncols,
                                                                const cpx<R>* __restrict__ twy)
{
    using S = YPassShape<R, LY>;
    __shared__ cpx<R> sh[S::NG * fft_region(LY)];
    const int tid = threadIdx.x, grp = tid / S::GT, g = tid % S::GT;
    const long long c0 = (long long)blockIdx.x * S::NG + grp;
    if constexpr (!S::WALK_FWD) {
        if (c0 >= ncols) return;
        const cpx<R>* src = in + c0 * n_in;
        cpx<R>* dst = out + c0 * LY;
        wave_fft<R, LY, false, true>(
            sh + grp * fft_region(LY), g, twy, 1,
            [&](int pos) -> cpx<R> { return pos < n_in ? src[pos] : cpx<R>{R(0), R(0)}; },
            [&](int pos, cpx<R> z) { dst[pos] = z; });
    } else {
        const long long step = (long long)gridDim.x * S::NG;
        Twiddles<R, LY> tw;
        tw.load(g, twy, 1);
        for (long long c = c0; c < ncols; c += step) {
            const cpx<R>* src = in + c * n_in;
            cpx<R>* dst = out + c * LY;
            cpx<R> v[S::V];
            fft_first_loads<R, LY, true>(v, g, [&](int pos) -> cpx<R> {
                return pos < n_in ? src[pos] : cpx<R>{R(0), R(0)};
            });
            wave_fft_pre<R, LY, false, true>(sh + grp * fft_region(LY), g, tw, v,
                                             [&](int pos, cpx<R> z) { dst[pos] = z; });
            wave_sync();
        }
    }
}

// LY spectrum values -> first n_out <= LY/2 values of the inverse transform
// (the last radix pass computes only that half); columns as in k_yfwd
template <typename R, int LY>
__global__ __launch_bounds__((YPassShape<R, LY>::NT)) void k_yinv(const cpx<R>* __restrict__ in,
                                                                cpx<R>* __restrict__ out, int n_out,
                                                                long long ncols,
                                                                const cpx<R>* __restrict__ twy)
{
    using S = YPassShape<R, LY>;
    __shared__ cpx<R> sh[S::NG * fft_region(LY)];
    const int tid = threadIdx.x, grp = tid / S::GT, g = tid % S::GT;
    const long long step = (long long)gridDim.x * S::NG;
    Twiddles<R, LY> tw;
    tw.load(g, twy, 1);
    for (long long c = (long long)blockIdx.x * S::NG + grp; c < ncols; c += step) {
        const cpx<R>* src = in + c * LY;
        cpx<R>* dst = out + c * n_out;
        cpx<R> v[S::V];
        fft_first_loads<R, LY>(v, g, [&](int pos) -> cpx<R> { return src[pos]; });
        wave_fft_pre<R, LY, true, false, true>(sh + grp * fft_region(LY), g, tw, v, [&](int pos, cpx<R> z) {
            if (pos < n_out) dst[pos] = z;
        });
        wave_sync();
    }
}

// One stored block (xx, yy, xy, xz, yz, and u = xx + yy - trace, so zz = -u)
// applied to a source in the rotated components (X, Y, iZ), in which the block
// is the real matrix [[xx, xy, xz], [xy, yy, yz], [-xz, -yz, zz]]; TR: the
// conjugate block of the transposed pair (xz, yz negated).
template <bool TR, typename R>
__device__ __forceinline__ void block_real(cpx<R> (&h)[3], cpx<R> X, cpx<R> Y, cpx<R> Z, const R (&q)[5], R u)
{
    const R xx = q[0], yy = q[1], xy = q[2], xz = TR ? -q[3] : q[3], yz = TR ? -q[4] : q[4];
    h[0].x = fma(xx, X.x, h[0].x); h[0].x = fma(xy, Y.x, h[0].x); h[0].x = fma(xz, Z.x, h[0].x);
    h[0].y = fma(xx, X.y, h[0].y); h[0].y = fma(xy, Y.y, h[0].y); h[0].y = fma(xz, Z.y, h[0].y);
    h[1].x = fma(xy, X.x, h[1].x); h[1].x = fma(yy, Y.x, h[1].x); h[1].x = fma(yz, Z.x, h[1].x);
    h[1].y = fma(xy, X.y, h[1].y); h[1].y = fma(yy, Y.y, h[1].y); h[1].y = fma(yz, Z.y, h[1].y);
    h[2].x = fma(-xz, X.x, h[2].x); h[2].x = fma(-yz, Y.x, h[2].x); h[2].x = fma(-u, Z.x, h[2].x);
    h[2].y = fma(-xz, X.y, h[2].y); h[2].y = fma(-yz, Y.y, h[2].y); h[2].y = fma(-u, Z.y, h[2].y);
}

// Five-pass z-mixing on full spectra (any nz), in place where Hh = Mh.
// A block takes one tile: 32 ky pairs of one kx column of one state, lanes l
// and 32 + l of every wave on the ky points t and LY - t (t = 0: ky = 0 and
// LY/2), which share one quadrant tensor entry.  The tile's spectra are staged
// once in LDS; each wave owns IB target layers, sums over all sources with its
// accumulators in registers, and requests the next source's entries while it
// applies the current one's.
// * Every entry of a layer pair is wanted by two waves, the owners of its two
//   layers: target groups g and g' take each other's sources in the same round
//   r (g + g' = r mod the group count), so the second request finds the line in
//   L1 or L2.  Blocks of more than 8 waves keep their rounds in step with a
//   barrier (64 layers: 1103 -> 995 us); smaller ones do not need it.
// * The two halves of a wave want the same entries, so each asks for one of two
//   targets' and halves() hands them over (10 loads for 20 entries).  That
//   does not hold for the first ky tile (t = 0 reads two different entries) nor
//   for the packed column (two different rows), which load every entry.
// * Each XCD (blocks go to the 8 XCDs in turn) runs a contiguous range of tiles,
//   the parts of a tile and the states first, then the ky tiles of a column: a
//   tile's 128-byte slices of the (odd-length) tensor rows straddle two lines,
//   and the states of one stack read the same entries.
// * In the rotated components (X, sg Y, iZ), sg = -1 on the points LY - t, where
//   xy and yz change sign, the block is the same real matrix for both points:
//   18 FMAs and one addition per direction.
// Bound by the stream of the tensor: per call 20 (FP64: 40) bytes per pair and
// quadrant frequency.  256 x 256 cells, FP32: 8 / 16 / 32 layers 54 / 115 / 406 ->
// 21 / 56 / 259 us (98, 280, 899 MB: 4.7, 5.0, 3.5 TB/s; 1.0 GB is fetched at 32
// layers), FP64, 8 layers 74 -> 37 us (196 MB from the Infinity Cache).  Before, one
// wave per target group read the spectra and entries of its tile on its own, 4.5
// times what is needed at 32 layers.
// Column 0 carries kx = 0 and Lx/2 packed as A + iB: lane p = 0 mixes A(t)
// with the kx = 0 row and lane p = 1 B(t) with the kx = Lx/2 row, and the pair
// repacks through a lane shuffle; at the self-mirrored points t = 0 (ky = 0 and
// LY/2) only xx, yy and zz are non-zero: the real part A takes the kx = 0 row
// and the imaginary part B, in a second sweep of that one tile, the kx = Lx/2 row.
// jc: layers staged at a time; parts: blocks that share a tile's target groups
// (not in place: they all read the tile); NT: the largest block.
template <typename R, int IB, int NT>
__global__ __launch_bounds__(NT) void k_mix_tile(const cpx<R>* Mh, cpx<R>* Hh, int nz, int M, int LY,
                                                 const R* __restrict__ Q, long long qcs,
                                                 const int* __restrict__ qslot, int QY,
                                                 const R* __restrict__ lp, int bpg, int adjoint,
                                                 int kx0, int ntile, int B, int jc, int parts)
{
    static_assert(IB % 2 == 0, "targets in pairs");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cpx<R>* sh = reinterpret_cast<cpx<R>*>(smem_raw);  // [3][jc][64]
    const int unit = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    // (integer divisions run on the vector unit: back to scalars)
    const int tile = __builtin_amdgcn_readfirstlane(unit / parts), part = unit - tile * parts;
    if (tile >= ntile) return;
    const int nkyb = (LY / 2 + 31) / 32, col = __builtin_amdgcn_readfirstlane(tile / B);
    const int b = tile - col * B, ck = __builtin_amdgcn_readfirstlane(col / nkyb);
    const int kyb = col - ck * nkyb, kx = kx0 + ck;
    const int geom = __builtin_amdgcn_readfirstlane(b / bpg);
    const int lane = threadIdx.x & 63, W = blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = kyb * 32 + (lane & 31), p = lane >> 5;
    const bool active = t0 < LY / 2;
    const int t = active ? t0 : 0;
    const int ky = p == 0 ? t : (t == 0 ? LY / 2 : LY - t);
    const int kq = p == 0 ? t : (t == 0 ? LY / 2 : t);
    const long long sst = (long long)M * LY;
    const cpx<R>* mb = Mh + ((long long)b * 3 * nz * M + kx) * LY + ky;
    cpx<R>* hb = Hh + ((long long)b * 3 * nz * M + kx) * LY + ky;
    const R* lpg = lp + (long long)geom * 2 * nz;
    const int* sl = qslot + (long long)geom * (nz * (nz + 1) / 2);  // the stack's pair slots
    const bool packed = kx == 0, mirror = packed && kyb == 0;
    const R sg = (!packed && p == 1 && t != 0) ? R(-1) : R(1);
    // a lane of the packed column reads row kx = 0 or kx = M (adjacent rows)
    const UniformBuf<R> qb(Q + (long long)tab_row(kx, M) * qcs,
                           (unsigned)((packed ? 2 : 1) * qcs * sizeof(R)));
    const int gi = part * W + w, i0 = gi * IB;   // this wave's target group
    const bool pace = W > 8;
    int rowbase[IB];   // pair (i, j >= i) is rowbase + j
#pragma unroll
    for (int k = 0; k < IB; ++k) {
        const int i = i0 + k < nz ? i0 + k : nz - 1;
        rowbase[k] = i * nz - i * (i - 1) / 2 - i;
    }

    cpx<R> H[IB][3];
#pragma unroll
    for (int k = 0; k < IB; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) H[k][c] = {R(0), R(0)};
    for (int step = 0; step < (mirror ? 2 : 1); ++step)
    for (int j0 = 0; j0 < nz; j0 += jc) {
        const int jn = nz - j0 < jc ? nz - j0 : jc;
        if (j0 > 0 || step > 0) __syncthreads();
        for (int lb = w * IB; lb < jn; lb += W * IB) {
            cpx<R> z[IB][3];
#pragma unroll
            for (int k = 0; k < IB; ++k)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    z[k][c] = mb[(c * nz + j0 + (lb + k < jn ? lb + k : jn - 1)) * sst];
#pragma unroll
            for (int k = 0; k < IB; ++k) {
                const int l = lb + k;
                if (l >= jn) break;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    cpx<R> v = z[k][c];
                    if (packed) {
                        // A(t) = (Z(t) + conj Z(-t)) / 2 on lane 0, B(t) = (Z(t) - conj Z(-t)) / (2i) on
                        // lane 1; the self-mirrored points take A, then iB
                        const cpx<R> o = {__shfl_xor(v.x, 32), __shfl_xor(v.y, 32)};
                        if (t != 0)
                            v = p == 0 ? cpx<R>{R(0.5) * (v.x + o.x), R(0.5) * (v.y - o.y)}
                                       : cpx<R>{R(0.5) * (o.y + v.y), R(0.5) * (v.x - o.x)};
                        else
                            v = step == 0 ? cpx<R>{v.x, R(0)} : cpx<R>{R(0), v.y};
                        if (step > 0 && t != 0) v = {R(0), R(0)};
                    }
                    if (adjoint) v = cscale(v, lpg[j0 + l]);
                    if (c == 1) v = cscale(v, sg);
                    if (c == 2) v = {-v.y, v.x};
                    sh[(c * jn + l) * 64 + lane] = v;
                }
            }
        }
        __syncthreads();
        // (second sweep: the self-mirrored points read row kx = M)
        const unsigned voff = (unsigned)(kq + (packed && ((p == 1 && t != 0) || step > 0) ? qcs : 0LL));

        // the sources of this chunk in rounds of IB
        const int nr = (jn + IB - 1) / IB;
        int sn[IB];   // table offsets of the source to fetch next
        auto slots = [&](int js) {
            const int j = j0 + (js < jn ? js : jn - 1), jrow = j * nz - j * (j - 1) / 2 - j;
#pragma unroll
            for (int k = 0; k < IB; ++k) {
                const int i = i0 + k < nz ? i0 + k : nz - 1;
                sn[k] = sl[i <= j ? rowbase[k] + j : jrow + i] * 5 * QY;
            }
        };
        auto rounds = [&](auto split) {
            constexpr bool SPLIT = decltype(split)::value;
            auto fetch = [&](R (&T)[IB][5]) {
                if constexpr (SPLIT) {
                    // each half-wave asks for the entries of one of two targets
#pragma unroll
                    for (int k = 0; k < IB; k += 2) {
                        const unsigned v = voff + (unsigned)(p == 0 ? sn[k] : sn[k + 1]);
#pragma unroll
                        for (int c = 0; c < 5; ++c) T[k][c] = qb.ld(v, (unsigned)(c * QY));
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < IB; ++k)
#pragma unroll
                        for (int c = 0; c < 5; ++c) T[k][c] = qb.ld(voff, (unsigned)(sn[k] + c * QY));
                }
            };
            auto apply = [&](int js, const R (&T)[IB][5]) {
                if (js >= jn) return;
                const int j = j0 + js;
                const cpx<R> X = sh[js * 64 + lane], Y = sh[(jn + js) * 64 + lane],
                             Z = sh[(2 * jn + js) * 64 + lane];
#pragma unroll
                for (int k = 0; k < IB; k += 2) {
                    R q[2][5];
#pragma unroll
                    for (int c = 0; c < 5; ++c) {
                        if constexpr (SPLIT) {
                            halves(T[k][c], q[0][c], q[1][c]);
                        } else {
                            q[0][c] = T[k][c];
                            q[1][c] = T[k + 1][c];
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int i = i0 + k + e;
                        R u = q[e][0] + q[e][1];
                        if (i == j) u -= lpg[nz + i];
                        if (i > j) block_real<true>(H[k + e], X, Y, Z, q[e], u);
                        else block_real<false>(H[k + e], X, Y, Z, q[e], u);
                    }
                }
            };
            R T[2][IB][5];
            int J = gi % nr;
            J = __builtin_amdgcn_readfirstlane(J == 0 ? 0 : nr - J);   // round 0: group -gi mod nr
            slots(J * IB);
            fetch(T[0]);
            slots(J * IB + 1);
            for (int r = 0; r < nr; ++r) {
                const int Jn = J + 1 == nr ? 0 : J + 1;
                if (pace) __builtin_amdgcn_s_barrier();
#pragma unroll
                for (int k = 0; k < IB; ++k) {
                    // (the last round fetches its successor's first source, unused)
                    fetch(T[(k + 1) % 2]);
                    slots(k + 2 < IB ? J * IB + k + 2 : Jn * IB + (k + 2 - IB));
                    apply(J * IB + k, T[k % 2]);
                }
                J = Jn;
            }
        };
        if (kyb != 0 && !packed) rounds(std::true_type{});
        else rounds(std::false_type{});
    }
    if (mirror) __syncthreads();  // (the second sweep read the tile again)
    // back to (X, Y, Z), scaled by 1/t (in place: only this block reads its
    // tile, and every layer has been staged)
#pragma unroll
    for (int k = 0; k < IB; ++k) {
        const int i = i0 + k;
        if (i >= nz) break;
        const R post = adjoint ? R(1) : lpg[i];
        const cpx<R> o[3] = {cscale(H[k][0], post), cscale(H[k][1], sg * post),
                             cpx<R>{post * H[k][2].y, -post * H[k][2].x}};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            cpx<R> v = o[c];
            if (packed) {
                // W(t) = HA + i HB on lane 0, W(-t) = conj(HA) + i conj(HB) on lane 1
                const cpx<R> e = {__shfl_xor(v.x, 32), __shfl_xor(v.y, 32)};
                if (t != 0) v = p == 0 ? cpx<R>{v.x - e.y, v.y + e.x} : cpx<R>{e.x + v.y, v.x - e.y};
            }
            if (active) hb[(c * nz + i) * sst] = v;
        }
    }
}

}  // namespace hfd
