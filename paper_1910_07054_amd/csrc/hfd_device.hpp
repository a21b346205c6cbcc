// Device-side building blocks for gfx950: complex arithmetic and a
// wavefront-local Stockham FFT engine.
//
// One FFT of length L is owned by a group of GT = L / V lanes of a single
// 64-wide wavefront; every lane holds V complex values in registers.  Passes
// use radix 8 (4 or 2 for the remainder).  Between passes the group exchanges
// data through its own LDS region of fft_region(L) slots (see Exchange);
// because the group never spans two wavefronts, no workgroup barrier is needed
// inside a transform.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hfd {

template <typename R>
struct alignas(2 * sizeof(R)) cpx {
    R x, y;
};

template <typename R>
__device__ __forceinline__ cpx<R> cadd(cpx<R> a, cpx<R> b) { return {a.x + b.x, a.y + b.y}; }
template <typename R>
__device__ __forceinline__ cpx<R> csub(cpx<R> a, cpx<R> b) { return {a.x - b.x, a.y - b.y}; }
template <typename R>
__device__ __forceinline__ cpx<R> cmul(cpx<R> a, cpx<R> b)
{
    return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename R>
__device__ __forceinline__ cpx<R> cconj(cpx<R> a) { return {a.x, -a.y}; }
template <typename R>
__device__ __forceinline__ cpx<R> cscale(cpx<R> a, R s) { return {a.x * s, a.y * s}; }
// multiply by -i (forward transforms) or +i (inverse transforms)
template <typename R, bool INV>
__device__ __forceinline__ cpx<R> mul_mi(cpx<R> a)
{
    return INV ? cpx<R>{-a.y, a.x} : cpx<R>{a.y, -a.x};
}

// Row order of the tensor tables (the Fourier tensor's pair slots and the
// derivative offsets): kx = 0, kx = M = Lx/2, then kx = 1 .. M - 1, so that
// the two rows the packed column 0 reads are adjacent.
__host__ __device__ inline int tab_row(int kx, int M) { return kx == 0 ? 0 : (kx == M ? 1 : kx + 1); }

// Ordering point for LDS traffic inside one wavefront.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Read-only view of `bytes` bytes at a wave-uniform base, loaded with raw buffer
// instructions: a per-lane 32-bit byte offset plus a wave-uniform (scalar) byte
// offset, so no per-lane 64-bit address arithmetic.  Loads beyond `bytes`
// return zero instead of touching memory.
template <typename R>
struct UniformBuf {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ UniformBuf(const R* base, unsigned bytes)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc((void*)uniform(base), (short)0,
                                                 (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000))
    {
    }
    // The base and the size pinned to scalar registers: where the compiler forms
    // either on the vector unit, a descriptor built from it counts as differing
    // between lanes, and every load becomes a loop over its distinct values.
    static __device__ __forceinline__ const R* uniform(const R* p)
    {
        const unsigned long long a = (unsigned long long)p;
        const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
        const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
        return (const R*)(((unsigned long long)hi << 32) | lo);
    }
    // element at (scalar element offset s) + (lane element offset v)
    __device__ __forceinline__ R ld(unsigned v, unsigned s) const
    {
        if constexpr (sizeof(R) == 4)
            return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(v * 4u),
                                                                              (int)(s * 4u), 0));
        else
            return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(v * 8u),
                                                                              (int)(s * 8u), 0));
    }
};

// a = the lower half-wave's v, b = the upper one's, in both halves
// (lane l gets the value of lane l % 32, or 32 + l % 32)
__device__ __forceinline__ void halves(float v, float& a, float& b)
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    a = __builtin_bit_cast(float, (unsigned)r[0]);
    b = __builtin_bit_cast(float, (unsigned)r[1]);
}
__device__ __forceinline__ void halves(double v, double& a, double& b)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    a = __builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]);
    b = __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]);
}

// values per lane for a transform of length L
__host__ __device__ constexpr int fft_vals(int L) { return L <= 8 ? L : (L <= 512 ? 8 : L / 64); }

// --- small DFTs in registers (natural order in and out) -------------------
template <typename R, bool INV>
__device__ __forceinline__ void dft2(cpx<R>* v)
{
    cpx<R> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <typename R, bool INV>
__device__ __forceinline__ void dft4(cpx<R>& a0, cpx<R>& a1, cpx<R>& a2, cpx<R>& a3)
{
    cpx<R> t0 = cadd(a0, a2), t1 = csub(a0, a2), t2 = cadd(a1, a3);
    cpx<R> t3 = mul_mi<R, INV>(csub(a1, a3));
    a0 = cadd(t0, t2);
    a2 = csub(t0, t2);
    a1 = cadd(t1, t3);
    a3 = csub(t1, t3);
}

template <typename R, bool INV>
__device__ __forceinline__ void dft8(cpx<R>* v)
{
    const R c = R(0.70710678118654752440084436210484903928);
    cpx<R> e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    cpx<R> o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4<R, INV>(e0, e1, e2, e3);
    dft4<R, INV>(o0, o1, o2, o3);
    // o_k *= w8^k (w8 = exp(-+ 2 pi i / 8))
    if (!INV) {
        o1 = {c * (o1.x + o1.y), c * (o1.y - o1.x)};
        o3 = {c * (o3.y - o3.x), -c * (o3.x + o3.y)};
    } else {
        o1 = {c * (o1.x - o1.y), c * (o1.x + o1.y)};
        o3 = {-c * (o3.x + o3.y), c * (o3.x - o3.y)};
    }
    o2 = mul_mi<R, INV>(o2);
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1);
    v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3);
    v[7] = csub(e3, o3);
}

// 16 = 4 x 4: DFT4 of x[b], x[4 + b], x[8 + b], x[12 + b], factors w16^(b k), DFT4 over b.
// The first step is left to `four`, which may know that its last two inputs are zero.
template <typename R, bool INV, class Four>
__device__ __forceinline__ void dft16(cpx<R>* v, Four four)
{
    const R c = R(0.70710678118654752440084436210484903928);
    const R c1 = R(0.92387953251128675612818318939678828682);  // cos(pi/8)
    const R s1 = R(0.38268343236508977172845998403039886676);  // sin(pi/8)
    cpx<R> y[4][4];  // [b][k]
#pragma unroll
    for (int b = 0; b < 4; ++b) four(v[b], v[4 + b], v[8 + b], v[12 + b], y[b]);
    const R d = INV ? R(-1) : R(1);
    // z exp(-+ i phi), (x, y) = (cos, sin) phi
    auto rot = [&](cpx<R> z, R x, R y) -> cpx<R> {
        y *= d;
        return {z.x * x + z.y * y, z.y * x - z.x * y};
    };
    auto eighth = [&](cpx<R> z) -> cpx<R> {  // exp(-+ i pi/4)
        return INV ? cpx<R>{c * (z.x - z.y), c * (z.x + z.y)} : cpx<R>{c * (z.x + z.y), c * (z.y - z.x)};
    };
    y[1][1] = rot(y[1][1], c1, s1);
    y[1][2] = eighth(y[1][2]);
    y[1][3] = rot(y[1][3], s1, c1);
    y[2][1] = eighth(y[2][1]);
    y[2][2] = mul_mi<R, INV>(y[2][2]);
    y[2][3] = mul_mi<R, INV>(eighth(y[2][3]));
    y[3][1] = rot(y[3][1], s1, c1);
    y[3][2] = mul_mi<R, INV>(eighth(y[3][2]));
    y[3][3] = rot(y[3][3], -c1, -s1);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        dft4<R, INV>(y[0][k], y[1][k], y[2][k], y[3][k]);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[k + 4 * q] = y[q][k];
    }
}

template <typename R, int RAD, bool INV>
__device__ __forceinline__ void dft(cpx<R>* v)
{
    if constexpr (RAD == 16) {
        dft16<R, INV>(v, [](cpx<R> a, cpx<R> b, cpx<R> c, cpx<R> d, cpx<R> (&y)[4]) {
            dft4<R, INV>(a, b, c, d);
            y[0] = a;
            y[1] = b;
            y[2] = c;
            y[3] = d;
        });
    } else if constexpr (RAD == 8) dft8<R, INV>(v);
    else if constexpr (RAD == 4) dft4<R, INV>(v[0], v[1], v[2], v[3]);
    else dft2<R, INV>(v);
}

// Radix-RAD DFT of inputs whose upper half v[RAD/2 ..] is zero (the first
// pass of a transform of a zero-padded sequence): the butterflies that only
// add zeros are dropped.
template <typename R, int RAD, bool INV>
__device__ __forceinline__ void dft_half_in(cpx<R>* v)
{
    // DFT4 of (a0, a1, 0, 0): (a0 + a1, a0 + rot(a1), a0 - a1, a0 - rot(a1)),
    // rot = multiplication by -i (forward) or +i (inverse)
    auto dft4h = [](cpx<R> a0, cpx<R> a1, cpx<R>& b0, cpx<R>& b1, cpx<R>& b2, cpx<R>& b3) {
        const cpx<R> t = mul_mi<R, INV>(a1);
        b0 = cadd(a0, a1);
        b2 = csub(a0, a1);
        b1 = cadd(a0, t);
        b3 = csub(a0, t);
    };
    if constexpr (RAD == 16) {
        dft16<R, INV>(v, [&](cpx<R> a, cpx<R> b, cpx<R>, cpx<R>, cpx<R> (&y)[4]) {
            dft4h(a, b, y[0], y[1], y[2], y[3]);
        });
    } else if constexpr (RAD == 8) {
        const R c = R(0.70710678118654752440084436210484903928);
        cpx<R> e0, e1, e2, e3, o0, o1, o2, o3;
        dft4h(v[0], v[2], e0, e1, e2, e3);
        dft4h(v[1], v[3], o0, o1, o2, o3);
        if (!INV) {
            o1 = {c * (o1.x + o1.y), c * (o1.y - o1.x)};
            o3 = {c * (o3.y - o3.x), -c * (o3.x + o3.y)};
        } else {
            o1 = {c * (o1.x - o1.y), c * (o1.x + o1.y)};
            o3 = {-c * (o3.x + o3.y), c * (o3.x - o3.y)};
        }
        o2 = mul_mi<R, INV>(o2);
        v[0] = cadd(e0, o0);
        v[4] = csub(e0, o0);
        v[1] = cadd(e1, o1);
        v[5] = csub(e1, o1);
        v[2] = cadd(e2, o2);
        v[6] = csub(e2, o2);
        v[3] = cadd(e3, o3);
        v[7] = csub(e3, o3);
    } else if constexpr (RAD == 4) {
        dft4h(v[0], v[1], v[0], v[1], v[2], v[3]);
    } else {
        v[1] = v[0];
    }
}

// LDS slots of the values between two passes.  A ds access of 8 bytes per
// lane serves 16 consecutive lanes at a time from 16 eight-byte slots, one of 16
// bytes 8 lanes from 8 (measured: 4.2 clocks per wave where every group's slots
// differ modulo 16, 8.1 where two lanes share one).  A pass that follows NS
// finished points writes pos = 8 j + r (first pass, lane j) or pos = 64 q + 8 r + k
// (NS = 8, j = 8 q + k), the next one reads consecutive positions.  The exchange after
// each pass has a layout of its own, slot(pos) = pos + (pos >> SHIFT) MULT:
//   8-byte values, NS = 1: pos + pos/16 (writes 8 (j & 1) + j / 2 mod 16, or j; reads aligned runs)
//   8-byte values, NS = 8: pos + 8 (pos/64) (writes k + 8 q mod 16)
//   NS > 8: as they are (both sides are runs of at least 16)
//   16-byte values: pos + pos/8 (writes 9 j and k mod 8), pos + pos/16 after a first pass of radix 16.
// With pos + pos/8 for both sizes the reads of 8-byte values took twice as long.
// A lane's positions differ by constants that do not carry into pos >> SHIFT, so
// their slots differ by compile-time constants and cost no address arithmetic.
// A transform of length L uses fft_region(L) slots.
template <typename R, int NS, int RAD>
struct Exchange {
    static constexpr bool WIDE = sizeof(R) == 8;
    static constexpr int SHIFT = NS == 1 && RAD == 16 ? 4 : WIDE ? 3 : (NS == 1 ? 4 : 6);
    static constexpr int MULT = WIDE ? 1 : (NS == 1 ? 1 : (NS == 8 ? 8 : 0));
    __host__ __device__ static constexpr int slot(int pos) { return pos + (pos >> SHIFT) * MULT; }
};
__host__ __device__ constexpr int fft_region(int L) { return L + (L >> 3); }

// --- Stockham engine -------------------------------------------------------
// X[k] = sum_n x[n] exp(-+2 pi i n k / L) (unnormalized in both directions).
// Twiddles: table of exp(-2 pi i m / (L * tws)) read at index m * tws,
// m in [0, L).  A lane's twiddles depend only on its position g in the group,
// so they are loaded once (Twiddles::load) and reused for every transform the
// lane runs; inverse transforms use their conjugates.
// load(pos) supplies x[pos] for the first pass; store(pos, v) receives X[pos]
// from the last pass; sh is the group's LDS region of fft_region(L) slots
// (the last pass stores through `store`, which may write the region's first
// L slots in natural order).
template <int L, int V, int NS>
struct PassShape {
    static constexpr int REM = L / NS;
    // radix 16 where it takes a pass less than 8 alone (128 = 16 8, 256 = 16 16,
    // 1024 = 16 8 8, 2048 = 16 16 8; not 4096, whose twiddles then spill more in FP64).
    // Each pass less is one exchange through LDS and one round of factors less, and the
    // kept factors take fewer registers: 64 states of 512 x 512 x 4 fused 2038 -> 1804 us,
    // 8 of 400 x 400 x 2 157 -> 102, 1024 x 1024 x 3 all transforms 175 -> 160, 128-point z
    // pass of 4 states of 128 x 64 x 40 123 -> 109.  16 values per lane for 128 and 256
    // points, where they are not there anyway, gain nothing.
    static constexpr bool R16 = V % 16 == 0 && (REM == 16 || REM == 128 || REM == 256 || REM == 1024 || REM == 2048);
    static constexpr int RAD = R16 ? 16 : (REM >= 8 && V % 8 == 0) ? 8 : ((REM >= 4 && V % 4 == 0) ? 4 : 2);
    static constexpr int NB = V / RAD;
    static constexpr bool LAST = (NS * RAD == L);
    static constexpr int NEXT = LAST ? L : NS * RAD;
};

// twiddle registers of all passes after the first, in pass order
template <int L, int V, int NS = 1>
struct TwCount {
    using P = PassShape<L, V, NS>;
    static constexpr int here = NS > 1 ? P::NB * (P::RAD - 1) : 0;
    static constexpr int value = here + (P::LAST ? 0 : TwCount<L, V, P::NEXT>::value);
};
template <int L, int V>
struct TwCount<L, V, L> {
    static constexpr int value = 0;
};

template <typename R, int L, int V = fft_vals(L)>
struct Twiddles {
    static constexpr int GT = L / V;
    static constexpr int N = TwCount<L, V>::value > 0 ? TwCount<L, V>::value : 1;
    cpx<R> w[N];

    template <int NS, int OFF>
    __device__ __forceinline__ void fill(int g, const cpx<R>* __restrict__ tw, int tws)
    {
        using P = PassShape<L, V, NS>;
        constexpr int here = NS > 1 ? P::NB * (P::RAD - 1) : 0;
        if constexpr (NS > 1) {
#pragma unroll
            for (int u = 0; u < P::NB; ++u) {
                const int j = g + GT * u;
                const int k = j & (NS - 1);
#pragma unroll
                for (int r = 1; r < P::RAD; ++r)
                    w[OFF + u * (P::RAD - 1) + r - 1] = tw[r * k * (L / (NS * P::RAD)) * tws];
            }
        }
        if constexpr (!P::LAST) fill<P::NEXT, OFF + here>(g, tw, tws);
    }
    __device__ __forceinline__ void load(int g, const cpx<R>* __restrict__ tw, int tws)
    {
        fill<1, 0>(g, tw, tws);
    }
};

// HIN: the input positions L/2 .. L-1 are zero (zero-padded sequence): the
// first pass neither loads nor transforms them.  HOUT: only the output
// positions 0 .. L/2-1 are wanted (cropped result): the last pass stores only
// those, and what feeds nothing else is not computed.
// XIn: layout of the values the pass before wrote.
template <typename R, int L, int V, bool INV, int NS, int OFF, bool PRE = false, bool HIN = false,
          bool HOUT = false, class XIn = Exchange<R, 1, 8>, class Load, class Store>
__device__ __forceinline__ void fft_pass(cpx<R> (&v)[V], cpx<R>* sh, int g, const cpx<R>* w,
                                         Load& load, Store& store)
{
    using P = PassShape<L, V, NS>;
    constexpr int GT = L / V;
    constexpr int RAD = P::RAD, NB = P::NB;
    constexpr int STRIDE = L / RAD;
    constexpr bool FIRST = (NS == 1);
    constexpr bool LAST = P::LAST;
    constexpr bool HALF_IN = FIRST && HIN;
    static_assert(L % (NS * RAD) == 0, "radix schedule");
    using XOut = Exchange<R, NS, RAD>;
    static_assert(FIRST || STRIDE % 8 == 0, "later passes read at multiples of 8");
    static_assert(LAST || RAD >= 8, "exchange layouts are for passes of radix 8 and 16");
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int j = g + GT * u;
        const int pj = XIn::slot(j);
#pragma unroll
        for (int r = 0; r < RAD; ++r) {
            if constexpr (FIRST) {
                // positions j + r STRIDE >= L/2 exactly when r >= RAD/2
                if constexpr (HALF_IN) {
                    if (r >= RAD / 2) {
                        v[u * RAD + r] = {R(0), R(0)};
                        continue;
                    }
                }
                if constexpr (!PRE) v[u * RAD + r] = load(j + r * STRIDE);
            } else {
                v[u * RAD + r] = sh[pj + XIn::slot(r * STRIDE)];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        if constexpr (NS > 1) {
#pragma unroll
            for (int r = 1; r < RAD; ++r) {
                cpx<R> t = w[OFF + u * (RAD - 1) + r - 1];
                if (INV) t.y = -t.y;
                v[u * RAD + r] = cmul(v[u * RAD + r], t);
            }
        }
        if constexpr (HALF_IN) dft_half_in<R, RAD, INV>(&v[u * RAD]);
        else dft<R, RAD, INV>(&v[u * RAD]);
    }
    if constexpr (!FIRST) wave_sync();
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        const int j = g + GT * u;
        const int k = j & (NS - 1);
        const int base = (j - k) * RAD + k;
        const int pb = XOut::slot(base);
#pragma unroll
        for (int r = 0; r < RAD; ++r) {
            if constexpr (LAST) {
                // positions base + r NS >= L/2 exactly when r >= RAD/2
                if (!HOUT || r < RAD / 2) store(base + r * NS, v[u * RAD + r]);
            } else {
                sh[pb + XOut::slot(r * NS)] = v[u * RAD + r];
            }
        }
    }
    if constexpr (!LAST) {
        wave_sync();
        constexpr int here = NS > 1 ? NB * (RAD - 1) : 0;
        fft_pass<R, L, V, INV, P::NEXT, OFF + here, false, false, HOUT, XOut>(v, sh, g, w, load, store);
    }
}

// The values a lane reads in the first pass, in register order, so that the
// input of several transforms can be requested before any of them starts
// (HIN: the zero upper half is not requested).
template <typename R, int L, bool HIN = false, int V, class Load>
__device__ __forceinline__ void fft_first_loads(cpx<R> (&v)[V], int g, Load load)
{
    constexpr int GT = L / V;
    using P = PassShape<L, V, 1>;
    constexpr int STRIDE = L / P::RAD;
#pragma unroll
    for (int u = 0; u < P::NB; ++u)
#pragma unroll
        for (int r = 0; r < P::RAD; ++r)
            v[u * P::RAD + r] = (HIN && r >= P::RAD / 2) ? cpx<R>{R(0), R(0)}
                                                           : load(g + GT * u + r * STRIDE);
}

// One transform whose first-pass values are already in v (fft_first_loads).
// sh: the group's LDS region of fft_region(L) values.
template <typename R, int L, bool INV, bool HIN = false, bool HOUT = false, int V, class Store>
__device__ __forceinline__ void wave_fft_pre(cpx<R>* sh, int g, const Twiddles<R, L, V>& tw,
                                             cpx<R> (&v)[V], Store store)
{
    static_assert(L / V <= 64, "one transform must fit in a wavefront");
    auto none = [](int) { return cpx<R>{R(0), R(0)}; };
    fft_pass<R, L, V, INV, 1, 0, true, HIN, HOUT>(v, sh, g, tw.w, none, store);
}

// One transform with preloaded twiddles.
template <typename R, int L, bool INV, bool HIN = false, bool HOUT = false, int V, class Load, class Store>
__device__ __forceinline__ void wave_fft(cpx<R>* sh, int g, const Twiddles<R, L, V>& tw, Load load,
                                         Store store)
{
    static_assert(L / V <= 64, "one transform must fit in a wavefront");
    cpx<R> v[V];
    fft_pass<R, L, V, INV, 1, 0, false, HIN, HOUT>(v, sh, g, tw.w, load, store);
}

// One transform loading its own twiddles (single-use callers).
template <typename R, int L, bool INV, bool HIN = false, bool HOUT = false, class Load, class Store>
__device__ __forceinline__ void wave_fft(cpx<R>* sh, int g, const cpx<R>* __restrict__ tw, int tws,
                                         Load load, Store store)
{
    Twiddles<R, L> t;
    t.load(g, tw, tws);
    wave_fft<R, L, INV, HIN, HOUT>(sh, g, t, load, store);
}

}  // namespace hfd
