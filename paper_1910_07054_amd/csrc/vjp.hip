// Thickness gradient of L = <g, h(m)> (h = -N * m) for every state.
//
// With T^{ij} = -DFT2(N^{ij}) / (Lx Ly) the field is H_i = sum_j T^{ij} M_j and
//   L = sum_k sum_{ij} conj(G_i(k)) . T^{ij}(k) M_j(k)   (full Lx x Ly grid),
// G, M the 2D DFTs of the zero-padded g and m.  N^{ij} depends on the four
// interfaces bot_i, top_i (target) and bot_j, top_j (source) through
// N = -1/(4 pi dx dy t_i) sum_c s_c Psi(zeta_c), zeta = {top_i - bot_j,
// bot_i - bot_j, top_i - top_j, bot_i - top_j}, s = {+1, -1, -1, +1}, Psi the
// lateral-stencilled Phi.  The sign s_c factors into a target sign (+1 top,
// -1 bottom) times a source sign (+1 bottom, -1 top), so with K(zeta) the
// normalized DFT of -Psi/(4 pi dx dy) and, per interface e of layer l,
//   Ghat_e = +-G_l / t_l (+ top, - bottom),  Mhat_e = -+M_l (- top, + bottom),
// the functional is a sum over interface pairs:
//   L = sum_{e,f} Re conj(Ghat_e) . K(z_e - z_f) Mhat_f.
// Interfaces that coincide (top_l touching bot_{l+1}) move together under
// every thickness change (gaps are fixed), so they are merged into one
// position p with summed Ghat_p, Mhat_p.  Moving position p alone changes L by
//   dL/dz_p = sum_q [P(p, q) - P(q, p)] + (1/t terms),
//   P(p, q) = Re conj(Ghat_p) . D(z_p - z_q) Mhat_q,
// D = dK/dzeta the normalized DFT of -1/(4 pi dx dy) dPsi/dz.  The 1/t_l
// factor of Ghat adds -L_l / t_l to the top of layer l and +L_l / t_l to its
// bottom, L_l = sum_j Re conj(G_l) . T^{lj} M_j the layer's share of L.
// In the rotated components (X, sg Y, iZ) (sg = -1 for ky < 0) D(zeta) is a real
// 3x3 matrix K per frequency and D(-zeta) is -K^T, so for z_p > z_q the pair's
// contribution is one number,
//   s = P(p, q) - P(q, p) = Ghat_p . (K Mhat_q) + Mhat_p . (K Ghat_q),
// added to p and subtracted from q (dot products over real and imaginary
// parts).  The stored tensor blocks S^{lj} = t_l T^{lj} are real in these components as
// well and S^{jl} is the transpose: S M_j and S G_j of a pair l <= j give its part
// of L_l and of L_j.  Each D and each S is read once per frequency, where a sum
// over ordered layer pairs and their four offsets reads D up to eight times.
// The half spectrum holds
// kx in [1, M) once (weight 2, the mirror -kx is the complex conjugate) and
// the packed column 0 carries kx = 0 and kx = Lx/2 (weight 1 each).
// Position p has rank r_p (r = l for bot_l, l + 1 for top_l) and
// dz_p/dt_k = [k < r_p].  D is stored for |zeta| only: dPsi/dz is odd in zeta
// for xx, yy, zz, xy and even for xz, yz, so D(-zeta) is D(zeta) with the
// first four negated (the table entry of a pair carries the sign).
#include "derivative_sizes.hpp"
#include "field_kernels.hpp"
#include "launch.hpp"

namespace hfd {

namespace {

// sum over the 64 lanes, the same bits in every lane (xor butterfly)
__device__ inline double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Re conj(g) . A m for the symmetric block A with real xx, yy, zz, xy and
// imaginary i xz, i yz entries; g, m = (re, im) x 3, arithmetic in double.
template <typename T>
__device__ inline double gAm(const double g[6], double xx, double yy, double zz, double xy,
                             double xz, double yz, const T mm[6])
{
    const double m[6] = {mm[0], mm[1], mm[2], mm[3], mm[4], mm[5]};
    const double vxr = xx * m[0] + xy * m[2] - xz * m[5];
    const double vxi = xx * m[1] + xy * m[3] + xz * m[4];
    const double vyr = xy * m[0] + yy * m[2] - yz * m[5];
    const double vyi = xy * m[1] + yy * m[3] + yz * m[4];
    const double vzr = zz * m[4] - xz * m[1] - yz * m[3];
    const double vzi = zz * m[5] + xz * m[0] + yz * m[2];
    return g[0] * vxr + g[1] * vxi + g[2] * vyr + g[3] * vyi + g[4] * vzr + g[5] * vzi;
}

// v = A m for a real block A = [[xx, xy, xz], [xy, yy, yz], [-xz, -yz, zz]] on the real and the
// imaginary parts of m (re, im of the three components), then g . v
__device__ __forceinline__ double dot_block(const double (&g)[6], double xx, double yy, double zz,
                                            double xy, double xz, double yz, const double (&m)[6])
{
    double s = 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const double X = m[h], Y = m[2 + h], Z = m[4 + h];
        s = fma(g[h], fma(xz, Z, fma(xy, Y, xx * X)), s);
        s = fma(g[2 + h], fma(yz, Z, fma(yy, Y, xy * X)), s);
        s = fma(g[4 + h], fma(-xz, X, fma(-yz, Y, zz * Z)), s);
    }
    return s;
}

}  // namespace

template <typename R>
struct alignas(4 * sizeof(R)) MG {
    cpx<R> m, g;
};

// One block per (state, kx, 32 lateral frequency pairs): lanes l and 32 + l of
// every wave take ky = t and LY - t (t = 0: ky = 0 and LY/2), which share every
// quadrant value of D and S; in the packed column lane p = 0 takes A(t) with row
// kx = 0 and lane p = 1 B(t) with row kx = M; the self-mirrored points t = 0 take
// A there, and B in an extra tile of their own.
// The tile's M and G spectra (rotated; in the packed column as they are, A and B
// are formed in FP64 where they are used) are staged in LDS and shared by the
// block's waves (1, 2 or 4), which take groups of QC source positions and of QC
// layers in turn: a group's spectra stay in registers (FP64) while the wave
// walks the positions above them, or the layers up to them, with the next one's
// D or S entries in flight.  The groups are dealt to `shares` (4, or 2 where 4 do not
// fit in LDS), each with per-position sums of its own in LDS, added up over shares and
// lanes at the end in a fixed order; a wave takes one share (ONE) or several, one after
// the other, so that the result does not depend on the waves per block.
// Block order: groups of 8 tiles, within a group every state of the launch,
// with the 8 tiles on consecutive block indices: the states of one tile are 8
// indices apart, so they run one after the other on one XCD and read that
// tile's slice of the offset table D (shared by every stack when stored) and
// of the tensor table through its L2.
// Bound by FP64 arithmetic: per tile 5 k fused multiply-adds of the products and
// 3.5 k conversions and sums.  16 states of 256 x 256 x 10: 1390 -> 1060 us (306 M
// vector instructions, 0.7 ms of issue; 2.4 GB fetched instead of 6.9), one state
// 64 x 64 x 3 in FP64 42 -> 16 us.  Groups of 2 take 1270 us (the conversions of the walked
// position are shared by fewer products), of 4 as much as of 3 (two blocks of 4 waves
// per CU either way).
// itab per geometry: see itab_layout.  D per geometry: [QX][nzt][6][QY], nzt D slots per row.
// lp per geometry: 1/t_l, then the trace term of the diagonal blocks.
// partial[b][2nz][tile]: the tile's position gradients.
template <typename R, bool ONE>
__global__ __launch_bounds__(256, 2) void k_tgrad(
    const cpx<R>* __restrict__ Mh, const cpx<R>* __restrict__ Gh, int nz, int M, int LY,
    const R* __restrict__ Q, long long qcs, const int* __restrict__ qslot, const R* __restrict__ D, int nzt,
    const int* __restrict__ itab, int itab_stride, const R* __restrict__ lp, int bpg, int QY, int b0, int nst,
    int ntiles, int nshare, double* __restrict__ partial)
{
    constexpr int QC = 3;
    const int L = blockIdx.x, r8 = L >> 3;
    const int tg = __builtin_amdgcn_readfirstlane(r8 / nst);
    const int slot = tg * 8 + (L & 7);
    if (slot >= ntiles) return;
    // the last tile: the self-mirrored points of the packed column with row kx = M
    const bool mirror = slot == ntiles - 1;
    const int tile = mirror ? 0 : slot;
    const int b = b0 + r8 - tg * nst;
    const int geom = __builtin_amdgcn_readfirstlane(b / bpg);
    const int half = LY >> 1, tpk = (half + 31) >> 5;
    const int kx = __builtin_amdgcn_readfirstlane(tile / tpk), kyb = tile - kx * tpk;
    const int lane = threadIdx.x & 63, W = blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), shares = ONE ? W : nshare;
    const int t0 = kyb * 32 + (lane & 31), p2 = lane >> 5;
    const bool active = t0 < half;
    const int t = active ? t0 : 0;
    const int ky = p2 == 0 ? t : (t == 0 ? half : LY - t);
    const int kq = p2 == 0 ? t : (t == 0 ? half : t);
    const bool packed = kx == 0;
    const R sg = (!packed && p2 == 1 && t != 0) ? R(-1) : R(1);
    // half spectrum: kx and -kx; packed column: ky and -ky except the self-mirrored points
    const double weight = !active || (mirror && t != 0) ? 0.0 : (packed && t == 0 ? 1.0 : 2.0);
    const int S3 = 3 * nz;
    const long long sst = (long long)M * LY;
    const cpx<R>* mb = Mh + ((long long)b * S3 * M + kx) * LY + ky;
    const cpx<R>* gb = Gh + ((long long)b * S3 * M + kx) * LY + ky;
    const int* sl = qslot + (long long)geom * (nz * (nz + 1) / 2);  // the stack's pair slots
    const R* lpg = lp + (long long)geom * 2 * nz;
    const int* it = itab + (long long)geom * itab_stride;
    const ITabLayout lay = itab_layout(nz);
    const int NI = it[0];
    const int* pinfo = it + lay.info;
    const int* pbot = it + lay.pbot;
    const int* ptop = it + lay.ptop;
    const int* zpq = it + lay.zpq;
    const long long drow = (long long)nzt * 6 * QY;
    const int trow = tab_row(kx, M);
    const UniformBuf<R> dbuf(D + (long long)trow * drow,
                             (unsigned)((packed ? 2 : 1) * drow * sizeof(R)));
    const UniformBuf<R> qbuf(Q + (long long)trow * qcs,
                             (unsigned)((packed ? 2 : 1) * qcs * sizeof(R)));

    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* acc0 = reinterpret_cast<double*>(smem_raw) + lane;  // [shares][NI][64]
    // (M, G) of component c, layer l: [nz][3][64]
    MG<R>* sm = reinterpret_cast<MG<R>*>(smem_raw + sizeof(double) * 64 * (size_t)shares * NI) + lane;
    for (int v = w; v < shares * NI; v += W) acc0[v * 64] = 0.0;

    const bool rowM = packed && ((p2 == 1 && t != 0) || mirror);
    const unsigned vd = (unsigned)(kq + (rowM ? drow : 0LL)), vq = (unsigned)(kq + (rowM ? qcs : 0LL));
    // three layers per wave at a time, all 18 values requested together
    for (int l0 = w * 3; l0 < nz; l0 += W * 3) {
        cpx<R> zm[3][3], zg[3][3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int s = c * nz + (l0 + k < nz ? l0 + k : nz - 1);
                zm[k][c] = mb[s * sst];
                zg[k][c] = gb[s * sst];
            }
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                cpx<R> vm = zm[k][c], vg = zg[k][c];
                if (!packed) {
                    if (c == 1) { vm = cscale(vm, sg); vg = cscale(vg, sg); }
                    if (c == 2) { vm = {-vm.y, vm.x}; vg = {-vg.y, vg.x}; }
                }
                if (l0 + k < nz) sm[((l0 + k) * 3 + c) * 64] = {vm, vg};
            }
    }
    __syncthreads();
    auto sweep = [&](auto column) {
        constexpr bool PACKED = decltype(column)::value;
        // layer l's spectra
        auto layer = [&](int l, double (&m)[6], double (&g)[6]) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const MG<R> v = sm[(l * 3 + c) * 64];
                m[2 * c] = v.m.x;
                m[2 * c + 1] = v.m.y;
                g[2 * c] = v.g.x;
                g[2 * c + 1] = v.g.y;
                if constexpr (PACKED) {
                    // A(t) = (Z(t) + conj Z(-t)) / 2 on lane 0, B(t) = (Z(t) - conj Z(-t)) / (2i) on lane 1;
                    // the self-mirrored points take A, then B
                    const MG<R> o = sm[(l * 3 + c) * 64 + (p2 == 0 ? 32 : -32)];
                    auto part = [&](cpx<R> z, cpx<R> n, double& x, double& y) {
                        if (t == 0) {
                            x = mirror ? z.y : z.x;
                            y = 0.0;
                        } else {
                            const double re = p2 == 0 ? (double)z.x + n.x : (double)n.y + z.y;
                            const double im = p2 == 0 ? (double)z.y - n.y : (double)z.x - n.x;
                            x = 0.5 * re;
                            y = 0.5 * im;
                        }
                        if (c == 2) {
                            const double r = x;
                            x = -y;
                            y = r;
                        }
                    };
                    part(v.m, o.m, m[2 * c], m[2 * c + 1]);
                    part(v.g, o.g, g[2 * c], g[2 * c + 1]);
                }
            }
        };
        // position p: Mhat = -M (top of rk - 1) + M (bottom of rk) in plan precision,
        // Ghat = G / t - G / t in FP64
        auto position = [&](int p, double (&m)[6], double (&g)[6]) {
            const int info = pinfo[p], rk = info >> 2;
            const int la = (info & 1) ? rk - 1 : rk, lb = (info & 2) ? rk : rk - 1;
            const R sa = (info & 1) ? R(-1) : R(0), sb = (info & 2) ? R(1) : R(0);
            const double wa = -(double)sa * (double)lpg[la], wb = -(double)sb * (double)lpg[lb];
            if constexpr (PACKED) {
                double ma[6], ga[6];
                layer(la, ma, ga);
                layer(lb, m, g);
#pragma unroll
                for (int c = 0; c < 6; ++c) {
                    m[c] = (R)((double)sa * ma[c] + (double)sb * m[c]);
                    g[c] = wa * ga[c] + wb * g[c];
                }
            } else if ((info & 3) == 3) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const MG<R> x = sm[(la * 3 + c) * 64], y = sm[(lb * 3 + c) * 64];
                    m[2 * c] = y.m.x - x.m.x;
                    m[2 * c + 1] = y.m.y - x.m.y;
                    g[2 * c] = fma(wa, (double)x.g.x, wb * (double)y.g.x);
                    g[2 * c + 1] = fma(wa, (double)x.g.y, wb * (double)y.g.y);
                }
            } else {
                const R sm1 = sa + sb;
                const double w1 = (info & 1) ? wa : wb;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const MG<R> x = sm[(la * 3 + c) * 64];
                    m[2 * c] = sm1 * x.m.x;
                    m[2 * c + 1] = sm1 * x.m.y;
                    g[2 * c] = w1 * (double)x.g.x;
                    g[2 * c + 1] = w1 * (double)x.g.y;
                }
            }
        };
        // groups u = 0, 1, .. of source positions from the lowest and of layers from the
        // highest, both by falling cost, dealt to the shares in turn and back
        const int ni = (NI + QC - 1) / QC, nl = (nz + QC - 1) / QC;
        for (int q = 0; q == 0 || (!ONE && q * W < shares); ++q)
        for (int r = 0; r * shares < 2 * (ni > nl ? ni : nl); ++r) {
            // this wave's share (two of four: w and 3 - w, which even out)
            const int h = (q & 1) ? (q + 1) * W - 1 - w : q * W + w;
            double* accw = acc0 + (size_t)h * NI * 64;
            const int e = r * shares + ((r & 1) ? shares - 1 - h : h), u = e >> 1;
            if ((e & 1) == 0) {
                if (u >= ni) continue;
                // source positions q0 .. q0 + QC - 1 against the positions above them
                const int q0 = u * QC;
                double mq[QC][6], gq[QC][6], aq[QC];
#pragma unroll
                for (int k = 0; k < QC; ++k) {
                    position(q0 + k < NI ? q0 + k : NI - 1, mq[k], gq[k]);
                    aq[k] = 0.0;
                }
                int sn[QC];   // table entries of the position to fetch next
                auto slots = [&](int p) {
#pragma unroll
                    for (int k = 0; k < QC; ++k)
                        sn[k] = zpq[(p < NI ? p : NI - 1) * lay.nsp + (q0 + k < NI ? q0 + k : NI - 1)];
                };
                auto fetch = [&](int p, R (&d)[QC][6]) {
#pragma unroll
                    for (int k = 0; k < QC; ++k)
#pragma unroll
                        for (int c = 0; c < 6; ++c) d[k][c] = dbuf.ld(vd, (unsigned)(((sn[k] >> 1) * 6 + c) * QY));
                    slots(p + 1);
                };
                auto apply = [&](int p, const R (&d)[QC][6]) {
                    double mp[6], gp[6], sp = 0.0;
                    position(p, mp, gp);
#pragma unroll
                    for (int k = 0; k < QC; ++k)
                        if (q0 + k < p) {
                            const double xx = d[k][0], yy = d[k][1], zz = d[k][2], xy = d[k][3], xz = d[k][4],
                                         yz = d[k][5];
                            const double s = dot_block(gp, xx, yy, zz, xy, xz, yz, mq[k]) +
                                             dot_block(mp, xx, yy, zz, xy, xz, yz, gq[k]);
                            sp += s;
                            aq[k] -= s;
                        }
                    accw[p * 64] += sp;
                };
                R d0[QC][6], d1[QC][6];
                slots(q0 + 1);
                fetch(q0 + 1, d0);
                for (int p = q0 + 1; p < NI; p += 2) {
                    fetch(p + 1, d1);
                    apply(p, d0);
                    if (p + 1 >= NI) break;
                    fetch(p + 2, d0);
                    apply(p + 1, d1);
                }
#pragma unroll
                for (int k = 0; k < QC; ++k)
                    if (q0 + k < NI) accw[(q0 + k) * 64] += aq[k];
            } else {
                if (u >= nl) continue;
                // the 1/t_l factor: top_l gets -L_l / t_l, bot_l gets +L_l / t_l; layers j0 .. j0 + QC - 1
                // against the layers up to them (the lowest group may reach below layer 0)
                const int j0 = nz - (u + 1) * QC, jn = j0 + QC;
                double mj[QC][6], gj[QC][6], aj[QC];
#pragma unroll
                for (int k = 0; k < QC; ++k) {
                    layer(j0 + k > 0 ? j0 + k : 0, mj[k], gj[k]);
                    if constexpr (PACKED)
#pragma unroll
                        for (int c = 0; c < 6; ++c) mj[k][c] = (R)mj[k][c];
                    aj[k] = 0.0;
                }
                int sn[QC];   // slots of the layer to fetch next
                auto slots = [&](int l) {
#pragma unroll
                    for (int k = 0; k < QC; ++k) {
                        const int j = j0 + k > 0 ? j0 + k : 0, a = l < j ? l : j;
                        sn[k] = sl[a * nz - a * (a - 1) / 2 + (j - a)];
                    }
                };
                auto fetch = [&](int l, R (&d)[QC][5]) {
#pragma unroll
                    for (int k = 0; k < QC; ++k)
#pragma unroll
                        for (int c = 0; c < 5; ++c) d[k][c] = qbuf.ld(vq, (unsigned)((sn[k] * 5 + c) * QY));
                    slots(l + 1);
                };
                auto add = [&](int l, double v) {
                    const double f = (double)lpg[l] * (double)lpg[l] * v;
                    accw[ptop[l] * 64] -= f;
                    accw[pbot[l] * 64] += f;
                };
                auto apply = [&](int l, const R (&d)[QC][5]) {
                    double ml[6], gl[6], x = 0.0;
                    layer(l, ml, gl);
                    if constexpr (PACKED)
#pragma unroll
                        for (int c = 0; c < 6; ++c) ml[c] = (R)ml[c];
#pragma unroll
                    for (int k = 0; k < QC; ++k) {
                        const int j = j0 + k;
                        if (j >= l) {
                            const double xx = d[k][0], yy = d[k][1], xy = d[k][2], xz = d[k][3], yz = d[k][4];
                            const double zz = -(xx + yy) + (l == j ? (double)lpg[nz + l] : 0.0);
                            x += dot_block(gl, xx, yy, zz, xy, xz, yz, mj[k]);
                            if (j > l) aj[k] += dot_block(ml, xx, yy, zz, xy, xz, yz, gj[k]);
                        }
                    }
                    add(l, x);
                };
                R d0[QC][5], d1[QC][5];
                slots(0);
                fetch(0, d0);
                for (int l = 0; l < jn; l += 2) {
                    fetch(l + 1, d1);
                    apply(l, d0);
                    if (l + 1 >= jn) break;
                    fetch(l + 2, d0);
                    apply(l + 1, d1);
                }
#pragma unroll
                for (int k = 0; k < QC; ++k)
                    if (j0 + k >= 0) add(j0 + k, aj[k]);
            }
        }
    };
    if (packed) sweep(std::true_type{});
    else sweep(std::false_type{});
    __syncthreads();
    double* out = partial + (long long)b * 2 * nz * ntiles + slot;
    for (int v = w; v < NI; v += W) {
        double sv = 0.0;
        for (int k = 0; k < shares; ++k) sv += acc0[(size_t)(k * NI + v) * 64];
        sv = wave_sum(sv * weight);
        if (lane == 0) out[(long long)v * ntiles] = sv;
    }
}

// four consecutive table entries from a 16-byte aligned address
__device__ inline void load_chunk(const int* __restrict__ src, int (&dst)[4])
{
    const int4 a = *reinterpret_cast<const int4*>(src);
    dst[0] = a.x;
    dst[1] = a.y;
    dst[2] = a.z;
    dst[3] = a.w;
}

// Stacks whose spectra do not fit in LDS: per-position gradient sums of one wave
// over its 64 frequencies of row kx
// (PACKED: the packed column, rows 0 and M from the unpacked pair A, B).
// Sources (interface positions, then layers) are taken in chunks of QC held
// in registers; for each target the loads of the next target are issued
// before the arithmetic of the current one (software pipelining), and no
// load sits behind a branch: the two layers of a position are always read
// (clamped index, weight 0 when absent), source slots past the end read a
// valid slot against a zero source.
template <typename R, int QC, bool PACKED>
__device__ inline void tgrad_row(const cpx<R>* __restrict__ mb, const cpx<R>* __restrict__ gb,
                                 long long sst, int nz, int M, int kx, int ky, int kyn, int kq,
                                 double sgy, double wgt0, const R* __restrict__ Q, long long qcs,
                                 const int* __restrict__ sl, const R* __restrict__ Dg, int nzt,
                                 const int* __restrict__ it,
                                 const R* __restrict__ lpg, int QY, double* __restrict__ acc)
{
    constexpr int NV = PACKED ? 2 : 1;  // raw spectrum values per entry (ky, and LY - ky)
    const int lane = threadIdx.x;
    const ITabLayout lay = itab_layout(nz);
    const int NI = it[0];
    const int* pinfo = it + lay.info;
    const int* pbot = it + lay.pbot;
    const int* ptop = it + lay.ptop;
    const int* zpq = it + lay.zpq;
    // acc[v][64]: lane-owned partial sums of position v (LDS, fire-and-forget adds)
    auto add_out = [&](int v, double val) { atomicAdd(&acc[v * 64 + lane], val); };
    for (int ps = 0; ps < NV; ++ps) {
        const int row = PACKED ? (ps ? M : 0) : kx;
        // rows of D ([QX][nzt][6][QY]) and of the tensor table ([QX][slots][5][QY])
        // as buffers: the lane offset is kq, the slot and component offsets are scalar
        const int trow = tab_row(row, M);
        const UniformBuf<R> dbuf(Dg + (long long)trow * nzt * 6 * QY, (unsigned)(nzt * 6 * QY * sizeof(R)));
        const UniformBuf<R> qbuf(Q + (long long)trow * qcs, (unsigned)(qcs * sizeof(R)));
        // component c of layer l: raw loads, then (re, im) at this point
        auto raw = [&](const cpx<R>* base, int c, int l, cpx<R> (&z)[NV]) {
            z[0] = base[(c * nz + l) * sst + ky];
            if (PACKED) z[NV - 1] = base[(c * nz + l) * sst + kyn];
        };
        auto comb = [&](const cpx<R> (&z)[NV], double& re, double& im) {
            if (!PACKED) {
                re = z[0].x;
                im = z[0].y;
            } else {
                const cpx<R> z1 = z[0], z2 = z[NV - 1];
                const double ar = 0.5 * ((double)z1.x + z2.x), ai = 0.5 * ((double)z1.y - z2.y);
                const double br = 0.5 * ((double)z1.y + z2.y), bi = 0.5 * ((double)z2.x - z1.x);
                re = ps ? br : ar;
                im = ps ? bi : ai;
            }
        };
        // ---- interface pairs ------------------------------------------------
        struct PosLoads {
            R d[QC][6];
            cpx<R> g[2][3][NV];
            int zi[QC];
        };
        for (int qc = 0; qc < NI; qc += QC) {
            R mh[QC][6];  // Mhat in plan precision
            {
                int pi[QC];
                load_chunk(pinfo + qc, pi);
                cpx<R> zm[QC][2][3][NV];
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const int rk = pi[q] >> 2;
                    const int la = rk > 0 ? rk - 1 : 0, lb = rk < nz ? rk : nz - 1;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        raw(mb, c, la, zm[q][0][c]);
                        raw(mb, c, lb, zm[q][1][c]);
                    }
                }
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const bool live = qc + q < NI;
                    const int info = pi[q];
                    const double wa = live && (info & 1) ? -1.0 : 0.0;  // top of rk - 1: -M
                    const double wb = live && (info & 2) ? 1.0 : 0.0;   // bottom of rk: +M
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        double ra, ia, rb, ib;
                        comb(zm[q][0][c], ra, ia);
                        comb(zm[q][1][c], rb, ib);
                        mh[q][2 * c] = (R)(wa * ra + wb * rb);
                        mh[q][2 * c + 1] = (R)(wa * ia + wb * ib);
                    }
                }
            }
            auto fetch = [&](int p, PosLoads& f) {
                const int rk = pinfo[p] >> 2;
                const int la = rk > 0 ? rk - 1 : 0, lb = rk < nz ? rk : nz - 1;
                load_chunk(zpq + p * lay.nsp + qc, f.zi);
#pragma unroll
                for (int q = 0; q < QC; ++q)
#pragma unroll
                    for (int c = 0; c < 6; ++c)
                        f.d[q][c] = dbuf.ld(kq, (unsigned)(((f.zi[q] >> 1) * 6 + c) * QY));
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    raw(gb, c, la, f.g[0][c]);
                    raw(gb, c, lb, f.g[1][c]);
                }
            };
            double gq[QC];
#pragma unroll
            for (int q = 0; q < QC; ++q) gq[q] = 0.0;
            PosLoads nxt;
            fetch(0, nxt);
            for (int p = 0; p < NI; ++p) {
                const PosLoads cur = nxt;
                if (p + 1 < NI) fetch(p + 1, nxt);
                const int info = pinfo[p], rk = info >> 2;
                const int la = rk > 0 ? rk - 1 : 0, lb = rk < nz ? rk : nz - 1;
                // top of rk - 1: +G / t; bottom of rk: -G / t (lp holds 1/t)
                const double wa = (info & 1) ? wgt0 * (double)lpg[la] : 0.0;
                const double wb = (info & 2) ? -wgt0 * (double)lpg[lb] : 0.0;
                double gh[6];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double ra, ia, rb, ib;
                    comb(cur.g[0][c], ra, ia);
                    comb(cur.g[1][c], rb, ib);
                    gh[2 * c] = wa * ra + wb * rb;
                    gh[2 * c + 1] = wa * ia + wb * ib;
                }
                double ga = 0.0;
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const R* d = cur.d[q];
                    // z_p < z_q: D(-zeta) = D(zeta) with xx, yy, zz, xy negated
                    const double sz = (cur.zi[q] & 1) ? -1.0 : 1.0;
                    const double pd = gAm(gh, sz * d[0], sz * d[1], sz * d[2], sz * sgy * (double)d[3],
                                          d[4], sgy * (double)d[5], mh[q]);
                    ga += pd;
                    gq[q] -= pd;
                }
                add_out(p, ga);
            }
#pragma unroll
            for (int q = 0; q < QC; ++q)
                if (qc + q < NI) add_out(qc + q, gq[q]);
        }
        // ---- the 1/t_l factor ----------------------------------------------
        // top_l gets -L_l / t_l, bot_l gets +L_l / t_l, L_l = sum_j
        // Re conj(G_l) . T^{lj} M_j; the stored blocks are t_l T^{lj}
        struct LayerLoads {
            R a[QC][5];
            cpx<R> g[3][NV];
        };
        for (int jc = 0; jc < nz; jc += QC) {
            R mj[QC][6];
            {
                cpx<R> zm[QC][3][NV];
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const int j = jc + q < nz ? jc + q : nz - 1;
#pragma unroll
                    for (int c = 0; c < 3; ++c) raw(mb, c, j, zm[q][c]);
                }
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const double w = jc + q < nz ? 1.0 : 0.0;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        double re, im;
                        comb(zm[q][c], re, im);
                        mj[q][2 * c] = (R)(w * re);
                        mj[q][2 * c + 1] = (R)(w * im);
                    }
                }
            }
            auto fetch = [&](int l, LayerLoads& f) {
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const int j = jc + q < nz ? jc + q : nz - 1;
                    const int a = l < j ? l : j, bq = l < j ? j : l;
                    const int slot = sl[a * nz - a * (a - 1) / 2 + (bq - a)];
#pragma unroll
                    for (int c = 0; c < 5; ++c) f.a[q][c] = qbuf.ld(kq, (unsigned)((slot * 5 + c) * QY));
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) raw(gb, c, l, f.g[c]);
            };
            LayerLoads nxt;
            fetch(0, nxt);
            for (int l = 0; l < nz; ++l) {
                const LayerLoads cur = nxt;
                if (l + 1 < nz) fetch(l + 1, nxt);
                const double it_l = lpg[l];  // lp holds 1/t
                const double w = wgt0 * it_l * it_l;
                const double trace = lpg[nz + l];
                double g6[6];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double re, im;
                    comb(cur.g[c], re, im);
                    g6[2 * c] = w * re;
                    g6[2 * c + 1] = w * im;
                }
                double sl = 0.0;
#pragma unroll
                for (int q = 0; q < QC; ++q) {
                    const int j = jc + q;
                    const double simag = l <= j ? 1.0 : -1.0;
                    const double xx = cur.a[q][0], yy = cur.a[q][1];
                    const double zz = -(xx + yy) + (l == j ? trace : 0.0);
                    sl += gAm(g6, xx, yy, zz, sgy * (double)cur.a[q][2], simag * (double)cur.a[q][3],
                              simag * sgy * (double)cur.a[q][4], mj[q]);
                }
                add_out(ptop[l], -sl);
                add_out(pbot[l], sl);
            }
        }
    }
}

// One wave per (state, kx, 32 lateral frequency pairs): lanes 2s and 2s+1 take
// ky = t and LY - t (t = ty*32 + s; lane 2s+1 of t = 0 takes ky = LY/2), which
// share every quadrant value of D and Q.  Each lane accumulates its own
// per-position sums in LDS; the block sums them over the lanes at the end.
// Block order and arguments as k_tgrad.
template <typename R, int QC>
__global__ __launch_bounds__(64) void k_tgrad_rows(const cpx<R>* __restrict__ Mh,
                                              const cpx<R>* __restrict__ Gh, int nz, int M, int LY,
                                              const R* __restrict__ Q, long long qcs,
                                              const int* __restrict__ qslot,
                                              const R* __restrict__ D, int nzt,
                                              const int* __restrict__ itab, int itab_stride,
                                              const R* __restrict__ lp, int bpg,
                                              int QY, int b0, int nst, int ntiles,
                                              double* __restrict__ partial)
{
    const int L = blockIdx.x, r8 = L >> 3;
    const int tile = (r8 / nst) * 8 + (L & 7);
    if (tile >= ntiles) return;
    const int b = b0 + r8 % nst;
    const int geom = b / bpg;
    const int half = LY >> 1;
    const int tpk = (half + 31) >> 5;
    const int kx = tile / tpk, ty = tile - kx * tpk;
    const int lane = threadIdx.x;
    const int t0 = ty * 32 + (lane >> 1);
    const bool active = t0 < half;
    const int t = active ? t0 : 0;
    const int ky = (lane & 1) == 0 ? t : (t == 0 ? half : LY - t);
    const int kq = ky <= half ? ky : LY - ky;
    const double sgy = ky <= half ? 1.0 : -1.0;
    const int kyn = (LY - ky) & (LY - 1);
    const int S = 3 * nz;
    const long long sst = (long long)M * LY;
    const cpx<R>* mb = Mh + ((long long)b * S * M + kx) * LY;
    const cpx<R>* gb = Gh + ((long long)b * S * M + kx) * LY;
    const int* sl = qslot + (long long)geom * (nz * (nz + 1) / 2);  // the stack's pair slots
    const R* lpg = lp + (long long)geom * 2 * nz;
    const int* it = itab + (long long)geom * itab_stride;
    const int NI = it[0], NS = 2 * nz;
    extern __shared__ double acc[];  // [NI][64]
    for (int v = 0; v < NI; ++v) acc[v * 64 + lane] = 0.0;
    if (kx == 0)
        tgrad_row<R, QC, true>(mb, gb, sst, nz, M, kx, ky, kyn, kq, sgy, active ? 1.0 : 0.0, Q, qcs,
                               sl, D, nzt, it, lpg, QY, acc);
    else
        tgrad_row<R, QC, false>(mb, gb, sst, nz, M, kx, ky, kyn, kq, sgy, active ? 2.0 : 0.0, Q,
                                qcs, sl, D, nzt, it, lpg, QY, acc);
    __syncthreads();
    double* out = partial + (long long)b * NS * (ntiles + 1) + tile;
    for (int v = 0; v < NI; ++v) {
        const double sv = wave_sum(acc[v * 64 + lane]);
        if (lane == 0) {
            out[(long long)v * (ntiles + 1)] = sv;
            // (k_tgrad's extra tile: its points are in tile 0 here)
            if (tile == 0) out[(long long)v * (ntiles + 1) + ntiles] = 0.0;
        }
    }
}

// Sum the tile partials of each position (fixed order) and apply the stacking
// chain rule dL/dt_k = sum_p [k < r_p] dL/dz_p.
__global__ __launch_bounds__(1024) void k_tgrad_finish(const double* __restrict__ partial, int nparts,
                                                       int nz, const int* __restrict__ itab,
                                                       int itab_stride, int bpg,
                                                       double* __restrict__ grad_t)
{
    __shared__ double gp[128];
    const int b = blockIdx.x, lane = threadIdx.x & 63;
    const int* it = itab + (long long)(b / bpg) * itab_stride;
    const int NI = it[0];
    // one wave per position, 16 partials per lane requested together (2048 tiles: 30 us
    // with 4 on half the waves)
    for (int v = threadIdx.x >> 6; v < NI; v += (int)(blockDim.x >> 6)) {
        const double* src = partial + ((long long)b * 2 * nz + v) * nparts;
        double t = 0.0;
        for (int k0 = 0; k0 < nparts; k0 += 1024) {
            double x[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int k = k0 + 64 * e + lane;
                x[e] = src[k < nparts ? k : nparts - 1];
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) t += k0 + 64 * e + lane < nparts ? x[e] : 0.0;
        }
        t = wave_sum(t);
        if (lane == 0) gp[v] = t;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nz; k += blockDim.x) {
        double s = 0.0;
        for (int p = 0; p < NI; ++p)
            if (k < (it[itab_layout(nz).info + p] >> 2)) s += gp[p];
        grad_t[(long long)b * nz + k] = s;
    }
}

int tgrad_tiles(int M, int LY)
{
    return M * ((LY / 2 + 31) / 32) + 1;
}

// LDS of k_tgrad: the sums of its shares and the staged spectra of M and G
template <typename R>
static size_t tgrad_lds(int shares, int nz, int ni)
{
    return sizeof(double) * 64 * (size_t)shares * ni + sizeof(MG<R>) * 64 * 3 * (size_t)nz;
}

// Shares of a tile's groups (see k_tgrad), by the plan alone: 4 where their sums fit in
// LDS, else 2, else none (0): one wave per tile without staging, which takes 3.2 and 3.5
// times as long at 64 x 64 x 24 and 32 in FP32, 4.7 at 18 in FP64.  Up to 3 layers have too
// few groups for 4.
template <typename R>
static int tgrad_shares(int nz, int ni_max)
{
    constexpr size_t kMax = 163840;
    if (nz > 3 && tgrad_lds<R>(4, nz, ni_max) <= kMax) return 4;
    return tgrad_lds<R>(2, nz, ni_max) <= kMax ? 2 : 0;
}

// Waves per tile, at most one per share: fewer where blocks queue up anyway.  A wave
// with several shares pays for their sums, and from 6 layers on for the blocks that
// their LDS keeps off a CU.  Whole calls with 1, 2 and 4 waves, a share each, and with 4
// shares on 2 waves:
//   250 x 250 x 3, 16 states  361, 403, 563 (2 shares on 1 wave: 370)   60 x 60 x 3  35, 27, 26
//   128 x 128 x 4, 4 states    74,  64,  71,   65                       60 x 60 x 4  43, 32, 29
//   250 x 250 x 5, 16 states  614, 637, 808,  667                      128 x 128 x 5 55, 42, 43
//   250 x 250 x 8, 16 states 1383, 1116, 1185, 1391                     60 x 60 x 8  77, 52, 38
static int tgrad_waves(int nz, unsigned nblk)
{
    if (nblk >= 4096) return nz <= 3 ? 1 : nz <= 5 ? 2 : 4;
    return nz <= 4 && nblk >= 512 ? 2 : 4;
}

template <typename R>
static hipError_t tgrad_r(const void* Mh, const void* Gh, int nz, int M, int LY, int b0, int nb, const void* Q,
                          long long qcs, const int* qslot, const void* D, int nzt, const int* itab,
                          int itab_stride, int ni_max, const void* lp, int bpg, int QY, int ntiles, unsigned nblk,
                          double* partial, hipStream_t s)
{
    const int shares = derivative_rows_fit(2, nzt, QY, sizeof(R)) ? tgrad_shares<R>(nz, ni_max) : 0;
    if (shares > 0) {
        const int waves = std::min(tgrad_waves(nz, nblk), shares);
        const auto kernel = waves == shares ? k_tgrad<R, true> : k_tgrad<R, false>;
        const size_t lds = tgrad_lds<R>(shares, nz, ni_max);
        const hipError_t e = ensure_lds_limit((const void*)kernel, lds > 65536 ? 163840 : 0);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(nblk), dim3(64 * waves), lds, s, (const cpx<R>*)Mh,
                           (const cpx<R>*)Gh, nz, M, LY, (const R*)Q, qcs, qslot, (const R*)D, nzt, itab,
                           itab_stride, (const R*)lp, bpg, QY, b0, nb, ntiles, shares, partial);
    } else {
        const size_t lds = sizeof(double) * 64 * (size_t)ni_max;
        hipLaunchKernelGGL((k_tgrad_rows<R, 4>), dim3(nblk), dim3(64), lds, s, (const cpx<R>*)Mh,
                           (const cpx<R>*)Gh, nz, M, LY, (const R*)Q, qcs, qslot, (const R*)D, nzt, itab,
                           itab_stride, (const R*)lp, bpg, QY, b0, nb, ntiles - 1, partial);
    }
    return hipGetLastError();
}

hipError_t launch_tgrad(bool fp64, const void* Mh, const void* Gh, int nz, int M, int LY, int b0,
                        int nb, const void* Q, long long qcs, const int* qslot, const void* D, int nzt,
                        const int* itab, int itab_stride, int ni_max, const void* lp, int bpg,
                        int QX, int QY, double* partial, hipStream_t s)
{
    if (nz < 1 || nz > 64 || ni_max < 1 || ni_max > 2 * nz || nb < 1 || bpg < 1 || nb % bpg || LY < 2 || (LY & (LY - 1)))
        return hipErrorInvalidValue;
    (void)QX;  // D and Q rows are addressed through nzt, qcs and QY
    // one row of D, two of Q (the packed column's) per descriptor; tgrad_r on two rows of D
    const long long rsz = fp64 ? 8 : 4;
    if (!derivative_rows_fit(1, nzt, QY, rsz) || 2 * qcs * rsz >= kDescriptorBytes) return hipErrorInvalidValue;
    const int ntiles = tgrad_tiles(M, LY);
    const long long nblk = (long long)((ntiles + 7) / 8) * 8 * nb;
    if (nblk > 0x7fffffffLL) return hipErrorInvalidValue;
    return fp64 ? tgrad_r<double>(Mh, Gh, nz, M, LY, b0, nb, Q, qcs, qslot, D, nzt, itab, itab_stride, ni_max,
                                  lp, bpg, QY, ntiles, (unsigned)nblk, partial, s)
                : tgrad_r<float>(Mh, Gh, nz, M, LY, b0, nb, Q, qcs, qslot, D, nzt, itab, itab_stride, ni_max,
                                 lp, bpg, QY, ntiles, (unsigned)nblk, partial, s);
}

hipError_t launch_tgrad_finish(const double* partial, int nparts, int B, int nz, const int* itab,
                               int itab_stride, int bpg, double* grad_t, hipStream_t s)
{
    if (nz < 1 || nz > 64 || B < 1 || bpg < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_tgrad_finish, dim3(B), dim3(1024), 0, s, partial, nparts, nz, itab,
                       itab_stride, bpg, grad_t);
    return hipGetLastError();
}

}  // namespace hfd
