// Transform kernels with the length compiled in (2^a 3^b from 16 to 1024),
// for gfx950.
//
// These passes are bound by HBM bandwidth, provided that the index
// arithmetic folds away: with the length taken from the arguments a value
// costs about 200 instructions (divisions per element, a branch around every
// stencil load, so one load in flight at a time): at 384x384x500 in FP32 the
// x forward pass with the divergence took 539 us so, 256 us here, the y passes
// 405 / 434 -> 141 / 149 us, the x inverse 307 -> 115 us (5.1 TB/s); the FP64
// residual pass at 256x256x384 455 -> 124 us.  Here a thread owns
// fixed columns (x) or a fixed column pair (y) for the whole tile, rows differ by
// constants, loads go out in batches before the first use, and the FFT's
// strides, radices and twiddle steps are constants.
//
// x tiles are x_len_rows consecutive rows of one z-plane (the last tile of a
// plane may be ragged: its missing rows load the last valid row and store
// nothing), two rows per complex sequence.  A group of threads has one thread
// per adjacent column pair (an odd length's last pair has one column) and
// marches down its rows, carrying the rows that the stencil needs twice.
#pragma once

#include "fsei_transforms.h"

namespace fsei {
namespace dev {

// two adjacent values: one vector access, or two where pairs are not aligned
// (d1: offset of the second value from the first)
template <bool VEC, typename T>
__device__ __forceinline__ typename Vec2T<T>::type ld_pair(const T* q, int d1 = 1) {
    if constexpr (VEC) {
        return *reinterpret_cast<const typename Vec2T<T>::type*>(q);
    } else {
        typename Vec2T<T>::type v;
        v.x = q[0];
        v.y = q[d1];
        return v;
    }
}
template <bool VEC, typename T>
__device__ __forceinline__ void st_pair(T* q, typename Vec2T<T>::type v, bool has1) {
    if constexpr (VEC) {
        *reinterpret_cast<typename Vec2T<T>::type*>(q) = v;
    } else {
        q[0] = v.x;
        if (has1) q[1] = v.y;
    }
}

template <int NF, typename T>
struct XGeom {
    static constexpr bool VEC = NF % 2 == 0;
    static constexpr int NP = (NF + 1) / 2;      // column pairs
    static constexpr int RG = x_len_groups(NF);  // thread groups
    static constexpr int NL = x_len_rows(NF);    // rows per tile
    static constexpr int RPG = NL / RG;          // rows per group
    static constexpr int NSQ = NL / 2;           // sequences per tile
    static constexpr int NTHR = x_len_threads(NF, (int)sizeof(T));
    static constexpr int SP = seq_stride(NF);
    static constexpr int E = NSQ * NF;
    static_assert(RPG % 2 == 0 && RPG * RG == NL, "whole row pairs per group");
};

// the rows of a ragged tile: nv valid rows from row j0 of a plane of ny rows
template <int NF>
struct TileRows {
    int j0, nv, ny;
    bool per;
    __device__ __forceinline__ int row(int l) const { return (l < nv ? l : nv - 1) * NF; }
    __device__ __forceinline__ int next(int l) const {   // row l + 1, wrapped
        return l + 1 < nv ? (l + 1) * NF : (j0 + nv < ny ? nv * NF : (per ? -j0 * NF : (nv - 1) * NF));
    }
    __device__ __forceinline__ int prev(int l) const {   // row l - 1, wrapped
        return l > 0 ? row(l - 1) : (j0 > 0 ? -NF : (per ? (ny - 1) * NF : 0));
    }
    __device__ __forceinline__ bool has_next(int l) const { return j0 + l + 1 < ny || per; }
    __device__ __forceinline__ bool has_prev(int l) const { return j0 + l > 0 || per; }
};

template <typename TI, typename TO, int PRO, int NF>
__global__ __launch_bounds__(x_len_threads(NF, (int)sizeof(TO))) void k_xfwd_len(XFwdArgs<TI, TO> a) {
    using G = XGeom<NF, TO>;
    constexpr int NP = G::NP, RG = G::RG, NL = G::NL, RPG = G::RPG, NTHR = G::NTHR, SP = G::SP;
    constexpr bool VEC = G::VEC;
    constexpr bool RES = PRO == PRO_RESID || PRO == PRO_RESID_F;
    using V = typename Vec2T<TI>::type;
    __shared__ TO sre[G::NSQ * SP];
    __shared__ TO sim[G::NSQ * SP];
    __shared__ TO twl[2 * NF];
    __shared__ double sred[3 * (NTHR / 64)];
    const int ny = a.ny, nz = a.nz;
    // tiles in (row tile, plane) order, plane fastest: the tile of the same
    // rows one plane up, whose rows of w (or p) this tile also reads, is the
    // next workgroup on the same XCD (an L2 hit)
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int jt = b / nz;
    const int k0 = b - jt * nz;
    const int j0 = jt * NL;
    const TileRows<NF> tr{j0, (ny - j0 < NL) ? ny - j0 : NL, ny, a.bcy == FSEI_BC_PERIODIC};
    const size_t base = ((size_t)k0 * ny + j0) * NF;
    // this thread: group g, column pair (i, i + 1)
    const bool act = threadIdx.x < NP * RG;
    const int g = (RG == 1 || !act) ? 0 : (int)threadIdx.x / NP;
    const int q = act ? (int)threadIdx.x - g * NP : 0;
    const int i = 2 * q, l0 = g * RPG;
    const bool perx = a.bcx == FSEI_BC_PERIODIC, wallx = !perx;
    const bool has1 = VEC || i + 1 < NF;
    const int i1 = has1 ? i + 1 : 0;             // second column (wrapped: the x neighbour of a lone last column)
    const int d1 = i1 - i;
    const int im = (i >= 1) ? i - 1 : NF - 1;
    const int ip2 = (i + 2 < NF) ? i + 2 : i + 2 - NF;
    const bool him = i >= 1 || perx, hip1 = has1 || perx, hip2 = i + 2 < NF || perx;
    const int lp0 = li(0, wallx ? mk_pos(i, NF) : i, SP);
    const int lp1 = li(0, wallx ? mk_pos(i1, NF) : i1, SP);
    const bool hzp = k0 + 1 < nz, hzm = k0 >= 1;
    const size_t plane = (size_t)NF * ny;
    TwiddleRegs<TO, NTHR, NF> twr;
    twr.load(a.twc, a.tws);
    // post-twiddles (cos, sin) of the outputs this thread stores (m = i,
    // i + 1), loaded before the rows and unconditionally (a periodic line
    // ignores them)
    const TO wr0 = a.dctc[i], ws0 = a.dcts[i], wr1 = a.dctc[i1], ws1 = a.dcts[i1];
    // rows per load batch (the residual stencil loads 8 values per cell: two
    // rows keep its registers within four waves per SIMD)
    constexpr int RB0 = (RES || (PRO == PRO_DIV && sizeof(TO) == 4)) ? 2 : 4;
    constexpr int RB = RPG < RB0 ? RPG : RB0;
    static_assert(RPG % RB == 0, "whole batches");
    double ss = 0.0, s1 = 0.0, sp = 0.0;
    V vcur;
    double2 pprev, pcur;
    if constexpr (PRO == PRO_DIV || PRO == PRO_DIV_ADJ) vcur = ld_pair<VEC>(a.v + base + tr.row(l0) + i, d1);
    const auto* __restrict__ pp = RES ? resid_iterate<PRO>(a) + base : nullptr;
    auto to_d2 = [](auto v) { return make_double2((double)v.x, (double)v.y); };
    if constexpr (RES) {
        pcur = to_d2(ld_pair<VEC>(pp + tr.row(l0) + i, d1));
        pprev = to_d2(ld_pair<VEC>(pp + tr.prev(l0) + i, d1));
    }
#pragma unroll
    for (int r0 = 0; r0 < RPG; r0 += RB) {
        TI val0[RB], val1[RB];
        if constexpr (RES) {
            // residual: the iterate's rows carried down the tile (rows l - 1
            // and l in registers, row l + 1 loaded), 6 loads per row not 8
            double2 pn[RB], pzp[RB], pzm[RB], fc[RB];
            double pxm[RB], pxp[RB];
#pragma unroll
            for (int lr = 0; lr < RB; ++lr) {
                const int l = l0 + r0 + lr;
                const auto* pr = pp + tr.row(l);
                pn[lr] = to_d2(ld_pair<VEC>(pp + tr.next(l) + i, d1));
                pzp[lr] = to_d2(ld_pair<VEC>(pr + (hzp ? plane : 0) + i, d1));
                pzm[lr] = to_d2(ld_pair<VEC>((hzm ? pr - plane : pr) + i, d1));
                fc[lr] = ld_pair<VEC>(a.f + base + tr.row(l) + i, d1);
                pxm[lr] = (double)pr[im];
                pxp[lr] = (double)pr[ip2];
            }
            const double zc = hzp ? a.zc[k0] : 0.0, za = hzm ? a.za[k0] : 0.0, mean = a.scal[0];
#pragma unroll
            for (int lr = 0; lr < RB; ++lr) {
                const int l = l0 + r0 + lr;
                const bool hyp = tr.has_next(l), hym = tr.has_prev(l);
                const double2 pc = pcur, pym = pprev, pyp = pn[lr];
                const double lx0 = (hip1 ? pc.y - pc.x : 0.0) + (him ? pxm[lr] - pc.x : 0.0);
                const double lx1 = (hip2 ? pxp[lr] - pc.y : 0.0) + (pc.x - pc.y);
                const double ly0 = (hyp ? pyp.x - pc.x : 0.0) + (hym ? pym.x - pc.x : 0.0);
                const double ly1 = (hyp ? pyp.y - pc.y : 0.0) + (hym ? pym.y - pc.y : 0.0);
                const double lz0 =
                    (hzp ? zc * (pzp[lr].x - pc.x) : 0.0) + (hzm ? za * (pzm[lr].x - pc.x) : 0.0);
                const double lz1 =
                    (hzp ? zc * (pzp[lr].y - pc.y) : 0.0) + (hzm ? za * (pzm[lr].y - pc.y) : 0.0);
                val0[lr] = (TI)((fc[lr].x - mean) - (lx0 * a.idx2 + ly0 * a.idy2 + lz0));
                val1[lr] = (TI)((fc[lr].y - mean) - (lx1 * a.idx2 + ly1 * a.idy2 + lz1));
                if (act && l < tr.nv) sp += pc.x + (has1 ? pc.y : 0.0);
                pprev = pc;
                pcur = pyp;
            }
        } else if constexpr (PRO == PRO_DIV || PRO == PRO_DIV_ADJ) {
            // divergence: v carried down the tile (row l + 1 of v is row l's
            // y+1 face), 5 loads per row
            V uc[RB], vn[RB], wc[RB], wh[RB], gv[RB];
            TI uh[RB];
#pragma unroll
            for (int lr = 0; lr < RB; ++lr) {
                const int l = l0 + r0 + lr;
                const size_t ro = base + tr.row(l);
                uc[lr] = ld_pair<VEC>(a.u + ro + i, d1);
                uh[lr] = a.u[ro + ip2];
                vn[lr] = ld_pair<VEC>(a.v + base + tr.next(l) + i, d1);
                wc[lr] = ld_pair<VEC>(a.w + ro + i, d1);
                wh[lr] = ld_pair<VEC>(a.w + ro + (hzp ? plane : 0) + i, d1);
                if constexpr (PRO == PRO_DIV_ADJ) {
                    if (a.gp) gv[lr] = ld_pair<VEC>(a.gp + ro + i, d1);
                }
            }
            const TI zk = a.zeta[k0], ek = a.eta[k0], zero = (TI)0;
#pragma unroll
            for (int lr = 0; lr < RB; ++lr) {
                const int l = l0 + r0 + lr;
                const bool hyp = tr.has_next(l), hym = tr.has_prev(l);
                const V vc = vcur, vh = vn[lr];
                TI x0 = ((hip1 ? uc[lr].y : zero) - (him ? uc[lr].x : zero)) * a.idx +
                        ((hyp ? vh.x : zero) - (hym ? vc.x : zero)) * a.idy +
                        (zk * (hzp ? wh[lr].x : zero) - ek * (hzm ? wc[lr].x : zero));
                TI x1 = ((hip2 ? uh[lr] : zero) - uc[lr].y) * a.idx +
                        ((hyp ? vh.y : zero) - (hym ? vc.y : zero)) * a.idy +
                        (zk * (hzp ? wh[lr].y : zero) - ek * (hzm ? wc[lr].y : zero));
                x0 *= a.alpha;
                x1 *= a.alpha;
                if constexpr (PRO == PRO_DIV_ADJ) {
                    if (a.gp) {
                        x0 += a.beta * gv[lr].x;
                        x1 += a.beta * gv[lr].y;
                    }
                }
                val0[lr] = x0;
                val1[lr] = x1;
                vcur = vh;
            }
        } else {
            double2 fc[RB];
#pragma unroll
            for (int lr = 0; lr < RB; ++lr) fc[lr] = ld_pair<VEC>(a.f + base + tr.row(l0 + r0 + lr) + i, d1);
#pragma unroll
            for (int lr = 0; lr < RB; ++lr) {
                val0[lr] = (TI)fc[lr].x;
                val1[lr] = (TI)fc[lr].y;
            }
        }
        if (r0 == 0) twr.store(twl);
#pragma unroll
        for (int lr = 0; lr < RB; ++lr) {
            const int l = l0 + r0 + lr;
            const bool in = l < tr.nv;
            const double v0 = in ? (double)val0[lr] : 0.0, v1 = (in && has1) ? (double)val1[lr] : 0.0;
            if (act) {
                if (a.out_f && in) st_pair<VEC>(a.out_f + base + l * NF + i, make_double2(v0, v1), has1);
                ss += v0 * v0 + v1 * v1;
                s1 += v0 + v1;
                TO* dst = (lr & 1) ? sim : sre;
                const int so = (l0 / 2 + (r0 + lr) / 2) * SP;
                dst[so + lp0] = (TO)v0;
                if (has1) dst[so + lp1] = (TO)v1;
            }
        }
    }
    if (a.partials) {
        // third sum: dz_k times the volume integral of the iterate (RES) or of v
        double s2 = a.dzw ? a.dzw[k0] * (RES ? sp : s1) : 0.0;
        block_sum3<NTHR>(ss, s1, s2, sred);
        if (threadIdx.x == 0) {
            a.partials[3 * blockIdx.x] = ss;
            a.partials[3 * blockIdx.x + 1] = s1;
            a.partials[3 * blockIdx.x + 2] = s2;
        }
    } else {
        __syncthreads();
    }
    if (a.out == nullptr) return;   // norm-only pass (uniform over the block)
    fft_fixed<TO, G::E, NTHR, -1, NF, 0, 1>(sre, sim, G::NSQ, twl, twl + NF);
    // outputs m = i, i + 1 of every line pair, stored as pairs
    TO* __restrict__ out = a.out + base;
    const int mm0 = (i == 0) ? 0 : NF - i, mm1 = (i1 == 0) ? 0 : NF - i1;
    const int o0 = li(0, i, SP), om0 = li(0, mm0, SP), o1 = li(0, i1, SP), om1 = li(0, mm1, SP);
    const bool lo0 = 2 * i <= NF, lo1 = 2 * i1 <= NF;
    if (act) {
#pragma unroll
        for (int t = 0; t < RPG / 2; ++t) {
            const int s = l0 / 2 + t;
            typename Vec2T<TO>::type xa, xb;
            post_fwd_v<TO>(a.bcx, lo0, sre[s * SP + o0], sim[s * SP + o0], sre[s * SP + om0], sim[s * SP + om0], wr0,
                           -ws0, xa.x, xb.x);
            post_fwd_v<TO>(a.bcx, lo1, sre[s * SP + o1], sim[s * SP + o1], sre[s * SP + om1], sim[s * SP + om1], wr1,
                           -ws1, xa.y, xb.y);
            if (2 * s < tr.nv) st_pair<VEC>(out + (2 * s) * NF + i, xa, has1);
            if (2 * s + 1 < tr.nv) st_pair<VEC>(out + (2 * s + 1) * NF + i, xb, has1);
        }
    }
}

template <typename T, typename TP, int EPI, int NF>
__global__ __launch_bounds__(x_len_threads(NF, (int)sizeof(T))) void k_xinv_len(XInvArgs<T, TP> a) {
    using G = XGeom<NF, T>;
    constexpr int NP = G::NP, RG = G::RG, NL = G::NL, RPG = G::RPG, NTHR = G::NTHR, SP = G::SP;
    constexpr bool VEC = G::VEC;
    __shared__ T sre[G::NSQ * SP];
    __shared__ T sim[G::NSQ * SP];
    __shared__ T twl[2 * NF];
    const int ny = a.ny;
    const int ntj = (ny + NL - 1) / NL;
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int k0 = b / ntj;
    const int j0 = (b - k0 * ntj) * NL;
    const int nv = (ny - j0 < NL) ? ny - j0 : NL;
    const size_t base = ((size_t)k0 * ny + j0) * NF;
    const T* in = a.in + base;   // not restrict: ACC_KEEP writes this field back (after every read of it)
    const bool act = threadIdx.x < NP * RG;
    const int g = (RG == 1 || !act) ? 0 : (int)threadIdx.x / NP;
    const int q = act ? (int)threadIdx.x - g * NP : 0;
    const int l0 = g * RPG;
    auto row = [&](int l) { return (l < nv ? l : nv - 1) * NF; };
    const bool wallx = a.bcx == FSEI_BC_WALL;
    TwiddleRegs<T, NTHR, NF> twr;
    twr.load(a.twc, a.tws);
    // each thread loads column m < (NF + 1) / 2 and its partner NF - m once and
    // forms both pre-twiddled values (m = 0 pairs with NF / 2 where that
    // exists; both of those use only their own column); the twiddles
    // cos/sin(pi m / 2NF) come before the rows and unconditionally (a
    // periodic line ignores them), at NF - m they are sin/cos at m
    const int m = q;
    const int nm = (m == 0) ? (VEC ? NF / 2 : 0) : NF - m;
    T cm = a.dctc[m], sm = a.dcts[m], c0 = a.dctc[NF / 2], s0 = a.dcts[NF / 2];
    T xam[RPG / 2], xanm[RPG / 2], xbm[RPG / 2], xbnm[RPG / 2];
#pragma unroll
    for (int t = 0; t < RPG / 2; ++t) {
        const T *ra = in + row(l0 + 2 * t), *rb = in + row(l0 + 2 * t + 1);
        xam[t] = ra[m];
        xanm[t] = ra[nm];
        xbm[t] = rb[m];
        xbnm[t] = rb[nm];
    }
    // (the twiddles are not used before the rows are requested)
    asm volatile("" : "+v"(cm), "+v"(sm), "+v"(c0), "+v"(s0));
    twr.store(twl);
    const T cn = (m == 0) ? c0 : sm, sn = (m == 0) ? s0 : cm;
    const int lm = li(0, m, SP), lnm = li(0, nm, SP);
    if (act) {
#pragma unroll
        for (int t = 0; t < RPG / 2; ++t) {
            const int s = l0 / 2 + t;
            const T pa = (m == 0) ? xanm[t] : xam[t], pb = (m == 0) ? xbnm[t] : xbm[t];
            T zr, zi;
            pre_inv_cs<T>(NF, m, a.bcx, xam[t], xanm[t], xbm[t], xbnm[t], cm, sm, zr, zi);
            sre[s * SP + lm] = zr;
            sim[s * SP + lm] = zi;
            if (VEC || m > 0) {
                pre_inv_cs<T>(NF, nm, a.bcx, xanm[t], pa, xbnm[t], pb, cn, sn, zr, zi);
                sre[s * SP + lnm] = zr;
                sim[s * SP + lnm] = zi;
            }
        }
    }
    // accumulating epilogues: the values the result is added to (the iterate,
    // or the FP32 field) are loaded before the transform and arrive while it runs
    const int i = 2 * q;
    const bool has1 = VEC || i + 1 < NF;
    const int i1 = has1 ? i + 1 : i;
    TP* __restrict__ out = a.out + base;
    constexpr bool ACC = EPI == EPI_ACC || EPI == EPI_ADDF || EPI == EPI_ACC_KEEP;
    typename Vec2T<TP>::type old[ACC ? RPG : 1];
    if constexpr (ACC) {
#pragma unroll
        for (int lr = 0; lr < RPG; ++lr) {
            const int o = row(l0 + lr) + i;
            if constexpr (EPI == EPI_ADDF) {
                const float2 f = ld_pair<VEC>(a.add32 + base + o, i1 - i);
                old[lr].x = (TP)f.x;
                old[lr].y = (TP)f.y;
            } else {
                old[lr] = ld_pair<VEC>(out + o, i1 - i);
            }
        }
    }
    __syncthreads();
    fft_fixed<T, G::E, NTHR, 1, NF, 0, 1>(sre, sim, G::NSQ, twl, twl + NF);
    const int ln0 = li(0, wallx ? mk_pos(i, NF) : i, SP), ln1 = li(0, wallx ? mk_pos(i1, NF) : i1, SP);
    const TP msub = (ACC && a.vsum) ? (TP)(a.vsum[0] * a.vscale) : (TP)0;
    if (act) {
#pragma unroll
        for (int lr = 0; lr < RPG; ++lr) {
            const int l = l0 + lr;
            const T* src = ((lr & 1) ? sim : sre) + (l0 / 2 + lr / 2) * SP;
            typename Vec2T<T>::type val;
            val.x = src[ln0];
            val.y = src[ln1];
            typename Vec2T<TP>::type r;
            if constexpr (ACC) {
                r.x = (old[lr].x - msub) + (TP)val.x;
                r.y = (old[lr].y - msub) + (TP)val.y;
            } else {
                r.x = (TP)val.x;
                r.y = (TP)val.y;
            }
            if (l < nv) {
                st_pair<VEC>(out + l * NF + i, r, has1);
                if constexpr (EPI == EPI_ACC_KEEP) st_pair<VEC>(a.keep + base + l * NF + i, val, has1);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// x inverse fused with the gradient correction (paper, Sec. 2.1, eq.
// NSdiscr0: the pressure term -dt grad p^{n+1} applied to the provisional
// velocity), even lengths:
//     p = inverse x transform of the y-inverted field,
//     u += cx (p_i - p_{i-1}),  v += cy (p_j - p_{j-1}),
//     w += sw (bk_k p_k - gk_k p_{k-1}),
// on active faces (wall faces written 0), p written once (optional) and never
// re-read: 64 bytes per FP64 cell (56 without p) against 72 in two passes.
// A workgroup owns GR = 8 rows j0..j0+7 (whole tiles only: row tests around
// the stores cost 40 registers) over a chunk of planes and marches up in z.  Each step inverts the 8
// rows plus row j0-1 (whose p the v update of row j0 needs) of one plane: 9
// real rows as 5 complex sequences, the last paired with a zero row.  RG
// groups of threads, one thread per column pair in each, share the rows of the
// gradient; the own rows' p of the previous plane stay in registers for the w
// update; the chunk's first step only produces them (it inverts the plane
// below the chunk).
// ---------------------------------------------------------------------------
template <int NF>
struct XgGeom {
    static constexpr int NP = NF / 2;
    static constexpr int RG = xg_len_groups(NF);
    static constexpr int RPG = kXgRows / RG;
    static constexpr int NTHR = xg_len_threads(NF);
    static constexpr int SP = seq_stride(NF);
};

template <typename T, int NF>
__global__ __launch_bounds__(XgGeom<NF>::NTHR) void k_xinv_grad_len(XInvGradArgs<T> a) {
    using G = XgGeom<NF>;
    using V = typename Vec2T<T>::type;
    constexpr int NP = G::NP, RG = G::RG, RPG = G::RPG, NTHR = G::NTHR, SP = G::SP;
    constexpr int GR = kXgRows, NSQ = kXgSeq;
    constexpr int GB = RPG < 4 ? RPG : 4;        // rows per batch of the gradient phase
    constexpr int NSG = (NSQ + RG - 1) / RG;     // sequences a group loads
    static_assert(NF % 2 == 0 && GR % RG == 0, "column pairs, whole groups");
    __shared__ T sre[NSQ * SP];
    __shared__ T sim[NSQ * SP];
    __shared__ T twl[2 * NF];
    const int ny = a.ny, nz = a.nz;
    const int ntj = ny / GR;
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int chunk = b / ntj;
    const int j0 = (b - chunk * ntj) * GR;
    const int kb = chunk * a.kc;
    const int ke = (kb + a.kc < nz) ? kb + a.kc : nz;
    const bool wallx = a.bcx == FSEI_BC_WALL, wally = a.bcy == FSEI_BC_WALL;
    stage_twiddles<T, NTHR>(twl, a.twc, a.tws, NF);
    const bool act = threadIdx.x < NP * RG;
    const int g = act ? (int)threadIdx.x / NP : 0;
    // pre-processing: column m and its partner nm of every row
    const int m = act ? (int)threadIdx.x - g * NP : 0;
    const int nm = (m == 0) ? NF / 2 : NF - m;
    const int lm = li(0, m, SP), lnm = li(0, nm, SP);
    T cm = (T)1, sm = (T)0, cn = (T)1, sn = (T)0;
    if (wallx) {
        cm = a.dctc[m];
        sm = a.dcts[m];
        cn = (m == 0) ? a.dctc[NF / 2] : sm;
        sn = (m == 0) ? a.dcts[NF / 2] : cm;
    }
    // gradient: this thread's column pair (i, i + 1) and the x neighbour i - 1
    const int i = 2 * m, l0g = g * RPG;
    const int ixm = (i > 0) ? i - 1 : NF - 1;
    const int q0 = li(0, wallx ? mk_pos(i, NF) : i, SP);
    const int q1 = li(0, wallx ? mk_pos(i + 1, NF) : i + 1, SP);
    const int qm = li(0, wallx ? mk_pos(ixm, NF) : ixm, SP);
    const size_t plane = (size_t)NF * ny;
    auto rowj = [&](int l) { return j0 + l; };
    // p of tile row r (r = 0: the halo row, r = 1..8: the own rows); the
    // sequence pairs rows 2s and 2s + 1
    auto pv = [&](int r, int q) -> T { return ((r & 1) ? sim : sre)[(r >> 1) * SP + q]; };
    V prev[RPG];
#pragma unroll
    for (int l = 0; l < RPG; ++l) prev[l].x = prev[l].y = (T)0;
    // input rows of one step: sequence s = g + t RG of this group's share
    T xa[NSG][2], xb[NSG][2];
    auto load_in = [&](int k) {
        const T* __restrict__ in = a.in + (size_t)k * plane;
#pragma unroll
        for (int t = 0; t < NSG; ++t) {
            const int s = g + t * RG < NSQ ? g + t * RG : NSQ - 1;
            const T* pa = in + (size_t)xg_in_row(s, 0, j0, ny) * NF;
            const T* pb = in + (size_t)xg_in_row(s, 1, j0, ny) * NF;
            xa[t][0] = pa[m];
            xa[t][1] = pa[nm];
            xb[t][0] = pb[m];
            xb[t][1] = pb[nm];
        }
    };
    for (int k = (kb > 0) ? kb - 1 : 0; k < ke; ++k) {
        if (act) {
            load_in(k);
#pragma unroll
            for (int t = 0; t < NSG; ++t) {
                const int s = g + t * RG;
                if (s < NSQ) {
                    const bool zb = s + 1 == NSQ;    // the last sequence has a zero row
                    const T b0 = zb ? (T)0 : xb[t][0], b1 = zb ? (T)0 : xb[t][1];
                    const T pa = (m == 0) ? xa[t][1] : xa[t][0], pb = (m == 0) ? b1 : b0;
                    T zr, zi;
                    pre_inv_cs<T>(NF, m, a.bcx, xa[t][0], xa[t][1], b0, b1, cm, sm, zr, zi);
                    sre[s * SP + lm] = zr;
                    sim[s * SP + lm] = zi;
                    pre_inv_cs<T>(NF, nm, a.bcx, xa[t][1], pa, b1, pb, cn, sn, zr, zi);
                    sre[s * SP + lnm] = zr;
                    sim[s * SP + lnm] = zi;
                }
            }
        }
        __syncthreads();
        fft_fixed<T, NSQ * NF, NTHR, 1, NF, 0, 1>(sre, sim, NSQ, twl, twl + NF);
        if (!act) {
        } else if (k >= kb) {   // not the chunk's first (halo) plane
            const T bkk = a.bk[k], gkk = a.gk[k];
            const size_t ro = (size_t)k * plane + (size_t)j0 * NF + i;
            V pym;
            pym.x = pv(l0g, q0);
            pym.y = pv(l0g, q1);
#pragma unroll
            for (int t0 = 0; t0 < RPG; t0 += GB) {
                V uo[GB], vo[GB], wo[GB];
#pragma unroll
                for (int t = 0; t < GB; ++t) {
                    const size_t o = (size_t)k * plane + (size_t)rowj(l0g + t0 + t) * NF + i;
                    uo[t] = *reinterpret_cast<const V*>(a.ui + o);
                    vo[t] = *reinterpret_cast<const V*>(a.vi + o);
                    wo[t] = *reinterpret_cast<const V*>(a.wi + o);
                }
#pragma unroll
                for (int t = 0; t < GB; ++t) {
                    const int l = l0g + t0 + t, r = l + 1;
                    V pc;
                    pc.x = pv(r, q0);
                    pc.y = pv(r, q1);
                    const T pxm = pv(r, qm);
                    const int j = j0 + l;
                    V un, vn, wn;
                    un.x = (wallx && i == 0) ? (T)0 : uo[t].x + a.cx * (pc.x - pxm);
                    un.y = uo[t].y + a.cx * (pc.y - pc.x);
                    const bool v0 = wally && j == 0;
                    vn.x = v0 ? (T)0 : vo[t].x + a.cy * (pc.x - pym.x);
                    vn.y = v0 ? (T)0 : vo[t].y + a.cy * (pc.y - pym.y);
                    wn.x = (k == 0) ? (T)0 : wo[t].x + a.sw * (bkk * pc.x - gkk * prev[t0 + t].x);
                    wn.y = (k == 0) ? (T)0 : wo[t].y + a.sw * (bkk * pc.y - gkk * prev[t0 + t].y);
                    // non-temporal: nothing here is read again soon
                    const size_t o = ro + (size_t)l * NF;
                    nt_store2(a.u + o, un);
                    nt_store2(a.v + o, vn);
                    nt_store2(a.w + o, wn);
                    if (a.p) nt_store2(a.p + o, pc);
                    prev[t0 + t] = pc;
                    pym = pc;
                }
                // keep the next batch's loads after this batch's stores
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int t = 0; t < RPG; ++t) {
                prev[t].x = pv(l0g + t + 1, q0);
                prev[t].y = pv(l0g + t + 1, q1);
            }
        }
        __syncthreads();   // the next step overwrites the tile
    }
}

// ---------------------------------------------------------------------------
// y transforms: a tile is y_len_pairs adjacent column pairs of one z-plane;
// a thread owns one pair s and the rows jr, jr + RPP, ...  VEC: pairs as one
// access (a switch inside the kernel makes the compiler merge both forms into
// single-value accesses, 15 % slower in FP32)
// ---------------------------------------------------------------------------
template <typename T, int NF>
struct YGeom {
    static constexpr int NSF = y_len_pairs(NF, (int)sizeof(T));
    static constexpr int NTHR = y_len_threads(NF, (int)sizeof(T));
    static constexpr int RPP = NTHR / NSF;             // rows per pass over the tile
    static constexpr int NPASS = (NF + RPP - 1) / RPP;
    static constexpr bool WHOLE = NF % RPP == 0;
    static constexpr int E = NSF * NF;
    static_assert(RPP * NSF == NTHR, "whole passes");
};

template <typename T, int NF, bool VEC>
__global__ __launch_bounds__(y_len_threads(NF, (int)sizeof(T)), y_len_waves(NF, (int)sizeof(T), false)) void k_yfwd_len(YArgs<T> a) {
    using G = YGeom<T, NF>;
    using V2 = typename Vec2T<T>::type;
    constexpr int NSF = G::NSF, NTHR = G::NTHR, RPP = G::RPP, NPASS = G::NPASS;
    constexpr int PS = y_len_pad((int)sizeof(T), false), SP = seq_stride(NF, PS);
    // FP32: both twiddle tables in LDS first (the tile's registers are the
    // limit: 1024 threads, two workgroups per CU); FP64: post-twiddles in
    // registers, the FFT twiddles' round trip overlaps the tile loads.  (A
    // table load between the stores would make every store wait for the
    // previous one.)
    constexpr bool TL = sizeof(T) == 4;
    __shared__ T sre[NSF * SP];
    __shared__ T sim[NSF * SP];
    __shared__ T twl[(TL ? 4 : 2) * NF];
    static_assert(sizeof(sre) + sizeof(sim) + sizeof(twl) == y_len_lds(NF, (int)sizeof(T), false), "as the bound has it");
    const int nx = a.nx;
    // tiles in XCD-contiguous runs: two neighbouring tiles that share
    // 128-byte lines meet in one L2
    const int bx = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int k = bx / a.ntile;
    const int i0 = (bx - k * a.ntile) * 2 * NSF;
    T* __restrict__ d = a.data + (size_t)k * nx * NF + i0;
    const int s = threadIdx.x % NSF, jr = threadIdx.x / NSF;
    const bool ok0 = i0 + 2 * s < nx, ok1 = i0 + 2 * s + 1 < nx;
    const unsigned lo = ok0 ? 2 * s : 0;    // columns beyond the plane read the tile's first pair
    const int d1 = (ok1 || (!ok0 && i0 + 1 < nx)) ? 1 : 0;
    // row r of the lane: a uniform row offset plus the lane's own (one
    // address register for all rows); the last pass of a ragged tile reads
    // row r * RPP where the lane's row is beyond the line
    const unsigned lane = (unsigned)(jr * nx) + lo, lane_last = (jr + (NPASS - 1) * RPP < NF) ? lane : lo;
    TwiddleRegs<T, NTHR, (TL ? 1 : NF)> twr;
    T wr[TL ? 1 : NPASS], wi[TL ? 1 : NPASS];
    if constexpr (TL) {
        stage_twiddles<T, NTHR>(twl, a.twc, a.tws, NF);
        stage_twiddles<T, NTHR>(twl + 2 * NF, a.dctc, a.dcts, NF);
    } else {
        twr.load(a.twc, a.tws);
#pragma unroll
        for (int r = 0; r < NPASS; ++r) {
            const int m = jr + r * RPP;
            wr[r] = a.dctc[G::WHOLE || m < NF ? m : 0];
            wi[r] = a.dcts[G::WHOLE || m < NF ? m : 0];
        }
    }
    V2 val[NPASS];
#pragma unroll
    for (int r = 0; r < NPASS; ++r) {
        const T* row = d + (size_t)(r * RPP) * nx;
        val[r] = ld_pair<VEC>(row + ((G::WHOLE || r < NPASS - 1) ? lane : lane_last), d1);
    }
    if constexpr (!TL) {
        // keep the post-twiddles in registers from here on (the compiler
        // would otherwise reload each next to its use, one wait per row)
#pragma unroll
        for (int r = 0; r < NPASS; ++r) asm volatile("" : "+v"(wr[r]), "+v"(wi[r]));
        twr.store(twl);
    }
#pragma unroll
    for (int r = 0; r < NPASS; ++r) {
        const int j = jr + r * RPP;
        if (G::WHOLE || j < NF) {
            const int o = s * SP + li<PS>(0, (a.bcy == FSEI_BC_WALL) ? mk_pos(j, NF) : j, SP);
            sre[o] = val[r].x;
            sim[o] = val[r].y;
        }
    }
    __syncthreads();
    fft_fixed<T, G::E, NTHR, -1, NF, 0, 1, PS>(sre, sim, NSF, twl, twl + NF);
#pragma unroll
    for (int r = 0; r < NPASS; ++r) {
        const int m = jr + r * RPP;
        if (G::WHOLE || m < NF) {
            const int mm = (m == 0) ? 0 : NF - m;
            const int om = s * SP + li<PS>(0, m, SP), omm = s * SP + li<PS>(0, mm, SP);
            V2 res;
            const T cr = TL ? twl[2 * NF + m] : wr[TL ? 0 : r];
            const T sr = TL ? twl[3 * NF + m] : wi[TL ? 0 : r];
            post_fwd_v<T>(a.bcy, 2 * m <= NF, sre[om], sim[om], sre[omm], sim[omm], cr, -sr, res.x, res.y);
            if (ok0) st_pair<VEC>(d + (size_t)(r * RPP) * nx + lane, res, ok1);
        }
    }
}

template <typename T, int NF, bool VEC>
__global__ __launch_bounds__(y_len_threads(NF, (int)sizeof(T)), y_len_waves(NF, (int)sizeof(T), true)) void k_yinv_len(YArgs<T> a) {
    using G = YGeom<T, NF>;
    using V2 = typename Vec2T<T>::type;
    constexpr int NSF = G::NSF, NTHR = G::NTHR, RPP = G::RPP, NPASS = G::NPASS;
    constexpr int SP = seq_stride(NF);
    constexpr int NM = (NF + 1) / 2;              // rows m with a partner NF - m (or none)
    constexpr int NH = (NM + RPP - 1) / RPP;
    constexpr bool WHOLE = NM % RPP == 0, EVEN = NF % 2 == 0;
    __shared__ T sre[NSF * SP];
    __shared__ T sim[NSF * SP];
    __shared__ T twl[2 * NF];
    static_assert(sizeof(sre) + sizeof(sim) + sizeof(twl) == y_len_lds(NF, (int)sizeof(T), true), "as the bound has it");
    const int nx = a.nx;
    const int bx = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int k = bx / a.ntile;
    const int i0 = (bx - k * a.ntile) * 2 * NSF;
    T* __restrict__ d = a.data + (size_t)k * nx * NF + i0;
    const int s = threadIdx.x % NSF, mr = threadIdx.x / NSF;
    const bool ok0 = i0 + 2 * s < nx, ok1 = i0 + 2 * s + 1 < nx;
    const unsigned lo = ok0 ? 2 * s : 0;
    const int d1 = (ok1 || (!ok0 && i0 + 1 < nx)) ? 1 : 0;
    TwiddleRegs<T, NTHR, NF> twr;
    twr.load(a.twc, a.tws);
    // each lane loads rows m < (NF + 1) / 2 and its partner NF - m once and
    // forms both pre-twiddled values (m = 0 pairs with NF/2 where that exists;
    // both of those use only their own row); pre-twiddles cos/sin(pi m / 2NF)
    // loaded before the data and unconditionally (a periodic line ignores
    // them; at NF - m they are sin/cos at m)
    auto mrow = [&](int r) { const int m = mr + r * RPP; return (WHOLE || m < NM) ? m : 0; };
    auto nrow = [&](int m) { return (m == 0) ? (EVEN ? NF / 2 : 0) : NF - m; };
    T c[NH], sn[NH];
#pragma unroll
    for (int r = 0; r < NH; ++r) {
        c[r] = a.dctc[mrow(r)];
        sn[r] = a.dcts[mrow(r)];
    }
    const T c0 = a.dctc[NF / 2], s0 = a.dcts[NF / 2];
    const unsigned lane = (unsigned)(mr * nx) + lo, laner = (unsigned)((RPP - 1 - mr) * nx) + lo;
    V2 A[NH], B[NH];
#pragma unroll
    for (int r = 0; r < NH; ++r) {
        // uniform row offset plus the lane's own, where the pass is whole
        const int m = mrow(r);
        if (WHOLE || r < NH - 1) A[r] = ld_pair<VEC>(d + (size_t)(r * RPP) * nx + lane, d1);
        else A[r] = ld_pair<VEC>(d + ((unsigned)(m * nx) + lo), d1);
        if (r > 0 && (WHOLE || r < NH - 1)) B[r] = ld_pair<VEC>(d + (size_t)(NF - (r + 1) * RPP + 1) * nx + laner, d1);
        else B[r] = ld_pair<VEC>(d + ((unsigned)(nrow(m) * nx) + lo), d1);
    }
    twr.store(twl);
#pragma unroll
    for (int r = 0; r < NH; ++r) {
        // opaque to the compiler, which would otherwise share products between
        // a row and its partner in the passes that cannot hold row 0 and
        // round those two rows together
        int m = mr + r * RPP;
        asm("" : "+v"(m));
        if (WHOLE || m < NM) {
            const int nm = nrow(m);
            const V2 Am = (m == 0) ? B[r] : A[r];
            const T cp = (m == 0) ? c0 : sn[r], sp = (m == 0) ? s0 : c[r];
            T zr, zi;
            pre_inv_cs<T>(NF, m, a.bcy, A[r].x, B[r].x, A[r].y, B[r].y, c[r], sn[r], zr, zi);
            sre[s * SP + li(0, m, SP)] = zr;
            sim[s * SP + li(0, m, SP)] = zi;
            if (EVEN || m > 0) {
                pre_inv_cs<T>(NF, nm, a.bcy, B[r].x, Am.x, B[r].y, Am.y, cp, sp, zr, zi);
                sre[s * SP + li(0, nm, SP)] = zr;
                sim[s * SP + li(0, nm, SP)] = zi;
            }
        }
    }
    __syncthreads();
    fft_fixed<T, G::E, NTHR, 1, NF, 0, 1>(sre, sim, NSF, twl, twl + NF);
#pragma unroll
    for (int r = 0; r < NPASS; ++r) {
        const int j = mr + r * RPP;
        if (G::WHOLE || j < NF) {
            const int o = s * SP + li(0, (a.bcy == FSEI_BC_WALL) ? mk_pos(j, NF) : j, SP);
            V2 res;
            res.x = sre[o];
            res.y = sim[o];
            if (ok0) st_pair<VEC>(d + (size_t)(r * RPP) * nx + lane, res, ok1);
        }
    }
}

// ---------------------------------------------------------------------------
// host side: the launchers of one compiled length
// ---------------------------------------------------------------------------
template <typename TI, typename TO>
using XFwdFn = void (*)(const XFwdArgs<TI, TO>&, unsigned, hipStream_t);
template <typename T, typename TP>
using XInvFn = void (*)(const XInvArgs<T, TP>&, unsigned, hipStream_t);
template <typename T>
using XgFn = void (*)(const XInvGradArgs<T>&, unsigned, hipStream_t);
template <typename T>
using YFn = void (*)(const YArgs<T>&, unsigned, hipStream_t);

struct LenOps {
    int x_rows;                 // rows per x tile
    int y_pairs_d, y_pairs_f;   // column pairs per y tile
    XFwdFn<double, double> xf_dd[PRO_KINDS];
    XFwdFn<float, float> xf_ff[PRO_KINDS];
    XFwdFn<double, float> xf_df[PRO_KINDS];
    XInvFn<double, double> xi_dd[EPI_KINDS];
    XInvFn<float, float> xi_ff[EPI_KINDS];
    XInvFn<float, double> xi_fd[EPI_KINDS];
    XgFn<double> xg_d;          // null where the fused kernel is not compiled
    YFn<double> yf_d[2], yi_d[2];   // [column pairs as one access]
    YFn<float> yf_f[2], yi_f[2];
    template <typename TI, typename TO>
    XFwdFn<TI, TO> xfwd(int pro) const {
        if constexpr (sizeof(TI) == 4) return xf_ff[pro];
        else if constexpr (sizeof(TO) == 4) return xf_df[pro];
        else return xf_dd[pro];
    }
    template <typename T, typename TP>
    XInvFn<T, TP> xinv(int epi) const {
        if constexpr (sizeof(T) == 8) return xi_dd[epi];
        else if constexpr (sizeof(TP) == 4) return xi_ff[epi];
        else return xi_fd[epi];
    }
    template <typename T>
    YFn<T> y(bool inverse, bool vec) const {
        if constexpr (sizeof(T) == 8) return (inverse ? yi_d : yf_d)[vec];
        else return (inverse ? yi_f : yf_f)[vec];
    }
};

#define FSEI_DECLARE_LEN(n) const LenOps& len_ops_##n();
FSEI_LENGTHS(FSEI_DECLARE_LEN)
#undef FSEI_DECLARE_LEN

}  // namespace dev
}  // namespace fsei
