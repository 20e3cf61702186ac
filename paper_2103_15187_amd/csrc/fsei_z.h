// The z solves of the pressure projection for gfx950 (MI355X): the batched
// tridiagonal solver of the mode lines, the near-singular lines and the
// singular zero mode, in one launch.
#pragma once

#include <hip/hip_runtime.h>

#include "fsei_fft.h"
#include "fsei_plan.h"
#include "fsei_transforms.h"

namespace fsei {
namespace dev {

// ---------------------------------------------------------------------------
// z: one tridiagonal per (kx, ky) mode,
//   a_k x_{k-1} + (b0_k + sigma) x_k + c_k x_{k+1} = scale * f_k,
// sigma = lambda_x + lambda_y.  A workgroup holds TXL modes (adjacent kx, same
// ky: coalesced rows of TXL elements) x P chunks of one z-line each.  Every
// thread keeps its chunk (<= LMAX rows) in registers, eliminates its interior
// rows in one downward sweep to express them through the two chunk-end
// unknowns, the chunk-end unknowns of a line are solved as a
// P x P tridiagonal in LDS, and each thread then back-substitutes its chunk.
// `transposed` solves T^T y = g through T^T = dz T dz^{-1} (scale by 1/dz_k on
// load and by dz_k on store).
// ---------------------------------------------------------------------------
// Reciprocal for the tridiagonal sweeps: the hardware estimate refined by
// Newton steps r <- r + r (1 - x r) (two in FP64, one in FP32), within a
// few ulp of 1/x for the well-scaled pivots of these systems (|x| between
// the smallest z coefficient and |lambda_x + lambda_y|).  The IEEE-exact
// division the compiler emits otherwise is a chain of ten dependent
// instructions on the critical path of every row.
__device__ __forceinline__ double zrcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ float zrcp(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}

template <typename TS, typename TC>
struct ZArgs {
    int nx, ny, nz, L, P, transposed;
    int gx;               // tiles per row of modes
    int form;             // the tiling (ZForm of fsei_z.hip)
    TS* data;
    TC scale;             // 1/(nx ny)
    // skip the lines with |lamx64 + lamy64| < sigma_thr, tested in FP64 on
    // the FP64 tables with the host's own expression, so that a line is
    // solved here exactly when the host left it out of its near-singular list
    double sigma_thr;
    const double* lamx64;
    const double* lamy64;
    const TC* za;
    const TC* zc;
    const TC* zb0;
    const TC* dz;
    const TC* inv_dz;
    const TC* lamx;
    const TC* lamy;
    // the zero mode and the near-singular lines, in FP64: nspec groups, taken
    // by the launch's first workgroups (group 0: the zero mode; group g: the
    // lines list[(g - 1) LN ...))
    int nspec, nlist;
    const int* list;      // line indices qy * nx + qx, ascending
    double scale64, lz;
    const double* za64;
    const double* zc64;
    const double* dz64;
    const double* inv_dz64;
    const double* h64;
    double* scal;         // scal[0] <- removed mean of the zero mode's right-hand side, or null
};

// ---------------------------------------------------------------------------
// Near-singular mode lines: |lambda_x + lambda_y| below the plan's threshold
// (condition 1 + 4 / (dz_min^2 |sigma|) above 1e4), in FP64 with the pivots in
// row-sum form.  With zero-flux walls every row of L_z + sigma sums to sigma,
// so the pivot d_k = b_k - a_k c_{k-1} / d_{k-1}, b_k = -(a_k + c_k) + sigma,
// equals g_k - c_k with g_k = sigma - a_k g_{k-1} / d_{k-1}, g_0 = sigma: every term
// has the sign of sigma, nothing cancels.  Forming b_k first rounds the small
// sigma against a_k + c_k, which costs up to ~1e-11 relative error at
// condition 1e8 in FP64 (768 x 768 x 1024, tanh 3.0).
//
// The recurrence is a chain over the rows, but each of its three parts composes:
//   pivots: q_k = g_k / d_k = (s + a q) / (s + a q + c), s = -sigma, a Moebius map
//     of q_{k-1} with the matrix [[a, s], [a, s + c]], whose entries and
//     products are all positive: products lose no accuracy (n, d kept in range by
//     powers of two).  With q = n / d, -d_k = d'/d for the mapped denominator d'.
//   forward y_k = (a_k / -d_k) y_{k-1} - f_k / -d_k and
//   backward x_k = y_k + (c_k / -d_k) x_{k+1}: affine maps with factors in [0, 1].
// So a line is cut into PS chunks of L rows, one per lane: compose the chunk,
// Kogge-Stone scan over the chunks (in LDS), then the chunk's rows from the
// value that enters it.  One lane per line walking all rows took 0.26 us per
// row (the latency of one chain): at 256 x 256 x 384 in FP32 100 us beside 50 us
// for all other lines, 57 us for both now; at 64^3 the z solve with the zero mode in a
// launch of its own on a second stream took about 40 us between its
// neighbours, 7 us now.
//
// LDS: ca (2 PS L doubles: the a_k, then the c_k) and ex ([4][NTS] doubles).
// Threads beyond NTS repeat the work of the first NTS (same values to the same
// slots) and do not store.
// ---------------------------------------------------------------------------
// n and d (or two columns of them) scaled by a common power of two, d near 1
__device__ __forceinline__ void renorm(double& n, double& d) {
    const int e = -__builtin_amdgcn_frexp_exp(d);
    n = __builtin_ldexp(n, e);
    d = __builtin_ldexp(d, e);
}
__device__ __forceinline__ void renorm2(double& n0, double& d0, double& n1, double& d1) {
    const int e = -__builtin_amdgcn_frexp_exp(d0 + d1);
    n0 = __builtin_ldexp(n0, e);
    d0 = __builtin_ldexp(d0, e);
    n1 = __builtin_ldexp(n1, e);
    d1 = __builtin_ldexp(d1, e);
}

template <int NT>
constexpr int zspec_threads() { return NT < 512 ? NT : 512; }
// chunks and rows per chunk of the special lines beside tiles of pmax chunks of
// l rows in nt threads: twice as many half as long for 8 rows and more (a lane
// holds two FP64 values per row; with 24 rows the tiles' kernels spilled), four
// times for 24 and more in the 128 registers of 1024 threads (FP32, 162 x 162 x
// 1800: 176 us without special lines, 257 beside chunks of half the rows)
constexpr int zspec_split(int l, int nt) { return l <= 4 ? 1 : nt == 1024 && l >= 24 ? 4 : 2; }
constexpr int zspec_chunks(int pmax, int l, int nt) { return pmax * zspec_split(l, nt); }
constexpr int zspec_rows(int l, int nt) { return l / zspec_split(l, nt); }
// Waves per SIMD that the tile code reaches by itself and that the special
// lines, compiled into the same kernel, must leave it (m modes per lane; 0: no
// bound needed): without a bound they took the registers of the FP32 kernels from
// 37-62 to 50-104 and a workgroup per CU with them (486 x 243 x 144, two
// modes per lane in 1024 threads: 47 -> 67 us).
constexpr int z_waves(int elem, int m, int l) {
    return elem == 8 ? (m == 1 && l == 4 ? 8 : 0)
                     : m == 1 ? (l <= 12 ? 8 : 0) : m == 2 ? (l <= 8 ? 8 : l == 12 ? 6 : 0) : 0;
}
// the bytes of their two LDS arrays
template <int NT>
constexpr int zspec_ex() { return 4 * zspec_threads<NT>() * (int)sizeof(double); }
template <int PMAX, int L>
constexpr int zspec_tab() { return 2 * PMAX * L * (int)sizeof(double); }

template <typename TS, typename TC, int PS, int L, int NT>
__device__ __forceinline__ void z_lines(const ZArgs<TS, TC>& a, int grp, double* ca, double* ex) {
    constexpr int NTS = zspec_threads<NT>(), LN = NTS / PS;
    static_assert(LN >= 1 && NTS % PS == 0 && NT % NTS == 0, "whole lines per group");
    double* cc = ca + PS * L;
    const int nz = a.nz;
    for (int k = threadIdx.x; k < PS * L; k += NT) {
        ca[k] = (k > 0 && k < nz) ? a.za64[k] : 0.0;
        cc[k] = (k + 1 < nz) ? a.zc64[k] : 0.0;
    }
    const int me = threadIdx.x % NTS;
    const int ln = me % LN, p = me / LN;
    const int li = grp * LN + ln;
    const bool own = li < a.nlist;
    const int line = a.list[own ? li : a.nlist - 1];
    const int qy = line / a.nx, qx = line - qy * a.nx;
    const double s = -(a.lamx64[qx] + a.lamy64[qy]);
    const size_t st = (size_t)a.nx * a.ny;
    TS* col = a.data + line;
    const int s0 = p * L;
    double f[L], r[L];
#pragma unroll
    for (int t = 0; t < L; ++t) {
        const int k = s0 + t < nz ? s0 + t : nz - 1;
        const double v = (double)col[(size_t)k * st];
        f[t] = s0 + t < nz ? v * (a.transposed ? a.scale64 * a.inv_dz64[k] : a.scale64) : 0.0;
    }
    __syncthreads();
    // the chunk's Moebius matrix, as the images of (n, d) = (1, 0) and (0, 1)
    double n0 = 1.0, d0 = 0.0, n1 = 0.0, d1 = 1.0;
#pragma unroll
    for (int t = 0; t < L; ++t) {
        const double A = ca[s0 + t], C = cc[s0 + t];
        n0 = A * n0 + s * d0;
        d0 = C * d0 + n0;
        n1 = A * n1 + s * d1;
        d1 = C * d1 + n1;
        if (t % 4 == 3) renorm2(n0, d0, n1, d1);
    }
    for (int o = 1; o < PS; o <<= 1) {
        __syncthreads();
        ex[me] = n0;
        ex[NTS + me] = d0;
        ex[2 * NTS + me] = n1;
        ex[3 * NTS + me] = d1;
        __syncthreads();
        if (p >= o) {
            const int w = me - o * LN;
            const double sn0 = ex[w], sd0 = ex[NTS + w], sn1 = ex[2 * NTS + w], sd1 = ex[3 * NTS + w];
            const double a0 = n0 * sn0 + n1 * sd0, b0 = d0 * sn0 + d1 * sd0;
            const double a1 = n0 * sn1 + n1 * sd1, b1 = d0 * sn1 + d1 * sd1;
            n0 = a0;
            d0 = b0;
            n1 = a1;
            d1 = b1;
            renorm2(n0, d0, n1, d1);
        }
    }
    __syncthreads();
    ex[me] = n0 + n1;          // the line starts from q = 1 (a_0 = 0: it has no effect)
    ex[NTS + me] = d0 + d1;
    __syncthreads();
    double n = 1.0, d = 1.0;
    if (p > 0) {
        n = ex[me - LN];
        d = ex[NTS + me - LN];
    }
    double Y = 0.0, Q = 1.0;   // the chunk's forward map: y_out = Q y_in + Y
#pragma unroll
    for (int t = 0; t < L; ++t) {
        const double A = ca[s0 + t], C = cc[s0 + t];
        const double t0 = A * n + s * d;
        const double dn = C * d + t0;
        r[t] = d * zrcp(dn);   // 1 / -d_k
        n = t0;
        d = dn;
        if (t % 4 == 3) renorm(n, d);
        const double al = A * r[t];
        Y = al * Y - f[t] * r[t];
        Q *= al;
    }
    for (int o = 1; o < PS; o <<= 1) {
        __syncthreads();
        ex[me] = Y;
        ex[NTS + me] = Q;
        __syncthreads();
        if (p >= o) {
            Y = Q * ex[me - o * LN] + Y;
            Q *= ex[NTS + me - o * LN];
        }
    }
    __syncthreads();
    ex[me] = Y;
    __syncthreads();
    double y = p > 0 ? ex[me - LN] : 0.0;
#pragma unroll
    for (int t = 0; t < L; ++t) {
        y = ca[s0 + t] * r[t] * y - f[t] * r[t];
        f[t] = y;
    }
    double X = 0.0;
    Q = 1.0;
#pragma unroll
    for (int t = L - 1; t >= 0; --t) {
        r[t] *= cc[s0 + t];    // c_k / -d_k from here on
        X = r[t] * X + f[t];
        Q *= r[t];
    }
    for (int o = 1; o < PS; o <<= 1) {
        __syncthreads();
        ex[me] = X;
        ex[NTS + me] = Q;
        __syncthreads();
        if (p + o < PS) {
            X = Q * ex[me + o * LN] + X;
            Q *= ex[NTS + me + o * LN];
        }
    }
    __syncthreads();
    ex[me] = X;
    __syncthreads();
    double x = p + 1 < PS ? ex[me + LN] : 0.0;
#pragma unroll
    for (int t = L - 1; t >= 0; --t) {
        x = r[t] * x + f[t];
        f[t] = x;
    }
    if (own && threadIdx.x < NTS) {
#pragma unroll
        for (int t = 0; t < L; ++t)
            if (s0 + t < nz) col[(size_t)(s0 + t) * st] = (TS)(a.transposed ? f[t] * a.dz64[s0 + t] : f[t]);
    }
    __syncthreads();           // the caller reuses the LDS
}

// ---------------------------------------------------------------------------
// (0,0) mode: singular z line (zero-flux walls).  Removes the dz-weighted
// mean of the scaled right-hand side (compatibility), integrates the flux
// F_k = sum_{k'<k} dz_k' f_k', sums p_k = sum_{k'<=k} h_k' F_k', and pins
// sum dz_k p_k = 0.  One workgroup, FP64, prefix sums by wave shuffles.
// ---------------------------------------------------------------------------
// sum of the values of all lower threads; total: of all threads
template <int NT>
__device__ __forceinline__ double block_exscan(double v, double* sh, double& total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    double inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double w = __shfl_up(inc, o, 64);
        if (lane >= o) inc += w;
    }
    double exc = __shfl_up(inc, 1, 64);
    if (lane == 0) exc = 0.0;
    __syncthreads();
    if (lane == 63) sh[wid] = inc;
    __syncthreads();
    double pre = 0.0;
    total = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        if (w == wid) pre = total;
        total += sh[w];
    }
    return pre + exc;
}

template <typename TS, typename TC, int NT>
__device__ __forceinline__ void z_zero_mode(const ZArgs<TS, TC>& a, double* sh) {
    constexpr int CMAX = (kMaxNz + NT - 1) / NT;
    const int nz = a.nz;
    const int c = (nz + NT - 1) / NT;
    const int k0 = threadIdx.x * c;
    const size_t st = (size_t)a.nx * a.ny;
    double f[CMAX], w[CMAX], h[CMAX];
    double loc = 0.0, total, total2;
#pragma unroll
    for (int r = 0; r < CMAX; ++r) {
        const int k = k0 + r;
        const bool in = r < c && k < nz;
        f[r] = in ? (double)a.data[(size_t)k * st] * (a.transposed ? a.scale64 * a.inv_dz64[k] : a.scale64) : 0.0;
        w[r] = in ? a.dz64[k] : 0.0;
        h[r] = in ? a.h64[k] : 0.0;   // h_0 = 0
        loc += w[r] * f[r];
    }
    block_exscan<NT>(loc, sh, total);
    const double mean = total / a.lz;
    loc = 0.0;
#pragma unroll
    for (int r = 0; r < CMAX; ++r) {
        f[r] -= mean;
        loc += w[r] * f[r];
    }
    double run = block_exscan<NT>(loc, sh, total2);   // flux entering this thread's first row
    loc = 0.0;
#pragma unroll
    for (int r = 0; r < CMAX; ++r) {
        h[r] *= run;
        run += w[r] * f[r];
        loc += h[r];
    }
    run = block_exscan<NT>(loc, sh, total2);
    loc = 0.0;
#pragma unroll
    for (int r = 0; r < CMAX; ++r) {
        run += h[r];
        f[r] = run;
        loc += w[r] * f[r];
    }
    block_exscan<NT>(loc, sh, total);
    const double pm = total / a.lz;
#pragma unroll
    for (int r = 0; r < CMAX; ++r) {
        const int k = k0 + r;
        if (r < c && k < nz) {
            double v = f[r] - pm;
            if (a.transposed) v *= w[r];
            a.data[(size_t)k * st] = (TS)v;
        }
    }
    if (threadIdx.x == 0 && a.scal) a.scal[0] = mean;
    __syncthreads();           // the caller reuses the LDS
}

// group g of the special lines, by a whole workgroup of a kernel whose tiles
// have PMAX chunks of L rows, in two of the tiles' LDS arrays.  (Two arrays and
// not one block: as parts of one block the compiler takes
// the tables and the exchange slots of the tile code for aliases, which spilled
// 30 registers more in the FP32 kernel of 32 rows.)
template <typename TS, typename TC, int PMAX, int L, int NT>
__device__ __forceinline__ void z_special(const ZArgs<TS, TC>& a, int g, void* tab, void* ex) {
    if (g == 0) z_zero_mode<TS, TC, NT>(a, static_cast<double*>(ex));
    else z_lines<TS, TC, zspec_chunks(PMAX, L, NT), zspec_rows(L, NT), NT>(a, g - 1, static_cast<double*>(tab),
                                                                       static_cast<double*>(ex));
}

// The special lines by themselves, where they are more than one group per CU:
// here two workgroups fit a CU, beside the tiles of long lines one (the solve
// of 768 x 768 x 1024, 14.5 thousand lines: 10.95 ms with them in the tiles'
// launch, 10.73 ms so)
template <typename TS, typename TC, int PS, int L>
__global__ __launch_bounds__(512, 4) void k_zspecial(ZArgs<TS, TC> a) {
    __shared__ double tab[2 * PS * L], ex[4 * 512];
    if (blockIdx.x == 0) z_zero_mode<TS, TC, 512>(a, ex);
    else z_lines<TS, TC, PS, L, 512>(a, blockIdx.x - 1, tab, ex);
}

template <typename TS, typename TC, int TXL, int L, int NT>
__global__ __launch_bounds__(NT, z_waves(sizeof(TC), 1, L)) void k_zsolve(ZArgs<TS, TC> a) {
    constexpr int PMAX = NT / TXL;
    __shared__ __align__(16) TC sh[4][NT];
    __shared__ __align__(16) TC tabs[6][PMAX * L];
    static_assert(sizeof(sh) >= zspec_ex<NT>() && sizeof(tabs) >= zspec_tab<PMAX, L>(), "the special lines fit");
    if ((int)blockIdx.x < a.nspec) {
        z_special<TS, TC, PMAX, L, NT>(a, blockIdx.x, tabs, sh);
        return;
    }
    TC *ta = tabs[0], *tc = tabs[1], *tb = tabs[2], *tm = tabs[3], *tsi = tabs[4], *tso = tabs[5];
    const int nx = a.nx, nz = a.nz, P = a.P;
    const int npad = P * L;
    // per-k coefficients staged in LDS, padded to P*L rows with decoupled
    // identity rows (a = c = 0, b = 1, f = 0); the scheduling barriers in the
    // sweeps keep each row's LDS reads next to their use, so the coefficients
    // are re-read per sweep instead of being held in registers
    // tsi: load scale 1/(nx ny) (times 1/dz_k when transposed);
    // tso: store scale 1 (dz_k when transposed)
    for (int k = threadIdx.x; k < npad; k += NT) {
        const bool in = k < nz;
        ta[k] = in ? a.za[k] : (TC)0;
        tc[k] = in ? a.zc[k] : (TC)0;
        tb[k] = in ? a.zb0[k] : (TC)1;   // diagonal b0_k + sigma * tm_k
        tm[k] = in ? (TC)1 : (TC)0;
        tsi[k] = in ? (a.transposed ? a.scale * a.inv_dz[k] : a.scale) : (TC)0;
        tso[k] = in ? (a.transposed ? a.dz[k] : (TC)1) : (TC)0;
    }
    const int ln = threadIdx.x % TXL;
    const int p = threadIdx.x / TXL;
    const size_t stride = (size_t)nx * a.ny;
    const int tile = (int)blockIdx.x - a.nspec;
    const int qy = tile / a.gx;
    const int qx = (tile - qy * a.gx) * TXL + ln;
    bool active = qx < nx;
    TC sigma = (TC)-1;
    if (active) {
        sigma = a.lamx[qx] + a.lamy[qy];
        if (qx == 0 && qy == 0) active = false;
        if (fabs(a.lamx64[qx] + a.lamy64[qy]) < a.sigma_thr) active = false;
        if (!active) sigma = (TC)-1;
    }
    const bool inrange = p < P;
    const int s0 = inrange ? p * L : 0;
    TS* __restrict__ col = a.data + (size_t)qy * nx + qx;
    const bool ld = active && inrange;

    TC F[L], Rr[L];
#pragma unroll
    for (int t = 0; t < L; ++t) {
        const int k = s0 + t;
        F[t] = (ld && k < nz) ? (TC)col[(size_t)k * stride] : (TC)0;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < L; ++t) F[t] *= tsi[s0 + t];
    // diagonal of row k: b0_k + sigma, 1 on padding rows (branch free)
#define ZDIAG(k) (tb[k] + sigma * tm[k])
    // One downward sweep over the interior rows s0..s0+L-2 (Dirichlet ends):
    // LU pivots r_t (kept), the eliminated right-hand side d' and the
    // sensitivity g to the left end value.  The back substitution of the
    // first interior row, x_s = sum_t d'_t pi_t with pi_t = prod_{j<t} (-c'_j),
    // is accumulated on the way, so no upward sweep is needed.
    TC cp = 0, dp = 0, g = 1, pi = 1, ysum = 0, gsum = 0;
#pragma unroll
    for (int t = 0; t < L - 1; ++t) {
        const int k = s0 + t;
        const TC A = ta[k], C = tc[k], B = ZDIAG(k);
        const TC r = zrcp(B - A * cp);
        Rr[t] = r;
        dp = (F[t] - A * dp) * r;
        g = -A * g * r;
        ysum += dp * pi;
        gsum += g * pi;
        cp = C * r;
        pi *= -cp;
    }
    const TC Ylast = dp, Glast = g, Hlast = -cp;
    const TC dh = ysum, ch = -gsum, hh = pi;
    const int me = threadIdx.x;
    // publish first-row expressions for the left neighbour chunk
    sh[0][me] = dh;    // Y_first
    sh[1][me] = -ch;   // G_first
    sh[2][me] = hh;    // H_first
    __syncthreads();
    // reduced row p: alpha x_{e(p-1)} + beta x_{e(p)} + gamma x_{e(p+1)} = phi
    TC al = 0, be = 1, ga = 0, ph = 0;
    if (inrange) {
        const int e = s0 + L - 1;
        const TC Ae = ta[e], Ce = tc[e], Be = ZDIAG(e);
        al = Ae * Glast;
        be = Be + Ae * Hlast;
        ph = F[L - 1] - Ae * Ylast;
        if (p + 1 < P) {
            const int nb = me + TXL;
            be += Ce * sh[1][nb];
            ga = Ce * sh[2][nb];
            ph -= Ce * sh[0][nb];
        }
    }
#undef ZDIAG
    // The P x P reduced system of each line is diagonally dominant like the
    // original; solve it by parallel cyclic reduction over the P threads of
    // the line: at stride s every row eliminates its couplings to rows p-s
    // and p+s (rows outside [0, P) act as identity rows), until all rows are
    // decoupled after ceil(log2 P) steps.
    for (int s = 1; s < P; s <<= 1) {
        __syncthreads();
        sh[0][me] = al;
        sh[1][me] = be;
        sh[2][me] = ga;
        sh[3][me] = ph;
        __syncthreads();
        if (inrange) {
            TC k1 = 0, k2 = 0, alm = 0, gam = 0, phm = 0, alp = 0, gap = 0, php = 0;
            if (p - s >= 0) {
                const int id = me - s * TXL;
                k1 = al * zrcp(sh[1][id]);
                alm = sh[0][id];
                gam = sh[2][id];
                phm = sh[3][id];
            }
            if (p + s < P) {
                const int id = me + s * TXL;
                k2 = ga * zrcp(sh[1][id]);
                alp = sh[0][id];
                gap = sh[2][id];
                php = sh[3][id];
            }
            be = be - k1 * gam - k2 * alp;
            ph = ph - k1 * phm - k2 * php;
            al = -k1 * alm;
            ga = -k2 * gap;
        }
    }
    __syncthreads();
    sh[0][me] = ph * zrcp(be);   // chunk-end value x_{e(p)}
    __syncthreads();
    const TC XR = sh[0][me];
    const TC XL = (p > 0) ? sh[0][me - TXL] : (TC)0;
    // sweep 3 (down) with the true left value, sweep 4 (up) from the right value
    TC prev = XL;
#pragma unroll
    for (int t = 0; t < L - 1; ++t) {
        prev = (F[t] - ta[s0 + t] * prev) * Rr[t];
        F[t] = prev;
    }
    F[L - 1] = XR;
    TC nxt = XR;
#pragma unroll
    for (int t = L - 2; t >= 0; --t) {
        nxt = F[t] - tc[s0 + t] * Rr[t] * nxt;
        F[t] = nxt;
    }
    if (ld) {
        // fresh base address (opaque to the compiler) so the per-row load
        // addresses are not kept alive until the stores
        TS* out = col + (size_t)s0 * stride;
        asm volatile("" : "+v"(out));
#pragma unroll
        for (int t = 0; t < L; ++t) {
            if (s0 + t < nz) out[(size_t)t * stride] = (TS)(F[t] * tso[s0 + t]);
        }
    }
}

// ---------------------------------------------------------------------------
// Same solver with M adjacent modes (qx .. qx+M-1) per lane: the global
// accesses become one M-wide vector (16 bytes for two FP64 or four FP32
// modes) and a workgroup row segment covers M*TXLM modes (256 B), which
// streams markedly better from HBM than 128-B segments; the M lines'
// recurrences also interleave.  Dense mode only; needs nx % M == 0.
// ---------------------------------------------------------------------------
// M adjacent values as one native vector (one 8- or 16-byte access)
template <typename T, int M> struct VecM;
template <> struct VecM<double, 1> { typedef double type __attribute__((ext_vector_type(1))); };
template <> struct VecM<double, 2> { typedef double type __attribute__((ext_vector_type(2))); };
template <> struct VecM<float, 2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct VecM<float, 4> { typedef float type __attribute__((ext_vector_type(4))); };

template <typename TS, typename TC, int M, int TXLM, int L, int NT>
__global__ __launch_bounds__(NT, z_waves(sizeof(TC), M, L)) void k_zsolvev(ZArgs<TS, TC> a) {
    using V = typename VecM<TS, M>::type;
    constexpr int PMAX = NT / TXLM;
    __shared__ __align__(16) TC sh[4][M * NT];
    __shared__ __align__(16) TC tabs[6][PMAX * L];
    static_assert(sizeof(sh) >= zspec_ex<NT>() && sizeof(tabs) >= zspec_tab<PMAX, L>(), "the special lines fit");
    if ((int)blockIdx.x < a.nspec) {
        z_special<TS, TC, PMAX, L, NT>(a, blockIdx.x, tabs, sh);
        return;
    }
    TC *ta = tabs[0], *tc = tabs[1], *tb = tabs[2], *tm = tabs[3], *tsi = tabs[4], *tso = tabs[5];
    const int nx = a.nx, nz = a.nz, P = a.P;
    const int npad = P * L;
    for (int k = threadIdx.x; k < npad; k += NT) {
        const bool in = k < nz;
        ta[k] = in ? a.za[k] : (TC)0;
        tc[k] = in ? a.zc[k] : (TC)0;
        tb[k] = in ? a.zb0[k] : (TC)1;   // diagonal b0_k + sigma * tm_k
        tm[k] = in ? (TC)1 : (TC)0;
        tsi[k] = in ? (a.transposed ? a.scale * a.inv_dz[k] : (TC)1) : (TC)0;
        tso[k] = in ? (a.transposed ? a.dz[k] : a.scale) : (TC)0;
    }
    const int ln = threadIdx.x % TXLM;
    const int p = threadIdx.x / TXLM;
    const int tile = (int)blockIdx.x - a.nspec;
    const int qy = tile / a.gx;
    const int qx0 = ((tile - qy * a.gx) * TXLM + ln) * M;
    const size_t strideV = (size_t)nx * a.ny / M;   // in vectors
    bool act[M];
    TC sigma[M];
    bool anyl = false, alll = true;
#pragma unroll
    for (int h = 0; h < M; ++h) {
        const int qx = qx0 + h;
        act[h] = qx < nx;
        sigma[h] = (TC)-1;
        if (act[h]) {
            sigma[h] = a.lamx[qx] + a.lamy[qy];
            if ((qx == 0 && qy == 0) || fabs(a.lamx64[qx] + a.lamy64[qy]) < a.sigma_thr) act[h] = false;
            if (!act[h]) sigma[h] = (TC)-1;
        }
        anyl = anyl || act[h];
        alll = alll && act[h];
    }
    const bool inrange = p < P;
    const int s0 = inrange ? p * L : 0;
    const bool anyact = anyl && inrange;
    const size_t coff = (size_t)qy * nx + (qx0 < nx ? qx0 : 0);   // element offset of the lane's column
    const V* __restrict__ col = reinterpret_cast<const V*>(a.data + coff);

    TC F[M][L], Rr[M][L];
#pragma unroll
    for (int t = 0; t < L; ++t) {
        const int k = s0 + t;
        V v = (V)(TS)0;
        if (anyact && k < nz) v = col[(size_t)k * strideV];
#pragma unroll
        for (int h = 0; h < M; ++h) F[h][t] = (TC)v[h];
    }
    __syncthreads();
    // the forward solve's uniform 1/(nx ny) is applied at the store (one
    // multiply fewer per value); the transposed solve's 1/dz_k here
    if (a.transposed) {
#pragma unroll
        for (int t = 0; t < L; ++t)
#pragma unroll
            for (int h = 0; h < M; ++h) F[h][t] *= tsi[s0 + t];
    }
    // downward sweep of the M lines (interleaved), first-row back
    // substitution accumulated as running sums (see k_zsolve)
    TC cp[M], dp[M], g[M], pi[M], ys[M], gs[M];
#pragma unroll
    for (int h = 0; h < M; ++h) {
        cp[h] = 0;
        dp[h] = 0;
        g[h] = 1;
        pi[h] = 1;
        ys[h] = 0;
        gs[h] = 0;
    }
#pragma unroll
    for (int t = 0; t < L - 1; ++t) {
        const int k = s0 + t;
        const TC A = ta[k], C = tc[k], B0 = tb[k], Mk = tm[k];
#pragma unroll
        for (int h = 0; h < M; ++h) {
            const TC r = zrcp(B0 + sigma[h] * Mk - A * cp[h]);
            Rr[h][t] = r;
            dp[h] = (F[h][t] - A * dp[h]) * r;
            g[h] = -A * g[h] * r;
            ys[h] += dp[h] * pi[h];
            gs[h] += g[h] * pi[h];
            cp[h] = C * r;
            pi[h] *= -cp[h];
        }
    }
    const int me = threadIdx.x;
    TC al[M], be[M], ga[M], ph[M];
#pragma unroll
    for (int h = 0; h < M; ++h) {
        sh[0][M * me + h] = ys[h];    // Y_first
        sh[1][M * me + h] = gs[h];    // G_first
        sh[2][M * me + h] = pi[h];    // H_first
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < M; ++h) {
        al[h] = 0;
        be[h] = 1;
        ga[h] = 0;
        ph[h] = 0;
        if (inrange) {
            const int e = s0 + L - 1;
            const TC Ae = ta[e], Ce = tc[e], Be = tb[e] + sigma[h] * tm[e];
            al[h] = Ae * g[h];
            be[h] = Be - Ae * cp[h];
            ph[h] = F[h][L - 1] - Ae * dp[h];
            if (p + 1 < P) {
                const int nb = M * (me + TXLM) + h;
                be[h] += Ce * sh[1][nb];
                ga[h] = Ce * sh[2][nb];
                ph[h] -= Ce * sh[0][nb];
            }
        }
    }
    // parallel cyclic reduction of the reduced systems of the M lines
    for (int s = 1; s < P; s <<= 1) {
        __syncthreads();
#pragma unroll
        for (int h = 0; h < M; ++h) {
            sh[0][M * me + h] = al[h];
            sh[1][M * me + h] = be[h];
            sh[2][M * me + h] = ga[h];
            sh[3][M * me + h] = ph[h];
        }
        __syncthreads();
        if (inrange) {
#pragma unroll
            for (int h = 0; h < M; ++h) {
                TC k1 = 0, k2 = 0, alm = 0, gam = 0, phm = 0, alp = 0, gap = 0, php = 0;
                if (p - s >= 0) {
                    const int id = M * (me - s * TXLM) + h;
                    k1 = al[h] * zrcp(sh[1][id]);
                    alm = sh[0][id];
                    gam = sh[2][id];
                    phm = sh[3][id];
                }
                if (p + s < P) {
                    const int id = M * (me + s * TXLM) + h;
                    k2 = ga[h] * zrcp(sh[1][id]);
                    alp = sh[0][id];
                    gap = sh[2][id];
                    php = sh[3][id];
                }
                be[h] = be[h] - k1 * gam - k2 * alp;
                ph[h] = ph[h] - k1 * phm - k2 * php;
                al[h] = -k1 * alm;
                ga[h] = -k2 * gap;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < M; ++h) sh[0][M * me + h] = ph[h] * zrcp(be[h]);
    __syncthreads();
    TC XR[M], prev[M];
#pragma unroll
    for (int h = 0; h < M; ++h) {
        XR[h] = sh[0][M * me + h];
        prev[h] = (p > 0) ? sh[0][M * (me - TXLM) + h] : (TC)0;   // x left of the chunk
    }
#pragma unroll
    for (int t = 0; t < L - 1; ++t) {
        const TC A = ta[s0 + t];
#pragma unroll
        for (int h = 0; h < M; ++h) {
            prev[h] = (F[h][t] - A * prev[h]) * Rr[h][t];
            F[h][t] = prev[h];
        }
    }
#pragma unroll
    for (int h = 0; h < M; ++h) F[h][L - 1] = XR[h];
#pragma unroll
    for (int t = L - 2; t >= 0; --t) {
        const TC C = tc[s0 + t];
#pragma unroll
        for (int h = 0; h < M; ++h) {
            XR[h] = F[h][t] - C * Rr[h][t] * XR[h];
            F[h][t] = XR[h];
        }
    }
    if (anyact) {
        // store addresses rebuilt from the field base (not kept live from the
        // loads), as whole-vector global stores
        size_t ooff = coff + (size_t)s0 * strideV * M;
        asm volatile("" : "+v"(ooff));
        V* out = reinterpret_cast<V*>(a.data + ooff);
        TS* outs = a.data + ooff;
#pragma unroll
        for (int t = 0; t < L; ++t) {
            if (s0 + t < nz) {
                const TC so = tso[s0 + t];
                if (alll) {
                    V v;
#pragma unroll
                    for (int h = 0; h < M; ++h) v[h] = (TS)(F[h][t] * so);
                    out[(size_t)t * strideV] = v;
                } else {
#pragma unroll
                    for (int h = 0; h < M; ++h)
                        if (act[h]) outs[(size_t)t * M * strideV + h] = (TS)(F[h][t] * so);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Persistent form of k_zsolvev (M = 1: of k_zsolve) for whole tiles of modes (nx
// a multiple of M TXLM, aligned to 16 bytes; P = NT / TXLM chunks of L rows, RAG: the last ones
// padded; TR: the transposed solve), one workgroup per CU: a workgroup walks tiles b, b +
// gridDim.x, ...; while it solves one tile, the first S rows of every chunk of
// its next tile come into LDS by direct global-to-LDS loads (no registers
// held), so the load phase of a tile covers only its last L - S rows and the
// rest of the tile's bytes arrive while the CU computes.  With S = L the next tile is
// waited for before the current tile's stores, so nothing waits for a store.
// Each wave reads back only the LDS slots its own loads wrote (slot = wave
// base + lane), so the buffer needs no barrier, only the wave's own counters.
// Same arithmetic, in the same order, as k_zsolvev.
// ---------------------------------------------------------------------------
template <typename TS, typename TC, int M, int TXLM, int L, int NT, int S, bool RAG, bool TR>
__global__ __launch_bounds__(NT) void k_zsolvev_pf(ZArgs<TS, TC> a) {
    using V = typename VecM<TS, M>::type;
    // one FP64 mode per lane: a direct load moves two modes, so one
    // instruction of a wave covers two rows of its chunks
    constexpr bool ONE = sizeof(V) == 8;
    static_assert(sizeof(V) == 16 || (ONE && TXLM == 16 && S % 2 == 0), "16-byte direct loads");
    static_assert(S >= 1 && S <= L, "prefetched rows");
    constexpr int P = NT / TXLM;
    constexpr int NZ = P * L;
    typedef __attribute__((address_space(3))) void* lds_void;
    typedef const __attribute__((address_space(1))) void* glb_void;
    // (one block here: as arrays of their own the FP64 transposed 768-row solve
    // took 700 us at 512 x 512 x 768 instead of 669, the FP32 one 5 % longer)
    struct Lds {
        TC sh[4][M * NT];
        TC tabs[TR ? 5 : 4][NZ];
        V pf[S][NT];
    };
    static_assert(sizeof(Lds::sh) >= zspec_ex<NT>() && sizeof(Lds::tabs) >= zspec_tab<P, L>(), "the special lines fit");
    __shared__ __align__(16) unsigned char lds[sizeof(Lds)];
    Lds& sm = *reinterpret_cast<Lds*>(lds);
    auto& sh = sm.sh;
    auto& pf = sm.pf;
    for (int g = blockIdx.x; g < a.nspec; g += gridDim.x) z_special<TS, TC, P, L, NT>(a, g, sm.tabs, sm.sh);
    TC *ta = sm.tabs[0], *tc = sm.tabs[1], *tb = sm.tabs[2], *tso = sm.tabs[3], *tsi = sm.tabs[TR ? 4 : 0];
    const int nx = a.nx, nz = RAG ? a.nz : NZ;
    for (int k = threadIdx.x; k < NZ; k += NT) {
        const bool in = k < nz;   // padding rows: decoupled, diagonal sigma - 1 (never 0)
        ta[k] = in ? a.za[k] : (TC)0;
        tc[k] = in ? a.zc[k] : (TC)0;
        tb[k] = in ? a.zb0[k] : (TC)-1;
        // the forward solve's uniform 1/(nx ny) is applied at the store
        tso[k] = in ? (TR ? a.dz[k] : a.scale) : (TC)0;
        if constexpr (TR) tsi[k] = in ? a.scale * a.inv_dz[k] : (TC)0;
    }
    const int ln = threadIdx.x % TXLM;
    const int p = threadIdx.x / TXLM;
    const int s0 = p * L;
    const int wbase = threadIdx.x & ~63;
    const int ntx = nx / (M * TXLM);
    const int ntiles = ntx * a.ny;
    const size_t strideV = (size_t)nx * a.ny / M;   // in vectors
    auto coff = [&](int b) -> size_t {              // element offset of the lane's column in tile b
        const int qy = b / ntx;
        return (size_t)qy * nx + (size_t)((b - qy * ntx) * TXLM + ln) * M;
    };
    auto row = [&](int t) { return s0 + t < nz ? s0 + t : nz - 1; };   // RAG: a valid row
    const int lane = threadIdx.x & 63;
    char* const pfw = reinterpret_cast<char*>(pf) + (ONE ? (threadIdx.x >> 6) * (S / 2) * 1024 : 0);
    auto slot = [&](int t) -> V {   // row t of the lane's chunk of the tile in LDS
        if constexpr (ONE) return *reinterpret_cast<const V*>(pfw + (t >> 1) * 1024 + (t & 1) * 512 + lane * 8);
        else return pf[t][threadIdx.x];
    };
    auto prefetch = [&](int b) {
        if constexpr (ONE) {
            // lane: row t2 + lane / 32 of the wave's chunk (lane / 8) % 4, modes 2 (lane % 8)
            const int qy = b / ntx;
            const TS* src = a.data + (size_t)qy * nx + (b - qy * ntx) * TXLM + 2 * (lane & 7);
            const int k0 = ((threadIdx.x >> 6) * 4 + ((lane >> 3) & 3)) * L + (lane >> 5);
#pragma unroll
            for (int t2 = 0; t2 < S / 2; ++t2) {
                int k = k0 + 2 * t2;
                if (RAG) k = k < nz ? k : nz - 1;
                __builtin_amdgcn_global_load_lds((glb_void)(src + (size_t)k * strideV), (lds_void)(pfw + t2 * 1024), 16, 0,
                                                 0);
            }
            return;
        }
        const V* src = reinterpret_cast<const V*>(a.data + coff(b)) + (RAG ? 0 : (size_t)s0 * strideV);
#pragma unroll
        for (int t = 0; t < S; ++t)
            __builtin_amdgcn_global_load_lds((glb_void)(src + (RAG ? (size_t)row(t) : (size_t)t) * strideV),
                                             (lds_void)&pf[t][wbase], 16, 0, 0);
    };
    prefetch(blockIdx.x);   // the host launches at most ntiles workgroups
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (int b = blockIdx.x; b < ntiles; b += gridDim.x) {
        const int qy = b / ntx;
        const int qx0 = (b - qy * ntx) * TXLM * M + ln * M;
        bool act[M];
        TC sigma[M];
        bool anyl = false, alll = true;
#pragma unroll
        for (int h = 0; h < M; ++h) {
            const int qx = qx0 + h;
            const double s64 = a.lamx64[qx] + a.lamy64[qy];
            const TC sg = a.lamx[qx] + a.lamy[qy];
            const bool off = ((qx | qy) == 0) | (fabs(s64) < a.sigma_thr);
            act[h] = !off;
            sigma[h] = off ? (TC)-1 : sg;
            anyl = anyl | act[h];
            alll = alll & act[h];
        }
        // the row stride re-read opaquely each tile, so the compiler rebuilds
        // the row addresses per tile instead of keeping 24 of them live
        size_t sv = strideV;
        asm volatile("" : "+s"(sv));
        const size_t cof = coff(b);
        const V* __restrict__ col = reinterpret_cast<const V*>(a.data + cof) + (RAG ? 0 : (size_t)s0 * sv);
        TC F[M][L], Rr[M][L];
#pragma unroll
        for (int t = S; t < L; ++t) {
            const V v = col[(RAG ? (size_t)row(t) : (size_t)t) * sv];
#pragma unroll
            for (int h = 0; h < M; ++h) F[h][t] = (TC)v[h];
        }
        // rows 0 .. S-1 from this wave's slots (its direct loads for this
        // tile were issued before every load above; where all rows come that
        // way, they were waited for before the last tile's stores)
        if constexpr (S < L) __builtin_amdgcn_s_waitcnt(imm_wait_vm(L - S));
#pragma unroll
        for (int t = 0; t < S; ++t) {
            const V v = slot(t);
#pragma unroll
            for (int h = 0; h < M; ++h) F[h][t] = (TC)v[h];
        }
        __builtin_amdgcn_s_waitcnt(imm_wait_lgkm0());   // buffer read: free for the next tile's rows
        const int nb0 = b + (int)gridDim.x;
        const int bnext = nb0 < ntiles ? nb0 : b;       // the last tile re-reads its own rows (never used)
        if constexpr (S == L) {
            __builtin_amdgcn_sched_barrier(0);
            prefetch(bnext);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (RAG || TR) {
#pragma unroll
            for (int t = 0; t < L; ++t) {
                const TC si = TR ? tsi[s0 + t] : (TC)1;
#pragma unroll
                for (int h = 0; h < M; ++h) {
                    if constexpr (RAG) F[h][t] = s0 + t < nz ? F[h][t] : (TC)0;
                    if constexpr (TR) F[h][t] *= si;
                }
            }
        }
        TC cp[M], dp[M], g[M], pi[M], ys[M], gs[M];
#pragma unroll
        for (int h = 0; h < M; ++h) {
            cp[h] = 0;
            dp[h] = 0;
            g[h] = 1;
            pi[h] = 1;
            ys[h] = 0;
            gs[h] = 0;
        }
#pragma unroll
        for (int t = 0; t < L - 1; ++t) {
            const int k = s0 + t;
            const TC A = ta[k], C = tc[k], B0 = tb[k];
#pragma unroll
            for (int h = 0; h < M; ++h) {
                const TC r = zrcp(B0 + sigma[h] - A * cp[h]);
                Rr[h][t] = r;
                dp[h] = (F[h][t] - A * dp[h]) * r;
                g[h] = -A * g[h] * r;
                ys[h] += dp[h] * pi[h];
                gs[h] += g[h] * pi[h];
                cp[h] = C * r;
                pi[h] *= -cp[h];
            }
        }
        // the next tile's first rows: issued once the downward sweep has used
        // every register row (a wait for a register row behind them would
        // wait for them too), in flight through the reduction and the sweeps
        if constexpr (S < L) {
            __builtin_amdgcn_sched_barrier(0);
            prefetch(bnext);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int me = threadIdx.x;
        TC al[M], be[M], ga[M], ph[M];
#pragma unroll
        for (int h = 0; h < M; ++h) {
            sh[0][M * me + h] = ys[h];
            sh[1][M * me + h] = gs[h];
            sh[2][M * me + h] = pi[h];
        }
        sync_lds_nofence();
#pragma unroll
        for (int h = 0; h < M; ++h) {
            const int e = s0 + L - 1;
            const TC Ae = ta[e], Ce = tc[e], Be = tb[e] + sigma[h];
            al[h] = Ae * g[h];
            be[h] = Be - Ae * cp[h];
            ph[h] = F[h][L - 1] - Ae * dp[h];
            ga[h] = 0;
            if (p + 1 < P) {
                const int nb = M * (me + TXLM) + h;
                be[h] += Ce * sh[1][nb];
                ga[h] = Ce * sh[2][nb];
                ph[h] -= Ce * sh[0][nb];
            }
        }
        for (int s = 1; s < P; s <<= 1) {
            sync_lds_nofence();
#pragma unroll
            for (int h = 0; h < M; ++h) {
                sh[0][M * me + h] = al[h];
                sh[1][M * me + h] = be[h];
                sh[2][M * me + h] = ga[h];
                sh[3][M * me + h] = ph[h];
            }
            sync_lds_nofence();
#pragma unroll
            for (int h = 0; h < M; ++h) {
                TC k1 = 0, k2 = 0, alm = 0, gam = 0, phm = 0, alp = 0, gap = 0, php = 0;
                if (p - s >= 0) {
                    const int id = M * (me - s * TXLM) + h;
                    k1 = al[h] * zrcp(sh[1][id]);
                    alm = sh[0][id];
                    gam = sh[2][id];
                    phm = sh[3][id];
                }
                if (p + s < P) {
                    const int id = M * (me + s * TXLM) + h;
                    k2 = ga[h] * zrcp(sh[1][id]);
                    alp = sh[0][id];
                    gap = sh[2][id];
                    php = sh[3][id];
                }
                be[h] = be[h] - k1 * gam - k2 * alp;
                ph[h] = ph[h] - k1 * phm - k2 * php;
                al[h] = -k1 * alm;
                ga[h] = -k2 * gap;
            }
        }
        sync_lds_nofence();
#pragma unroll
        for (int h = 0; h < M; ++h) sh[0][M * me + h] = ph[h] * zrcp(be[h]);
        sync_lds_nofence();
        TC XR[M], prev[M];
#pragma unroll
        for (int h = 0; h < M; ++h) {
            XR[h] = sh[0][M * me + h];
            prev[h] = (p > 0) ? sh[0][M * (me - TXLM) + h] : (TC)0;
        }
#pragma unroll
        for (int t = 0; t < L - 1; ++t) {
            const TC A = ta[s0 + t];
#pragma unroll
            for (int h = 0; h < M; ++h) {
                prev[h] = (F[h][t] - A * prev[h]) * Rr[h][t];
                F[h][t] = prev[h];
            }
        }
#pragma unroll
        for (int h = 0; h < M; ++h) F[h][L - 1] = XR[h];
#pragma unroll
        for (int t = L - 2; t >= 0; --t) {
            const TC C = tc[s0 + t];
#pragma unroll
            for (int h = 0; h < M; ++h) {
                XR[h] = F[h][t] - C * Rr[h][t] * XR[h];
                F[h][t] = XR[h];
            }
        }
        if constexpr (S == L) __builtin_amdgcn_s_waitcnt(imm_wait_vm(0));   // the next tile's rows are in LDS
        if (anyl) {
            size_t ooff = cof + (size_t)s0 * strideV * M;
            asm volatile("" : "+v"(ooff));
            V* out = reinterpret_cast<V*>(a.data + ooff);
            TS* outs = a.data + ooff;
#pragma unroll
            for (int t = 0; t < L; ++t) {
                const TC so = tso[s0 + t];
                if (RAG && s0 + t >= nz) continue;
                if (alll) {
                    V v;
#pragma unroll
                    for (int h = 0; h < M; ++h) v[h] = (TS)(F[h][t] * so);
                    out[(size_t)t * strideV] = v;
                } else {
#pragma unroll
                    for (int h = 0; h < M; ++h)
                        if (act[h]) outs[(size_t)t * M * strideV + h] = (TS)(F[h][t] * so);
                }
            }
        }
        sync_lds_nofence();   // sh is rewritten by the next tile
    }
    __builtin_amdgcn_s_waitcnt(0);   // the last direct loads land before the workgroup's LDS is released
}

// host side (fsei_z.hip, compiled once per type): z_tiling chooses the tiling
// and says whether the special lines go in a launch of their own, ahead of the
// tiles (z_launch_special, then z_launch)
template <typename T>
bool z_tiling(ZArgs<T, T>* a, int cus);
template <typename T>
void z_launch_special(const ZArgs<T, T>& a, hipStream_t st);
template <typename T>
void z_launch(const ZArgs<T, T>& a, hipStream_t st, int cus);

}  // namespace dev
}  // namespace fsei
