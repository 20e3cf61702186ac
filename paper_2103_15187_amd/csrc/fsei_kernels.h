// HIP kernels of the pressure projection for gfx950 (MI355X): the gradient
// correction, the residual norm and the partial-sum reduction.  The transform
// kernels are in fsei_lengths.h and fsei_transforms.h, the z solves in fsei_z.h.
//
// Pass structure of one projection (fields are (nz, ny, nx), x fastest):
//   k_xfwd   : per pair of x-rows, the cell divergence of u* (or the
//              transposed gradient for the adjoint, or the FP64 residual in
//              refinement) fused with the forward x transform
//   k_yfwd   : per tile of x-columns of one z-plane, forward y transform
//   k_zsolve : per (kx, ky) mode, the z tridiagonal, partitioned over the
//              threads of a workgroup (no global scratch); the near-singular
//              lines and the singular (0,0) mode in the same launch
//   k_yinv, k_xinv : inverse transforms (x inverse writes or accumulates p)
//   k_grad   : gradient correction of the three velocity components
#pragma once

#include <hip/hip_runtime.h>

#include "fsei_fft.h"
#include "fsei_plan.h"
#include "fsei_transforms.h"

namespace fsei {
namespace dev {

// ---------------------------------------------------------------------------
// gradient correction on the faces:
//   u += cx (p_i - p_{i-1}),  v += cy (p_j - p_{j-1}),
//   w += sw (bk_k p_k - gk_k p_{k-1});  wall faces written 0.
// forward: cx = -dt/dx, cy = -dt/dy, sw = -dt, bk = gk = 1/h_k
// adjoint (u* <- u - D^T s): cx = 1/dx, cy = 1/dy, sw = 1, bk = 1/dz_k,
//   gk = 1/dz_{k-1}
// ---------------------------------------------------------------------------
template <typename TIO, typename TP>
struct GradArgs {
    int nx, ny, nz, bcx, bcy;
    const TIO* ui;   // velocity in; each the output below or an array that overlaps no output
    const TIO* vi;
    const TIO* wi;
    TIO* u;          // velocity out
    TIO* v;
    TIO* w;
    const TP* p;
    TIO cx, cy, sw;
    const TIO* bk;
    const TIO* gk;
};

template <typename TIO, typename TP, int B>
__global__ __launch_bounds__(256) void k_grad(GradArgs<TIO, TP> a) {
    // one x-row (k, j) per workgroup in XCD-contiguous order.  When ny is a
    // multiple of GJ the rows go in tiles of GJ rows, plane by plane inside a
    // tile: the k-1 row of p was read GJ workgroups earlier and the j-1 row
    // one workgroup earlier on the same XCD (L2 hits), except at tile edges
    constexpr int GJ = 8;
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int nx = a.nx, ny = a.ny;
    int k, j;
    if (ny % GJ == 0) {
        const int per = a.nz * GJ;
        const int jt = b / per;
        const int rem = b - jt * per;
        k = rem / GJ;
        j = jt * GJ + (rem - k * GJ);
    } else {
        k = b / ny;
        j = b - k * ny;
    }
    const long row = (long)k * ny + j;
    const size_t base = (size_t)row * nx;
    const TP* __restrict__ p = a.p;
    const TIO bk = a.bk[k], gk = a.gk[k];
    const size_t jm = (j > 0) ? (size_t)nx : (size_t)0 - (size_t)(ny - 1) * nx;   // offset to row j-1
    // B columns per thread and batch, every load before the first store (the
    // outputs may be the inputs, so the compiler cannot move them)
    for (int i0 = threadIdx.x; i0 < nx; i0 += B * 256) {
        TIO pc[B], px[B], py[B], pz[B], uo[B], vo[B], wo[B];
#pragma unroll
        for (int t = 0; t < B; ++t) {
            const int i = i0 + t * 256;
            if (i < nx) {
                const size_t idx = base + i;
                pc[t] = (TIO)p[idx];
                px[t] = (TIO)p[(i > 0) ? idx - 1 : idx + nx - 1];
                py[t] = (TIO)p[idx - jm];
                pz[t] = (k > 0) ? (TIO)p[idx - (size_t)nx * ny] : (TIO)0;
                uo[t] = a.ui[idx];
                vo[t] = a.vi[idx];
                wo[t] = a.wi[idx];
            }
        }
#pragma unroll
        for (int t = 0; t < B; ++t) {
            const int i = i0 + t * 256;
            if (i < nx) {
                const size_t idx = base + i;
                a.u[idx] = (a.bcx == FSEI_BC_WALL && i == 0) ? (TIO)0 : uo[t] + a.cx * (pc[t] - px[t]);
                a.v[idx] = (a.bcy == FSEI_BC_WALL && j == 0) ? (TIO)0 : vo[t] + a.cy * (pc[t] - py[t]);
                a.w[idx] = (k == 0) ? (TIO)0 : wo[t] + a.sw * (bk * pc[t] - gk * pz[t]);
            }
        }
    }
}

// One x-row per workgroup, one cell pair per lane (NT >= nx / 2): the
// simplest streaming shape, which runs closest to the HBM ceiling.  Rows in
// tiles of GJ rows (ny % GJ == 0), plane by plane inside a tile (as k_grad).
template <typename TIO, typename TP, int NT, int GJ>
__global__ __launch_bounds__(NT) void k_grad_row2(GradArgs<TIO, TP> a) {
    using V = typename Vec2T<TIO>::type;
    using VP = typename Vec2T<TP>::type;
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int nx = a.nx, ny = a.ny;
    const int per = a.nz * GJ;
    const int jt = b / per;
    const int rem = b - jt * per;
    const int k = rem / GJ;
    const int j = jt * GJ + (rem - k * GJ);
    const unsigned i = 2u * threadIdx.x;
    if (i >= (unsigned)nx) return;
    const size_t nxy = (size_t)nx * ny;
    const size_t ro = (size_t)k * nxy + (size_t)j * nx;
    const TP* __restrict__ pr = a.p + ro;
    const TP* __restrict__ py = (j > 0) ? pr - nx : pr + (size_t)(ny - 1) * nx;   // j-1, wrapped
    const TP* __restrict__ pz = (k > 0) ? pr - nxy : pr;                           // unused at k = 0
    const unsigned im = (i > 0) ? i - 1 : (unsigned)nx - 1;
    const VP pc = *reinterpret_cast<const VP*>(pr + i);
    const TP pxm = pr[im];
    const VP pyv = *reinterpret_cast<const VP*>(py + i);
    const VP pzv = *reinterpret_cast<const VP*>(pz + i);
    TIO* u = a.u + ro;
    TIO* v = a.v + ro;
    TIO* w = a.w + ro;
    const V uo = *reinterpret_cast<const V*>(a.ui + ro + i);
    const V vo = *reinterpret_cast<const V*>(a.vi + ro + i);
    const V wo = *reinterpret_cast<const V*>(a.wi + ro + i);
    const TIO bk = a.bk[k], gk = a.gk[k];
    V un, vn, wn;
    un.x = (a.bcx == FSEI_BC_WALL && i == 0) ? (TIO)0 : uo.x + a.cx * ((TIO)pc.x - (TIO)pxm);
    un.y = uo.y + a.cx * ((TIO)pc.y - (TIO)pc.x);
    const bool v0 = a.bcy == FSEI_BC_WALL && j == 0;
    vn.x = v0 ? (TIO)0 : vo.x + a.cy * ((TIO)pc.x - (TIO)pyv.x);
    vn.y = v0 ? (TIO)0 : vo.y + a.cy * ((TIO)pc.y - (TIO)pyv.y);
    wn.x = (k == 0) ? (TIO)0 : wo.x + a.sw * (bk * (TIO)pc.x - gk * (TIO)pzv.x);
    wn.y = (k == 0) ? (TIO)0 : wo.y + a.sw * (bk * (TIO)pc.y - gk * (TIO)pzv.y);
    *reinterpret_cast<V*>(u + i) = un;
    *reinterpret_cast<V*>(v + i) = vn;
    *reinterpret_cast<V*>(w + i) = wn;
}

// ---------------------------------------------------------------------------
// FP64 residual norm of the refinement, r = (f - mean) - L p: per-block
// (sum r^2, sum r, sum dz_k p) partials.  The third sum is the volume
// integral of the iterate (over dx dy): the residual is blind to constants,
// so this is what lets a correction pin the V-mean of p in FP64.  Lanes own
// two adjacent x-cells (16-byte accesses), workgroups RJ rows of one
// z-plane, tiles plane-fastest (the k-1 rows of p were read by the previous
// workgroup on the same XCD); the j-1 / j+1 rows rotate through registers.
// ---------------------------------------------------------------------------
template <typename TPP>
struct ResArgs {
    int nx, ny, nz, bcx, bcy;
    const double* f;
    const TPP* p;         // pressure iterate (FP64, or the first FP32 solve)
    double idx2, idy2;
    const double* za;
    const double* zc;
    const double* scal;   // scal[0] = removed mean
    const double* dz;     // cell widths dz_k (third partial)
    double* partials;
};

// two adjacent values of T as a double2
template <typename T>
__device__ __forceinline__ double2 ld2d(const T* q) {
    const auto v = *reinterpret_cast<const typename Vec2T<T>::type*>(q);
    return make_double2((double)v.x, (double)v.y);
}

template <int NT, int RJ, typename TPP, int RB = 2>   // RB: rows per load batch
__global__ __launch_bounds__(NT) void k_resid_pairs(ResArgs<TPP> a) {
    static_assert(RJ % RB == 0, "whole batches");
    __shared__ double sred[3 * (NT / 64)];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int jt = b / nz;
    const int k = b - jt * nz;
    const int j0 = jt * RJ;
    const size_t nxy = (size_t)nx * ny;
    const TPP* __restrict__ pk = a.p + (size_t)k * nxy;
    const TPP* __restrict__ pkm = (k > 0) ? pk - nxy : pk;
    const TPP* __restrict__ pkp = (k + 1 < nz) ? pk + nxy : pk;
    const double* __restrict__ fk = a.f + (size_t)k * nxy;
    const double czm = (k > 0) ? a.za[k] : 0.0, czp = (k + 1 < nz) ? a.zc[k] : 0.0;
    const bool hzm = k > 0, hzp = k + 1 < nz;
    const bool pery = a.bcy == FSEI_BC_PERIODIC, perx = a.bcx == FSEI_BC_PERIODIC;
    const double mean = a.scal[0];
    double ss = 0.0, s1 = 0.0, sp = 0.0;
    for (int c = threadIdx.x; 2 * c < nx; c += NT) {
        const unsigned i = 2u * (unsigned)c;
        // x neighbours of the pair: i - 1 and i + 2 (wrapped)
        const unsigned im = (i > 0) ? i - 1 : (unsigned)nx - 1;
        const unsigned ip = (i + 2 < (unsigned)nx) ? i + 2 : 0u;
        const bool him = (i > 0) || perx, hip = (i + 2 < (unsigned)nx) || perx;
        const int jm0 = (j0 > 0) ? j0 - 1 : ny - 1;
        double2 pm = ld2d(pk + (size_t)jm0 * nx + i);
        double2 pc = ld2d(pk + (size_t)j0 * nx + i);
#pragma unroll
        for (int l0 = 0; l0 < RJ; l0 += RB) {
            double2 pn[RB], pzm[RB], pzp[RB], fc[RB];
            double pxm[RB], pxp[RB];
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int j = j0 + l0 + r;
                const size_t ro = (size_t)j * nx;
                const int jn = (j + 1 < ny) ? j + 1 : 0;
                pn[r] = ld2d(pk + (size_t)jn * nx + i);
                pxm[r] = (double)pk[ro + im];
                pxp[r] = (double)pk[ro + ip];
                pzm[r] = ld2d(pkm + ro + i);
                pzp[r] = ld2d(pkp + ro + i);
                fc[r] = *reinterpret_cast<const double2*>(fk + ro + i);
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int j = j0 + l0 + r;
                const bool hym = (j > 0) || pery, hyp = (j + 1 < ny) || pery;
                // cell i: x neighbours i+1 (= pc.y) and i-1; cell i+1: i+2 and i
                const double lx0 = (pc.y - pc.x) + (him ? pxm[r] - pc.x : 0.0);
                const double lx1 = (hip ? pxp[r] - pc.y : 0.0) + (pc.x - pc.y);
                const double ly0 = (hyp ? pn[r].x - pc.x : 0.0) + (hym ? pm.x - pc.x : 0.0);
                const double ly1 = (hyp ? pn[r].y - pc.y : 0.0) + (hym ? pm.y - pc.y : 0.0);
                const double lz0 = (hzp ? czp * (pzp[r].x - pc.x) : 0.0) + (hzm ? czm * (pzm[r].x - pc.x) : 0.0);
                const double lz1 = (hzp ? czp * (pzp[r].y - pc.y) : 0.0) + (hzm ? czm * (pzm[r].y - pc.y) : 0.0);
                const double r0 = (fc[r].x - mean) - (lx0 * a.idx2 + ly0 * a.idy2 + lz0);
                const double r1 = (fc[r].y - mean) - (lx1 * a.idx2 + ly1 * a.idy2 + lz1);
                ss += r0 * r0 + r1 * r1;
                s1 += r0 + r1;
                sp += pc.x + pc.y;
                pm = pc;
                pc = pn[r];
            }
        }
    }
    double s2 = a.dz[k] * sp;   // every row of the block is in plane k
    block_sum3<NT>(ss, s1, s2, sred);
    if (threadIdx.x == 0) {
        a.partials[3 * blockIdx.x] = ss;
        a.partials[3 * blockIdx.x + 1] = s1;
        a.partials[3 * blockIdx.x + 2] = s2;
    }
}

// ---------------------------------------------------------------------------
// Gradient correction fused with the FP64 residual norm of the refinement's
// current pressure iterate: u += cx (g_i - g_{i-1}), v += cy (g_j - g_{j-1}),
// w += sw (bk_k g_k - gk_k g_{k-1}) with g = p (or, DELTA, with g = the last
// correction c, applied on top of an earlier update), and the partials
// (sum r^2, sum r, 0) of r = (f - mean) - L p.  Pair tiling as
// k_resid_pairs.  The convergence check of the last correction then costs no
// pass of its own.
// ---------------------------------------------------------------------------
struct GradResArgs {
    int nx, ny, nz, bcx, bcy;
    const double* ui;     // velocity in (the outputs, or arrays that overlap none)
    const double* vi;
    const double* wi;
    double* u;            // velocity out
    double* v;
    double* w;
    const double* p;      // current iterate (residual; gradient unless DELTA)
    const float* c;       // DELTA: the correction whose gradient is applied
    double cx, cy, sw;
    const double* bk;
    const double* gk;
    const double* f;
    double idx2, idy2;
    const double* za;
    const double* zc;
    const double* scal;   // scal[0] = removed mean
    double* partials;
};

template <int NT, int RJ, bool DELTA>
__global__ __launch_bounds__(NT) void k_grad_resid(GradResArgs a) {
    constexpr int RB = 2;   // rows per load batch (20 doubles per row in flight)
    static_assert(RJ % RB == 0, "whole batches");
    __shared__ double sred[3 * (NT / 64)];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int jt = b / nz;
    const int k = b - jt * nz;
    const int j0 = jt * RJ;
    const size_t nxy = (size_t)nx * ny;
    const size_t pl = (size_t)k * nxy;
    const double* __restrict__ pk = a.p + pl;
    const double* __restrict__ pkm = (k > 0) ? pk - nxy : pk;
    const double* __restrict__ pkp = (k + 1 < nz) ? pk + nxy : pk;
    const float* __restrict__ ck = DELTA ? a.c + pl : nullptr;
    const float* __restrict__ ckm = (DELTA && k > 0) ? ck - nxy : ck;
    const double* __restrict__ fk = a.f + pl;
    const double* ui = a.ui + pl;
    const double* vi = a.vi + pl;
    const double* wi = a.wi + pl;
    double* uk = a.u + pl;
    double* vk = a.v + pl;
    double* wk = a.w + pl;
    const double czm = (k > 0) ? a.za[k] : 0.0, czp = (k + 1 < nz) ? a.zc[k] : 0.0;
    const bool hzm = k > 0, hzp = k + 1 < nz;
    const bool pery = a.bcy == FSEI_BC_PERIODIC, perx = a.bcx == FSEI_BC_PERIODIC;
    const bool wallx = !perx, wally = !pery;
    const double mean = a.scal[0];
    const double bkk = a.bk[k], gkk = a.gk[k];
    double ss = 0.0, s1 = 0.0;
    for (int c = threadIdx.x; 2 * c < nx; c += NT) {
        const unsigned i = 2u * (unsigned)c;
        const unsigned im = (i > 0) ? i - 1 : (unsigned)nx - 1;
        const unsigned ip = (i + 2 < (unsigned)nx) ? i + 2 : 0u;
        const bool him = (i > 0) || perx, hip = (i + 2 < (unsigned)nx) || perx;
        const int jm0 = (j0 > 0) ? j0 - 1 : ny - 1;
        double2 pm = ld2d(pk + (size_t)jm0 * nx + i);
        double2 pc = ld2d(pk + (size_t)j0 * nx + i);
        double2 cm = make_double2(0.0, 0.0);
        if constexpr (DELTA) cm = ld2d(ck + (size_t)jm0 * nx + i);
#pragma unroll
        for (int l0 = 0; l0 < RJ; l0 += RB) {
            double2 pn[RB], pzm[RB], pzp[RB], fc[RB], uo[RB], vo[RB], wo[RB], cc[RB], czk[RB];
            double pxm[RB], pxp[RB], cxm[RB];
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int j = j0 + l0 + r;
                const size_t ro = (size_t)j * nx;
                const int jn = (j + 1 < ny) ? j + 1 : 0;
                pn[r] = ld2d(pk + (size_t)jn * nx + i);
                pxm[r] = pk[ro + im];
                pxp[r] = pk[ro + ip];
                pzm[r] = ld2d(pkm + ro + i);
                pzp[r] = ld2d(pkp + ro + i);
                fc[r] = ld2d(fk + ro + i);
                uo[r] = ld2d(ui + ro + i);
                vo[r] = ld2d(vi + ro + i);
                wo[r] = ld2d(wi + ro + i);
                if constexpr (DELTA) {
                    cc[r] = ld2d(ck + ro + i);
                    cxm[r] = (double)ck[ro + im];
                    czk[r] = ld2d(ckm + ro + i);
                }
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
                const int j = j0 + l0 + r;
                const size_t ro = (size_t)j * nx;
                const bool hym = (j > 0) || pery, hyp = (j + 1 < ny) || pery;
                // residual of the current iterate (as k_resid_pairs)
                const double lx0 = (pc.y - pc.x) + (him ? pxm[r] - pc.x : 0.0);
                const double lx1 = (hip ? pxp[r] - pc.y : 0.0) + (pc.x - pc.y);
                const double ly0 = (hyp ? pn[r].x - pc.x : 0.0) + (hym ? pm.x - pc.x : 0.0);
                const double ly1 = (hyp ? pn[r].y - pc.y : 0.0) + (hym ? pm.y - pc.y : 0.0);
                const double lz0 = (hzp ? czp * (pzp[r].x - pc.x) : 0.0) + (hzm ? czm * (pzm[r].x - pc.x) : 0.0);
                const double lz1 = (hzp ? czp * (pzp[r].y - pc.y) : 0.0) + (hzm ? czm * (pzm[r].y - pc.y) : 0.0);
                const double r0 = (fc[r].x - mean) - (lx0 * a.idx2 + ly0 * a.idy2 + lz0);
                const double r1 = (fc[r].y - mean) - (lx1 * a.idx2 + ly1 * a.idy2 + lz1);
                ss += r0 * r0 + r1 * r1;
                s1 += r0 + r1;
                // gradient of g = p, or of the correction c
                const double2 gc = DELTA ? cc[r] : pc;
                const double2 gm = DELTA ? cm : pm;
                const double gxm = DELTA ? cxm[r] : pxm[r];
                const double2 gz = DELTA ? czk[r] : pzm[r];
                double2 un, vn, wn;
                un.x = (wallx && i == 0) ? 0.0 : uo[r].x + a.cx * (gc.x - gxm);
                un.y = uo[r].y + a.cx * (gc.y - gc.x);
                const bool v0 = wally && j == 0;
                vn.x = v0 ? 0.0 : vo[r].x + a.cy * (gc.x - gm.x);
                vn.y = v0 ? 0.0 : vo[r].y + a.cy * (gc.y - gm.y);
                wn.x = (k == 0) ? 0.0 : wo[r].x + a.sw * (bkk * gc.x - gkk * gz.x);
                wn.y = (k == 0) ? 0.0 : wo[r].y + a.sw * (bkk * gc.y - gkk * gz.y);
                *reinterpret_cast<double2*>(uk + ro + i) = un;
                *reinterpret_cast<double2*>(vk + ro + i) = vn;
                *reinterpret_cast<double2*>(wk + ro + i) = wn;
                pm = pc;
                pc = pn[r];
                if constexpr (DELTA) cm = cc[r];
            }
            // keep the next batch's loads after this batch's stores (bounds
            // the registers to one batch)
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    double s2 = 0.0;
    block_sum3<NT>(ss, s1, s2, sred);
    if (threadIdx.x == 0) {
        a.partials[3 * blockIdx.x] = ss;
        a.partials[3 * blockIdx.x + 1] = s1;
        a.partials[3 * blockIdx.x + 2] = 0.0;
    }
}

// out = (double) in, n values (grid-stride)
__global__ __launch_bounds__(256) void k_widen(const float* __restrict__ in, double* __restrict__ out, size_t n) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
        out[i] = (double)in[i];
}

// deterministic sum of the per-block partial triples: one workgroup of NT
// threads, 8 triples in flight per thread, fixed summation order; optionally
// also mean_out = (third sum) * mean_scale
template <int NT>
__global__ __launch_bounds__(NT) void k_sum_partials(const double* part, int nblk, double* out, double* mean_out,
                                                    double mean_scale) {
    __shared__ double sh[3 * (NT / 64)];
    double a = 0.0, b = 0.0, c = 0.0;
    for (int t0 = threadIdx.x; t0 < nblk; t0 += 8 * NT) {
        double v[8][3];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int t = t0 + r * NT;
#pragma unroll
            for (int q = 0; q < 3; ++q) v[r][q] = (t < nblk) ? part[3 * t + q] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            a += v[r][0];
            b += v[r][1];
            c += v[r][2];
        }
    }
    block_sum3<NT>(a, b, c, sh);
    if (threadIdx.x == 0) {
        out[0] = a;
        out[1] = b;
        out[2] = c;
        if (mean_out) *mean_out = c * mean_scale;
    }
}

// first stage of the two-stage sum: workgroup g sums the triples
// [g * chunk, min(nblk, (g + 1) * chunk)) in a fixed order into grp[3 g ..]
__global__ __launch_bounds__(256) void k_sum_partials_grp(const double* part, int nblk, int chunk, double* grp) {
    __shared__ double sh[3 * 4];
    const int lo = blockIdx.x * chunk;
    const int hi = (lo + chunk < nblk) ? lo + chunk : nblk;
    double a = 0.0, b = 0.0, c = 0.0;
    for (int t0 = lo + (int)threadIdx.x; t0 < hi; t0 += 4 * 256) {
        double v[4][3];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = t0 + r * 256;
#pragma unroll
            for (int q = 0; q < 3; ++q) v[r][q] = (t < hi) ? part[3 * t + q] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            a += v[r][0];
            b += v[r][1];
            c += v[r][2];
        }
    }
    block_sum3<256>(a, b, c, sh);
    if (threadIdx.x == 0) {
        grp[3 * blockIdx.x] = a;
        grp[3 * blockIdx.x + 1] = b;
        grp[3 * blockIdx.x + 2] = c;
    }
}

}  // namespace dev
}  // namespace fsei
