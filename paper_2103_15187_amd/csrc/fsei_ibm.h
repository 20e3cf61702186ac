// fsei_ibm.h -- immersed-boundary moving-least-squares (IB-MLS) transfer
// between Lagrangian markers and one staggered velocity component.
//
// Paper, Sec. 2.1 (eq. interpv, Fig. mls): each marker x_b has a support of
// 3 x 3 x 3 nodes of the component's own lattice; the velocity at the marker
// is sum_k phi_k u_k with moving-least-squares operators on the linear basis
// [1, x, y, z] and an exponential weight centred on the marker; the force
// computed at the marker goes back to the same nodes as a distributed forcing.
//
//     A = sum_k W_k p_k p_k^T,  p_k = [1, x_k - x_b, y_k - y_b, z_k - z_b],
//     phi_k = W_k (A^-1 e_0) . p_k,
//     W_k = exp(-(dx_k/dx)^2 - (dy_k/dy)^2 - (dz_k/hz)^2),
//
// hz the z extent of the support's middle node (cell width for centre
// values, centre distance for w faces).  Supports are the three nodes around
// the nearest one, shifted inwards at walls and wrapped in periodic
// directions (displacements to the nearest periodic image).  One lane per
// marker.  The weight is a product over the axes, so A is diagonal in the basis
// centred on the weighted means: with n the weights of an axis over their sum,
// m = sum n d the mean displacement and v = sum n (d - m)^2,
//     phi = n_x n_y n_z (1 - g_x - g_y - g_z),   g = m (d - m) / v
// (sum phi = 1, sum phi d = 0 on each axis).
#pragma once

#include <hip/hip_runtime.h>

#include "fsei_plan.h"

namespace fsei {
namespace dev {

struct IbArgs {
    int nx, ny, nz, perx, pery, comp;
    long nb;
    double dx, dy;
    const double* zn;    // z of the component's nodes (faces for w, centres otherwise), nz
    const double* hz;    // z extent of each node's control volume, nz
    const double* xb;    // markers (nb, 3)
    double* field;       // interpolate: read; spread: += (atomic)
    double* ub;          // interpolate: out (nb)
    const double* fb;    // spread: marker values (nb)
    const double* dvb;   // spread: marker volumes (nb)
};

// support along a uniform axis: first index and displacements of its 3 nodes
__device__ __forceinline__ void ib_axis(double xb, double x0, double d, int n, bool per, int (&idx)[3],
                                        double (&dis)[3]) {
    double t = (xb - x0) / d;
    if (!(t == t)) t = 0.0;                       // NaN position: any in-grid support
    t = fmin(fmax(t, -1.0e9), 1.0e9);
    long m = (long)floor(t + 0.5);
    const double L = d * n;
    if (per) {
        m = ((m % n) + n) % n;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int i = (int)((m + q - 1 + n) % n);
            double dd = x0 + i * d - xb;
            dd -= L * rint(dd / L);
            idx[q] = i;
            dis[q] = dd;
        }
    } else {
        m = m < 1 ? 1 : (m > n - 2 ? n - 2 : m);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            idx[q] = (int)(m + q - 1);
            dis[q] = x0 + idx[q] * d - xb;
        }
    }
}

// support along z: nearest node by bisection on the node coordinates
__device__ __forceinline__ int ib_zmid(const double* __restrict__ zn, int n, double zb) {
    int lo = 0, hi = n - 1;   // zn increasing
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (zn[mid] <= zb) lo = mid;
        else hi = mid;
    }
    int m = (fabs(zn[hi] - zb) < fabs(zn[lo] - zb)) ? hi : lo;
    return m < 1 ? 1 : (m > n - 2 ? n - 2 : m);
}

// one axis of a marker's support: node indices, n and g of the three nodes
struct IbAxis {
    int idx[3];
    double n[3], g[3];
    // Deviations and variance from the differences of the nodes, and the
    // weights over that of the nearest one: exact to rounding also for markers
    // far beyond a wall, whose nearest node has all but 1e-9 of the weight at ten cells
    // (taken from the mean, they lost all digits at 16 cells).
    __device__ __forceinline__ void weigh(const double (&dis)[3], double scale) {
        double e[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const double r = dis[q] / scale;
            e[q] = r * r;
        }
        const double least = fmin(fmin(e[0], e[1]), e[2]);
#pragma unroll
        for (int q = 0; q < 3; ++q) e[q] = exp(least - e[q]);
        const double rs = 1.0 / (e[0] + e[1] + e[2]);
        double mean = 0.0;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            n[q] = e[q] * rs;
            mean += n[q] * dis[q];
        }
        const double d10 = dis[1] - dis[0], d20 = dis[2] - dis[0], d21 = dis[2] - dis[1];
        g[0] = -(n[1] * d10 + n[2] * d20);
        g[1] = n[0] * d10 - n[2] * d21;
        g[2] = n[0] * d20 + n[1] * d21;
        const double mv = mean / (n[0] * (n[1] * d10 * d10 + n[2] * d20 * d20) + n[1] * n[2] * d21 * d21);
#pragma unroll
        for (int q = 0; q < 3; ++q) g[q] *= mv;
    }
};

struct IbSupport {
    IbAxis x, y, z;
};

__device__ __forceinline__ IbSupport ib_support(const IbArgs& a, long b) {
    IbSupport s;
    double dis[3];
    const double xbx = a.xb[3 * b], xby = a.xb[3 * b + 1], xbz = a.xb[3 * b + 2];
    const int mz = ib_zmid(a.zn, a.nz, (xbz == xbz) ? xbz : 0.0);
    ib_axis(xbx, a.comp == 0 ? 0.0 : 0.5 * a.dx, a.dx, a.nx, a.perx, s.x.idx, dis);
    s.x.weigh(dis, a.dx);
    ib_axis(xby, a.comp == 1 ? 0.0 : 0.5 * a.dy, a.dy, a.ny, a.pery, s.y.idx, dis);
    s.y.weigh(dis, a.dy);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        s.z.idx[q] = mz + q - 1;
        dis[q] = a.zn[s.z.idx[q]] - xbz;
    }
    s.z.weigh(dis, a.hz[mz]);
    return s;
}

// flat offset of node (0, jj, kk) of the support's row, without x; IT: 32-bit
// offsets when the field has fewer than 2^32 cells, else 64-bit
template <typename IT>
__device__ __forceinline__ IT ib_row(const IbArgs& a, const IbSupport& s, int jj, int kk) {
    return ((IT)s.z.idx[kk] * (IT)a.ny + (IT)s.y.idx[jj]) * (IT)a.nx;
}

// u(x_b) = sum_k phi_k u_k: two sums per x row (sum n u and sum n (1 - g_x) u),
// combined with the row's weight and g_y + g_z.  Bound by the 27 gathers.
// Weights, moments and a Cholesky factor per node and marker (27 exponentials
// instead of 9) made it instruction bound: 80 us for 998 200 surface markers at
// 512x512x768, 50 us now.
template <typename IT>
__global__ __launch_bounds__(256) void k_ib_interpolate(IbArgs a) {
    const long b = (long)blockIdx.x * 256 + threadIdx.x;
    if (b >= a.nb) return;
    const IbSupport s = ib_support(a, b);
    double val[9][3];
#pragma unroll
    for (int r = 0; r < 9; ++r) {
        const IT row = ib_row<IT>(a, s, r % 3, r / 3);
#pragma unroll
        for (int ii = 0; ii < 3; ++ii) val[r][ii] = a.field[row + (IT)s.x.idx[ii]];
    }
    double wx[3], u = 0.0;
#pragma unroll
    for (int ii = 0; ii < 3; ++ii) wx[ii] = s.x.n[ii] * (1.0 - s.x.g[ii]);
#pragma unroll
    for (int r = 0; r < 9; ++r) {
        const int jj = r % 3, kk = r / 3;
        const double t0 = s.x.n[0] * val[r][0] + s.x.n[1] * val[r][1] + s.x.n[2] * val[r][2];
        const double t1 = wx[0] * val[r][0] + wx[1] * val[r][1] + wx[2] * val[r][2];
        u += s.y.n[jj] * s.z.n[kk] * (t1 - (s.y.g[jj] + s.z.g[kk]) * t0);
    }
    a.ub[b] = u;
}

// the contribution of a marker of strength f to node (ii, jj, kk); wr: the
// row's n_y n_z f / hz_k
__device__ __forceinline__ double ib_share(const IbSupport& s, double wr, int ii, int jj, int kk) {
    return s.x.n[ii] * wr * (1.0 - s.x.g[ii] - (s.y.g[jj] + s.z.g[kk]));
}

// f_k += phi_k F_b dV_b / (dx dy hz_k), one global atomic per node and marker
template <typename IT>
__global__ __launch_bounds__(256) void k_ib_spread(IbArgs a) {
    const long b = (long)blockIdx.x * 256 + threadIdx.x;
    if (b >= a.nb) return;
    const IbSupport s = ib_support(a, b);
    const double f = a.fb[b] * a.dvb[b] / (a.dx * a.dy);
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) {
        const double fk = f / a.hz[s.z.idx[kk]] * s.z.n[kk];   // over the z extent of the plane's nodes
#pragma unroll
        for (int jj = 0; jj < 3; ++jj) {
            const IT row = ib_row<IT>(a, s, jj, kk);
#pragma unroll
            for (int ii = 0; ii < 3; ++ii)
                atomicAdd(a.field + row + (IT)s.x.idx[ii], ib_share(s, fk * s.y.n[jj], ii, jj, kk));
        }
    }
}

// Spreading with the adds of one workgroup's markers combined in LDS first.
// Markers that come in mesh order (neighbours on the surface next to each
// other) share most of their support nodes: a workgroup's 256 x 27
// contributions land on about 6 nodes per marker, in about 2.3 aligned runs of
// four nodes (32 bytes).  An open-addressing table of runs (run number, four
// sums; bounded linear probing, a contribution that finds no slot goes
// straight to the global atomic) collects them, and its sums are then added to
// the field by four adjacent lanes per run: the L2 takes the atomics of one
// instruction to one line together, where sums kept per node in hash order
// cost one line each (2.3e10 atomics/s; 309 us for 998 200 surface markers at
// 512x512x768, 137 us now with the cheaper weights; runs of 8 and 16 nodes,
// whose tables leave two workgroups per CU, 144 and 176 us).  Markers that share
// no nodes: 1.23 -> 1.06 ms per million.  Needs 32-bit offsets: the empty key
// is no run number.
//
// FEW: at most one workgroup per CU, so that the launch takes as long as one
// marker's chain of probes, and longest where markers share no nodes and the
// table overflows.  There a probe is one compare-and-swap (no read first), four
// probes look for a slot, and a marker that found none adds the rest of its runs
// directly.  Markers apart / on one
// surface / at one point, 4000 each, us: 18 / 17 / 19 (as for many markers 37 /
// 37 / 18, and 34 / 34 / 23 with a key per node).  With many markers the reads
// and the eight probes are the faster: 998 200 on the surface 131 against 157.
constexpr int kIbRun = 4;
constexpr int kIbSlots = 1024;   // runs in the table: 36 KB, four workgroups per CU
constexpr unsigned kIbEmpty = 0xFFFFFFFFu;

template <bool FEW>
__global__ __launch_bounds__(256) void k_ib_spread_lds(IbArgs a) {
    constexpr int PROBES = FEW ? 4 : 8;
    __shared__ unsigned skey[kIbSlots];
    __shared__ double sval[kIbSlots * kIbRun];
    for (int t = threadIdx.x; t < kIbSlots; t += 256) skey[t] = kIbEmpty;
    for (int t = threadIdx.x; t < kIbSlots * kIbRun; t += 256) sval[t] = 0.0;
    __syncthreads();
    // slot of a run, or -1
    auto find = [&](unsigned run) -> int {
        unsigned h = (run * 2654435761u) / (unsigned)(0x100000000ull / kIbSlots);
        for (int pr = 0; pr < PROBES; ++pr) {
            unsigned old = FEW ? kIbEmpty : *(volatile unsigned*)&skey[h];   // (many: most finds meet their run)
            if (old == kIbEmpty) old = atomicCAS(&skey[h], kIbEmpty, run);
            if (old == kIbEmpty || old == run) return (int)h;
            h = (h + 1) % kIbSlots;
        }
        return -1;
    };
    const long b = (long)blockIdx.x * 256 + threadIdx.x;
    if (b < a.nb) {
        const IbSupport s = ib_support(a, b);
        const double f = a.fb[b] * a.dvb[b] / (a.dx * a.dy);
        bool look = true;
#pragma unroll
        for (int kk = 0; kk < 3; ++kk) {
            const double fk = f / a.hz[s.z.idx[kk]] * s.z.n[kk];
#pragma unroll
            for (int jj = 0; jj < 3; ++jj) {
                const unsigned row = ib_row<unsigned>(a, s, jj, kk);
                unsigned run = kIbEmpty;
                int slot = -1;
#pragma unroll
                for (int ii = 0; ii < 3; ++ii) {
                    const unsigned key = row + (unsigned)s.x.idx[ii];
                    const double v = ib_share(s, fk * s.y.n[jj], ii, jj, kk);
                    if (key / kIbRun != run) {
                        run = key / kIbRun;
                        slot = look ? find(run) : -1;
                        if (FEW) look = slot >= 0;
                    }
                    if (slot >= 0) atomicAdd(&sval[slot * kIbRun + key % kIbRun], v);
                    else atomicAdd(a.field + key, v);
                }
            }
        }
    }
    __syncthreads();
    // a sum that is exactly 0 (a node of the run that no marker reached, among
    // them any beyond the field's end) adds nothing
    for (int t = threadIdx.x; t < kIbSlots * kIbRun; t += 256) {
        const double v = sval[t];
        const unsigned run = skey[t / kIbRun];
        if (run != kIbEmpty && v != 0.0) atomicAdd(a.field + (size_t)run * kIbRun + t % kIbRun, v);
    }
}

}  // namespace dev
}  // namespace fsei
