// Transform kernels of the pressure projection for gfx950 (MI355X): the x
// transforms (fused with the divergence / transposed-gradient / residual
// stencils on the way in and the pressure write or accumulation on the way
// out) and the y transforms.
//
// Transforms (paper, Program summary: FFTW in the homogeneous directions):
// two real lines a, b travel as one complex sequence z = a + i b through a
// length-N FFT.  Walls use the DCT-II basis cos(pi q (i+1/2)/N), computed from
// the even/odd reordering v_n = x_{2n}, v_{N-1-n} = x_{2n+1} and a post-twiddle
// exp(-i pi q / 2N) (Makhoul's method); periodic directions use the real DFT
// in half-complex layout (real parts at rows 0..N/2, imaginary parts of mode
// m at row N-m).  Both inverses are unnormalised (they return N times the
// input); the z solve folds in the factor 1/(nx ny).
//
// The kernels here take the length from the arguments: they serve the lengths
// below 16 and above 1024 and fields that are not aligned to column pairs; the
// other lengths have kernels compiled for them (fsei_lengths.h).  Tile loops
// have compile-time trip counts and are unrolled; addresses are 32-bit offsets
// from per-workgroup base pointers.
#pragma once

#include <hip/hip_runtime.h>

#include "fsei_fft.h"
#include "fsei_plan.h"

namespace fsei {
namespace dev {

// position of element i in the even/odd reordered sequence (walls)
__device__ __forceinline__ int mk_pos(int i, int N) { return (i & 1) ? N - 1 - (i >> 1) : (i >> 1); }

// Workgroups are handed to the 8 XCDs of the chip round-robin (workgroup i
// runs on XCD i % 8), and each XCD has its own L2.  This bijection of
// [0, n) gives XCD x a contiguous run of logical blocks, so blocks that
// touch neighbouring rows and planes (stencil halos) share an L2.
constexpr int kXcds = 8;
__device__ __forceinline__ long xcd_remap(long i, long n) {
    const long q = n / kXcds, r = n % kXcds;
    const long x = i % kXcds, t = i / kXcds;
    return x * q + (x < r ? x : r) + t;
}

// deterministic block sum of three values (result valid in thread 0)
template <int NTHR>
__device__ __forceinline__ void block_sum3(double& a, double& b, double& c, double* sh) {
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
        c += __shfl_down(c, off, 64);
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) {
        sh[3 * wid] = a;
        sh[3 * wid + 1] = b;
        sh[3 * wid + 2] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sa = 0.0, sb = 0.0, sc = 0.0;
        for (int w = 0; w < NTHR / 64; ++w) {
            sa += sh[3 * w];
            sb += sh[3 * w + 1];
            sc += sh[3 * w + 2];
        }
        a = sa;
        b = sb;
        c = sc;
    }
    __syncthreads();
}

// the length-N twiddle table exp(2 pi i t / N) in LDS (2 N values, in the
// kernel's dynamic LDS)
template <typename T>
__device__ __forceinline__ T* lds_twiddle_ptr() {
    extern __shared__ __align__(16) unsigned char dyn_lds[];
    return reinterpret_cast<T*>(dyn_lds);
}

// copies the twiddle table into LDS; visible after the next barrier.  The
// compile-time-length kernels call this after issuing their first field
// loads, so that the table's round trip overlaps theirs.
template <typename T, int NTHR>
__device__ __forceinline__ void stage_twiddles(T* twl, const T* __restrict__ twc, const T* __restrict__ tws, int N) {
    for (int t = threadIdx.x; t < N; t += NTHR) {
        twl[t] = twc[t];
        twl[N + t] = tws[t];
    }
}

// Compile-time length: the table is read into registers first (before the
// kernel's field loads are issued) and written to LDS after them, so its
// round trip overlaps theirs instead of preceding it.
template <typename T, int NTHR, int NF>
struct TwiddleRegs {
    static constexpr int IT = (NF + NTHR - 1) / NTHR;
    T c[IT], s[IT];
    __device__ __forceinline__ void load(const T* __restrict__ twc, const T* __restrict__ tws) {
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int t = threadIdx.x + r * NTHR;
            c[r] = (t < NF) ? twc[t] : (T)0;
            s[r] = (t < NF) ? tws[t] : (T)0;
        }
    }
    __device__ __forceinline__ void store(T* twl) const {
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int t = threadIdx.x + r * NTHR;
            if (t < NF) {
                twl[t] = c[r];
                twl[NF + t] = s[r];
            }
        }
    }
};

template <typename T, int NTHR>
__device__ __forceinline__ T* lds_twiddles(const T* __restrict__ twc, const T* __restrict__ tws, int N) {
    T* twl = lds_twiddle_ptr<T>();
    stage_twiddles<T, NTHR>(twl, twc, tws, N);
    return twl;
}

// forward post-processing of pair s: the two real outputs at row m
template <typename T, int PS = kPadShift>
__device__ __forceinline__ void post_fwd(const T* re, const T* im, int s, int SP, int N, int m, int bc,
                                         const T* __restrict__ dctc, const T* __restrict__ dcts, T& xa,
                                         T& xb) {
    const T half = (T)0.5;
    if (bc == FSEI_BC_WALL) {
        const int mm = (m == 0) ? 0 : N - m;
        const T zr = re[li<PS>(s, m, SP)], zi = im[li<PS>(s, m, SP)];
        const T cr = re[li<PS>(s, mm, SP)], ci = im[li<PS>(s, mm, SP)];
        const T ar = (zr + cr) * half, ai = (zi - ci) * half;
        const T br = (zi + ci) * half, bi = (cr - zr) * half;
        const T wr = dctc[m], wi = -dcts[m];
        xa = wr * ar - wi * ai;
        xb = wr * br - wi * bi;
    } else {
        if (2 * m <= N) {
            const int mm = (m == 0) ? 0 : N - m;
            xa = (re[li<PS>(s, m, SP)] + re[li<PS>(s, mm, SP)]) * half;
            xb = (im[li<PS>(s, m, SP)] + im[li<PS>(s, mm, SP)]) * half;
        } else {
            const int q = N - m;
            xa = (im[li<PS>(s, q, SP)] - im[li<PS>(s, m, SP)]) * half;
            xb = (re[li<PS>(s, m, SP)] - re[li<PS>(s, q, SP)]) * half;
        }
    }
}

// inverse pre-processing: complex input Z[m] of the pair from the rows m and
// N-m of the two transformed lines
template <typename T>
__device__ __forceinline__ void pre_inv_cs(int N, int m, int bc, T xam, T xanm, T xbm, T xbnm, T c, T s, T& zr,
                                           T& zi) {
    if (bc == FSEI_BC_WALL) {
        if (m == 0) {
            xanm = (T)0;
            xbnm = (T)0;
        }
        const T var = c * xam + s * xanm, vai = s * xam - c * xanm;
        const T vbr = c * xbm + s * xbnm, vbi = s * xbm - c * xbnm;
        zr = var - vbi;
        zi = vai + vbr;
    } else {
        T ra, ia, rb, ib;
        if (2 * m <= N) {
            ra = xam;
            rb = xbm;
            const bool hasim = (m != 0) && (2 * m != N);
            ia = hasim ? xanm : (T)0;
            ib = hasim ? xbnm : (T)0;
        } else {
            ra = xanm;
            rb = xbnm;
            ia = -xam;
            ib = -xbm;
        }
        zr = ra - ib;
        zi = ia + rb;
    }
}

// as pre_inv_cs with the twiddle pair read from the tables
template <typename T>
__device__ __forceinline__ void pre_inv(int N, int m, int bc, T xam, T xanm, T xbm, T xbnm,
                                        const T* __restrict__ dctc, const T* __restrict__ dcts, T& zr, T& zi) {
    T c = (T)1, s = (T)0;
    if (bc == FSEI_BC_WALL) {
        c = dctc[m];
        s = dcts[m];
    }
    pre_inv_cs<T>(N, m, bc, xam, xanm, xbm, xbnm, c, s, zr, zi);
}

// (k, j) of row j0 + l of plane k0 (rows wrap into the following planes)
__device__ __forceinline__ void row_kj(int k0, int j0, int l, int ny, int& k, int& j) {
    j = j0 + l;
    k = k0;
    if (j >= ny) {
        k += j / ny;
        j -= (j / ny) * ny;
    }
}

// forward post-processing from the four values at rows m and mm = (N - m) % N
// of one pair (selects instead of branches; same arithmetic as post_fwd)
template <typename T>
__device__ __forceinline__ void post_fwd_v(int bc, bool lo, T zr, T zi, T cr, T ci, T wr, T wi, T& xa, T& xb) {
    const T half = (T)0.5;
    if (bc == FSEI_BC_WALL) {
        const T ar = (zr + cr) * half, ai = (zi - ci) * half;
        const T br = (zi + ci) * half, bi = (cr - zr) * half;
        xa = wr * ar - wi * ai;
        xb = wr * br - wi * bi;
    } else {
        xa = lo ? (zr + cr) * half : (ci - zi) * half;
        xb = lo ? (zi + ci) * half : (zr - cr) * half;
    }
}

// s_waitcnt immediates (vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt
// 11:8): wait until at most n vector-memory operations of this wave are
// outstanding; wait for this wave's LDS operations only
__device__ constexpr int imm_wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
__device__ constexpr int imm_wait_lgkm0() { return 15 | (3 << 14) | (7 << 4); }
// Workgroup barrier for LDS exchanges while direct global-to-LDS loads may
// still be in flight: this wave's LDS accesses complete, then the barrier,
// with no memory fence (a fence would wait for the direct loads too); the
// empty asm keeps the compiler from moving memory accesses across it.
__device__ __forceinline__ void sync_lds_nofence() {
    __builtin_amdgcn_s_waitcnt(imm_wait_lgkm0());
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// two adjacent values of a field as one vector access
template <typename T>
struct Vec2T;
template <>
struct Vec2T<double> {
    using type = double2;
};
template <>
struct Vec2T<float> {
    using type = float2;
};

// ---------------------------------------------------------------------------
// x forward: prologue (divergence / transposed gradient / residual / copy)
// fused with the forward x transform
// ---------------------------------------------------------------------------
// RESID: the FP64 residual (f - mean) - L p of an FP64 iterate p; RESID_F: of
// an FP32 iterate p32 (the first solve of the refinement), read as FP32 and
// evaluated in FP64
enum { PRO_COPY = 0, PRO_DIV = 1, PRO_DIV_ADJ = 2, PRO_RESID = 3, PRO_RESID_F = 4, PRO_KINDS = 5 };

template <typename TI, typename TO>
struct XFwdArgs {
    int nx, ny, nz, bcx, bcy, nseq;
    FftPlan fp;
    // prologue inputs
    const TI* u;
    const TI* v;
    const TI* w;
    const TI* gp;       // adjoint: dLoss/dp or null
    const double* f;    // COPY (double input) and RESID
    const double* p;    // RESID
    const float* p32;   // RESID_F
    TI alpha, beta, idx, idy;
    const TI* zeta;     // coefficient of w_{k+1}
    const TI* eta;      // coefficient of w_k
    double idx2, idy2;  // RESID
    const double* za;   // RESID
    const double* zc;   // RESID
    const double* scal; // RESID: scal[0] = removed mean
    // outputs
    TO* out;
    double* out_f;      // optional FP64 copy of the prologue value
    double* partials;   // optional per-block (sum v^2, sum v, sum dzw_k v)
    const double* dzw;  // with partials: z weights of the third sum (dz_k), or null;
                        // RESID: the third sum is sum dzw_k p (the iterate, not r)
    const TO* twc;
    const TO* tws;
    const TO* dctc;
    const TO* dcts;
};

// the pressure iterate a residual prologue reads
template <int PRO, typename TI, typename TO>
__device__ __forceinline__ auto resid_iterate(const XFwdArgs<TI, TO>& a) {
    if constexpr (PRO == PRO_RESID_F) return a.p32;
    else return a.p;
}

// The stencil value at cell (k, j, i); `o` is the cell's offset from the
// workgroup base `base` (first cell of its first row), so all accesses are
// 32-bit offsets from base pointers.
template <typename TI, typename TO, int PRO>
__device__ __forceinline__ TI x_prologue(const XFwdArgs<TI, TO>& a, size_t base, int k, int j, int i, int o,
                                         int N) {
    const int nx = N, ny = a.ny, nz = a.nz;
    const int nxy = nx * ny;
    if constexpr (PRO == PRO_COPY) {
        return (TI)a.f[base + o];
    } else if constexpr (PRO == PRO_RESID || PRO == PRO_RESID_F) {
        const auto* __restrict__ p = resid_iterate<PRO>(a) + base;
        const double pc = (double)p[o];
        double lx = 0.0, ly = 0.0, lz = 0.0;
        if (i + 1 < nx) lx += (double)p[o + 1] - pc;
        else if (a.bcx == FSEI_BC_PERIODIC) lx += (double)p[o + 1 - nx] - pc;
        if (i >= 1) lx += (double)p[o - 1] - pc;
        else if (a.bcx == FSEI_BC_PERIODIC) lx += (double)p[o + nx - 1] - pc;
        if (j + 1 < ny) ly += (double)p[o + nx] - pc;
        else if (a.bcy == FSEI_BC_PERIODIC) ly += (double)p[o - (ny - 1) * nx] - pc;
        if (j >= 1) ly += (double)p[o - nx] - pc;
        else if (a.bcy == FSEI_BC_PERIODIC) ly += (double)p[o + (ny - 1) * nx] - pc;
        if (k + 1 < nz) lz += a.zc[k] * ((double)p[o + nxy] - pc);
        if (k >= 1) lz += a.za[k] * ((double)p[o - nxy] - pc);
        const double lap = lx * a.idx2 + ly * a.idy2 + lz;
        return (TI)((a.f[base + o] - a.scal[0]) - lap);
    } else {
        const TI* __restrict__ u = a.u + base;
        const TI* __restrict__ v = a.v + base;
        const TI* __restrict__ w = a.w + base;
        const TI zero = (TI)0;
        const TI uc = (a.bcx == FSEI_BC_WALL && i == 0) ? zero : u[o];
        const TI uh = (i + 1 < nx) ? u[o + 1] : ((a.bcx == FSEI_BC_PERIODIC) ? u[o + 1 - nx] : zero);
        const TI vc = (a.bcy == FSEI_BC_WALL && j == 0) ? zero : v[o];
        const TI vh = (j + 1 < ny) ? v[o + nx] : ((a.bcy == FSEI_BC_PERIODIC) ? v[o - (ny - 1) * nx] : zero);
        const TI wc = (k == 0) ? zero : w[o];
        const TI wh = (k + 1 < nz) ? w[o + nxy] : zero;
        TI val = (uh - uc) * a.idx + (vh - vc) * a.idy + (a.zeta[k] * wh - a.eta[k] * wc);
        val *= a.alpha;
        if constexpr (PRO == PRO_DIV_ADJ) {
            if (a.gp) val += a.beta * a.gp[base + o];
        }
        return val;
    }
}

template <typename TI, typename TO, int PRO, int EMAX, int NTHR>
__global__ __launch_bounds__(NTHR) void k_xfwd(XFwdArgs<TI, TO> a) {
    __shared__ TO sre[lds_elems(EMAX)];
    __shared__ TO sim[lds_elems(EMAX)];
    __shared__ double sred[3 * (NTHR / 64)];
    const int N = a.nx;
    const int SP = seq_stride(N);
    const int nseq = a.nseq;
    const int nl = 2 * nseq;
    const long nrows = (long)a.ny * a.nz;
    const long row0 = xcd_remap(blockIdx.x, gridDim.x) * nl;
    const int k0 = (int)(row0 / a.ny);
    const int j0 = (int)(row0 - (long)k0 * a.ny);
    const size_t base = (size_t)row0 * N;
    TO* twl = lds_twiddles<TO, NTHR>(a.twc, a.tws, N);
    double* __restrict__ out_f = a.out_f;
    double ss = 0.0, s1 = 0.0, s2 = 0.0;
    const int total = nl * N;
    constexpr int PER = 2 * EMAX / NTHR;   // elements per thread, >= total / NTHR
    constexpr int BAT = (PER % 4 == 0) ? 4 : 1;
    for (int r0 = 0; r0 < PER; r0 += BAT) {
        TI val[BAT];
#pragma unroll
        for (int r = 0; r < BAT; ++r) {
            const int e = threadIdx.x + (r0 + r) * NTHR;
            val[r] = (TI)0;
            if (e < total) {
                const int l = e / N;
                const int i = e - l * N;
                if (row0 + l < nrows) {
                    int k, j;
                    row_kj(k0, j0, l, a.ny, k, j);
                    val[r] = x_prologue<TI, TO, PRO>(a, base, k, j, i, e, N);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < BAT; ++r) {
            const int e = threadIdx.x + (r0 + r) * NTHR;
            if (e < total) {
                const int l = e / N;
                const int i = e - l * N;
                if (row0 + l < nrows) {
                    if (out_f) out_f[base + e] = (double)val[r];
                    ss += (double)val[r] * (double)val[r];
                    s1 += (double)val[r];
                    if (a.dzw) {
                        int k, j;
                        row_kj(k0, j0, l, a.ny, k, j);
                        constexpr bool RES = PRO == PRO_RESID || PRO == PRO_RESID_F;
                        s2 += a.dzw[k] * (RES ? (double)resid_iterate<PRO>(a)[base + e] : (double)val[r]);
                    }
                }
                const int n = (a.bcx == FSEI_BC_WALL) ? mk_pos(i, N) : i;
                if (l & 1) sim[li(l >> 1, n, SP)] = (TO)val[r];
                else sre[li(l >> 1, n, SP)] = (TO)val[r];
            }
        }
    }
    if (a.partials) {
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
    fft_lds<TO, EMAX, NTHR, -1>(sre, sim, N, nseq, a.fp, twl, twl + N);
    TO* __restrict__ out = a.out + base;
    constexpr int PST = EMAX / NTHR;
#pragma unroll
    for (int r = 0; r < PST; ++r) {
        const int e = threadIdx.x + r * NTHR;
        if (e < nseq * N) {
            const int s = e / N;
            const int m = e - s * N;
            TO xa, xb;
            post_fwd<TO>(sre, sim, s, SP, N, m, a.bcx, a.dctc, a.dcts, xa, xb);
            if (row0 + 2 * s < nrows) out[2 * s * N + m] = xa;
            if (row0 + 2 * s + 1 < nrows) out[(2 * s + 1) * N + m] = xb;
        }
    }
}

// ---------------------------------------------------------------------------
// x inverse: unnormalised inverse x transform of row pairs; writes (STORE)
// or adds (ACC) the result into the output field
// ---------------------------------------------------------------------------
// STORE: out = result; ACC: out += result; ADDF: out = add32 + result;
// ACC_KEEP: out += result and the result is also written back over the input
enum { EPI_STORE = 0, EPI_ACC = 1, EPI_ADDF = 2, EPI_ACC_KEEP = 3, EPI_KINDS = 4 };

template <typename T, typename TP>
struct XInvArgs {
    int nx, ny, nz, bcx, nseq;
    FftPlan fp;
    const T* in;
    TP* out;
    const float* add32;   // EPI_ADDF: FP32 field added to the result
    T* keep;              // EPI_ACC_KEEP: receives the result (the input field itself)
    const double* vsum;   // ACC / ADDF: if set, vsum[0] * vscale is subtracted from
    double vscale;        //   every output (the V-mean of the previous iterate)
    const T* twc;
    const T* tws;
    const T* dctc;
    const T* dcts;
};

template <typename T, typename TP, int EPI, int EMAX, int NTHR>
__global__ __launch_bounds__(NTHR) void k_xinv(XInvArgs<T, TP> a) {
    __shared__ T sre[lds_elems(EMAX)];
    __shared__ T sim[lds_elems(EMAX)];
    const int N = a.nx;
    const int SP = seq_stride(N);
    const int nseq = a.nseq;
    const int nl = 2 * nseq;
    const long row0 = xcd_remap(blockIdx.x, gridDim.x) * nl;
    const long nrows = (long)a.ny * a.nz;
    const size_t base = (size_t)row0 * N;
    const T* in = a.in + base;   // not restrict: ACC_KEEP writes this field back (after every read of it)
    T* twl = lds_twiddles<T, NTHR>(a.twc, a.tws, N);
    constexpr int PLD = EMAX / NTHR;
#pragma unroll
    for (int r = 0; r < PLD; ++r) {
        const int e = threadIdx.x + r * NTHR;
        if (e < nseq * N) {
            const int s = e / N;
            const int m = e - s * N;
            const int nm = (m == 0) ? 0 : N - m;
            T xam = 0, xanm = 0, xbm = 0, xbnm = 0;
            if (row0 + 2 * s < nrows) {
                xam = in[2 * s * N + m];
                xanm = in[2 * s * N + nm];
            }
            if (row0 + 2 * s + 1 < nrows) {
                xbm = in[(2 * s + 1) * N + m];
                xbnm = in[(2 * s + 1) * N + nm];
            }
            T zr, zi;
            pre_inv<T>(N, m, a.bcx, xam, xanm, xbm, xbnm, a.dctc, a.dcts, zr, zi);
            sre[li(s, m, SP)] = zr;
            sim[li(s, m, SP)] = zi;
        }
    }
    TP* __restrict__ out = a.out + base;
    __syncthreads();
    fft_lds<T, EMAX, NTHR, 1>(sre, sim, N, nseq, a.fp, twl, twl + N);
    constexpr int PST = 2 * EMAX / NTHR;
    const TP msub = (EPI != EPI_STORE && a.vsum) ? (TP)(a.vsum[0] * a.vscale) : (TP)0;
#pragma unroll
    for (int r = 0; r < PST; ++r) {
        const int e = threadIdx.x + r * NTHR;
        if (e < nl * N) {
            const int l = e / N;
            const int i = e - l * N;
            if (row0 + l < nrows) {
                const int n = (a.bcx == FSEI_BC_WALL) ? mk_pos(i, N) : i;
                const T val = (l & 1) ? sim[li(l >> 1, n, SP)] : sre[li(l >> 1, n, SP)];
                if constexpr (EPI == EPI_ACC) out[e] = (out[e] - msub) + (TP)val;
                else if constexpr (EPI == EPI_ADDF) out[e] = ((TP)a.add32[base + e] - msub) + (TP)val;
                else if constexpr (EPI == EPI_ACC_KEEP) {
                    out[e] = (out[e] - msub) + (TP)val;
                    a.keep[base + e] = val;
                } else out[e] = (TP)val;
            }
        }
    }
}

// two adjacent doubles as one non-temporal 16-byte store
__device__ __forceinline__ void nt_store2(double* q, double2 v) {
    __builtin_nontemporal_store(v.x, q);
    __builtin_nontemporal_store(v.y, q + 1);
}
__device__ __forceinline__ void nt_store2(float* q, float2 v) {
    __builtin_nontemporal_store(v.x, q);
    __builtin_nontemporal_store(v.y, q + 1);
}

// the fused x inverse + gradient correction (k_xinv_grad_len)
template <typename T>
struct XInvGradArgs {
    int ny, nz, bcx, bcy, kc;   // kc: planes per chunk
    const T* in;                // y-inverted field (transform space in x)
    T* p;                       // pressure out, or null
    const T* ui;                // velocity in (the outputs, or arrays that overlap none)
    const T* vi;
    const T* wi;
    T* u;                       // velocity out
    T* v;
    T* w;
    T cx, cy, sw;
    const T* bk;
    const T* gk;
    const T* twc;
    const T* tws;
    const T* dctc;
    const T* dcts;
};

// ---------------------------------------------------------------------------
// The first correction of the FP32 + FP64 refinement fused with the gradient
// correction and the convergence check (one pass instead of the x inverse
// with the ADDF epilogue followed by the gradient + residual kernel):
//     delta = FP32 inverse x transform of the y-inverted correction,
//     p = (p32 - m) + delta        in FP64 (m: V-mean of the first solve),
//     u += cx (p_i - p_{i-1}),  v += cy (p_j - p_{j-1}),
//     w += sw (bk_k p_k - gk_k p_{k-1})        (wall faces written 0),
//     r = (f - mean) - L p,  per-workgroup partials of sum r^2 and sum r,
// p written once.  The marching of k_xinv_grad_len, with 10 rows per plane
// (halo rows j0-1 and j0+8, both needed by the Laplacian) as 5 complex FP32
// sequences.  The residual of plane k needs p of plane k+1: its part
// without that term is kept in registers and completed one step later (the
// chunk's march takes one plane beyond its end when there is one).
// Every p is formed from p32 and delta exactly as the ADDF epilogue forms it.
// ---------------------------------------------------------------------------
struct XInvGradResArgs {
    int ny, nz, bcx, bcy, kc;
    const float* in;        // y-inverted correction (transform space in x), FP32
    const float* p32;       // first solve
    const double* vsum;     // vsum[0] * vscale is subtracted from p32
    double vscale;
    double* p;              // pressure out (FP64)
    const double* ui;       // velocity in (the outputs, or arrays that overlap none)
    const double* vi;
    const double* wi;
    double* u;              // velocity out
    double* v;
    double* w;
    double cx, cy, sw;
    const double* bk;
    const double* gk;
    const double* f;        // FP64 right-hand side
    double idx2, idy2;
    const double* za;
    const double* zc;
    const double* scal;     // scal[0] = removed mean of f
    double* partials;       // per workgroup: sum r^2, sum r, 0
    const float* twc;
    const float* tws;
    const float* dctc;
    const float* dcts;
};

// threads of k_xinv_grad_resid: one per column pair at 512 (two workgroups
// per CU fit the registers), one per radix-8 butterfly at 768
template <int NF>
constexpr int xgr_threads() { return NF == 512 ? NF / 2 : kXgSeq * NF / 8; }

template <int NF>
__global__ __launch_bounds__(xgr_threads<NF>()) void k_xinv_grad_resid(XInvGradResArgs a) {
    constexpr int NTHR = xgr_threads<NF>();
    constexpr int GR = kXgRows, NSQ = kXgSeq, EMAX = NSQ * NF;
    static_assert(NTHR >= NF / 2, "a column pair per thread");
    constexpr int SP = seq_stride(NF);
    constexpr int GB = 2;   // rows per batch of the gradient phase
    static_assert(NSQ * SP <= lds_elems(EMAX), "tile fits");
    static_assert(2 * NSQ == GR + 2, "two halo rows + own rows");
    static_assert(GR % GB == 0, "whole batches");
    static_assert(NF / 2 <= 64 * (NTHR / 64), "the column-owning threads are in the waves block_sum3 adds");
    __shared__ float sre[lds_elems(EMAX)];
    __shared__ float sim[lds_elems(EMAX)];
    __shared__ double sred[3 * (NTHR / 64 + 1)];
    const int ny = a.ny, nz = a.nz;
    const int ntj = ny / GR;
    const int b = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int chunk = b / ntj;
    const int jt = b - chunk * ntj;
    const int j0 = jt * GR;
    const int kb = chunk * a.kc;
    const int ke = (kb + a.kc < nz) ? kb + a.kc : nz;
    const int kend = (ke < nz) ? ke + 1 : ke;   // one plane beyond the chunk for its last residual
    const int jh = (j0 > 0) ? j0 - 1 : ny - 1;            // halo rows (wrapped; a y wall never uses them)
    const int jn = (j0 + GR < ny) ? j0 + GR : 0;
    const bool wallx = a.bcx == FSEI_BC_WALL, wally = a.bcy == FSEI_BC_WALL;
    float* twl = lds_twiddles<float, NTHR>(a.twc, a.tws, NF);
    const bool colt = threadIdx.x < NF / 2;   // owns a column (pair)
    const int m = colt ? threadIdx.x : 0;
    const int nm = (m == 0) ? NF / 2 : NF - m;
    const int lm = li(0, m, SP), lnm = li(0, nm, SP);
    float cm = 1.0f, sm = 0.0f, cn = 1.0f, sn = 0.0f;
    if (wallx) {
        cm = a.dctc[m];
        sm = a.dcts[m];
        cn = (m == 0) ? a.dctc[NF / 2] : sm;
        sn = (m == 0) ? a.dcts[NF / 2] : cm;
    }
    // this thread's column pair (i, i + 1) and its x neighbours i - 1, i + 2
    const int i = 2 * m;
    const int ixm = (i > 0) ? i - 1 : NF - 1;
    const int ixp = (i + 2 < NF) ? i + 2 : 0;
    const bool perx = !wallx, pery = !wally;
    const bool him = (i > 0) || perx, hip = (i + 2 < NF) || perx;
    const int q0 = li(0, wallx ? mk_pos(i, NF) : i, SP);
    const int q1 = li(0, wallx ? mk_pos(i + 1, NF) : i + 1, SP);
    const int qm = li(0, wallx ? mk_pos(ixm, NF) : ixm, SP);
    const int qp = li(0, wallx ? mk_pos(ixp, NF) : ixp, SP);
    const size_t plane = (size_t)NF * ny;
    const double msub = a.vsum ? a.vsum[0] * a.vscale : 0.0;
    const double mean = a.scal[0];
    auto rowj = [&](int r) { return (r == 0) ? jh : ((r <= GR) ? j0 + r - 1 : jn); };
    // step input: the correction's rows (tile row r = 0: row j0 - 1, 1..8:
    // own rows, 9: row j0 + 8; sequence s pairs rows 2s and 2s + 1)
    float xa[NSQ][2], xb[NSQ][2];
    auto load_in = [&](int k) {
        const float* __restrict__ in = a.in + (size_t)k * plane;
#pragma unroll
        for (int s = 0; s < NSQ; ++s) {
            const float* pa = in + (size_t)rowj(2 * s) * NF;
            const float* pb = in + (size_t)rowj(2 * s + 1) * NF;
            xa[s][0] = pa[m];
            xa[s][1] = pa[nm];
            xb[s][0] = pb[m];
            xb[s][1] = pb[nm];
        }
    };
    auto dl = [&](int r, int q) -> double { return (double)((r & 1) ? sim : sre)[(r >> 1) * SP + q]; };
    // p of tile row r at the thread's pair, from that row's p32 pair: (p32 - m) + delta, in FP64
    auto pair_p = [&](int r, float2 q) {
        return make_double2(((double)q.x - msub) + dl(r, q0), ((double)q.y - msub) + dl(r, q1));
    };
    double2 prev[GR];    // p of the plane below, own rows
    double2 rpart[GR];   // residual of the plane below without its z+1 term
#pragma unroll
    for (int l = 0; l < GR; ++l) {
        prev[l] = make_double2(0.0, 0.0);
        rpart[l] = make_double2(0.0, 0.0);
    }
    double ss = 0.0, s1 = 0.0;
    int k = (kb > 0) ? kb - 1 : 0;
    for (; k < kend; ++k) {
        if (colt) load_in(k);
#pragma unroll
        for (int s = 0; s < NSQ && colt; ++s) {
            const float pa = (m == 0) ? xa[s][1] : xa[s][0], pb = (m == 0) ? xb[s][1] : xb[s][0];
            float zr, zi;
            pre_inv_cs<float>(NF, m, a.bcx, xa[s][0], xa[s][1], xb[s][0], xb[s][1], cm, sm, zr, zi);
            sre[s * SP + lm] = zr;
            sim[s * SP + lm] = zi;
            pre_inv_cs<float>(NF, nm, a.bcx, xa[s][1], pa, xb[s][1], pb, cn, sn, zr, zi);
            sre[s * SP + lnm] = zr;
            sim[s * SP + lnm] = zi;
        }
        __syncthreads();
        fft_fixed<float, EMAX, NTHR, 1, NF, 0, 1>(sre, sim, NSQ, twl, twl + NF);
        // uniform over the workgroup: this plane's own rows get the gradient
        // (grad), complete the residual of the plane below (lag), or only
        // provide p for the next plane (the chunk's halo plane)
        const bool grad = k >= kb && k < ke;
        const bool lag = k - 1 >= kb && k - 1 < ke;
        if (colt) {
            const float* __restrict__ p3 = a.p32 + (size_t)k * plane + i;
            const size_t ro = (size_t)k * plane + (size_t)j0 * NF + i;
            const double bkk = a.bk[k], gkk = a.gk[k];
            const double czm = (k > 0) ? a.za[k] : 0.0;
            const double czl = (k > 0) ? a.zc[k - 1] : 0.0;   // z+1 coefficient of the plane below
            const bool hzm = k > 0, hzp = k + 1 < nz;
            double2 pym = make_double2(0.0, 0.0);
            if (grad) pym = pair_p(0, *reinterpret_cast<const float2*>(p3 + (size_t)jh * NF));
#pragma unroll
            for (int l0 = 0; l0 < GR; l0 += GB) {
                // p32 of tile rows l0+1 .. l0+GB+1 (the last one is the next
                // batch's first row, needed here for the y Laplacian)
                float2 q32[GB + 1];
                float qxm[GB], qxp[GB];
                double2 uo[GB], vo[GB], wo[GB], fo[GB];
#pragma unroll
                for (int t = 0; t <= GB; ++t) {
                    const int r = l0 + t + 1;
                    if (t < GB || grad) q32[t] = *reinterpret_cast<const float2*>(p3 + (size_t)rowj(r) * NF);
                }
                if (grad) {
#pragma unroll
                    for (int t = 0; t < GB; ++t) {
                        const size_t o = ro + (size_t)(l0 + t) * NF;
                        const float* pr = a.p32 + (o - i);
                        qxm[t] = pr[ixm];
                        qxp[t] = pr[ixp];
                        uo[t] = *reinterpret_cast<const double2*>(a.ui + o);
                        vo[t] = *reinterpret_cast<const double2*>(a.vi + o);
                        wo[t] = *reinterpret_cast<const double2*>(a.wi + o);
                        fo[t] = *reinterpret_cast<const double2*>(a.f + o);
                    }
                }
#pragma unroll
                for (int t = 0; t < GB; ++t) {
                    const int l = l0 + t, r = l + 1;
                    const int j = j0 + l;
                    const double2 pc = pair_p(r, q32[t]);
                    if (lag) {   // the residual of the plane below, completed with this plane's p
                        const double r0 = rpart[l].x - czl * (pc.x - prev[l].x);
                        const double r1 = rpart[l].y - czl * (pc.y - prev[l].y);
                        ss += r0 * r0 + r1 * r1;
                        s1 += r0 + r1;
                    }
                    if (grad) {
                        const double2 pyp = pair_p(r + 1, q32[t + 1]);
                        const double pxm = ((double)qxm[t] - msub) + dl(r, qm);
                        const double pxp = ((double)qxp[t] - msub) + dl(r, qp);
                        // gradient correction
                        double2 un, vn, wn;
                        un.x = (wallx && i == 0) ? 0.0 : uo[t].x + a.cx * (pc.x - pxm);
                        un.y = uo[t].y + a.cx * (pc.y - pc.x);
                        const bool v0 = wally && j == 0;
                        vn.x = v0 ? 0.0 : vo[t].x + a.cy * (pc.x - pym.x);
                        vn.y = v0 ? 0.0 : vo[t].y + a.cy * (pc.y - pym.y);
                        wn.x = (k == 0) ? 0.0 : wo[t].x + a.sw * (bkk * pc.x - gkk * prev[l].x);
                        wn.y = (k == 0) ? 0.0 : wo[t].y + a.sw * (bkk * pc.y - gkk * prev[l].y);
                        // residual without the z+1 term
                        const bool hym = (j > 0) || pery, hyp = (j + 1 < ny) || pery;
                        const double lx0 = (pc.y - pc.x) + (him ? pxm - pc.x : 0.0);
                        const double lx1 = (hip ? pxp - pc.y : 0.0) + (pc.x - pc.y);
                        const double ly0 = (hyp ? pyp.x - pc.x : 0.0) + (hym ? pym.x - pc.x : 0.0);
                        const double ly1 = (hyp ? pyp.y - pc.y : 0.0) + (hym ? pym.y - pc.y : 0.0);
                        const double lz0 = hzm ? czm * (prev[l].x - pc.x) : 0.0;
                        const double lz1 = hzm ? czm * (prev[l].y - pc.y) : 0.0;
                        const double r0 = (fo[t].x - mean) - (lx0 * a.idx2 + ly0 * a.idy2 + lz0);
                        const double r1 = (fo[t].y - mean) - (lx1 * a.idx2 + ly1 * a.idy2 + lz1);
                        if (hzp) {
                            rpart[l] = make_double2(r0, r1);
                        } else {
                            ss += r0 * r0 + r1 * r1;
                            s1 += r0 + r1;
                        }
                        const size_t o = ro + (size_t)l * NF;
                        nt_store2(a.u + o, un);
                        nt_store2(a.v + o, vn);
                        nt_store2(a.w + o, wn);
                        nt_store2(a.p + o, pc);
                    }
                    prev[l] = pc;
                    pym = pc;
                }
                // keep the next batch's loads after this batch's stores
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();   // the next step overwrites the tile
    }
    double s2 = 0.0;
    block_sum3<NTHR>(ss, s1, s2, sred);
    if (threadIdx.x == 0) {
        a.partials[3 * blockIdx.x] = ss;
        a.partials[3 * blockIdx.x + 1] = s1;
        a.partials[3 * blockIdx.x + 2] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// y transforms, in place, on tiles of TX = 2*nseq adjacent x-columns of one
// z-plane (each column pair is one complex sequence)
// ---------------------------------------------------------------------------
template <typename T>
struct YArgs {
    int nx, ny, nz, bcy, nseq, ntile;
    FftPlan fp;
    T* data;
    const T* twc;
    const T* tws;
    const T* dctc;
    const T* dcts;
};

template <typename T, int EMAX, int NTHR>
__global__ __launch_bounds__(NTHR) void k_yfwd(YArgs<T> a) {
    __shared__ T sre[lds_elems(EMAX)];
    __shared__ T sim[lds_elems(EMAX)];
    const int N = a.ny;
    const int SP = seq_stride(N);
    const int nx = a.nx;
    const int nseq = a.nseq;
    const int TX = 2 * nseq;
    // tiles in XCD-contiguous runs: neighbouring tiles share an L2
    const int bx = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int k = bx / a.ntile;
    const int tile = bx - k * a.ntile;
    const int i0 = tile * TX;
    T* __restrict__ d = a.data + (size_t)k * nx * N + i0;
    T* twl = lds_twiddles<T, NTHR>(a.twc, a.tws, N);
    constexpr int PLD = 2 * EMAX / NTHR;
    T val[PLD];
#pragma unroll
    for (int r = 0; r < PLD; ++r) {
        const int e = threadIdx.x + r * NTHR;
        const int j = e / TX;
        const int c = e - j * TX;
        val[r] = (e < TX * N && i0 + c < nx) ? d[j * nx + c] : (T)0;
    }
#pragma unroll
    for (int r = 0; r < PLD; ++r) {
        const int e = threadIdx.x + r * NTHR;
        if (e < TX * N) {
            const int j = e / TX;
            const int c = e - j * TX;
            const int n = (a.bcy == FSEI_BC_WALL) ? mk_pos(j, N) : j;
            if (c & 1) sim[li(c >> 1, n, SP)] = val[r];
            else sre[li(c >> 1, n, SP)] = val[r];
        }
    }
    __syncthreads();
    fft_lds<T, EMAX, NTHR, -1>(sre, sim, N, nseq, a.fp, twl, twl + N);
    constexpr int PST = EMAX / NTHR;
#pragma unroll
    for (int r = 0; r < PST; ++r) {
        const int e = threadIdx.x + r * NTHR;
        if (e < nseq * N) {
            const int m = e / nseq;
            const int s = e - m * nseq;
            T xa, xb;
            post_fwd<T>(sre, sim, s, SP, N, m, a.bcy, a.dctc, a.dcts, xa, xb);
            if (i0 + 2 * s < nx) d[m * nx + 2 * s] = xa;
            if (i0 + 2 * s + 1 < nx) d[m * nx + 2 * s + 1] = xb;
        }
    }
}

template <typename T, int EMAX, int NTHR>
__global__ __launch_bounds__(NTHR) void k_yinv(YArgs<T> a) {
    __shared__ T sre[lds_elems(EMAX)];
    __shared__ T sim[lds_elems(EMAX)];
    const int N = a.ny;
    const int SP = seq_stride(N);
    const int nx = a.nx;
    const int nseq = a.nseq;
    const int TX = 2 * nseq;
    // tiles in XCD-contiguous runs: neighbouring tiles share an L2
    const int bx = (int)xcd_remap(blockIdx.x, gridDim.x);
    const int k = bx / a.ntile;
    const int tile = bx - k * a.ntile;
    const int i0 = tile * TX;
    T* __restrict__ d = a.data + (size_t)k * nx * N + i0;
    T* twl = lds_twiddles<T, NTHR>(a.twc, a.tws, N);
    constexpr int PLD = EMAX / NTHR;
#pragma unroll
    for (int r = 0; r < PLD; ++r) {
        const int e = threadIdx.x + r * NTHR;
        if (e < nseq * N) {
            const int m = e / nseq;
            const int s = e - m * nseq;
            const int nm = (m == 0) ? 0 : N - m;
            T xam = 0, xanm = 0, xbm = 0, xbnm = 0;
            if (i0 + 2 * s < nx) {
                xam = d[m * nx + 2 * s];
                xanm = d[nm * nx + 2 * s];
            }
            if (i0 + 2 * s + 1 < nx) {
                xbm = d[m * nx + 2 * s + 1];
                xbnm = d[nm * nx + 2 * s + 1];
            }
            T zr, zi;
            pre_inv<T>(N, m, a.bcy, xam, xanm, xbm, xbnm, a.dctc, a.dcts, zr, zi);
            sre[li(s, m, SP)] = zr;
            sim[li(s, m, SP)] = zi;
        }
    }
    __syncthreads();
    fft_lds<T, EMAX, NTHR, 1>(sre, sim, N, nseq, a.fp, twl, twl + N);
    constexpr int PST = 2 * EMAX / NTHR;
#pragma unroll
    for (int r = 0; r < PST; ++r) {
        const int e = threadIdx.x + r * NTHR;
        if (e < TX * N) {
            const int j = e / TX;
            const int c = e - j * TX;
            if (i0 + c < nx) {
                const int n = (a.bcy == FSEI_BC_WALL) ? mk_pos(j, N) : j;
                d[j * nx + c] = (c & 1) ? sim[li(c >> 1, n, SP)] : sre[li(c >> 1, n, SP)];
            }
        }
    }
}

}  // namespace dev
}  // namespace fsei
