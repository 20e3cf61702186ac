// Batched mixed-radix Stockham FFT in LDS for gfx950: radices 8, 4, 3, 2 for
// lengths taken from the arguments, 16, 12, 9, 8, 6, 4, 3, 2 for compiled lengths.
//
// A workgroup transforms `nseq` complex sequences of length N held in LDS as
// split real/imaginary arrays.  Element n of sequence s sits at
//     s * SP + n + n / 16,      SP = N + N / 16 + 1,
// i.e. one pad slot every 16 elements (breaks the power-of-two strides of a
// stage's scatter) and an odd stride between sequences (threads that walk
// across sequences at a fixed n hit different banks).  Each radix-R stage
// reads R inputs at stride N/R, applies the twiddles exp(SIGN 2 pi i t / N),
// does a length-R DFT in registers and writes the outputs to their
// self-sorting positions, so the result is in natural order without a
// bit-reversal pass.  A stage is done in place: every thread gathers all of
// its butterflies into registers, the workgroup synchronises, then scatters.
//
// For a compiled length (fft_fixed) the stage loop is unrolled with constant
// radices and strides, so no integer division remains.
#pragma once

#include <hip/hip_runtime.h>

#include "fsei_plan.h"

namespace fsei {
namespace dev {

// seq_stride, lds_elems and tile_nseq (the tile geometry) live in fsei_plan.h
template <int PS = kPadShift>
__device__ __forceinline__ int li(int s, int n, int SP) { return s * SP + n + (n >> PS); }

template <typename T>
__device__ __forceinline__ void cmul(T& ar, T& ai, T br, T bi) {
    const T t = ar * br - ai * bi;
    ai = ar * bi + ai * br;
    ar = t;
}

// ---- length-R DFTs in registers, y_q = sum_r x_r exp(SIGN 2 pi i r q / R)
template <typename T, int SIGN>
__device__ __forceinline__ void dft2(T* xr, T* xi) {
    const T ar = xr[0] + xr[1], ai = xi[0] + xi[1];
    xr[1] = xr[0] - xr[1];
    xi[1] = xi[0] - xi[1];
    xr[0] = ar;
    xi[0] = ai;
}

template <typename T, int SIGN>
__device__ __forceinline__ void dft4v(T x0r, T x0i, T x1r, T x1i, T x2r, T x2i, T x3r, T x3i,
                                      T* yr, T* yi) {
    const T ar = x0r + x2r, ai = x0i + x2i;
    const T br = x0r - x2r, bi = x0i - x2i;
    const T cr = x1r + x3r, ci = x1i + x3i;
    const T dr = x1r - x3r, di = x1i - x3i;
    yr[0] = ar + cr;
    yi[0] = ai + ci;
    yr[2] = ar - cr;
    yi[2] = ai - ci;
    // y1 = b + SIGN i d, y3 = b - SIGN i d
    yr[1] = br - SIGN * di;
    yi[1] = bi + SIGN * dr;
    yr[3] = br + SIGN * di;
    yi[3] = bi - SIGN * dr;
}

template <typename T, int SIGN>
__device__ __forceinline__ void dft4(T* xr, T* xi) {
    T yr[4], yi[4];
    dft4v<T, SIGN>(xr[0], xi[0], xr[1], xi[1], xr[2], xi[2], xr[3], xi[3], yr, yi);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        xr[q] = yr[q];
        xi[q] = yi[q];
    }
}

template <typename T, int SIGN>
__device__ __forceinline__ void dft8(T* xr, T* xi) {
    T er[4], ei[4], orr[4], oi[4];
    dft4v<T, SIGN>(xr[0], xi[0], xr[2], xi[2], xr[4], xi[4], xr[6], xi[6], er, ei);
    dft4v<T, SIGN>(xr[1], xi[1], xr[3], xi[3], xr[5], xi[5], xr[7], xi[7], orr, oi);
    const T h = (T)0.70710678118654752440084436210484903928;
    // w^q O_q with w = exp(SIGN i pi / 4)
    T tr[4], ti[4];
    tr[0] = orr[0];
    ti[0] = oi[0];
    tr[1] = h * (orr[1] - SIGN * oi[1]);
    ti[1] = h * (oi[1] + SIGN * orr[1]);
    tr[2] = -SIGN * oi[2];
    ti[2] = SIGN * orr[2];
    tr[3] = h * (-orr[3] - SIGN * oi[3]);
    ti[3] = h * (-oi[3] + SIGN * orr[3]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        xr[q] = er[q] + tr[q];
        xi[q] = ei[q] + ti[q];
        xr[q + 4] = er[q] - tr[q];
        xi[q + 4] = ei[q] - ti[q];
    }
}

template <typename T, int SIGN>
__device__ __forceinline__ void dft3(T* xr, T* xi) {
    const T s3 = (T)0.86602540378443864676372317075293618347;
    const T tr = xr[1] + xr[2], ti = xi[1] + xi[2];
    const T ur = xr[1] - xr[2], ui = xi[1] - xi[2];
    const T mr = xr[0] - (T)0.5 * tr, mi = xi[0] - (T)0.5 * ti;
    xr[0] = xr[0] + tr;
    xi[0] = xi[0] + ti;
    xr[1] = mr - SIGN * s3 * ui;
    xi[1] = mi + SIGN * s3 * ur;
    xr[2] = mr + SIGN * s3 * ui;
    xi[2] = mi - SIGN * s3 * ur;
}

// cos and sin of 2 pi k / R for the inner twiddles of the composite radices
__host__ __device__ constexpr double root_c(int R, int k) {
    const int e = k * (144 / R);   // in units of 2 pi / 144
    return e == 0     ? 1.0
           : e == 9   ? 0.92387953251128675613   // 16: 1
           : e == 12  ? 0.86602540378443864676   // 12: 1
           : e == 16  ? 0.76604444311897803520   // 9: 1
           : e == 18  ? 0.70710678118654752440   // 16: 2
           : e == 24  ? 0.5                      // 6: 1, 12: 2
           : e == 27  ? 0.38268343236508977173   // 16: 3
           : e == 32  ? 0.17364817766693034885   // 9: 2
           : e == 36  ? 0.0                      // 12: 3, 16: 4
           : e == 48  ? -0.5                     // 6: 2, 12: 4
           : e == 54  ? -0.70710678118654752440  // 16: 6
           : e == 64  ? -0.93969262078590838405  // 9: 4
           : e == 72  ? -1.0                     // 12: 6
           : e == 81  ? -0.92387953251128675613  // 16: 9
                      : 2.0;                     // not an inner twiddle
}
__host__ __device__ constexpr double root_s(int R, int k) {
    const int e = k * (144 / R);
    return e == 0     ? 0.0
           : e == 9   ? 0.38268343236508977173
           : e == 12  ? 0.5
           : e == 16  ? 0.64278760968653932632
           : e == 18  ? 0.70710678118654752440
           : e == 24  ? 0.86602540378443864676
           : e == 27  ? 0.92387953251128675613
           : e == 32  ? 0.98480775301220805937
           : e == 36  ? 1.0
           : e == 48  ? 0.86602540378443864676
           : e == 54  ? 0.70710678118654752440
           : e == 64  ? 0.34202014332566873304
           : e == 72  ? 0.0
           : e == 81  ? -0.38268343236508977173
                      : 2.0;
}

template <typename T, int R, int SIGN>
__device__ __forceinline__ void dftR(T* xr, T* xi);

// radix A B: A-point DFTs over the elements n = B n1 + n2 of each n2, the
// twiddles exp(SIGN 2 pi i n2 k1 / (A B)), B-point DFTs over n2; output
// k1 + A k2
template <typename T, int A, int B, int SIGN>
__device__ __forceinline__ void dft_ab(T* xr, T* xi) {
    constexpr int R = A * B;
    T tr[B][A], ti[B][A];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) {
            tr[n2][n1] = xr[B * n1 + n2];
            ti[n2][n1] = xi[B * n1 + n2];
        }
        dftR<T, A, SIGN>(tr[n2], ti[n2]);
#pragma unroll
        for (int k1 = 1; k1 < A; ++k1)
            if (n2 > 0) cmul(tr[n2][k1], ti[n2][k1], (T)root_c(R, n2 * k1), (T)SIGN * (T)root_s(R, n2 * k1));
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
        T vr[B], vi[B];
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) {
            vr[n2] = tr[n2][k1];
            vi[n2] = ti[n2][k1];
        }
        dftR<T, B, SIGN>(vr, vi);
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) {
            xr[k1 + A * k2] = vr[k2];
            xi[k1 + A * k2] = vi[k2];
        }
    }
}

template <typename T, int R, int SIGN>
__device__ __forceinline__ void dftR(T* xr, T* xi) {
    if constexpr (R == 2) dft2<T, SIGN>(xr, xi);
    else if constexpr (R == 3) dft3<T, SIGN>(xr, xi);
    else if constexpr (R == 4) dft4<T, SIGN>(xr, xi);
    else if constexpr (R == 6) dft_ab<T, 3, 2, SIGN>(xr, xi);
    else if constexpr (R == 8) dft8<T, SIGN>(xr, xi);
    else if constexpr (R == 9) dft_ab<T, 3, 3, SIGN>(xr, xi);
    else if constexpr (R == 12) dft_ab<T, 4, 3, SIGN>(xr, xi);
    else dft_ab<T, 4, 4, SIGN>(xr, xi);
}

// One Stockham stage of radix R over all nseq sequences.  MAXB bounds the
// butterflies per thread: nseq*N/R <= MAXB*blockDim.x.  N and Ns are
// compile-time constants when the caller's are.
template <typename T, int R, int MAXB, int SIGN, int NTHR, int PS = kPadShift>
__device__ __forceinline__ void fft_stage(T* __restrict__ re, T* __restrict__ im, int N, int SP, int nseq, int Ns,
                                          const T* __restrict__ twc, const T* __restrict__ tws) {
    const int NR = N / R;
    const int nb = nseq * NR;
    const int tstep = N / (Ns * R);
    T vr[MAXB][R], vi[MAXB][R];
    int dst[MAXB];
#pragma unroll
    for (int b = 0; b < MAXB; ++b) {
        const int w = threadIdx.x + b * NTHR;
        dst[b] = -1;
        if (w < nb) {
            const int s = w / NR;
            const int j = w - s * NR;
            const int k = j % Ns;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int o = li<PS>(s, j + r * NR, SP);
                vr[b][r] = re[o];
                vi[b][r] = im[o];
            }
            if (Ns > 1) {
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    const int t = k * r * tstep;
                    cmul(vr[b][r], vi[b][r], twc[t], (T)SIGN * tws[t]);
                }
            }
            dftR<T, R, SIGN>(vr[b], vi[b]);
            dst[b] = s * (1 << 20) + (j - k) * R + k;   // (sequence, position) packed
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < MAXB; ++b) {
        if (dst[b] >= 0) {
            const int s = dst[b] >> 20;
            const int pos = dst[b] & ((1 << 20) - 1);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int o = li<PS>(s, pos + r * Ns, SP);
                re[o] = vr[b][r];
                im[o] = vi[b][r];
            }
        }
    }
    __syncthreads();
}

__host__ __device__ constexpr int cdiv(int a, int b) { return (a + b - 1) / b; }

// Radix schedule of a compiled length: the fewest stages (each costs an LDS
// round trip of the tile and two barriers), among those the smallest sum of
// radices; powers of two first, the larger first (the first stage has no
// twiddles, and scatters with the stride of its radix: 768 points as 12 8 8
// instead of 8 8 12 took 3-5 % longer).
constexpr int kNoSchedule = 1 << 20;
__host__ __device__ constexpr int sched_cost(int n, int stages) {
    if (stages == 0) return n == 1 ? 0 : kNoSchedule;
    constexpr int rad[8] = {16, 12, 9, 8, 6, 4, 3, 2};
    int best = kNoSchedule;
    for (int r : rad)
        if (n % r == 0) {
            const int c = r + sched_cost(n / r, stages - 1);
            if (c < best) best = c;
        }
    return best;
}
__host__ __device__ constexpr int num_stages(int n) {
    int s = 1;
    while (sched_cost(n, s) >= kNoSchedule) ++s;
    return s;
}
__host__ __device__ constexpr int stage_radix(int n, int st) {
    constexpr int rad[8] = {16, 8, 4, 2, 12, 9, 6, 3};
    int left = num_stages(n);
    for (;;) {
        const int want = sched_cost(n, left);
        for (int r : rad)
            if (n % r == 0 && r + sched_cost(n / r, left - 1) == want) {
                if (st == 0) return r;
                n /= r;
                break;
            }
        --st;
        --left;
    }
}

template <typename T, int EMAX, int NTHR, int SIGN, int NF, int ST, int NS, int PS = kPadShift>
__device__ __forceinline__ void fft_fixed(T* re, T* im, int nseq, const T* __restrict__ twc,
                                          const T* __restrict__ tws) {
    if constexpr (ST < num_stages(NF)) {
        constexpr int R = stage_radix(NF, ST);
        fft_stage<T, R, cdiv(EMAX, NTHR * R), SIGN, NTHR, PS>(re, im, NF, seq_stride(NF, PS), nseq, NS, twc, tws);
        fft_fixed<T, EMAX, NTHR, SIGN, NF, ST + 1, NS * R, PS>(re, im, nseq, twc, tws);
    }
}

// Full transform of nseq sequences (nseq*N <= EMAX) with NTHR threads, the
// length from the arguments.
template <typename T, int EMAX, int NTHR, int SIGN>
__device__ __forceinline__ void fft_lds(T* re, T* im, int N, int nseq, const FftPlan& pl,
                                        const T* __restrict__ twc, const T* __restrict__ tws) {
    const int SP = seq_stride(N);
    int Ns = 1;
    for (int st = 0; st < pl.nstages; ++st) {
        const int R = pl.radix[st];
        if (R == 8)
            fft_stage<T, 8, cdiv(EMAX, NTHR * 8), SIGN, NTHR>(re, im, N, SP, nseq, Ns, twc, tws);
        else if (R == 4)
            fft_stage<T, 4, cdiv(EMAX, NTHR * 4), SIGN, NTHR>(re, im, N, SP, nseq, Ns, twc, tws);
        else if (R == 2)
            fft_stage<T, 2, cdiv(EMAX, NTHR * 2), SIGN, NTHR>(re, im, N, SP, nseq, Ns, twc, tws);
        else
            fft_stage<T, 3, cdiv(EMAX, NTHR * 3), SIGN, NTHR>(re, im, N, SP, nseq, Ns, twc, tws);
        Ns *= R;
    }
}

}  // namespace dev
}  // namespace fsei
