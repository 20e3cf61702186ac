// Tilings and launches of the z solve for one type: this file is compiled
// twice, with -DFSEI_REAL=double and -DFSEI_REAL=float.
#include <cstdint>

#include "fsei_z.h"

namespace fsei {
namespace dev {

namespace {

using T = FSEI_REAL;
using Args = ZArgs<T, T>;
constexpr bool F32 = sizeof(T) == 4;

// All forms do the same arithmetic.  ZPF: the persistent kernel; ZV: adjacent
// modes per lane as one vector; Z1: one mode per lane; the number: chunks.
enum ZForm { ZPF1, ZPF32, ZV32_HALF, ZV32, ZV32_WIDE, ZV64, Z1_32, Z1_64 };

// chunking of the z lines: P chunks of exactly L rows (L one of the compiled
// sizes), the last chunk padded with decoupled rows; P <= pmax
constexpr int next_rows(int l) { return l < 16 ? l + 4 : l + 8; }   // 4, 8, 12, 16, 24, 32
bool choose_chunks(Args* a, int pmax) {
    for (int l = 4; l <= 32; l = next_rows(l)) {
        const int pc = (a->nz + l - 1) / l;
        if (pc <= pmax) {
            a->L = l;
            a->P = pc;
            return true;
        }
    }
    return false;
}

// lanes per tile row of the persistent kernel (16 bytes each)
constexpr int pf_lanes(int l) { return l >= 24 ? 16 : 8; }
int pf_modes(const Args& a) { return pf_lanes(a.L) * 16 / (int)sizeof(T); }

// groups of special lines beside tiles of pmax chunks in workgroups of nt threads
int groups(const Args& a, int pmax, int nt) {
    const int ln = (nt < 512 ? nt : 512) / zspec_chunks(pmax, a.L, nt);
    return 1 + (a.nlist + ln - 1) / ln;
}

template <int L, int S, bool RAG, bool TR>
void launch_pf(const Args& a, hipStream_t st, int cus) {
    constexpr int TXLM = pf_lanes(L);
    const long ntiles = (long)a.gx * a.ny, want = (long)cus * (16 / TXLM);
    const unsigned g = (unsigned)(ntiles < want ? ntiles : want);
    constexpr int M = L == 32 ? 1 : 16 / (int)sizeof(T);
    hipLaunchKernelGGL((k_zsolvev_pf<T, T, M, TXLM, L, 32 * TXLM, S, RAG, TR>), dim3(g), dim3(32 * TXLM), 0, st, a);
}
template <int L, int S>
void launch_pf_any(const Args& a, hipStream_t st, int cus) {
    const bool rag = a.nz != 32 * L;
    if (a.transposed) {
        if (rag) launch_pf<L, S, true, true>(a, st, cus);
        else launch_pf<L, S, false, true>(a, st, cus);
    } else {
        if (rag) launch_pf<L, S, true, false>(a, st, cus);
        else launch_pf<L, S, false, false>(a, st, cus);
    }
}

// LO .. HI: the rows per chunk that the tiling gives a form
template <int M, int TXLM, int NT, int LO, int HI, int L = LO>
void launch_v(const Args& a, hipStream_t st) {
    if (L < HI && a.L != L) {
        if constexpr (L < HI) launch_v<M, TXLM, NT, LO, HI, next_rows(L)>(a, st);
        return;
    }
    const dim3 g((unsigned)a.nspec + (unsigned)a.gx * (unsigned)a.ny), b(NT);
    hipLaunchKernelGGL((k_zsolvev<T, T, M, TXLM, L, NT>), g, b, 0, st, a);
}

template <int TXL, int NT, int LO, int HI, int L = LO>
void launch_1(const Args& a, hipStream_t st) {
    if (L < HI && a.L != L) {
        if constexpr (L < HI) launch_1<TXL, NT, LO, HI, next_rows(L)>(a, st);
        return;
    }
    const dim3 g((unsigned)a.nspec + (unsigned)a.gx * (unsigned)a.ny), b(NT);
    hipLaunchKernelGGL((k_zsolve<T, T, TXL, L, NT>), g, b, 0, st, a);
}

template <int PS, int L>
void launch_spec(const Args& a, hipStream_t st) {
    constexpr int LN = 512 / PS;
    hipLaunchKernelGGL((k_zspecial<T, T, PS, L>), dim3(1u + (unsigned)((a.nlist + LN - 1) / LN)), dim3(512), 0, st, a);
}

// FP32: 16 lanes x 2 modes (128-B rows) in 512 threads against the forms after it
// in z_tiling's list.  It needs half the registers of the four-mode form and has
// twice its waves (us: 384 x 384 x 144 54 -> 44, 512 x 512 x 64 58 -> 50, 1024 x
// 1024 x 64 207 -> 181, 128 x 128 x 192 17.7 -> 15.9), which it loses in many
// rounds of 12 and 16 rows per chunk (1024 x 1024 x 384 853 -> 918; 512 x 512 x
// 500 247 -> 265, but 288 x 288 x 500 78 -> 67).  Where nx / 2 is odd the
// two-mode form in 1024 threads is as fast or faster up to 8 rows (486 x 486 x
// 256 121 against 145, x 128 82 against 86) but for few tiles (54 x 54 x 200 12.4
// against 10.8) or few chunks (162 x 162 x 12 10.8 against 9.2).
bool two_modes_512(const Args& a, int cus) {
    const long tiles = (long)((a.nx + 31) / 32) * a.ny;
    if (a.L > 16 || a.nx % 2 != 0) return false;
    if (a.L >= 12) return tiles <= (a.L == 12 ? 100L : 20L) * cus;
    if (a.nx % 4 == 0) return true;
    return a.L == 4 ? (a.P <= 12 || tiles <= 2L * cus) : tiles <= cus;
}

}  // namespace

// Adjacent modes per lane as one vector where nx allows, at most 32 chunks per
// line; lines longer than 768 rows (chunks of 32 rows) keep one FP64 mode per
// lane or take 64 FP32 chunks of at most 16 rows, which avoids register spills.
//
// The persistent kernel where it was the faster (us, forward, against the form
// below it in the list):
//   FP64, 12 or 16 rows per chunk, tiles of 16 modes in 256 threads, two
//     workgroups per CU: 256 x 256 x 384 98 -> 83, 288 x 288 x 467 168 -> 142,
//     384 x 384 x 500 294 -> 271 (tiles of 32 modes in 512 threads, one per CU:
//     104, 157, 257); needs a few tiles per workgroup (128 x 96 x 400, 1.5 of
//     them: 29.3 -> 31.7).  8 rows: slower (256 x 256 x 250: 58 -> 65).
//   FP64, 32 rows: 768 x 768 x 1024 2651 -> 2318, 512 x 256 x 900 585 -> 428.
//   24 rows: whole 768-row lines, FP64 also transposed (512 x 512 x 768: 857 ->
//     673); padded chunks spill registers there (384 x 256 x 513: 226 -> 302).
//   FP32 otherwise not: 256 x 256 x 384 53 -> 61 to 71.
template <>
bool z_tiling<T>(Args* a, int cus) {
    const int nx = a->nx;
    int pmax = 32, nt = 512, tx;
    const bool c32 = choose_chunks(a, 32);
    const bool al16 = reinterpret_cast<uintptr_t>(a->data) % 16 == 0;
    const bool pf = a->nz == 768 ? (!F32 || !a->transposed)
                                 : !F32 && (a->L == 12 || a->L == 16) &&
        (long)(nx / 16) * a->ny >= 4L * cus;
    if (c32 && pf && nx % pf_modes(*a) == 0 && al16) {
        a->form = ZPF32;
        tx = pf_modes(*a);
        nt = 32 * pf_lanes(a->L);
    } else if (F32 && c32 && two_modes_512(*a, cus)) {
        a->form = ZV32_HALF;
        tx = 32;
    } else if (c32 && a->L <= 24 && nx % (16 / (int)sizeof(T)) == 0) {
        // FP64: 16 lanes x 2 modes (256-B rows) in 512 threads.  FP32: 8 lanes
        // x 4 modes (128-B rows) in 256 threads, two workgroups per CU, one
        // solving while the other loads (11 % faster than 16 lanes in 512
        // threads, one per CU, at 512 x 512 x 768; the FP64 kernel the other
        // way round, 18 % slower)
        a->form = ZV32;
        nt = F32 ? 256 : 512;
        tx = 32;
    } else if (F32 && c32 && a->L <= 24 && nx % 2 == 0) {
        a->form = ZV32_WIDE;
        nt = 1024;
        tx = 64;
    } else if (F32 && nx % 2 == 0 && choose_chunks(a, 64)) {
        a->form = ZV64;
        pmax = 64;
        nt = 1024;
        tx = 32;
    } else if (!F32 && c32 && a->L == 32 && nx % 16 == 0 && al16 && (long)(nx / 16) * a->ny >= 3L * cus) {
        a->form = ZPF1;
        tx = 16;
    } else if (c32) {
        a->form = Z1_32;
        nt = F32 ? 1024 : 512;
        tx = F32 ? 32 : 16;
    } else {
        choose_chunks(a, 64);
        a->form = Z1_64;
        pmax = 64;
        nt = F32 ? 1024 : 512;
        tx = F32 ? 16 : 8;
    }
    a->gx = (nx + tx - 1) / tx;
    a->nspec = groups(*a, pmax, nt);
    // special lines that would take the tiles' launch more than one round of
    // the CUs go ahead in a launch of their own
    if (a->nspec <= cus) return false;
    a->nspec = 0;
    return true;
}

// Chunks of a line by its length: with 64 for every line up to 256 rows a
// workgroup held 8 lines whatever their length (262 thousand lines of 4, 16, 64
// rows, us: 221, 307, 312 so, 11, 25, 87 here; one lane per line 48, 89, 229)
template <>
void z_launch_special<T>(const Args& a, hipStream_t st) {
    if (a.nz <= 8) launch_spec<2, 4>(a, st);
    else if (a.nz <= 16) launch_spec<4, 4>(a, st);
    else if (a.nz <= 32) launch_spec<8, 4>(a, st);
    else if (a.nz <= 64) launch_spec<16, 4>(a, st);
    else if (a.nz <= 128) launch_spec<32, 4>(a, st);
    else if (a.nz <= 256) launch_spec<64, 4>(a, st);
    else if (a.nz <= 512) launch_spec<64, 8>(a, st);
    else if (a.nz <= 1024) launch_spec<64, 16>(a, st);
    else launch_spec<128, 16>(a, st);
}

template <>
void z_launch<T>(const Args& a, hipStream_t st, int cus) {
    switch (a.form) {
        case ZPF1:
            if constexpr (!F32) launch_pf_any<32, 26>(a, st, cus);
            break;
        case ZPF32:
            // rows of each chunk staged in LDS for the next tile: all where the
            // tile fits beside the tables, else what fits
            if constexpr (F32) {
                launch_pf<24, 12, false, false>(a, st, cus);
            } else {
                if (a.L == 12) launch_pf_any<12, 12>(a, st, cus);
                else if (a.L == 16) launch_pf_any<16, 11>(a, st, cus);
                else if (a.transposed) launch_pf<24, 12, false, true>(a, st, cus);
                else launch_pf<24, 12, false, false>(a, st, cus);
            }
            break;
        case ZV32_HALF:
            if constexpr (F32) launch_v<2, 16, 512, 4, 16>(a, st);
            break;
        case ZV32:
            if constexpr (F32) launch_v<4, 8, 256, 12, 24>(a, st);   // up to 8 rows: ZV32_HALF
            else launch_v<2, 16, 512, 4, 24>(a, st);
            break;
        case ZV32_WIDE:
            if constexpr (F32) launch_v<2, 32, 1024, 4, 24>(a, st);
            break;
        case ZV64:
            if constexpr (F32) launch_v<2, 16, 1024, 16, 32>(a, st);   // from 769 rows
            break;
        case Z1_32:
            if constexpr (F32) launch_1<32, 1024, 4, 32>(a, st);
            else launch_1<16, 512, 4, 32>(a, st);
            break;
        default:
            if constexpr (F32) launch_1<16, 1024, 24, 32>(a, st);   // from 1025 rows
            else launch_1<8, 512, 24, 32>(a, st);
            break;
    }
}

}  // namespace dev
}  // namespace fsei
