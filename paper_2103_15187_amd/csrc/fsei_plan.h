// Internal plan structure shared by the host-only plan code (fsei_plan.cpp)
// and the HIP entry points (fsei_api.hip).  No HIP types appear here, so the
// plan logic builds and runs on a machine without a GPU.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "../../include/fsei.h"

namespace fsei {

constexpr int kMaxStages = 16;
constexpr int kMaxN = 2048;     // longest x/y transform
constexpr int kMaxNz = 2048;    // longest z line
constexpr size_t kAlign = 256;
constexpr int kSumGroups = 64;   // first-stage workgroups of the two-stage partial sums
// complex elements per x-transform workgroup (8 per thread; 256 threads, 384
// at length 768 so that the tile holds four sequences there too): small
// tiles keep several workgroups resident per CU so loads, LDS transforms and
// stores of different workgroups overlap
inline int x_emax(int nx) { return nx == 768 ? 3072 : 2048; }

// LDS tile geometry shared by the host (launch sizes) and the kernels:
// sequence s of length N starts at s * seq_stride(N); one array of a tile of
// emax complex elements holds lds_elems(emax) slots.
// One pad slot every 2^ps elements (ps = kPadShift unless a kernel picks its
// own: the best pad depends on the kernel's access pattern and is measured).
constexpr int kPadShift = 4;
constexpr int seq_stride(int N, int ps = kPadShift) { return N + (N >> ps) + 1; }
constexpr int lds_elems(int emax, int ps = kPadShift) { return emax + (emax >> ps) + 16; }
constexpr int tile_nseq(int emax, int N, int ps = kPadShift) {
    return (emax / N < lds_elems(emax, ps) / seq_stride(N, ps)) ? emax / N : lds_elems(emax, ps) / seq_stride(N, ps);
}
inline int x_nseq(int nx) { return tile_nseq(x_emax(nx), nx) > 0 ? tile_nseq(x_emax(nx), nx) : 1; }

// Lengths with kernels compiled for them (fsei_len.hip): every 2^a 3^b from
// kLenMin to kLenMax, as listed in FSEI_LENGTHS; other lengths, and fields
// that are not aligned to column pairs, take the kernels with the length from
// the arguments.
constexpr int kLenMin = 16;
constexpr int kLenMax = 1024;
#define FSEI_LENGTHS(X)                                                                                     \
    X(16) X(18) X(24) X(27) X(32) X(36) X(48) X(54) X(64) X(72) X(81) X(96) X(108) X(128) X(144) X(162)     \
    X(192) X(216) X(243) X(256) X(288) X(324) X(384) X(432) X(486) X(512) X(576) X(648) X(729) X(768) X(864) \
    X(972) X(1024)

// Tile of the compiled x kernels: RG groups of threads, one thread per column
// pair of the line in each, side by side over x_len_rows rows of one z-plane;
// enough groups that the whole waves are at least 3/4 used, or as well used
// as they can be.  A group takes up to eight rows (the same number of complex
// elements per thread as a radix-8 butterfly), fewer where the groups are
// many (short lines: small grids need the workgroups) or the line is long
// (two FP64 workgroups of 1024-point lines must fit the CU's LDS).
//
// Threads (x and y): where LDS leaves two or three workgroups per CU, whole
// sets of four waves, one per SIMD; a workgroup of five, six, seven, nine or
// eleven waves loads the SIMDs unevenly and streams up to 40 % slower
// (measured at 80 M cells, TB/s: y FP64 384 points 6 waves 3.3, 8 waves 5.5;
// y FP32 432 points 14 waves 2.7, 16 waves 4.5; x FP64 768 points 6 waves
// 3.9, 8 waves 4.9).  FP32 x tiles leave room for four and more workgroups, which
// balance by themselves (768 points: 6 waves 4.36, 8 waves 4.17).
constexpr int round64(int n) { return (n + 63) / 64 * 64; }
constexpr int round_waves(int threads) { return threads <= 256 ? round64(threads) : (threads + 255) / 256 * 256; }
constexpr int x_len_groups(int n) {
    const int np = (n + 1) / 2;
    int best = 1;
    for (int rg = 1; rg <= 8; rg *= 2) {
        if (4 * np * rg >= 3 * round64(np * rg)) return rg;
        if (np * rg * round64(np * best) > np * best * round64(np * rg)) best = rg;
    }
    return best;
}
constexpr int x_len_rows(int n) { return x_len_groups(n) > 1 ? 16 : n > 768 ? 4 : 8; }
constexpr int x_len_threads(int n, int elem) {
    const int t = (n + 1) / 2 * x_len_groups(n);
    return (elem == 4 && n <= 768) ? round64(t) : round_waves(t);
}

// The fused x inverse + gradient kernel (FP64): even lengths from 256 to 768.
// Two thread groups, one thread per column pair in each, divide its eight rows
// up to 512 points; enough threads for a radix-8 stage of its five sequences.
constexpr bool xg_len(int n) { return n % 2 == 0 && n >= 256 && n <= 768; }
constexpr int xg_len_groups(int n) { return n <= 512 ? 2 : 1; }
constexpr int xg_len_threads(int n) {
    const int t = n / 2 * xg_len_groups(n), b = 5 * n / 8;
    return n <= 512 ? round64(t) : round_waves(t > b ? t : b);
}

// Own rows and complex sequences per step of the fused x inverses, and the row
// of a plane that sequence s (0 .. kXgSeq - 1) of the x inverse + gradient reads
// as its first (half 0) or second (half 1) line, for the tile of rows j0 ..
// j0 + 7: sequence 0 starts with the halo row j0 - 1 (wrapped); the last one's
// second line is a zero row, for which a valid row is addressed.
constexpr int kXgRows = 8;
constexpr int kXgSeq = 5;
constexpr int xg_in_row(int s, int half, int j0, int ny) {
    return half == 0 ? (s == 0 ? (j0 > 0 ? j0 - 1 : ny - 1) : j0 + 2 * s - 1)
                     : j0 + (2 * s < kXgRows ? 2 * s : kXgRows - 1);
}

// Tile of the compiled y kernels: column pairs per tile (rows of 128 bytes;
// 64 for lines beyond 512, two of whose workgroups then fit a CU, but for 1024
// points in FP64 and in the FP32 forward kernel, which reads four tables), about
// eight complex elements per thread
constexpr int y_len_pairs(int n, int elem) { return (n <= 512 ? 64 : 32) / elem; }
constexpr int y_len_threads(int n, int elem) { return round_waves(y_len_pairs(n, elem) * n / 8); }
// pad of the kernels' LDS sequences: FP32 forward tiles run fastest with one
// slot per 64 elements, the others with one per 16 (measured)
constexpr int y_len_pad(int elem, bool inverse) { return elem == 4 && !inverse ? 6 : kPadShift; }
// their LDS: the tile's two arrays, the FFT twiddles and (FP32 forward) the
// post-twiddles
constexpr int y_len_lds(int n, int elem, bool inverse) {
    return (2 * y_len_pairs(n, elem) * seq_stride(n, y_len_pad(elem, inverse)) + (elem == 4 && !inverse ? 4 : 2) * n) * elem;
}
// waves per SIMD that two workgroups per CU need, where two fit (the kernels'
// register bound)
constexpr int y_len_waves(int n, int elem, bool inverse) {
    return ((2 * y_len_lds(n, elem, inverse) <= 160 * 1024 ? 2 : 1) * y_len_threads(n, elem) + 255) / 256;
}

// Line solves of the implicit viscous step: every line is cut into
// kViscPmax chunks of L rows (L one of the compiled sizes), so lines of up
// to kViscPmax * 32 rows are supported.  One table block per (component,
// direction) holds visc_tab_elems(L) doubles (layout in fsei_viscous.h).
constexpr int kViscPmax = 32;
constexpr int kViscLv = 5;   // Kogge-Stone levels over the chunks, log2(kViscPmax)
constexpr int kViscMaxN = kViscPmax * 32;
constexpr int visc_tab_elems(int L) { return 6 * kViscPmax * L + 2 * kViscLv * kViscPmax + 2; }
// chunk length for a line of n rows (0: too long)
constexpr int visc_chunk(int n) {
    return n <= kViscPmax * 4    ? 4
           : n <= kViscPmax * 8  ? 8
           : n <= kViscPmax * 12 ? 12
           : n <= kViscPmax * 16 ? 16
           : n <= kViscPmax * 24 ? 24
           : n <= kViscPmax * 32 ? 32
                                 : 0;
}

// The x kernel of the line solves: tiles of kViscXLines lines, one lane per
// (line, chunk), each workgroup walking up to kViscXTiles consecutive tiles with
// the tables staged once.
constexpr int kViscXLines = 8;
constexpr int kViscXTiles = 4;
// its workgroups per CU, by LDS (tables, scan slots and the tile) and threads
constexpr long visc_x_per_cu(int n, int L) {
    const long lds = 8L * (visc_tab_elems(L) + 2 * kViscXLines * kViscPmax + 2 * kViscXLines + kViscXLines * (n + 2));
    const long fit = 160L * 1024 / lds, thr = 2048 / (kViscXLines * kViscPmax);
    return fit < thr ? fit : thr;
}
// Twice the time of nlines lines with t tiles per workgroup, in tiles: the
// tables and the first tile's round trip cost about 2.5 tiles more per workgroup
// (measured one round: 96 rows 5.1 + 1.5 t us, 512 rows 7.3 + 2.8 t, 768 rows
// 9.8 + 3.8 t)
constexpr long visc_x_cost(long nlines, int t, int n, int L, int cus) {
    const long per = (long)kViscXLines * t, slots = visc_x_per_cu(n, L) * cus;
    const long groups = (nlines + per - 1) / per;
    return (groups + slots - 1) / slots * (2 * t + 5);
}
// Tiles per workgroup: the fewest such tiles in all rounds of the CUs.  (us
// with 1, 2, 3, 4 tiles: 7968 lines of 768 rows, one workgroup per CU, 47.0,
// 38.7, 43.9, 30.3; 24000 lines of 512 rows 47.1, 47.4, 42.2, 45.4; 9360 lines
// of 96 rows 11, 12, 13, 15.)
constexpr int visc_x_tiles(long nlines, int n, int L, int cus) {
    int best = 1;
    for (int t = 2; t <= kViscXTiles; ++t)
        if (visc_x_cost(nlines, t, n, L, cus) < visc_x_cost(nlines, best, n, L, cus)) best = t;
    return best;
}

// Radix schedule of one complex FFT length (radices 8, 4, 2, 3).
struct FftPlan {
    int n = 0;
    int nstages = 0;
    int radix[kMaxStages] = {0};
};

// Names of the per-k / per-mode / twiddle tables stored on the device, each
// in double and in float.  The order is the order inside the table block.
enum TableId {
    T_ZA = 0,      // a_k  = 1/(dz_k h_k), k>=1; a_0 = 0            (nz)
    T_ZC,          // c_k  = 1/(dz_k h_{k+1}), k<=nz-2; c_{nz-1}=0  (nz)
    T_ZB0,         // -(a_k + c_k)                                    (nz)
    T_DZ,          // dz_k                                            (nz)
    T_INV_DZ,      // 1/dz_k                                          (nz)
    T_INV_H,       // 1/h_k, k>=1; 0 at k=0                           (nz)
    T_H,           // h_k = zm_k - zm_{k-1}, k>=1; 0 at k=0          (nz)
    T_ZETA_ADJ,    // 1/h_{k+1} for k<=nz-2, 0 at nz-1                (nz)
    T_GAM_ADJ,     // 1/dz_{k-1} for k>=1, 0 at k=0                   (nz)
    T_ZF,          // z of face k (zc_k), k < nz                     (nz)
    T_ZM,          // z of cell centre k, (zc_k + zc_{k+1})/2         (nz)
    T_HF,          // z extent of the w-face volumes: h_k, k>=1; dz_0/2 (nz)
    T_LAMX,        // modified wavenumbers of x rows                  (nx)
    T_LAMY,        // modified wavenumbers of y rows                  (ny)
    T_TWX_C,       // cos(2 pi t / nx)                                (nx)
    T_TWX_S,       // sin(2 pi t / nx)                                (nx)
    T_DCTX_C,      // cos(pi m / (2 nx))                              (nx)
    T_DCTX_S,      // sin(pi m / (2 nx))                              (nx)
    T_TWY_C,       // cos(2 pi t / ny)                                (ny)
    T_TWY_S,       // sin(2 pi t / ny)                                (ny)
    T_DCTY_C,      // cos(pi m / (2 ny))                              (ny)
    T_DCTY_S,      // sin(pi m / (2 ny))                              (ny)
    T_COUNT
};

// Kernel slots for per-kernel timing.
enum KernelSlot {
    K_XFWD = 0, K_YFWD, K_ZSOLVE, K_YINV, K_XINV, K_GRAD, K_RESID_XFWD, K_XINV_ACC,
    K_NORM, K_PREP, K_SLOT_COUNT
};

struct fsei_plan_impl {
    int nx = 0, ny = 0, nz = 0, bcx = 0, bcy = 0;
    double dx = 0, dy = 0;
    std::vector<double> zc, dz, h;   // h[0] unused (0)
    double lz = 0;
    double dzmin = 0;

    FftPlan fx, fy;

    int precision = FSEI_PREC_FP64;
    double rtol = 1e-10;
    int max_iter = 4;
    double kappa_star = 1e4;

    // host copies of the device tables
    std::vector<double> tab_d;
    std::vector<float> tab_f;
    size_t tab_off[T_COUNT] = {0};   // element offsets inside tab_d / tab_f
    size_t tab_elems = 0;

    // workspace layout (byte offsets)
    size_t ws_tab_d = 0, ws_tab_f = 0, ws_scalars = 0, ws_partials = 0;
    size_t ws_field = 0, ws_field_bytes = 0;       // main intermediate field
    size_t ws_field2 = 0, ws_field2_bytes = 0;     // second field (refine: FP32 work field)
    size_t ws_field3 = 0, ws_field3_bytes = 0;     // refine: FP64 pressure when the caller passes none
    size_t ws_field4 = 0, ws_field4_bytes = 0;     // refine: FP32 pressure of the first solve
    size_t ws_list = 0, ws_list_bytes = 0;         // near-singular mode lines
    // implicit viscous step: chunk length per direction (x, y, z; 0 when a
    // line is longer than kViscMaxN), the table blocks of the three
    // components (x, y, z blocks each), and the beta each component's
    // tables were last built for (NaN: not built for this workspace)
    int visc_L[3] = {0, 0, 0};
    size_t ws_visc = 0, ws_visc_comp = 0;           // region offset, bytes per component
    double visc_beta[3] = {0, 0, 0};
    std::vector<double> visc_host[3];
    size_t ws_total = 0;
    size_t n_partials = 0;                          // per-block partial sums (triples)
    static constexpr int kScalars = 64;

    // lines with |lambda_x + lambda_y| < sigma_thr (condition number above
    // kappa_star) are solved in FP64 with row-sum pivots
    double sigma_thr = 0.0;
    std::vector<int> list_host;
    int nlist = 0;

    void* ws = nullptr;
    size_t ws_bytes = 0;
    void* stream = nullptr;
    // timing
    bool timing = false;
    double t_ms[FSEI_NUM_KERNEL_SLOTS] = {0};
    long t_count[FSEI_NUM_KERNEL_SLOTS] = {0};
    std::vector<void*> ev_pool;          // hipEvent_t pairs, recorded lazily
    std::vector<int> ev_slot;            // pending (start, stop) pairs -> slot
    size_t ev_used = 0;

    size_t ncells() const { return (size_t)nx * ny * nz; }
};

// Host-side helpers (fsei_plan.cpp).
bool factor_radices(int n, FftPlan* out);
void compute_layout(fsei_plan_impl* p);
// Tables of the viscous line solves of component comp (0 u, 1 v, 2 w) for
// beta, x, y and z blocks one after the other (ws_visc_comp bytes).
void build_visc_tables(const fsei_plan_impl* p, int comp, double beta, double* out);

}  // namespace fsei

struct fsei_plan : fsei::fsei_plan_impl {};
