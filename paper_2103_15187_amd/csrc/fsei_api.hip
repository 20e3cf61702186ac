// HIP side of the C ABI: workspace upload, kernel launches on the plan's
// stream, precision modes, refinement loop, per-kernel event timing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <atomic>
#include <mutex>
#include <type_traits>
#include <vector>

#include "fsei_kernels.h"
#include "fsei_lengths.h"
#include "fsei_z.h"
#include "fsei_plan.h"
#include "fsei_viscous.h"
#include "fsei_momentum.h"
#include "fsei_ibm.h"

using namespace fsei;
using namespace fsei::dev;

namespace {



const char* kSlotNames[FSEI_NUM_KERNEL_SLOTS] = {
    "xfwd", "yfwd", "zsolve", "yinv", "xinv", "grad", "resid_xfwd", "xinv_acc", "norm", "zero_mode",
    "zsolve_fp64_lines", "resid_norm", "resid", "xfwd_r", "grad_resid", "visc_x", "visc_y", "visc_z", "momentum_rhs", "ib_transfer",
    "xinv_grad", "xinv_grad_resid"};
constexpr int K_ZLIST = 10;
constexpr int K_RESNORM = 11;
constexpr int K_RESID_PAIRS = 12;
constexpr int K_XFWD_R = 13;
constexpr int K_GRAD_RESID = 14;
constexpr int K_VISC_X = 15;
constexpr int K_VISC_Y = 16;
constexpr int K_VISC_Z = 17;
constexpr int K_MOM_RHS = 18;
constexpr int K_IB = 19;
constexpr int K_XINV_GRAD = 20;
constexpr int K_XINV_GRAD_RESID = 21;

struct PendingEv {
    hipEvent_t a, b;
    int slot;
};

struct TimingState {
    std::vector<PendingEv> pending;
    std::vector<hipEvent_t> free_ev;
};

TimingState& tstate(fsei_plan* p) {
    // one state per plan, owned through ev_pool[0]
    if (p->ev_pool.empty()) p->ev_pool.push_back(new TimingState());
    return *static_cast<TimingState*>(p->ev_pool[0]);
}

hipEvent_t get_event(TimingState& ts) {
    if (!ts.free_ev.empty()) {
        hipEvent_t e = ts.free_ev.back();
        ts.free_ev.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    (void)hipEventCreate(&e);
    return e;
}

void harvest(fsei_plan* p) {
    TimingState& ts = tstate(p);
    for (auto& pe : ts.pending) {
        (void)hipEventSynchronize(pe.b);
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, pe.a, pe.b);
        p->t_ms[pe.slot] += ms;
        p->t_count[pe.slot] += 1;
        ts.free_ev.push_back(pe.a);
        ts.free_ev.push_back(pe.b);
    }
    ts.pending.clear();
}

// Brackets one launch with events when timing is on.
struct Timed {
    fsei_plan* p;
    int slot;
    hipStream_t st;
    hipEvent_t a = nullptr, b = nullptr;
    Timed(fsei_plan* pl, int s) : p(pl), slot(s), st((hipStream_t)pl->stream) {
        if (p->timing) {
            TimingState& ts = tstate(p);
            if (ts.pending.size() > 4096) harvest(p);
            a = get_event(ts);
            b = get_event(ts);
            (void)hipEventRecord(a, st);
        }
    }
    ~Timed() {
        if (p->timing) {
            (void)hipEventRecord(b, st);
            tstate(p).pending.push_back({a, b, slot});
        }
    }
};

template <typename T>
const T* tab(const fsei_plan* p, int id);
template <>
const double* tab<double>(const fsei_plan* p, int id) {
    return reinterpret_cast<const double*>((const char*)p->ws + p->ws_tab_d) + p->tab_off[id];
}
template <>
const float* tab<float>(const fsei_plan* p, int id) {
    return reinterpret_cast<const float*>((const char*)p->ws + p->ws_tab_f) + p->tab_off[id];
}

double* scalars(const fsei_plan* p) { return reinterpret_cast<double*>((char*)p->ws + p->ws_scalars); }
double* partials(const fsei_plan* p) { return reinterpret_cast<double*>((char*)p->ws + p->ws_partials); }
void* field1(const fsei_plan* p) { return (char*)p->ws + p->ws_field; }
void* field2(const fsei_plan* p) { return (char*)p->ws + p->ws_field2; }
void* field3(const fsei_plan* p) { return (char*)p->ws + p->ws_field3; }
void* field4(const fsei_plan* p) { return (char*)p->ws + p->ws_field4; }
int* zlist(const fsei_plan* p) { return reinterpret_cast<int*>((char*)p->ws + p->ws_list); }

int nseq_x(const fsei_plan* p) { return x_nseq(p->nx); }

long xblocks(const fsei_plan* p) {
    const long nl = 2L * nseq_x(p);
    return ((long)p->ny * p->nz + nl - 1) / nl;
}

// pair kernels (gradient, residual norm): lanes own two adjacent x-cells,
// workgroups kPairRows rows of one plane
constexpr int kPairRows = 8;
bool pair_tiles(const fsei_plan* p) { return p->nx % 2 == 0 && p->ny % kPairRows == 0; }
bool aligned16(const void* q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; }
bool al16(const void* q) { return q == nullptr || aligned16(q); }   // optional pointer

// compute units of the current device (cached per device; 256 if the query fails)
int cus_of_current_device() {
    constexpr int kDevs = 64;
    static std::atomic<int> cus[kDevs];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevs) return 256;
    int n = cus[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cus[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// the kernels compiled for length n, or null
const LenOps* len_ops(int n) {
    switch (n) {
#define FSEI_CASE(n) \
    case n: return &len_ops_##n();
        FSEI_LENGTHS(FSEI_CASE)
#undef FSEI_CASE
        default: return nullptr;
    }
}

// The compiled x kernels read and write even lengths as aligned column pairs
// (odd lengths by single values): fields off the 16-byte alignment take the
// kernels with the length from the arguments.
const LenOps* x_ops(const fsei_plan* p, bool aligned) {
    return (p->nx % 2 != 0 || aligned) ? len_ops(p->nx) : nullptr;
}
// their workgroups: tiles of x_len_rows rows of one plane
long x_len_blocks(const fsei_plan* p, const LenOps* o) {
    return (long)((p->ny + o->x_rows - 1) / o->x_rows) * p->nz;
}

hipStream_t S(const fsei_plan* p) { return (hipStream_t)p->stream; }

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// returns the number of workgroups (with a.partials: of partial sums)
template <typename TI, typename TO, int PRO>
long launch_xfwd(fsei_plan* p, XFwdArgs<TI, TO> a, int slot) {
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.bcx = p->bcx;
    a.bcy = p->bcy;
    a.nseq = nseq_x(p);
    a.fp = p->fx;
    a.twc = tab<TO>(p, T_TWX_C);
    a.tws = tab<TO>(p, T_TWX_S);
    a.dctc = tab<TO>(p, T_DCTX_C);
    a.dcts = tab<TO>(p, T_DCTX_S);
    const bool al = al16(a.u) && al16(a.v) && al16(a.w) && al16(a.gp) && al16(a.f) && al16(a.p) &&
                    al16(a.p32) && al16(a.out) && al16(a.out_f);
    Timed t(p, slot);
    const LenOps* o = x_ops(p, al);
    // without room for a partial sum per tile (some plans of lines beyond 768
    // and ny no multiple of 4): the kernel whose tiles run on across planes
    if (o && a.partials && x_len_blocks(p, o) > (long)p->n_partials) o = nullptr;
    if (o) {
        const long nb = x_len_blocks(p, o);
        o->xfwd<TI, TO>(PRO)(a, (unsigned)nb, S(p));
        return nb;
    }
    const size_t dyn = 2 * p->nx * sizeof(TO);
    const long nb = xblocks(p);
    if (x_emax(p->nx) == 3072)
        hipLaunchKernelGGL((k_xfwd<TI, TO, PRO, 3072, 384>), dim3((unsigned)nb), dim3(384), dyn, S(p), a);
    else
        hipLaunchKernelGGL((k_xfwd<TI, TO, PRO, 2048, 256>), dim3((unsigned)nb), dim3(256), dyn, S(p), a);
    return nb;
}

template <typename T, typename TP, int EPI>
void launch_xinv(fsei_plan* p, const T* in, TP* out, int slot, const float* add32 = nullptr, T* keep = nullptr,
                 const double* vsum = nullptr) {
    XInvArgs<T, TP> a{};
    a.add32 = add32;
    a.keep = keep;
    a.vsum = vsum;
    a.vscale = 1.0 / ((double)p->nx * (double)p->ny * p->lz);
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.bcx = p->bcx;
    a.nseq = nseq_x(p);
    a.fp = p->fx;
    a.in = in;
    a.out = out;
    a.twc = tab<T>(p, T_TWX_C);
    a.tws = tab<T>(p, T_TWX_S);
    a.dctc = tab<T>(p, T_DCTX_C);
    a.dcts = tab<T>(p, T_DCTX_S);
    const bool al = al16(in) && al16(out) && al16(add32) && al16(keep);
    Timed t(p, slot);
    if (const LenOps* o = x_ops(p, al)) {
        o->xinv<T, TP>(EPI)(a, (unsigned)x_len_blocks(p, o), S(p));
        return;
    }
    const size_t dyn = 2 * p->nx * sizeof(T);
    const dim3 grid((unsigned)xblocks(p));
    if (x_emax(p->nx) == 3072)
        hipLaunchKernelGGL((k_xinv<T, TP, EPI, 3072, 384>), grid, dim3(384), dyn, S(p), a);
    else
        hipLaunchKernelGGL((k_xinv<T, TP, EPI, 2048, 256>), grid, dim3(256), dyn, S(p), a);
}

// The velocity a gradient correction reads and the one it writes: the same
// three arrays (in place), or outputs that overlap none of the inputs: a
// caller that keeps its input then needs no copy of it, 48 B/cell of FP64
// traffic less (autograd projection, FP32+refine at 512x512x768: 9.52 -> 7.44
// ms; FP64 forward + adjoint at 256x256x384: 2.59 -> 2.12 ms)
template <typename T>
struct Vel {
    const T *ui, *vi, *wi;
    T *u, *v, *w;
    bool aligned() const {
        return aligned16(ui) && aligned16(vi) && aligned16(wi) && aligned16(u) && aligned16(v) && aligned16(w);
    }
    // a further correction of the outputs
    Vel onto() const { return {u, v, w, u, v, w}; }
};
template <typename T>
Vel<T> in_place(T* u, T* v, T* w) {
    return {u, v, w, u, v, w};
}
template <typename Args, typename T>
void set_vel(Args* a, const Vel<T>& q) {
    a->ui = q.ui;
    a->vi = q.vi;
    a->wi = q.wi;
    a->u = q.u;
    a->v = q.v;
    a->w = q.w;
}

// the stencil weights of a gradient correction, or of its adjoint
template <typename Args>
void set_grad(const fsei_plan* p, Args* a, bool adjoint, double dt) {
    using T = decltype(a->cx);
    if (!adjoint) {
        a->cx = (T)(-dt / p->dx);
        a->cy = (T)(-dt / p->dy);
        a->sw = (T)(-dt);
        a->bk = tab<T>(p, T_INV_H);
        a->gk = tab<T>(p, T_INV_H);
    } else {
        a->cx = (T)(1.0 / p->dx);
        a->cy = (T)(1.0 / p->dy);
        a->sw = (T)1;
        a->bk = tab<T>(p, T_INV_DZ);
        a->gk = tab<T>(p, T_GAM_ADJ);
    }
}

// most planes per workgroup of the fused x inverses
constexpr int kXgPlanes = 32;

// Fused x inverse + gradient (FP64): a length it is compiled for, whole 8-row
// tiles, every field aligned to column pairs, and a grid of at least 32 planes
// of one tile per CU (two passes, us: 256 x 256 x 384 294 -> 274, its adjoint
// 290 -> 255; 384 x 384 x 500 1002 -> 921, adjoint 1002 -> 834; on small grids
// the intermediate stays in cache and the two passes are the faster: 128 x 128
// x 192 42 against 47, 512 x 64 x 64 33 against 231 in 32-plane chunks; in FP32
// too, 384 x 384 x 500 496 against 590)
const LenOps* xg_ops(const fsei_plan* p, const void* in, const void* pout, const Vel<double>& q) {
    const bool ok = xg_len(p->nx) && p->ny % kXgRows == 0 && aligned16(in) && al16(pout) && q.aligned() &&
                    (long)(p->ny / kXgRows) * p->nz >= 32L * cus_of_current_device();
    return ok ? len_ops(p->nx) : nullptr;
}

// Planes per workgroup: the fewest plane steps in all rounds of the CUs, each
// chunk with `extra` steps more for planes beyond its ends (576 x 384 x 384: 12
// planes, six whole rounds, 1.10 ms; 18 planes, 4.1 rounds, 1.24 ms)
int xg_planes(const fsei_plan* p, int per_cu, int extra) {
    const long slots = (long)per_cu * cus_of_current_device();   // workgroups at a time
    const long ntj = p->ny / kXgRows;
    long best = 0;
    int kc = kXgPlanes;
    for (int c = kXgPlanes; c >= 6; --c) {
        const long rounds = (ntj * ((p->nz + c - 1) / c) + slots - 1) / slots;
        if (best == 0 || rounds * (c + extra) < best) {
            best = rounds * (c + extra);
            kc = c;
        }
    }
    return kc;
}

void launch_xinv_grad(fsei_plan* p, const LenOps* ops, const double* in, double* pout, const Vel<double>& q,
                      bool adjoint, double dt) {
    using T = double;
    XInvGradArgs<T> a{};
    a.ny = p->ny;
    a.nz = p->nz;
    a.bcx = p->bcx;
    a.bcy = p->bcy;
    a.in = in;
    a.p = pout;
    set_vel(&a, q);
    set_grad(p, &a, adjoint, dt);
    a.twc = tab<T>(p, T_TWX_C);
    a.tws = tab<T>(p, T_TWX_S);
    a.dctc = tab<T>(p, T_DCTX_C);
    a.dcts = tab<T>(p, T_DCTX_S);
    const int ntj = p->ny / kXgRows;
    a.kc = xg_planes(p, p->nx <= 256 ? 2 : 1, 1);
    const int nchunk = (p->nz + a.kc - 1) / a.kc;
    Timed t(p, K_XINV_GRAD);
    ops->xg_d(a, (unsigned)(ntj * nchunk), S(p));
}

// First refinement correction fused with the gradient and the convergence
// check (FP32 correction, FP64 p): the two lengths it is compiled for, whole 8-row
// tiles, every field 16-byte aligned; returns the number of partials written.
// Other lengths take two passes of 80 B/cell instead of 72 (256 x 256 x 384 to
// 648 x 648 x 300: 4.6 to 5.1 TB/s).  The grid's size is not looked at: against
// the two passes 512 x 512 x 768 takes 2.88 ms instead of 3.14, 512 x 256 x 256
// 480 us instead of 514 and 768 x 128 x 128 182 instead of 203, but 512 x 64 x 64
// 74 instead of 36 and 768 x 64 x 64 82 instead of 48.
bool xgr_ok(const fsei_plan* p, const void* in, const void* p32, const void* p64, const void* f,
            const Vel<double>& q) {
    return (p->nx == 512 || p->nx == 768) && p->ny % kXgRows == 0 && aligned16(in) && aligned16(p32) &&
           aligned16(p64) && aligned16(f) && q.aligned();
}

long launch_xinv_grad_resid(fsei_plan* p, const float* in, const float* p32, const double* vsum, double* p64,
                            const Vel<double>& q, const double* f, double dt) {
    XInvGradResArgs a{};
    a.ny = p->ny;
    a.nz = p->nz;
    a.bcx = p->bcx;
    a.bcy = p->bcy;
    a.kc = xg_planes(p, p->nx == 512 ? 2 : 1, 2);
    a.in = in;
    a.p32 = p32;
    a.vsum = vsum;
    a.vscale = 1.0 / ((double)p->nx * (double)p->ny * p->lz);
    a.p = p64;
    set_vel(&a, q);
    a.cx = -dt / p->dx;
    a.cy = -dt / p->dy;
    a.sw = -dt;
    a.bk = tab<double>(p, T_INV_H);
    a.gk = tab<double>(p, T_INV_H);
    a.f = f;
    a.idx2 = 1.0 / (p->dx * p->dx);
    a.idy2 = 1.0 / (p->dy * p->dy);
    a.za = tab<double>(p, T_ZA);
    a.zc = tab<double>(p, T_ZC);
    a.scal = scalars(p);
    a.partials = partials(p);
    a.twc = tab<float>(p, T_TWX_C);
    a.tws = tab<float>(p, T_TWX_S);
    a.dctc = tab<float>(p, T_DCTX_C);
    a.dcts = tab<float>(p, T_DCTX_S);
    const int nchunk = (p->nz + a.kc - 1) / a.kc;
    const long nb = (long)(p->ny / kXgRows) * nchunk;
    Timed t(p, K_XINV_GRAD_RESID);
    if (p->nx == 768)
        hipLaunchKernelGGL((k_xinv_grad_resid<768>), dim3((unsigned)nb), dim3(xgr_threads<768>()),
                           2 * 768 * sizeof(float), S(p), a);
    else
        hipLaunchKernelGGL((k_xinv_grad_resid<512>), dim3((unsigned)nb), dim3(xgr_threads<512>()),
                           2 * 512 * sizeof(float), S(p), a);
    return nb;
}

template <typename T, int EMAX, int NTHR>
void launch_y_cfg(fsei_plan* p, YArgs<T> a, bool inverse) {
    a.nseq = std::max(1, std::min(tile_nseq(EMAX, p->ny), (p->nx + 1) / 2));
    // whole 128-byte row segments per tile where the tile holds at least one
    // (16 doubles / 32 floats = 8 / 16 column pairs)
    constexpr int kSeqLine = 64 / (int)sizeof(T);
    if (a.nseq > kSeqLine) a.nseq -= a.nseq % kSeqLine;
    const int tx = 2 * a.nseq;
    a.ntile = (p->nx + tx - 1) / tx;
    const dim3 grid((unsigned)(a.ntile * p->nz));
    const size_t dyn = 2 * p->ny * sizeof(T);
    if (inverse)
        hipLaunchKernelGGL((k_yinv<T, EMAX, NTHR>), grid, dim3(NTHR), dyn, S(p), a);
    else
        hipLaunchKernelGGL((k_yfwd<T, EMAX, NTHR>), grid, dim3(NTHR), dyn, S(p), a);
}

template <typename T>
void launch_y(fsei_plan* p, T* data, bool inverse) {
    YArgs<T> a{};
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.bcy = p->bcy;
    a.fp = p->fy;
    a.data = data;
    a.twc = tab<T>(p, T_TWY_C);
    a.tws = tab<T>(p, T_TWY_S);
    a.dctc = tab<T>(p, T_DCTY_C);
    a.dcts = tab<T>(p, T_DCTY_S);
    Timed t(p, inverse ? K_YINV : K_YFWD);
    if (const LenOps* o = len_ops(p->ny)) {
        const bool vec = p->nx % 2 == 0 && reinterpret_cast<uintptr_t>(data) % (2 * sizeof(T)) == 0;
        const int tx = 2 * (sizeof(T) == 8 ? o->y_pairs_d : o->y_pairs_f);
        a.ntile = (p->nx + tx - 1) / tx;
        o->y<T>(inverse, vec)(a, (unsigned)(a.ntile * p->nz), S(p));
        return;
    }
    // lengths below 16 and above 1024: the workgroup's LDS holds enough
    // columns that a row segment covers 128 B (16 doubles / 32 floats) where
    // the tile (2 arrays, padded) plus the 2 ny twiddles fit the 160 KB
    const long want = (long)(64 / sizeof(T)) * p->ny;
    const bool fits = (2L * lds_elems(8192) + 2L * p->ny) * (long)sizeof(T) <= 160L * 1024;
    if (want <= 2048) launch_y_cfg<T, 2048, 256>(p, a, inverse);
    else if (sizeof(T) == 4 || fits) launch_y_cfg<T, 8192, 1024>(p, a, inverse);
    else if constexpr (sizeof(T) == 8) launch_y_cfg<T, 4096, 512>(p, a, inverse);
}

template <typename TS, typename TC>
ZArgs<TS, TC> zargs(const fsei_plan* p, TS* data, int transposed, bool record_mean) {
    ZArgs<TS, TC> a{};
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.transposed = transposed;
    a.data = data;
    a.scale = (TC)(1.0 / ((double)p->nx * (double)p->ny));
    a.za = tab<TC>(p, T_ZA);
    a.zc = tab<TC>(p, T_ZC);
    a.zb0 = tab<TC>(p, T_ZB0);
    a.dz = tab<TC>(p, T_DZ);
    a.inv_dz = tab<TC>(p, T_INV_DZ);
    a.lamx = tab<TC>(p, T_LAMX);
    a.lamy = tab<TC>(p, T_LAMY);
    a.lamx64 = tab<double>(p, T_LAMX);
    a.lamy64 = tab<double>(p, T_LAMY);
    a.sigma_thr = p->sigma_thr;   // the host's threshold, compared in FP64
    a.nlist = p->nlist;
    a.list = zlist(p);
    a.scale64 = 1.0 / ((double)p->nx * (double)p->ny);
    a.lz = p->lz;
    a.za64 = tab<double>(p, T_ZA);
    a.zc64 = tab<double>(p, T_ZC);
    a.dz64 = tab<double>(p, T_DZ);
    a.inv_dz64 = tab<double>(p, T_INV_DZ);
    a.h64 = tab<double>(p, T_H);
    a.scal = (record_mean && !transposed) ? scalars(p) : nullptr;
    return a;
}

// z solve of every mode line of `data` (in place), zero mode included
template <typename T>
void launch_z(fsei_plan* p, T* data, int transposed, bool record_mean) {
    ZArgs<T, T> a = zargs<T, T>(p, data, transposed, record_mean);
    const int cus = cus_of_current_device();
    if (z_tiling<T>(&a, cus)) {
        Timed t(p, K_ZLIST);
        z_launch_special<T>(a, S(p));
    }
    Timed t(p, K_ZSOLVE);
    z_launch<T>(a, S(p), cus);
}

// k_grad_row2 with the smallest workgroup that gives every cell pair of a
// row a lane (np = nx / 2 <= 512 pairs)
template <typename TIO, typename TP, int GJ>
void launch_grad_row2(fsei_plan* p, const GradArgs<TIO, TP>& a, dim3 grid, int np) {
    if (np > 384)
        hipLaunchKernelGGL((k_grad_row2<TIO, TP, 512, GJ>), grid, dim3(512), 0, S(p), a);
    else if (np > 256)
        hipLaunchKernelGGL((k_grad_row2<TIO, TP, 384, GJ>), grid, dim3(384), 0, S(p), a);
    else if (np > 128)
        hipLaunchKernelGGL((k_grad_row2<TIO, TP, 256, GJ>), grid, dim3(256), 0, S(p), a);
    else if (np > 64)
        hipLaunchKernelGGL((k_grad_row2<TIO, TP, 128, GJ>), grid, dim3(128), 0, S(p), a);
    else
        hipLaunchKernelGGL((k_grad_row2<TIO, TP, 64, GJ>), grid, dim3(64), 0, S(p), a);
}

template <typename TIO, typename TP>
void launch_grad(fsei_plan* p, const Vel<TIO>& q, const TP* pr, bool adjoint, double dt) {
    GradArgs<TIO, TP> a{};
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.bcx = p->bcx;
    a.bcy = p->bcy;
    set_vel(&a, q);
    a.p = pr;
    set_grad(p, &a, adjoint, dt);
    Timed t(p, K_GRAD);
    const bool al = q.aligned() && aligned16(pr);
    const int np = p->nx / 2;
    if (p->nx % 2 == 0 && np <= 512 && p->ny % 8 == 0 && al) {
        // one row per workgroup, one cell pair per lane; rows in 16-row
        // tiles when ny allows (fewer re-read halo rows), else 8
        const dim3 grid((unsigned)((long)p->ny * p->nz));
        if (p->ny % 16 == 0)
            launch_grad_row2<TIO, TP, 16>(p, a, grid, np);
        else
            launch_grad_row2<TIO, TP, 8>(p, a, grid, np);
        return;
    }
    // a row of up to 256 columns has one per thread: registers for four cost it
    // waves (us, FP64: 27 x 1296 x 315 224 with two, 289 with four; 81 x 432 x 514
    // 216 and 271); longer rows keep more loads in flight with four (384 x 324 x
    // 300 386 against 397)
    const dim3 grid((unsigned)((long)p->ny * p->nz));
    if (p->nx <= 256)
        hipLaunchKernelGGL((k_grad<TIO, TP, 2>), grid, dim3(256), 0, S(p), a);
    else
        hipLaunchKernelGGL((k_grad<TIO, TP, 4>), grid, dim3(256), 0, S(p), a);
}

// FP64 residual norm pass of the refinement (partials of sum r^2, sum r,
// sum dz_k p); returns the number of partials written
template <typename TPP>
long launch_resid_pairs(fsei_plan* p, const double* f, const TPP* pr) {
    ResArgs<TPP> a{};
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.bcx = p->bcx;
    a.bcy = p->bcy;
    a.f = f;
    a.p = pr;
    a.idx2 = 1.0 / (p->dx * p->dx);
    a.idy2 = 1.0 / (p->dy * p->dy);
    a.za = tab<double>(p, T_ZA);
    a.zc = tab<double>(p, T_ZC);
    a.scal = scalars(p);
    a.dz = tab<double>(p, T_DZ);
    a.partials = partials(p);
    const long nb = (long)(p->ny / kPairRows) * p->nz;
    const dim3 grid((unsigned)nb);
    const int np = p->nx / 2;
    Timed t(p, K_RESNORM);
    if (np == 384)
        hipLaunchKernelGGL((k_resid_pairs<384, kPairRows, TPP>), grid, dim3(384), 0, S(p), a);
    else if (np >= 256)
        hipLaunchKernelGGL((k_resid_pairs<256, kPairRows, TPP>), grid, dim3(256), 0, S(p), a);
    else if (np > 64)
        hipLaunchKernelGGL((k_resid_pairs<128, kPairRows, TPP>), grid, dim3(128), 0, S(p), a);
    else
        hipLaunchKernelGGL((k_resid_pairs<64, kPairRows, TPP>), grid, dim3(64), 0, S(p), a);
    return nb;
}

// Gradient correction of (u, v, w) fused with the residual norm partials of
// the iterate p64 (DELTA: the gradient of the correction c32 instead of p64);
// returns the number of partials written
template <bool DELTA>
long launch_grad_resid(fsei_plan* p, const Vel<double>& q, const double* f, const double* p64, const float* c32,
                       double dt) {
    GradResArgs a{};
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.bcx = p->bcx;
    a.bcy = p->bcy;
    set_vel(&a, q);
    a.p = p64;
    a.c = c32;
    a.cx = -dt / p->dx;
    a.cy = -dt / p->dy;
    a.sw = -dt;
    a.bk = tab<double>(p, T_INV_H);
    a.gk = tab<double>(p, T_INV_H);
    a.f = f;
    a.idx2 = 1.0 / (p->dx * p->dx);
    a.idy2 = 1.0 / (p->dy * p->dy);
    a.za = tab<double>(p, T_ZA);
    a.zc = tab<double>(p, T_ZC);
    a.scal = scalars(p);
    a.partials = partials(p);
    // 16-row tiles halve the re-read halo rows (j-1 of the first row, j+1 of
    // the last) against 8-row tiles when ny allows
    const int rows = (p->ny % 16 == 0) ? 16 : kPairRows;
    const long nb = (long)(p->ny / rows) * p->nz;
    const dim3 grid((unsigned)nb);
    const int np = p->nx / 2;
    Timed t(p, K_GRAD_RESID);
    if (rows == 16) {
        if (np == 384)
            hipLaunchKernelGGL((k_grad_resid<384, 16, DELTA>), grid, dim3(384), 0, S(p), a);
        else if (np >= 256)
            hipLaunchKernelGGL((k_grad_resid<256, 16, DELTA>), grid, dim3(256), 0, S(p), a);
        else if (np > 64)
            hipLaunchKernelGGL((k_grad_resid<128, 16, DELTA>), grid, dim3(128), 0, S(p), a);
        else
            hipLaunchKernelGGL((k_grad_resid<64, 16, DELTA>), grid, dim3(64), 0, S(p), a);
        return nb;
    }
    if (np == 384)
        hipLaunchKernelGGL((k_grad_resid<384, kPairRows, DELTA>), grid, dim3(384), 0, S(p), a);
    else if (np >= 256)
        hipLaunchKernelGGL((k_grad_resid<256, kPairRows, DELTA>), grid, dim3(256), 0, S(p), a);
    else if (np > 64)
        hipLaunchKernelGGL((k_grad_resid<128, kPairRows, DELTA>), grid, dim3(128), 0, S(p), a);
    else
        hipLaunchKernelGGL((k_grad_resid<64, kPairRows, DELTA>), grid, dim3(64), 0, S(p), a);
    return nb;
}

template <typename TI, typename TO>
XFwdArgs<TI, TO> div_args(const fsei_plan* p, const TI* u, const TI* v, const TI* w, const TI* gp, bool adjoint,
                          double dt) {
    XFwdArgs<TI, TO> a{};
    a.u = u;
    a.v = v;
    a.w = w;
    a.gp = gp;
    a.idx = (TI)(1.0 / p->dx);
    a.idy = (TI)(1.0 / p->dy);
    if (!adjoint) {
        a.alpha = (TI)(1.0 / dt);
        a.beta = (TI)0;
        a.zeta = tab<TI>(p, T_INV_DZ);
        a.eta = tab<TI>(p, T_INV_DZ);
    } else {
        a.alpha = (TI)-1;
        a.beta = (TI)(-1.0 / dt);
        a.zeta = tab<TI>(p, T_ZETA_ADJ);
        a.eta = tab<TI>(p, T_INV_H);
    }
    return a;
}

fsei_status check_hip() {
    return (hipGetLastError() == hipSuccess) ? FSEI_OK : FSEI_ERR_HIP;
}

// ---------------------------------------------------------------------------
// implicit viscous step: line solves along x (LDS-staged), y and z (strided)
// ---------------------------------------------------------------------------
template <int L>
void launch_visc_x_L(fsei_plan* p, ViscArgs a) {
    a.tiles = visc_x_tiles(a.nlines, a.n, L, cus_of_current_device());
    const long per = (long)kViscXLines * a.tiles;
    const unsigned nb = (unsigned)((a.nlines + per - 1) / per);
    const int dyn = kViscXLines * (a.n + 2) * (int)sizeof(double);
    static bool attr = false;   // allow the tile beyond the default dynamic LDS limit
    if (!attr) {
        (void)hipFuncSetAttribute((const void*)k_visc_x<L>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  kViscXLines * (kViscMaxN + 2) * (int)sizeof(double));
        attr = true;
    }
    hipLaunchKernelGGL((k_visc_x<L>), dim3(nb), dim3(kViscXLines * kViscPmax), dyn, S(p), a);
}

void launch_visc_x(fsei_plan* p, const ViscArgs& a, int L) {
    switch (L) {
        case 4: launch_visc_x_L<4>(p, a); break;
        case 8: launch_visc_x_L<8>(p, a); break;
        case 12: launch_visc_x_L<12>(p, a); break;
        case 16: launch_visc_x_L<16>(p, a); break;
        case 24: launch_visc_x_L<24>(p, a); break;
        default: launch_visc_x_L<32>(p, a); break;
    }
}

template <int M>
void launch_visc_s_M(fsei_plan* p, const ViscArgs& a, int L, unsigned groups) {
    const dim3 g((unsigned)((a.ncol + 16 * M - 1) / (16 * M)), groups);
    const dim3 b(16 * kViscPmax);
    switch (L) {
        case 4: hipLaunchKernelGGL((k_visc_strided<M, 4>), g, b, 0, S(p), a); break;
        case 8: hipLaunchKernelGGL((k_visc_strided<M, 8>), g, b, 0, S(p), a); break;
        case 12: hipLaunchKernelGGL((k_visc_strided<M, 12>), g, b, 0, S(p), a); break;
        case 16: hipLaunchKernelGGL((k_visc_strided<M, 16>), g, b, 0, S(p), a); break;
        case 24: hipLaunchKernelGGL((k_visc_strided<M, 24>), g, b, 0, S(p), a); break;
        default: hipLaunchKernelGGL((k_visc_strided<M, 32>), g, b, 0, S(p), a); break;
    }
}

void launch_visc_strided(fsei_plan* p, const ViscArgs& a, int L, unsigned groups) {
    const bool al = aligned16(a.data) && (a.add == nullptr || aligned16(a.add));
    if (L == 24 && a.n == kViscPmax * 24 && a.ncol % 32 == 0 && al) {
        // whole tiles of 768-row lines: the persistent kernel, the next tile's
        // first 12 rows of each chunk staged in LDS, one workgroup per CU (z
        // pass at 512x512x768: 0.69 -> 0.63 ms per component)
        const int ngx = a.ncol / 32;
        const long ntiles = (long)ngx * groups;
        const int cus = cus_of_current_device();
        const unsigned g = (unsigned)(ntiles < cus ? ntiles : cus);
        hipLaunchKernelGGL((k_visc_strided_pf<24, 12>), dim3(g), dim3(16 * kViscPmax), 0, S(p), a, ngx, (int)ntiles);
        return;
    }
    // two adjacent columns per lane (16-byte accesses) when the rows allow
    if (a.ncol % 2 == 0 && al)
        launch_visc_s_M<2>(p, a, L, groups);
    else
        launch_visc_s_M<1>(p, a, L, groups);
}

fsei_status ready(const fsei_plan* p) {
    if (!p) return FSEI_ERR_ARG;
    if (!p->ws || p->ws_bytes < p->ws_total) return FSEI_ERR_WORKSPACE;
    return FSEI_OK;
}

bool good_dt(double dt) { return std::isfinite(dt) && dt > 0.0; }

// Whether some output of an out-of-place call shares memory with an input other
// than its own, with another output or with p (its own input: the same array, or
// none of its memory).  A kernel would read there what another tile has written.
// dLoss/dp of the adjoint may lie anywhere: it is read before the first output.
template <typename T>
bool overlaps(const fsei_plan* p, const Vel<T>& q, const T* pout) {
    const size_t bytes = p->ncells() * sizeof(T);
    auto meet = [&](const void* a, const void* b) {
        const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
        return a != nullptr && b != nullptr && (x < y ? y - x : x - y) < bytes;
    };
    const T* in[3] = {q.ui, q.vi, q.wi};
    const T* out[3] = {q.u, q.v, q.w};
    for (int i = 0; i < 3; ++i) {
        if (meet(pout, in[i]) || meet(pout, out[i])) return true;
        for (int j = 0; j < 3; ++j) {
            if (j != i && (meet(out[i], in[j]) || meet(out[i], out[j]))) return true;
            if (j == i && out[i] != in[i] && meet(out[i], in[i])) return true;
        }
    }
    return false;
}

// the argument checks every projection entry point shares
template <typename T>
fsei_status check_vel(const fsei_plan* p, const Vel<T>& q, double dt) {
    fsei_status st = ready(p);
    if (st != FSEI_OK) return st;
    if (!q.ui || !q.vi || !q.wi || !q.u || !q.v || !q.w) return FSEI_ERR_ARG;
    if (!good_dt(dt)) return FSEI_ERR_ARG;
    constexpr bool f32 = std::is_same<T, float>::value;
    if ((p->precision == FSEI_PREC_FP32) != f32) return FSEI_ERR_PRECISION;
    return FSEI_OK;
}

fsei_status read_scalars(fsei_plan* p, double* host, int n) {
    if (hipMemcpyAsync(host, scalars(p), n * sizeof(double), hipMemcpyDeviceToHost, S(p)) != hipSuccess)
        return FSEI_ERR_HIP;
    if (hipStreamSynchronize(S(p)) != hipSuccess) return FSEI_ERR_HIP;
    return FSEI_OK;
}

// sums of the last xfwd pass with partials (sum v^2, sum v, sum dz_k v) into
// scalars[off..off+2]; with `vmean`, also scalars[0] = the V-mean of v,
// sum dz_k v / (nx ny lz)
void reduce_partials(fsei_plan* p, int off, long nblk, bool vmean = false) {
    Timed t(p, K_NORM);
    const double scale = 1.0 / ((double)p->nx * (double)p->ny * p->lz);
    double* out = scalars(p) + off;
    double* mean = vmean ? scalars(p) : nullptr;
    if (nblk <= 4 * kSumGroups) {
        hipLaunchKernelGGL(k_sum_partials<1024>, dim3(1), dim3(1024), 0, S(p), (const double*)partials(p), (int)nblk,
                           out, mean, scale);
        return;
    }
    // two stages: kSumGroups workgroups over contiguous chunks, then one
    // small workgroup over their triples (the group sums follow the
    // partials in the workspace)
    const int chunk = (int)((nblk + kSumGroups - 1) / kSumGroups);
    double* grp = partials(p) + 3 * p->n_partials;
    hipLaunchKernelGGL(k_sum_partials_grp, dim3(kSumGroups), dim3(256), 0, S(p), (const double*)partials(p),
                       (int)nblk, chunk, grp);
    hipLaunchKernelGGL(k_sum_partials<64>, dim3(1), dim3(64), 0, S(p), (const double*)grp, kSumGroups, out, mean,
                       scale);
}

// ---------------------------------------------------------------------------
// FP32 + FP64 iterative refinement.  f (FP64) is the right-hand side; on
// return p64 holds the pressure.
//   p0 = solve32(f); repeat: r = (f - mean) - L p (FP64 stencil), stop when
//   ||r|| <= rtol ||f - mean||, else p += solve32(r).
// ---------------------------------------------------------------------------
// Projection target of a refined solve: with the pair tiling and rtol > 0 the
// gradient correction is fused with the convergence check of each
// correction (the first applies the gradient of p, later ones the gradient of
// their own correction); `applied` tells the caller whether it still has to
// apply the gradient of the final p.
struct RefineGrad {
    Vel<double> q;
    double dt;
    bool applied;
};

template <int PRO>
fsei_status refine_solve(fsei_plan* p, XFwdArgs<double, float> first, double* p64, fsei_info* info,
                         RefineGrad* g = nullptr) {
    float* w32 = static_cast<float*>(field2(p));
    double* f64 = static_cast<double*>(field1(p));
    first.out = w32;
    first.out_f = f64;
    first.partials = partials(p);
    first.dzw = tab<double>(p, T_DZ);
    const long nfirst = launch_xfwd<double, float, PRO>(p, first, K_XFWD);
    // scalars[5..7] = sum f^2, sum f, sum dz_k f; scalars[0] = V-mean of f in
    // FP64 (the FP32 zero-mode solve removes its own FP32 mean to stay
    // compatible, but the residual must use the exact one: a constant left in
    // the residual is in the null space of L and no correction removes it)
    reduce_partials(p, 5, nfirst, true);
    launch_y<float>(p, w32, false);
    launch_z<float>(p, w32, 0, false);
    launch_y<float>(p, w32, true);
    // With the pair tiling the first solve's pressure stays in FP32 (its
    // error is FP32-level anyway; the residual is evaluated exactly in FP64
    // from those values and the first correction writes p = p32 + delta in
    // FP64), saving 4 bytes per cell in each of three passes.  Otherwise it is
    // written to p64 directly.
    float* p32 = static_cast<float*>(field4(p));
    const bool pairs = pair_tiles(p) && aligned16(f64) && aligned16(p64) && aligned16(w32) && aligned16(p32);
    if (pairs)
        launch_xinv<float, float, EPI_STORE>(p, w32, p32, K_XINV);
    else
        launch_xinv<float, double, EPI_STORE>(p, w32, p64, K_XINV);
    bool p_in_32 = pairs;   // the current iterate is p32 (before the first correction)
    const double N = (double)p->ncells();
    auto rel_from = [&](const double* h) {
        // ||f - mean||^2 = sum f^2 - 2 mean sum f + N mean^2; h[1] = sum r^2
        const double mean = h[0];
        double fn2 = h[5] - 2.0 * mean * h[6] + N * mean * mean;
        if (fn2 <= 0.0) fn2 = h[5];
        return (fn2 > 0.0) ? std::sqrt(h[1] / fn2) : 0.0;
    };
    XFwdArgs<double, float> r{};
    r.f = f64;
    r.p = p64;
    r.idx2 = 1.0 / (p->dx * p->dx);
    r.idy2 = 1.0 / (p->dy * p->dy);
    r.za = tab<double>(p, T_ZA);
    r.zc = tab<double>(p, T_ZC);
    r.scal = scalars(p);
    r.partials = partials(p);
    r.dzw = tab<double>(p, T_DZ);   // third partial: sum dz_k p of the iterate
    int it = 0;
    double rel = -1.0, rel_prev = -1.0;
    bool converged = false;
    bool floor = false;      // a correction no longer halved the residual
    bool measured = false;   // rel belongs to the current iterate
    long nres = 0;    // partials of the last residual pass
    // The first solve's residual norm is reduced into scalars[8..10] but not
    // read back on its own: it is fetched with the first corrected iterate's
    // norm, so the common one-correction case waits on the host once.  (A
    // first solve that already meets rtol then still gets one correction.)
    bool first_pending = false;
    double vmean = 0.0;
    auto residual_norm = [&]() -> fsei_status {
        reduce_partials(p, 1, nres);   // scalars[1..3]: sum r^2, sum r, (sum dz_k p or 0)
        double h[11];
        fsei_status st = read_scalars(p, h, first_pending ? 11 : 8);
        if (st != FSEI_OK) return st;
        vmean = h[0];
        if (first_pending) {
            double h0[8];
            std::copy(h, h + 8, h0);
            h0[1] = h[8];
            rel = rel_from(h0);
            first_pending = false;
        }
        rel_prev = rel;
        rel = rel_from(h);
        measured = true;
        converged = p->rtol > 0.0 && rel <= p->rtol;
        // the FP64 residual cannot fall below the rounding floor of the
        // stencil applied to this p: stop once a correction gains < 2x
        floor = !converged && rel_prev >= 0.0 && rel > 0.5 * rel_prev;
        return FSEI_OK;
    };
    // Residual passes.  A pass that feeds a correction is the x-forward
    // kernel with the FP64 residual stencil as its prologue (reading the FP32
    // first solve, or the FP64 iterate), writing the FP32 transform of r and
    // the partial sums; a norm-only pass is the pair residual kernel (with
    // the pair tiling) or the same x-forward prologue without output.
    auto norm_pass = [&]() {
        if (pairs) {
            nres = p_in_32 ? launch_resid_pairs(p, f64, (const float*)p32)
                           : launch_resid_pairs(p, f64, (const double*)p64);
        } else {
            r.out = nullptr;
            nres = launch_xfwd<double, float, PRO_RESID>(p, r, K_RESNORM);
        }
    };
    auto resid_pass = [&]() {
        if (p_in_32) {
            XFwdArgs<double, float> r32 = r;
            r32.p = nullptr;
            r32.p32 = p32;
            r32.out = w32;
            nres = launch_xfwd<double, float, PRO_RESID_F>(p, r32, K_RESID_XFWD);
        } else {
            r.out = w32;
            nres = launch_xfwd<double, float, PRO_RESID>(p, r, K_RESID_XFWD);
        }
    };
    resid_pass();
    if (p->max_iter > 0) {
        // scalars[8..10]: the first solve's sum r^2, sum r and sum dz_k p.
        // The last is its V-integral: the first correction subtracts the
        // V-mean it gives, so p is pinned in FP64 (later corrections are
        // solves of residuals, whose V-mean is zero).
        reduce_partials(p, 8, nres);
        first_pending = p->rtol > 0.0;
    } else if (p->rtol > 0.0) {
        fsei_status st = residual_norm();
        if (st != FSEI_OK) return st;
    }
    const double* vsum0 = scalars(p) + 10;
    const bool fuse = g != nullptr && pairs && p->rtol > 0.0 && g->q.aligned();
    while (!converged && it < p->max_iter) {
        launch_y<float>(p, w32, false);
        launch_z<float>(p, w32, 0, false);
        launch_y<float>(p, w32, true);
        const double* vsum = (it == 0) ? vsum0 : nullptr;
        bool checked = false;   // the gradient and the residual partials of this iterate are done
        if (p_in_32) {
            // p64 = (p32 - its V-mean) + delta; with a projection, in the pass
            // that also applies the gradient of p64 and takes its residual
            if (fuse && xgr_ok(p, w32, p32, p64, f64, g->q)) {
                nres = launch_xinv_grad_resid(p, w32, p32, vsum, p64, g->q, f64, g->dt);
                g->applied = true;
                checked = true;
            } else {
                launch_xinv<float, double, EPI_ADDF>(p, w32, p64, K_XINV_ACC, p32, nullptr, vsum);
            }
            p_in_32 = false;
        } else if (fuse && g->applied) {
            // p64 += delta, and delta itself kept (in w32) for its gradient
            launch_xinv<float, double, EPI_ACC_KEEP>(p, w32, p64, K_XINV_ACC, nullptr, w32, vsum);
        } else {
            launch_xinv<float, double, EPI_ACC>(p, w32, p64, K_XINV_ACC, nullptr, nullptr, vsum);
        }
        ++it;
        measured = false;
        bool transformed = false;   // the next correction's transformed residual is in w32
        if (p->rtol > 0.0) {
            // convergence check of the corrected iterate: for a projection
            // fused with the gradient correction; for a solve that may take
            // another correction, the residual pass of that correction (its
            // partials are this iterate's norm: r is evaluated once, and the
            // transform is wasted only on the last iteration); else norm only
            if (checked) {
            } else if (fuse) {
                nres = g->applied ? launch_grad_resid<true>(p, g->q.onto(), f64, p64, w32, g->dt)
                                  : launch_grad_resid<false>(p, g->q, f64, p64, nullptr, g->dt);
                g->applied = true;
            } else if (it < p->max_iter) {
                resid_pass();
                transformed = true;
            } else {
                norm_pass();
            }
            fsei_status st = residual_norm();
            if (st != FSEI_OK) return st;
            if (converged || floor) break;
        }
        // residual again, transformed for the next correction
        if (it < p->max_iter && !transformed) resid_pass();
    }
    if (p_in_32) {
        // no correction ran (max_iter = 0, or the first solve already met
        // rtol): the iterate is the FP32 first solve
        const size_t n = p->ncells();
        Timed t(p, K_XINV_ACC);
        hipLaunchKernelGGL(k_widen, dim3((unsigned)std::min<size_t>((n + 255) / 256, 65536)), dim3(256), 0, S(p),
                           (const float*)p32, p64, n);
        p_in_32 = false;
    }
    if (info != nullptr && !measured) {
        norm_pass();
        fsei_status st = residual_norm();
        if (st != FSEI_OK) return st;
    }
    if (info) {
        if (!measured) {
            double h[1];
            fsei_status st = read_scalars(p, h, 1);
            if (st != FSEI_OK) return st;
            vmean = h[0];
        }
        info->iterations = it;
        info->rel_residual = rel;
        info->rhs_vmean_removed = vmean;
        info->floor_reached = floor ? 1 : 0;
    }
    fsei_status st = check_hip();
    if (st != FSEI_OK) return st;
    if (p->rtol > 0.0 && !converged) return FSEI_ERR_NOT_CONVERGED;
    return FSEI_OK;
}

}  // namespace

extern "C" {

void fsei_poisson_plan_destroy(fsei_plan* p) {
    if (!p) return;
    if (!p->ev_pool.empty()) {
        TimingState* ts = static_cast<TimingState*>(p->ev_pool[0]);
        for (auto& pe : ts->pending) {
            (void)hipEventDestroy(pe.a);
            (void)hipEventDestroy(pe.b);
        }
        for (auto e : ts->free_ev) (void)hipEventDestroy(e);
        delete ts;
    }
    delete p;
}

fsei_status fsei_plan_set_workspace(fsei_plan* p, void* dev, size_t bytes) {
    if (!p || !dev) return FSEI_ERR_ARG;
    if (((uintptr_t)dev % kAlign) != 0 || bytes < p->ws_total) return FSEI_ERR_WORKSPACE;
    if (hipMemcpy((char*)dev + p->ws_tab_d, p->tab_d.data(), p->tab_d.size() * sizeof(double),
                  hipMemcpyHostToDevice) != hipSuccess)
        return FSEI_ERR_HIP;
    if (hipMemcpy((char*)dev + p->ws_tab_f, p->tab_f.data(), p->tab_f.size() * sizeof(float),
                  hipMemcpyHostToDevice) != hipSuccess)
        return FSEI_ERR_HIP;
    if (!p->list_host.empty()) {
        if (hipMemcpy((char*)dev + p->ws_list, p->list_host.data(), p->list_host.size() * sizeof(int),
                      hipMemcpyHostToDevice) != hipSuccess)
            return FSEI_ERR_HIP;
    }
    if (hipMemset((char*)dev + p->ws_scalars, 0, fsei_plan_impl::kScalars * sizeof(double)) != hipSuccess)
        return FSEI_ERR_HIP;
    p->ws = dev;
    p->ws_bytes = bytes;
    for (double& b : p->visc_beta) b = 0.0;   // viscous tables live in the workspace: rebuild on next use
    return FSEI_OK;
}

fsei_status fsei_plan_set_stream(fsei_plan* p, void* stream) {
    if (!p) return FSEI_ERR_ARG;
    p->stream = stream;
    return FSEI_OK;
}

fsei_status fsei_poisson_solve(fsei_plan* p, const double* f, double* out, fsei_info* info) {
    fsei_status st = ready(p);
    if (st != FSEI_OK) return st;
    if (!f || !out) return FSEI_ERR_ARG;
    if (p->precision == FSEI_PREC_FP32) return FSEI_ERR_PRECISION;
    if (p->precision == FSEI_PREC_FP32_REFINE) {
        XFwdArgs<double, float> a{};
        a.f = f;
        return refine_solve<PRO_COPY>(p, a, out, info);
    }
    XFwdArgs<double, double> a{};
    a.f = f;
    a.out = out;
    launch_xfwd<double, double, PRO_COPY>(p, a, K_XFWD);
    launch_y<double>(p, out, false);
    launch_z<double>(p, out, 0, true);
    launch_y<double>(p, out, true);
    launch_xinv<double, double, EPI_STORE>(p, out, out, K_XINV);
    st = check_hip();
    if (st != FSEI_OK) return st;
    if (info) {
        double h[1];
        st = read_scalars(p, h, 1);
        if (st != FSEI_OK) return st;
        info->iterations = 0;
        info->rel_residual = -1.0;
        info->rhs_vmean_removed = h[0];
        info->floor_reached = 0;
    }
    return FSEI_OK;
}

}  // extern "C"

namespace {

// the projection on the plan's current workspace (arguments checked by the caller)
fsei_status project_impl(fsei_plan* p, const Vel<double>& q, double* pout, double dt, fsei_info* info) {
    fsei_status st = FSEI_OK;
    if (p->precision == FSEI_PREC_FP32_REFINE) {
        double* p64 = pout ? pout : static_cast<double*>(field3(p));
        XFwdArgs<double, float> a = div_args<double, float>(p, q.ui, q.vi, q.wi, nullptr, false, dt);
        RefineGrad g{q, dt, false};
        st = refine_solve<PRO_DIV>(p, a, p64, info, &g);
        if (st != FSEI_OK && st != FSEI_ERR_NOT_CONVERGED) return st;
        if (!g.applied) launch_grad<double, double>(p, q, p64, false, dt);
        fsei_status st2 = check_hip();
        return (st2 != FSEI_OK) ? st2 : st;
    }
    // the transform chain runs in the workspace field when the x inverse is
    // fused with the gradient (its halo rows must not be overwritten by a
    // neighbouring tile's p), else in the caller's p when given
    double* ws1 = static_cast<double*>(field1(p));
    const LenOps* xg = xg_ops(p, ws1, pout, q);
    double* buf = (pout && !xg) ? pout : ws1;
    XFwdArgs<double, double> a = div_args<double, double>(p, q.ui, q.vi, q.wi, nullptr, false, dt);
    a.out = buf;
    launch_xfwd<double, double, PRO_DIV>(p, a, K_XFWD);
    launch_y<double>(p, buf, false);
    launch_z<double>(p, buf, 0, true);
    launch_y<double>(p, buf, true);
    if (xg) {
        launch_xinv_grad(p, xg, buf, pout, q, false, dt);
    } else {
        launch_xinv<double, double, EPI_STORE>(p, buf, buf, K_XINV);
        launch_grad<double, double>(p, q, buf, false, dt);
    }
    st = check_hip();
    if (st != FSEI_OK) return st;
    if (info) {
        double h[1];
        st = read_scalars(p, h, 1);
        if (st != FSEI_OK) return st;
        info->iterations = 0;
        info->rel_residual = -1.0;
        info->rhs_vmean_removed = h[0];
        info->floor_reached = 0;
    }
    return FSEI_OK;
}

// ---------------------------------------------------------------------------
// Device-resident scratch of the allocation-free projection: one copy per
// GPU, held until the process ends.  Host code never uses the array's name
// as an address: the device address comes from hipGetSymbolAddress, once per
// device, and is kept in scratch_ptr.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)128 << 20;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_ptr[kMaxDevices] = {};

__global__ __launch_bounds__(256) void k_zero(double* __restrict__ q, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) q[i] = 0.0;
}

fsei_status scratch_of_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return FSEI_ERR_HIP;
    if (dev >= kMaxDevices) return FSEI_ERR_HIP;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (scratch_ptr[dev] == nullptr) {
        void* q = nullptr;
        if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || q == nullptr) return FSEI_ERR_HIP;
        scratch_ptr[dev] = q;
    }
    *out = scratch_ptr[dev];
    return FSEI_OK;
}

}  // namespace

extern "C" {

fsei_status fsei_project(fsei_plan* p, double* u, double* v, double* w, double* pout, double dt, fsei_info* info) {
    const Vel<double> q = in_place(u, v, w);
    fsei_status st = check_vel(p, q, dt);
    return st == FSEI_OK ? project_impl(p, q, pout, dt, info) : st;
}

fsei_status fsei_project_to(fsei_plan* p, const double* u, const double* v, const double* w, double* ou, double* ov,
                            double* ow, double* pout, double dt, fsei_info* info) {
    const Vel<double> q{u, v, w, ou, ov, ow};
    if (p && overlaps(p, q, (const double*)pout)) return FSEI_ERR_ARG;
    fsei_status st = check_vel(p, q, dt);
    return st == FSEI_OK ? project_impl(p, q, pout, dt, info) : st;
}

size_t fsei_project_noalloc_max_bytes(void) { return kScratchBytes; }

fsei_status fsei_project_noalloc(fsei_plan* p, double* u, double* v, double* w, double* pout, double dt,
                                 fsei_info* info) {
    if (!p || !u || !v || !w) return FSEI_ERR_ARG;
    if (!good_dt(dt)) return FSEI_ERR_ARG;
    if (p->precision == FSEI_PREC_FP32) return FSEI_ERR_PRECISION;
    if (p->ws_total > kScratchBytes) return FSEI_ERR_SCRATCH;
    void* sp = nullptr;
    fsei_status st = scratch_of_current_device(&sp);
    if (st != FSEI_OK) return st;
    // this plan's tables (and FP64 line list) into the shared scratch, the
    // scalars cleared by a kernel; everything on the plan's stream, so the
    // copies are ordered before the kernels that read them
    hipStream_t s = S(p);
    if (hipMemcpyAsync((char*)sp + p->ws_tab_d, p->tab_d.data(), p->tab_d.size() * sizeof(double),
                       hipMemcpyHostToDevice, s) != hipSuccess)
        return FSEI_ERR_HIP;
    if (hipMemcpyAsync((char*)sp + p->ws_tab_f, p->tab_f.data(), p->tab_f.size() * sizeof(float),
                       hipMemcpyHostToDevice, s) != hipSuccess)
        return FSEI_ERR_HIP;
    if (!p->list_host.empty() &&
        hipMemcpyAsync((char*)sp + p->ws_list, p->list_host.data(), p->list_host.size() * sizeof(int),
                       hipMemcpyHostToDevice, s) != hipSuccess)
        return FSEI_ERR_HIP;
    constexpr int nsc = fsei_plan_impl::kScalars;
    hipLaunchKernelGGL(k_zero, dim3((nsc + 255) / 256), dim3(256), 0, s,
                       reinterpret_cast<double*>((char*)sp + p->ws_scalars), nsc);
    void* ws0 = p->ws;
    const size_t bytes0 = p->ws_bytes;
    p->ws = sp;
    p->ws_bytes = kScratchBytes;
    st = check_hip();
    if (st == FSEI_OK) st = project_impl(p, in_place(u, v, w), pout, dt, info);
    p->ws = ws0;
    p->ws_bytes = bytes0;
    return st;
}

}  // extern "C"

namespace {

fsei_status backward_impl(fsei_plan* p, const Vel<double>& q, const double* gp, double dt) {
    double* buf = static_cast<double*>(field1(p));
    XFwdArgs<double, double> a = div_args<double, double>(p, q.ui, q.vi, q.wi, gp, true, dt);
    a.out = buf;
    launch_xfwd<double, double, PRO_DIV_ADJ>(p, a, K_XFWD);
    launch_y<double>(p, buf, false);
    launch_z<double>(p, buf, 1, false);
    launch_y<double>(p, buf, true);
    if (const LenOps* xg = xg_ops(p, buf, nullptr, q)) {
        launch_xinv_grad(p, xg, buf, nullptr, q, true, dt);
    } else {
        launch_xinv<double, double, EPI_STORE>(p, buf, buf, K_XINV);
        launch_grad<double, double>(p, q, buf, true, dt);
    }
    return check_hip();
}

fsei_status project_f32_impl(fsei_plan* p, const Vel<float>& q, float* pout, float dt) {
    float* buf = pout ? pout : static_cast<float*>(field1(p));
    XFwdArgs<float, float> a = div_args<float, float>(p, q.ui, q.vi, q.wi, nullptr, false, dt);
    a.out = buf;
    launch_xfwd<float, float, PRO_DIV>(p, a, K_XFWD);
    launch_y<float>(p, buf, false);
    launch_z<float>(p, buf, 0, true);
    launch_y<float>(p, buf, true);
    launch_xinv<float, float, EPI_STORE>(p, buf, buf, K_XINV);
    launch_grad<float, float>(p, q, buf, false, dt);
    return check_hip();
}

fsei_status backward_f32_impl(fsei_plan* p, const Vel<float>& q, const float* gp, float dt) {
    float* buf = static_cast<float*>(field1(p));
    XFwdArgs<float, float> a = div_args<float, float>(p, q.ui, q.vi, q.wi, gp, true, dt);
    a.out = buf;
    launch_xfwd<float, float, PRO_DIV_ADJ>(p, a, K_XFWD);
    launch_y<float>(p, buf, false);
    launch_z<float>(p, buf, 1, false);
    launch_y<float>(p, buf, true);
    launch_xinv<float, float, EPI_STORE>(p, buf, buf, K_XINV);
    launch_grad<float, float>(p, q, buf, true, dt);
    return check_hip();
}

}  // namespace

extern "C" {

fsei_status fsei_project_backward(fsei_plan* p, double* gu, double* gv, double* gw, const double* gp, double dt) {
    const Vel<double> q = in_place(gu, gv, gw);
    fsei_status st = check_vel(p, q, dt);
    return st == FSEI_OK ? backward_impl(p, q, gp, dt) : st;
}

fsei_status fsei_project_backward_to(fsei_plan* p, const double* gu, const double* gv, const double* gw,
                                     const double* gp, double* ou, double* ov, double* ow, double dt) {
    const Vel<double> q{gu, gv, gw, ou, ov, ow};
    if (p && overlaps(p, q, (const double*)nullptr)) return FSEI_ERR_ARG;
    fsei_status st = check_vel(p, q, dt);
    return st == FSEI_OK ? backward_impl(p, q, gp, dt) : st;
}

fsei_status fsei_project_f32(fsei_plan* p, float* u, float* v, float* w, float* pout, float dt) {
    const Vel<float> q = in_place(u, v, w);
    fsei_status st = check_vel(p, q, dt);
    return st == FSEI_OK ? project_f32_impl(p, q, pout, dt) : st;
}

fsei_status fsei_project_to_f32(fsei_plan* p, const float* u, const float* v, const float* w, float* ou, float* ov,
                                float* ow, float* pout, float dt) {
    const Vel<float> q{u, v, w, ou, ov, ow};
    if (p && overlaps(p, q, (const float*)pout)) return FSEI_ERR_ARG;
    fsei_status st = check_vel(p, q, dt);
    return st == FSEI_OK ? project_f32_impl(p, q, pout, dt) : st;
}

fsei_status fsei_project_backward_f32(fsei_plan* p, float* gu, float* gv, float* gw, const float* gp, float dt) {
    const Vel<float> q = in_place(gu, gv, gw);
    fsei_status st = check_vel(p, q, dt);
    return st == FSEI_OK ? backward_f32_impl(p, q, gp, dt) : st;
}

fsei_status fsei_project_backward_to_f32(fsei_plan* p, const float* gu, const float* gv, const float* gw,
                                         const float* gp, float* ou, float* ov, float* ow, float dt) {
    const Vel<float> q{gu, gv, gw, ou, ov, ow};
    if (p && overlaps(p, q, (const float*)nullptr)) return FSEI_ERR_ARG;
    fsei_status st = check_vel(p, q, dt);
    return st == FSEI_OK ? backward_f32_impl(p, q, gp, dt) : st;
}

static fsei_status viscous_solve(fsei_plan* p, int comp, double* q, double beta, double* add);

fsei_status fsei_viscous_solve(fsei_plan* p, int comp, double* q, double beta) {
    return viscous_solve(p, comp, q, beta, nullptr);
}

fsei_status fsei_viscous_solve_add(fsei_plan* p, int comp, double* rhs, double* u, double beta) {
    if (p && !u) return FSEI_ERR_ARG;
    if (u && u == rhs) return FSEI_ERR_ARG;
    return viscous_solve(p, comp, rhs, beta, u);
}

static fsei_status viscous_solve(fsei_plan* p, int comp, double* q, double beta, double* add) {
    fsei_status st = ready(p);
    if (st != FSEI_OK) return st;
    if (!q || comp < 0 || comp > 2 || !std::isfinite(beta) || !(beta > 0.0)) return FSEI_ERR_ARG;
    if (p->ws_visc_comp == 0) return FSEI_ERR_SIZE;
    double* tab = reinterpret_cast<double*>((char*)p->ws + p->ws_visc + comp * p->ws_visc_comp);
    if (p->visc_beta[comp] != beta) {
        // new tables for this component: drain the stream first so that no
        // earlier solve still reads the old ones, and keep the host copy
        // alive in the plan until the next rebuild (which drains again)
        if (hipStreamSynchronize(S(p)) != hipSuccess) return FSEI_ERR_HIP;
        std::vector<double>& h = p->visc_host[comp];
        h.assign(p->ws_visc_comp / sizeof(double), 0.0);
        build_visc_tables(p, comp, beta, h.data());
        if (hipMemcpyAsync(tab, h.data(), p->ws_visc_comp, hipMemcpyHostToDevice, S(p)) != hipSuccess)
            return FSEI_ERR_HIP;
        p->visc_beta[comp] = beta;
    }
    ViscArgs a{};
    a.data = q;
    // x: contiguous lines
    a.tab = tab;
    a.n = p->nx;
    a.cyc = p->bcx == FSEI_BC_PERIODIC;
    a.nlines = (long)p->ny * p->nz;
    a.vec = (p->nx % 2 == 0 && aligned16(q)) ? 1 : 0;
    {
        Timed t(p, K_VISC_X);
        launch_visc_x(p, a, p->visc_L[0]);
    }
    // y: lines of stride nx inside each z-plane
    a.tab = tab + visc_tab_elems(p->visc_L[0]);
    a.n = p->ny;
    a.cyc = p->bcy == FSEI_BC_PERIODIC;
    a.ncol = p->nx;
    a.rstride = (size_t)p->nx;
    a.bstride = (size_t)p->nx * p->ny;
    a.remap = 1;
    {
        Timed t(p, K_VISC_Y);
        launch_visc_strided(p, a, p->visc_L[1], (unsigned)p->nz);
    }
    // z: lines of stride nx*ny, one group per y row
    a.tab = tab + visc_tab_elems(p->visc_L[0]) + visc_tab_elems(p->visc_L[1]);
    a.n = p->nz;
    a.cyc = 0;
    a.rstride = (size_t)p->nx * p->ny;
    a.bstride = (size_t)p->nx;
    a.remap = 0;
    a.add = add;   // the last pass adds its result to `add` when given
    {
        Timed t(p, K_VISC_Z);
        launch_visc_strided(p, a, p->visc_L[2], (unsigned)p->ny);
    }
    return check_hip();
}

fsei_status fsei_momentum_rhs(fsei_plan* p, const double* u, const double* v, const double* w, double* nu,
                              double* nv, double* nw, double* ru, double* rv, double* rw, double dt, double re,
                              double gamma, double rho) {
    fsei_status st = ready(p);
    if (st != FSEI_OK) return st;
    if (!u || !v || !w || !nu || !nv || !nw || !ru || !rv || !rw) return FSEI_ERR_ARG;
    if (!good_dt(dt) || !std::isfinite(re) || !(re > 0.0) || !std::isfinite(gamma) || !std::isfinite(rho))
        return FSEI_ERR_ARG;
    MomArgs a{};
    a.nx = p->nx;
    a.ny = p->ny;
    a.nz = p->nz;
    a.perx = p->bcx == FSEI_BC_PERIODIC;
    a.pery = p->bcy == FSEI_BC_PERIODIC;
    a.u = u;
    a.v = v;
    a.w = w;
    a.nu = nu;
    a.nv = nv;
    a.nw = nw;
    a.ru = ru;
    a.rv = rv;
    a.rw = rw;
    a.idx = 1.0 / p->dx;
    a.idy = 1.0 / p->dy;
    a.idx2 = a.idx * a.idx;
    a.idy2 = a.idy * a.idy;
    a.dt = dt;
    a.inv_re = 1.0 / re;
    a.gamma = gamma;
    a.rho = rho;
    a.dz = tab<double>(p, T_DZ);
    a.inv_dz = tab<double>(p, T_INV_DZ);
    a.inv_h = tab<double>(p, T_INV_H);
    a.za = tab<double>(p, T_ZA);
    a.zc = tab<double>(p, T_ZC);
    {
        Timed t(p, K_MOM_RHS);
        const unsigned nb = (unsigned)((long)p->ny * p->nz);
        // cell pairs as 16-byte accesses when the rows allow
        const bool pairs = p->nx % 2 == 0 && aligned16(u) && aligned16(v) && aligned16(w) && aligned16(nu) &&
                           aligned16(nv) && aligned16(nw) && aligned16(ru) && aligned16(rv) && aligned16(rw);
        const bool t16 = p->ny % 16 == 0;
        // one wave per row (measured fastest at 512x512x768: 64 lanes 4.49 ms, 128 4.61, 256 5.15),
        // outputs stored non-temporally (nothing re-reads them in this pass)
        if (pairs && t16)
            hipLaunchKernelGGL((k_momentum_rhs_pairs<64, 16, true>), dim3(nb), dim3(64), 0, S(p), a);
        else if (pairs)
            hipLaunchKernelGGL((k_momentum_rhs_pairs<64, 1, true>), dim3(nb), dim3(64), 0, S(p), a);
        else if (t16)
            hipLaunchKernelGGL((k_momentum_rhs<256, 16>), dim3(nb), dim3(256), 0, S(p), a);
        else
            hipLaunchKernelGGL((k_momentum_rhs<256, 1>), dim3(nb), dim3(256), 0, S(p), a);
    }
    return check_hip();
}

fsei_status ib_setup(fsei_plan* p, int comp, const double* xb, long nb, IbArgs* a) {
    fsei_status st = ready(p);
    if (st != FSEI_OK) return st;
    if (comp < 0 || comp > 2 || nb < 0 || (nb > 0 && !xb)) return FSEI_ERR_ARG;
    if (p->nx < 3 || p->ny < 3 || p->nz < 3) return FSEI_ERR_SIZE;
    *a = IbArgs{};
    a->nx = p->nx;
    a->ny = p->ny;
    a->nz = p->nz;
    a->perx = p->bcx == FSEI_BC_PERIODIC;
    a->pery = p->bcy == FSEI_BC_PERIODIC;
    a->comp = comp;
    a->nb = nb;
    a->dx = p->dx;
    a->dy = p->dy;
    a->zn = tab<double>(p, comp == 2 ? T_ZF : T_ZM);
    a->hz = tab<double>(p, comp == 2 ? T_HF : T_DZ);
    a->xb = xb;
    return FSEI_OK;
}

fsei_status fsei_ib_interpolate(fsei_plan* p, int comp, const double* field, const double* xb, long nb,
                                double* ub) {
    IbArgs a;
    fsei_status st = ib_setup(p, comp, xb, nb, &a);
    if (st != FSEI_OK) return st;
    if (nb > 0 && (!field || !ub)) return FSEI_ERR_ARG;
    if (nb == 0) return FSEI_OK;
    a.field = const_cast<double*>(field);
    a.ub = ub;
    {
        Timed t(p, K_IB);
        if (p->ncells() < ((size_t)1 << 32))
            hipLaunchKernelGGL(k_ib_interpolate<uint32_t>, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, S(p), a);
        else
            hipLaunchKernelGGL(k_ib_interpolate<size_t>, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, S(p), a);
    }
    return check_hip();
}

fsei_status fsei_ib_spread(fsei_plan* p, int comp, double* field, const double* xb, const double* fb,
                           const double* dvb, long nb) {
    IbArgs a;
    fsei_status st = ib_setup(p, comp, xb, nb, &a);
    if (st != FSEI_OK) return st;
    if (nb > 0 && (!field || !fb || !dvb)) return FSEI_ERR_ARG;
    if (nb == 0) return FSEI_OK;
    a.field = field;
    a.fb = fb;
    a.dvb = dvb;
    {
        Timed t(p, K_IB);
        const dim3 grid((unsigned)((nb + 255) / 256));
        // the LDS table's 32-bit keys must hold the node offsets
        if (p->ncells() > (size_t)0xFFFFFFFEu)
            hipLaunchKernelGGL(k_ib_spread<size_t>, grid, dim3(256), 0, S(p), a);
        else if (nb <= 256L * cus_of_current_device())
            hipLaunchKernelGGL(k_ib_spread_lds<true>, grid, dim3(256), 0, S(p), a);
        else
            hipLaunchKernelGGL(k_ib_spread_lds<false>, grid, dim3(256), 0, S(p), a);
    }
    return check_hip();
}

fsei_status fsei_plan_set_timing(fsei_plan* p, int enable) {
    if (!p) return FSEI_ERR_ARG;
    p->timing = enable != 0;
    return FSEI_OK;
}

fsei_status fsei_plan_reset_timing(fsei_plan* p) {
    if (!p) return FSEI_ERR_ARG;
    harvest(p);
    for (int s = 0; s < FSEI_NUM_KERNEL_SLOTS; ++s) {
        p->t_ms[s] = 0.0;
        p->t_count[s] = 0;
    }
    return FSEI_OK;
}

fsei_status fsei_plan_kernel_time(fsei_plan* p, int slot, double* total_ms, long* launches, const char** name) {
    if (!p || slot < 0 || slot >= FSEI_NUM_KERNEL_SLOTS) return FSEI_ERR_ARG;
    harvest(p);
    if (total_ms) *total_ms = p->t_ms[slot];
    if (launches) *launches = p->t_count[slot];
    if (name) *name = kSlotNames[slot];
    return FSEI_OK;
}

}  // extern "C"
