// The transform kernels of one compiled length: this file is compiled once
// per length of FSEI_LENGTHS, with -DFSEI_LEN=<length>.
#include "fsei_lengths.h"

namespace fsei {
namespace dev {

namespace {

constexpr int N = FSEI_LEN;

template <typename TI, typename TO, int PRO>
void xfwd(const XFwdArgs<TI, TO>& a, unsigned grid, hipStream_t st) {
    hipLaunchKernelGGL((k_xfwd_len<TI, TO, PRO, N>), dim3(grid), dim3(x_len_threads(N, (int)sizeof(TO))), 0, st, a);
}
template <typename T, typename TP, int EPI>
void xinv(const XInvArgs<T, TP>& a, unsigned grid, hipStream_t st) {
    hipLaunchKernelGGL((k_xinv_len<T, TP, EPI, N>), dim3(grid), dim3(x_len_threads(N, (int)sizeof(T))), 0, st, a);
}
template <typename T>
void xinv_grad(const XInvGradArgs<T>& a, unsigned grid, hipStream_t st) {
    hipLaunchKernelGGL((k_xinv_grad_len<T, N>), dim3(grid), dim3(XgGeom<N>::NTHR), 0, st, a);
}
template <typename T, bool VEC>
void yfwd(const YArgs<T>& a, unsigned grid, hipStream_t st) {
    hipLaunchKernelGGL((k_yfwd_len<T, N, VEC>), dim3(grid), dim3(y_len_threads(N, (int)sizeof(T))), 0, st, a);
}
template <typename T, bool VEC>
void yinv(const YArgs<T>& a, unsigned grid, hipStream_t st) {
    hipLaunchKernelGGL((k_yinv_len<T, N, VEC>), dim3(grid), dim3(y_len_threads(N, (int)sizeof(T))), 0, st, a);
}

LenOps make() {
    LenOps o{};
    o.x_rows = x_len_rows(N);
    o.y_pairs_d = y_len_pairs(N, 8);
    o.y_pairs_f = y_len_pairs(N, 4);
    o.xf_dd[PRO_COPY] = xfwd<double, double, PRO_COPY>;
    o.xf_dd[PRO_DIV] = xfwd<double, double, PRO_DIV>;
    o.xf_dd[PRO_DIV_ADJ] = xfwd<double, double, PRO_DIV_ADJ>;
    o.xf_ff[PRO_DIV] = xfwd<float, float, PRO_DIV>;
    o.xf_ff[PRO_DIV_ADJ] = xfwd<float, float, PRO_DIV_ADJ>;
    o.xf_df[PRO_COPY] = xfwd<double, float, PRO_COPY>;
    o.xf_df[PRO_DIV] = xfwd<double, float, PRO_DIV>;
    o.xf_df[PRO_RESID] = xfwd<double, float, PRO_RESID>;
    o.xf_df[PRO_RESID_F] = xfwd<double, float, PRO_RESID_F>;
    o.xi_dd[EPI_STORE] = xinv<double, double, EPI_STORE>;
    o.xi_ff[EPI_STORE] = xinv<float, float, EPI_STORE>;
    o.xi_fd[EPI_STORE] = xinv<float, double, EPI_STORE>;
    o.xi_fd[EPI_ACC] = xinv<float, double, EPI_ACC>;
    o.xi_fd[EPI_ADDF] = xinv<float, double, EPI_ADDF>;
    o.xi_fd[EPI_ACC_KEEP] = xinv<float, double, EPI_ACC_KEEP>;
    if constexpr (xg_len(N)) o.xg_d = xinv_grad<double>;
    o.yf_d[0] = yfwd<double, false>;
    o.yf_d[1] = yfwd<double, true>;
    o.yi_d[0] = yinv<double, false>;
    o.yi_d[1] = yinv<double, true>;
    o.yf_f[0] = yfwd<float, false>;
    o.yf_f[1] = yfwd<float, true>;
    o.yi_f[0] = yinv<float, false>;
    o.yi_f[1] = yinv<float, true>;
    return o;
}

}  // namespace

#define FSEI_CAT_(a, b) a##b
#define FSEI_CAT(a, b) FSEI_CAT_(a, b)
const LenOps& FSEI_CAT(len_ops_, FSEI_LEN)() {
    static const LenOps o = make();
    return o;
}

}  // namespace dev
}  // namespace fsei
