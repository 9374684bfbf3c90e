// pn.hip -- the post-Newtonian terms (pn.h) as a kernel of their own: the
// initialisation and steps whose end does not add them itself.
#include "pn.h"

namespace nb {
namespace {

// One lane per leading row of the active list (the hard particles come
// first in an ordered list): for a hard particle i, the terms of every pair
// (i, k) with k < n_hard, k != i, added to its acceleration and jerk, and to
// its snap and crackle when those outputs are given (orders 6 and 8).
template <int P>
__global__ void __launch_bounds__(64)
k_pn(int64_t n, int64_t n_hard, int rows, const double *__restrict__ m, const double *__restrict__ x,
     const double *__restrict__ v, PnDs ds, const int64_t *__restrict__ t_tick_of, int64_t t,
     double c, int terms, const int32_t *__restrict__ act, int64_t n_act, double *__restrict__ acc,
     double *__restrict__ jrk, double *__restrict__ snp, double *__restrict__ crk)
{
    const int q = int(blockIdx.x) * 64 + int(threadIdx.x);
    if (q >= rows) return;
    const int64_t i = act[q];
    if (i < 0 || i >= n_hard) return;
    double w[4][3];
    pn_row<P>(n, n_hard, i, m, x, v, ds, t_tick_of, t, c, terms, w);
    double *outs[4] = {acc, jrk, snp, crk};
#pragma unroll
    for (int o = 0; o < 4; ++o)
        if (outs[o])
#pragma unroll
            for (int l = 0; l < 3; ++l) outs[o][l * n_act + q] += w[o][l];
}

}  // namespace

hipError_t launch_pn(const nbody_config &c, const nbody_state &st, const int64_t *t_tick_of, int64_t t_tick,
                     const int32_t *act, int64_t n_act, double *acc, double *jrk, double *snp, double *crk,
                     hipStream_t s)
{
    const int64_t nh = c.n_hard < c.n ? c.n_hard : c.n;
    const int rows = int(n_act < nh ? n_act : nh);
    if (rows <= 0) return hipSuccess;
    const dim3 g(unsigned((rows + 63) / 64));
    const PnDs ds{{st.d[0], st.d[1], st.d[2], st.d[3], st.d[4], st.d[5]}};
#define NB_PN(P)                                                                                              \
    hipLaunchKernelGGL((k_pn<P>), g, dim3(64), 0, s, c.n, nh, rows, st.m, st.x, st.v, ds, t_tick_of, t_tick, \
                       c.c_light, int(c.pn_terms), act, n_act, acc, jrk, snp, crk)
    if (c.order == 4) NB_PN(4);
    else if (c.order == 6) NB_PN(6);
    else NB_PN(8);
#undef NB_PN
    return hipGetLastError();
}

}  // namespace nb
