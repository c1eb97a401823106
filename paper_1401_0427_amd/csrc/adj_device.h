// Node arithmetic of the discrete adjoint (formulas in adjoint.hip) and the partial
// sums of dL/ds, shared by the one-step and multi-step adjoint kernels.
#pragma once

#include "internal.h"

namespace lbm {

// mu = J^T l at W = (h, qx, qy), J = d f^eq / d W; ih = 1 / h.  The adjoint steps take
// lbm_rcp(h), which their f^eq has computed already; the gradient at a caller's W0, whose
// heights nothing has checked, the division.
__device__ __forceinline__ void adj_mu(const double *l, double h, double ih, double qx, double qy,
                                       const Phys &P, double &mh, double &mx, double &my)
{
    const double u = qx * ih, v = qy * ih, gh = P.g * h;
    const double L0h = (l[0] + l[2]) + (l[1] + l[3]);
    const double Lxh = l[0] - l[2], Lyh = l[1] - l[3];
    const double L0x = (l[4] + l[6]) + (l[5] + l[7]);
    const double Lxx = l[4] - l[6], Lyx = l[5] - l[7];
    const double L0y = (l[8] + l[10]) + (l[9] + l[11]);
    const double Lxy = l[8] - l[10], Lyy = l[9] - l[11];
    const double cross = Lyx + Lxy;
    mh = 0.25 * L0h + P.c * (Lxx * (gh - u * u) - cross * (u * v) + Lyy * (gh - v * v));
    mx = P.c * Lxh + 0.25 * L0x + P.c * (2.0 * u * Lxx + v * cross);
    my = P.c * Lyh + 0.25 * L0y + P.c * (2.0 * v * Lyy + u * cross);
}

// The collision's transpose at one 2D node: l holds lam^{n+1} on entry and vt on exit
// (not rounded); returns the node's share of dL/ds, lam^{n+1} . (f^eq(W(v)) - v).
template <typename T>
__device__ __forceinline__ double adj_node2d(const double *v, double *l, const Phys &P)
{
    double h, qx, qy, e[12], mu[3];
    moments2d(v, h, qx, qy);
    feq2d<T>(h, qx, qy, P, e);
    adj_mu(l, h, lbm_rcp(h), qx, qy, P, mu[0], mu[1], mu[2]);
    double acc[3] = {0.0, 0.0, 0.0};  // one chain per component
#pragma unroll
    for (int pl = 0; pl < 12; ++pl)
        acc[pl >> 2] = __builtin_fma(l[pl], e[pl] - v[pl], acc[pl >> 2]);
    // (products and sums of lambda stay apart: float storage rounds it at every step, and
    // a fused form, though no less exact, moves a 500-step gradient by 1e-7)
    const double oms = 1.0 - P.s;
#pragma unroll
    for (int pl = 0; pl < 12; ++pl) l[pl] = oms * l[pl] + P.s * mu[pl >> 2];
    return (acc[0] + acc[1]) + acc[2];
}

// dL/ds of all-periodic 2D grids is summed per row and group of kAdjGroup columns: one FP64 slot per
// group, accumulated step by step.  Groups this narrow let every adjoint kernel,
// whatever its tiling, add exactly the same numbers in the same order, with two
// cross-lane additions and no LDS.  group_sum: the sum over the lane's aligned group of
// four lanes, on each of them: (a0 + a1) + (a2 + a3).
constexpr int kAdjGroup = 4;
template <int CTRL>
__device__ __forceinline__ double adj_quad(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double group_sum(double a)
{
    a = a + adj_quad<0xb1>(a);     // quad_perm [1, 0, 3, 2]
    return a + adj_quad<0x4e>(a);  // quad_perm [2, 3, 0, 1]
}
__host__ __device__ inline long adj_slots_row(int nx) { return (nx + kAdjGroup - 1) / kAdjGroup; }
__device__ __forceinline__ long adj_slot(int nx, int x, int y)
{
    return y * adj_slots_row(nx) + x / kAdjGroup;
}

} // namespace lbm
