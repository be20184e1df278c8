// The collision of one node (Eq. fiexp and the general operator of Eq. mrtlbe; the formulas stand at the top
// of lbm_lattice_impl.h), shared by the single-step kernel and the marching kernels.  Products and sums are
// fused as written and nowhere else, so every kernel that collides a node with the same values gets the
// same bits: a run does not depend on which of them took a step.
#pragma once

#include "lbm_device.h"

namespace lbm {

__device__ __forceinline__ float fm(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fm(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <class T> struct Node {
    T drho, jx, jy, jz, pxx, pyy, pzz, pxy, pxz, pyz;
};

// Moments over opposite pairs (i, i + 1): the pair sum feeds the even moments (mass, second moments),
// the difference the odd ones (momentum).  Each sum starts at its first term.
template <class T> __device__ __forceinline__ Node<T> moments_of(const T (&f)[NQ])
{
    Node<T> m{f[0], 0, 0, 0, 0, 0, 0, 0, 0, 0};
    bool s_jx = false, s_jy = false, s_jz = false, s_pxx = false, s_pyy = false, s_pzz = false, s_pxy = false,
         s_pxz = false, s_pyz = false;
#pragma unroll
    for (int i = 1; i < NQ; i += 2) {
        const T sm = f[i] + f[i + 1], df = f[i] - f[i + 1];
        const int cx = cvel(i, 0), cy = cvel(i, 1), cz = cvel(i, 2);
        m.drho += sm;
        if (cx != 0) { acc_first(m.jx, s_jx, cx > 0 ? df : -df); acc_first(m.pxx, s_pxx, sm); }
        if (cy != 0) { acc_first(m.jy, s_jy, cy > 0 ? df : -df); acc_first(m.pyy, s_pyy, sm); }
        if (cz != 0) { acc_first(m.jz, s_jz, cz > 0 ? df : -df); acc_first(m.pzz, s_pzz, sm); }
        if (cx * cy != 0) acc_first(m.pxy, s_pxy, cx * cy > 0 ? sm : -sm);
        if (cx * cz != 0) acc_first(m.pxz, s_pxz, cx * cz > 0 ? sm : -sm);
        if (cy * cz != 0) acc_first(m.pyz, s_pyz, cy * cz > 0 ? sm : -sm);
    }
    return m;
}

// Force density of one point, whose stencil starts at (bx, by, bz), at node (x, y, z), added to (gx, gy, gz) (Sec. III).
// Rows the point's stencil misses take nothing from it and are skipped (a branch taken by whole waves when y and
// z are wave-uniform; otherwise waves whose lanes all miss skip it).
template <class T>
__device__ __forceinline__ void add_point(const Geom& G, int bx, int by, int bz, const PRec<T>& r, int x, int y, int z, T& gx,
                                          T& gy, T& gz)
{
    int dy = y - by, dz = z - bz;
    if (dy < 0) dy += G.ny;
    if (dz < 0) dz += G.nz;
    if (dy > 3 || dz > 3) return;
    const T w = stencil_w<T>(x, bx, G.nx, r.wx) * stencil_w<T>(y, by, G.ny, r.wy) * stencil_w<T>(z, bz, G.nz, r.wz);
    gx = fm(r.f[0], w, gx);
    gy = fm(r.f[1], w, gy);
    gz = fm(r.f[2], w, gz);
}

// What the collision needs of a box, in the arithmetic type.
template <class T> struct Rates {
    T rho0, tau, om;      // reference density, tau, 1 / (tau + 1/2)
    T tb, omb;            // general operator: bulk mode
};

template <int COLL, class T> __device__ __forceinline__ Rates<T> rates_of(const Geom& G, const BoxDev& B)
{
    Rates<T> r{T(G.rho0), T(B.tau), T(B.omega), T(0), T(0)};
    if constexpr (COLL != 0) {
        r.tb = T(B.tau_b);
        r.omb = T(B.omega_b);
    }
    return r;
}

// Velocity u and the ten pieces of the post-collision state (order of MomPlane) from the moments and the
// force density g.  COLL != 0: the trace of the stress relaxes at omega_b (bulk mode).
template <int COLL, class T>
__device__ __forceinline__ void pieces_of(const Node<T>& m, const T (&g)[3], const Rates<T>& R, T (&p)[MP_N], T (&u)[3])
{
#pragma clang fp contract(off)
    const T half = T(0.5), third = T(1.0 / 3.0);
    const T rho = R.rho0 + m.drho, ir = T(1) / rho;
    const T hx = fm(half, g[0], m.jx), hy = fm(half, g[1], m.jy), hz = fm(half, g[2], m.jz);
    const T ux = hx * ir, uy = hy * ir, uz = hz * ir;
    u[0] = ux;
    u[1] = uy;
    u[2] = uz;
    const T sxx = fm(-third, m.drho, m.pxx), syy = fm(-third, m.drho, m.pyy), szz = fm(-third, m.drho, m.pzz);
    // rho u_a u_b + tau (u_a g_b + g_a u_b) as u_b (rho u_a + tau g_a) + u_a tau g_b with rho u_a = h_a
    const T tgx = R.tau * g[0], tgy = R.tau * g[1], tgz = R.tau * g[2];
    const T qx = hx + tgx, qy = hy + tgy, qz = hz + tgz;
    const T dxx = fm(-ux, qx + tgx, sxx), dyy = fm(-uy, qy + tgy, syy), dzz = fm(-uz, qz + tgz, szz);
    T Bxx, Byy, Bzz;
    if constexpr (COLL != 0) {
        const T trs = ((dxx + dyy) + dzz) * third;
        const T uu = fm(uz, uz, fm(uy, uy, ux * ux)), ug = fm(uz, g[2], fm(uy, g[1], ux * g[0]));
        const T trb = fm(T(-2) * R.tb, ug, fm(-rho, uu, (sxx + syy) + szz)) * third;
        Bxx = fm(-R.omb, trb, fm(-R.om, dxx - trs, sxx));
        Byy = fm(-R.omb, trb, fm(-R.om, dyy - trs, syy));
        Bzz = fm(-R.omb, trb, fm(-R.om, dzz - trs, szz));
    } else {
        Bxx = fm(-R.om, dxx, sxx);
        Byy = fm(-R.om, dyy, syy);
        Bzz = fm(-R.om, dzz, szz);
    }
    const T Bxy = fm(-R.om, m.pxy - fm(ux, tgy, uy * qx), m.pxy);
    const T Bxz = fm(-R.om, m.pxz - fm(ux, tgz, uz * qx), m.pxz);
    const T Byz = fm(-R.om, m.pyz - fm(uy, tgz, uz * qy), m.pyz);
    p[MP_R0] = fm(T(-1.5), (Bxx + Byy) + Bzz, m.drho);
    p[MP_AX] = T(3) * (m.jx + g[0]);
    p[MP_AY] = T(3) * (m.jy + g[1]);
    p[MP_AZ] = T(3) * (m.jz + g[2]);
    p[MP_BXX] = T(4.5) * Bxx;
    p[MP_BYY] = T(4.5) * Byy;
    p[MP_BZZ] = T(4.5) * Bzz;
    p[MP_BXY] = T(9) * Bxy;
    p[MP_BXZ] = T(9) * Bxz;
    p[MP_BYZ] = T(9) * Byz;
}

// Whether the moments and the force of a node are finite.
template <class T> __device__ __forceinline__ bool finite_node(const Node<T>& m, const T (&g)[3])
{
    const T chk = m.drho + m.jx + m.jy + m.jz + m.pxx + m.pyy + m.pzz + g[0] + g[1] + g[2];
    return fabs(chk) <= T(sizeof(T) == 4 ? 3.0e38 : 1.0e300);
}

// Post-collision populations from the pieces (projected operator).  Rounded as if stored: the product is never fused
// into the sums of a pull that takes the value from a register.
template <class T> __device__ __forceinline__ void populations_of(const T (&p)[MP_N], T (&f)[NQ])
{
#pragma clang fp contract(off)
    f[0] = T(wgt(0)) * p[MP_R0];
#pragma unroll
    for (int i = 1; i < NQ; i += 2) {
        T bp, bm;
        rebuild_pair(p, i, bp, bm);
        f[i] = T(wgt(i)) * bp;
        f[i + 1] = T(wgt(i)) * bm;
    }
}

}  // namespace lbm
