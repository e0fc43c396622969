// Point-wise arithmetic of the FR right-hand side shared by the kernels
// that evaluate it (the solution-point kernel, the fused gradient kernel and
// the interface kernels), so that every path computes the same bits.
// Internal header (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace frd {
namespace {

// Multiply-adds are written out and the compiler's own contraction is off in
// this file: which of two products of a difference it would fuse depends on
// the code around, and a kernel that keeps a value in a register would then
// differ in the last bit from one that stores it and reads it back.
#pragma clang fp contract(off)

template <typename T>
__device__ __forceinline__ T madd(T a, T b, T c) { return __builtin_elementwise_fma(a, b, c); }

// a b - c d
template <typename T>
__device__ __forceinline__ T diff2(T a, T b, T c, T d) { return madd(a, b, -(c * d)); }

// a . b of three values each
template <typename T>
__device__ __forceinline__ T dot3(T a0, T a1, T a2, T b0, T b1, T b2) { return madd(a2, b2, madd(a1, b1, a0 * b0)); }

// ---------------------------------------------------------------------------
// Geometry at a solution point from the Jacobian coefficients.
// Tet: constant columns c0..c2.  Prism: dx/dxi = A1 + C1 z,
// dx/deta = B1 + C2 z, dx/dzeta = C0 + C1 x + C2 y.  Hexahedron (trilinear
// map, coefficients c1..c7): dx/dr = c1 + c4 s + c5 t + c7 st,
// dx/ds = c2 + c4 r + c6 t + c7 rt, dx/dt = c3 + c5 r + c6 s + c7 rs.
// adj[k][j] = J dxi_k/dx_j (rows are cross products of the columns).
// ---------------------------------------------------------------------------
template <typename T, int ET>
__device__ __forceinline__ T metric(const T *__restrict__ g, int64_t ld, int64_t e,
                                    const T *__restrict__ xi, T adj[3][3]) {
    T c[3][3];
    if (ET == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int d = 0; d < 3; ++d) c[k][d] = g[(3 * k + d) * ld + e];
    } else if (ET == 2) {
        const T r = xi[0], sv = xi[1], t = xi[2];
        const T st = sv * t, rt = r * t, rs = r * sv;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const T c1 = g[d * ld + e], c2 = g[(3 + d) * ld + e], c3 = g[(6 + d) * ld + e];
            const T c4 = g[(9 + d) * ld + e], c5 = g[(12 + d) * ld + e], c6 = g[(15 + d) * ld + e];
            const T c7 = g[(18 + d) * ld + e];
            c[0][d] = madd(c7, st, madd(c5, t, madd(c4, sv, c1)));
            c[1][d] = madd(c7, rt, madd(c6, t, madd(c4, r, c2)));
            c[2][d] = madd(c7, rs, madd(c6, sv, madd(c5, r, c3)));
        }
    } else {
        const T x = xi[0], y = xi[1], z = xi[2];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const T A1 = g[d * ld + e], B1 = g[(3 + d) * ld + e], C0 = g[(6 + d) * ld + e];
            const T C1 = g[(9 + d) * ld + e], C2 = g[(12 + d) * ld + e];
            c[0][d] = madd(C1, z, A1);
            c[1][d] = madd(C2, z, B1);
            c[2][d] = madd(C2, y, madd(C1, x, C0));
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int k1 = (k + 1) % 3, k2 = (k + 2) % 3;
        adj[k][0] = diff2(c[k1][1], c[k2][2], c[k1][2], c[k2][1]);
        adj[k][1] = diff2(c[k1][2], c[k2][0], c[k1][0], c[k2][2]);
        adj[k][2] = diff2(c[k1][0], c[k2][1], c[k1][1], c[k2][0]);
    }
    return dot3(c[0][0], c[0][1], c[0][2], adj[0][0], adj[0][1], adj[0][2]);
}

// Inviscid flux F[j][v] of the conserved state u, with the constant
// reference pressure pref taken out of the momentum flux's pressure term
// (pref = 0: the plain flux; p returns the full pressure).  A constant flux
// has zero discrete divergence on a mesh that preserves a uniform state, so
// every residual is unchanged in exact arithmetic when the volume and the
// interface fluxes both leave pref out, while single precision no longer
// rounds the large constant part of the pressure at low Mach number.
template <typename T>
__device__ __forceinline__ void euler_flux(const T u[5], T gamma, T pref, T F[3][5], T &p) {
    const T rinv = T(1) / u[0];
    const T v[3] = {u[1] * rinv, u[2] * rinv, u[3] * rinv};
    p = (gamma - T(1)) * madd(T(-0.5), dot3(u[1], u[2], u[3], v[0], v[1], v[2]), u[4]);
    const T pm = p - pref;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        F[j][0] = u[1 + j];
#pragma unroll
        for (int i = 0; i < 3; ++i) F[j][1 + i] = i == j ? madd(u[1 + i], v[j], pm) : u[1 + i] * v[j];
        F[j][4] = (u[4] + p) * v[j];
    }
}

// Viscous flux Fv[j][v] from the state u and the physical gradient q[j][v]:
// tau = mu (grad v + grad v^T - 2/3 div v I), heat flux from grad(p/rho) with
// conductivity mu gamma / (Pr (gamma - 1)).
template <typename T>
__device__ __forceinline__ void viscous_flux(const T u[5], const T q[3][5], T gamma, T mu,
                                             T prandtl, T Fv[3][5]) {
    const T rinv = T(1) / u[0];
    const T v[3] = {u[1] * rinv, u[2] * rinv, u[3] * rinv};
    const T e = u[4] * rinv;
    T dv[3][3], dT[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
#pragma unroll
        for (int i = 0; i < 3; ++i) dv[i][j] = madd(-v[i], q[j][0], q[j][1 + i]) * rinv;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j)
        dT[j] = (gamma - T(1)) * madd(madd(-e, q[j][0], q[j][4]), rinv,
                                      -dot3(v[0], v[1], v[2], dv[0][j], dv[1][j], dv[2][j]));
    const T div = dv[0][0] + dv[1][1] + dv[2][2];
    const T kappa = mu * gamma / (prandtl * (gamma - T(1)));
    const T mdiv = mu * T(2.0 / 3.0) * div;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        Fv[j][0] = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            Fv[j][1 + i] = i == j ? madd(mu, dv[i][j] + dv[j][i], -mdiv) : mu * (dv[i][j] + dv[j][i]);
        Fv[j][4] = madd(kappa, dT[j], dot3(v[0], v[1], v[2], Fv[j][1], Fv[j][2], Fv[j][3]));
    }
}

// Physical gradient q = adj^T qt / J at one solution point.
template <typename T>
__device__ __forceinline__ void upts_gradient(const T qt[3][5], const T adj[3][3], T Jinv, T q[3][5]) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int v = 0; v < 5; ++v)
            q[j][v] = dot3(adj[0][j], adj[1][j], adj[2][j], qt[0][v], qt[1][v], qt[2][v]) * Jinv;
}

// Transformed flux Ft = adj (F_inv(u) - F_vis(u, q)) at one solution point
// (NS false: the inviscid flux alone, q unused).
template <typename T, bool NS>
__device__ __forceinline__ void upts_flux(const T u[5], const T q[3][5], const T adj[3][3], T gamma, T mu, T prandtl,
                                          T pref, T Ft[3][5]) {
    T F[3][5], p;
    euler_flux(u, gamma, pref, F, p);
    if (NS) {
        T Fv[3][5];
        viscous_flux(u, q, gamma, mu, prandtl, Fv);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int v = 1; v < 5; ++v) F[j][v] -= Fv[j][v];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int v = 0; v < 5; ++v) Ft[k][v] = dot3(adj[k][0], adj[k][1], adj[k][2], F[0][v], F[1][v], F[2][v]);
}

// Work at one solution point: the physical gradient (NS) and the
// transformed flux.  Section 3.4: compressible Navier-Stokes with constant
// viscosity; Section 2.1: the point-wise step between the operator products.
template <typename T, bool NS>
__device__ __forceinline__ void upts_point(const T u[5], const T qt[3][5], const T adj[3][3], T Jinv, T gamma,
                                           T mu, T prandtl, T pref, T q[3][5], T Ft[3][5]) {
    if (NS) upts_gradient(qt, adj, Jinv, q);
    upts_flux<T, NS>(u, q, adj, gamma, mu, prandtl, pref, Ft);
}

#pragma clang fp contract(fast)   // as the files that include this one

}  // namespace
}  // namespace frd
