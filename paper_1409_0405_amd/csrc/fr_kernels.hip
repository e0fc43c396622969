// HIP kernels of the FR right-hand side for gfx950 (CDNA4).
//
// Paper, Section 2.1: an FR step is mostly products C <- A B of a small
// constant operator A with very wide row-major state matrices B (block-by-
// panel shape), plus point-wise operations at solution and flux points.
// Section 3.4: DG-type scheme, Rusanov interface flux, compressible
// Navier-Stokes with constant viscosity.
//
// State layout per element type: [point][field][ld], element index fastest,
// so every point-wise access of a wavefront is one contiguous segment and the
// operator products see B as K rows of (fields x ld) contiguous columns.
//
// The operator products live in fr_opmul.hpp, instantiated per element type
// and precision in fr_opmul_*.hip.
#include <hip/hip_runtime.h>

#include <cmath>

#include "fr_device.hpp"
#include "fr_opmul.hpp"
#include "fr_pointwise.hpp"

namespace frd {

// instantiated in fr_opmul_*.hip
FR_OPMUL_EXTERN(float, 0) FR_OPMUL_EXTERN(double, 0)
FR_SPLIT_EXTERN(false, 0) FR_SPLIT_EXTERN(true, 0)
FR_OPMUL_EXTERN(float, 1) FR_OPMUL_EXTERN(double, 1)
FR_SPLIT_EXTERN(false, 1) FR_SPLIT_EXTERN(true, 1)
FR_OPMUL_EXTERN(float, 2) FR_OPMUL_EXTERN(double, 2)
FR_SPLIT_EXTERN(false, 2) FR_SPLIT_EXTERN(true, 2)
FR_OPMUL_EXTERN(float, 3) FR_OPMUL_EXTERN(double, 3)
FR_SPLIT_EXTERN(false, 3) FR_SPLIT_EXTERN(true, 3)
FR_OPMUL_EXTERN(float, 4) FR_OPMUL_EXTERN(double, 4)
FR_SPLIT_EXTERN(false, 4) FR_SPLIT_EXTERN(true, 4)
FR_OPMUL_EXTERN(float, 5) FR_OPMUL_EXTERN(double, 5)
FR_SPLIT_EXTERN(false, 5) FR_SPLIT_EXTERN(true, 5)
FR_OPMUL_EXTERN(float, 6) FR_OPMUL_EXTERN(double, 6)
FR_SPLIT_EXTERN(false, 6) FR_SPLIT_EXTERN(true, 6)
FR_OPMUL_EXTERN(float, 7) FR_OPMUL_EXTERN(double, 7)
FR_SPLIT_EXTERN(false, 7) FR_SPLIT_EXTERN(true, 7)
FR_OPMUL_EXTERN(float, 8) FR_OPMUL_EXTERN(double, 8)
FR_SPLIT_EXTERN(false, 8) FR_SPLIT_EXTERN(true, 8)
FR_OPMUL_EXTERN(float, 9) FR_OPMUL_EXTERN(double, 9)
FR_SPLIT_EXTERN(false, 9) FR_SPLIT_EXTERN(true, 9)
FR_OPMUL_EXTERN(float, 10) FR_OPMUL_EXTERN(double, 10)
FR_SPLIT_EXTERN(false, 10) FR_SPLIT_EXTERN(true, 10)
FR_OPMUL_EXTERN(float, 11) FR_OPMUL_EXTERN(double, 11)
FR_SPLIT_EXTERN(false, 11) FR_SPLIT_EXTERN(true, 11)

namespace {

// ---------------------------------------------------------------------------
// Point-wise solution-point kernel: physical gradient and transformed flux.
// One thread per (element, solution point); blockIdx.y is the point.
// ---------------------------------------------------------------------------
template <typename T, int ET, bool NS>
__global__ __launch_bounds__(256) void upts_kernel(UptsArgs<T> a) {
    const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int i = blockIdx.y;
    if (e >= a.nelem) return;
    const int64_t ld = a.ld;
    T adj[3][3], Jinv;
    if (a.padj) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) adj[k][j] = a.padj[(int64_t(3 * k + j) * a.nu + i) * ld + e];
        Jinv = a.pjinv[int64_t(i) * ld + e];
    } else {
        Jinv = T(1) / metric<T, ET>(a.geom, ld, e, a.xi + 3 * i, adj);
    }
    T u[5], qt[3][5], q[3][5], Ft[3][5];
#pragma unroll
    for (int v = 0; v < 5; ++v) u[v] = a.U[(int64_t(i) * 5 + v) * ld + e];
    if (NS) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v)
                qt[k][v] = a.Qt[((int64_t(k) * a.nu + i) * 5 + v) * ld + e];
    }
    upts_point<T, NS>(u, qt, adj, Jinv, a.gamma, a.mu, a.prandtl, a.pref, q, Ft);
    if (NS) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int v = 0; v < 5; ++v) a.Q[(int64_t(i) * 15 + j * 5 + v) * ld + e] = q[j][v];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int v = 0; v < 5; ++v) a.Ft[((int64_t(k) * a.nu + i) * 5 + v) * ld + e] = Ft[k][v];
}

// Per-type kernel argument of an element type t in {0, 1, 2}, selected
// without indexing the argument block (which would be a memory load per
// thread).
template <typename P>
__device__ __forceinline__ P pick(const P (&v)[NTYPE], int t) {
    return t == 0 ? v[0] : (t == 1 ? v[1] : v[2]);
}

// Side word: element (22 bits) | flux point << 22 (8 bits) | type << 30.
__device__ __forceinline__ void unpack(uint32_t s, int64_t &e, int &f, int &t) {
    e = s & 0x3fffffu;
    f = (s >> 22) & 0xff;
    t = s >> 30;
}

// Jump to the common solution of the LDG scheme at each paired flux point,
// C = (1/2 - beta) U_L + (1/2 + beta) U_R, stored per side as D = C - U_f:
//   D_L = (1/2 + beta) (U_R - U_L),   D_R = (1/2 - beta) (U_L - U_R).
// A side whose weight is zero keeps the zeros the buffer was created with.
template <typename T>
__global__ __launch_bounds__(256) void common_solution_kernel(PairArgs<T> a) {
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= a.npairs) return;
    int64_t eL, eR;
    int fL, fR, tL, tR;
    unpack(a.sideL[p], eL, fL, tL);
    unpack(a.sideR[p], eR, fR, tR);
    const int64_t ldL = pick(a.ld, tL), ldR = pick(a.ld, tR);
    const T wL = T(0.5) + a.beta, wR = T(0.5) - a.beta;
    const T *__restrict__ uL = pick(a.Uf, tL) + int64_t(fL) * 5 * ldL + eL;
    const T *__restrict__ uR = pick(a.Uf, tR) + int64_t(fR) * 5 * ldR + eR;
    T jump[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) jump[v] = uR[v * ldR] - uL[v * ldL];     // all loads first
    if (wL != T(0)) {
        T *dL = pick(a.Cf, tL) + int64_t(fL) * 5 * ldL + eL;
#pragma unroll
        for (int v = 0; v < 5; ++v) dL[v * ldL] = wL * jump[v];
    }
    if (wR != T(0)) {
        T *dR = pick(a.Cf, tR) + int64_t(fR) * 5 * ldR + eR;
#pragma unroll
        for (int v = 0; v < 5; ++v) dR[v * ldR] = -wR * jump[v];
    }
}

// Common transformed normal flux at each paired flux point:
//   f = Rusanov(U_L, U_R; n) [- ((1/2+beta) Fv_L + (1/2-beta) Fv_R).n
//       + tau (U_L - U_R)]   (NS terms in brackets)
// side L stores sL f, side R stores -sR f.
template <typename T, bool NS>
__global__ __launch_bounds__(256) void common_flux_kernel(PairArgs<T> a) {
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= a.npairs) return;
    int64_t eL, eR;
    int fL, fR, tL, tR;
    unpack(a.sideL[p], eL, fL, tL);
    unpack(a.sideR[p], eR, fR, tR);
    const int64_t ldL = pick(a.ld, tL), ldR = pick(a.ld, tR);
    const int64_t P = a.npairs;
    const T n[3] = {a.geo[p], a.geo[P + p], a.geo[2 * P + p]};
    const T sL = a.geo[3 * P + p], sR = a.geo[4 * P + p];
    T uL[5], uR[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        uL[v] = pick(a.Uf, tL)[(int64_t(fL) * 5 + v) * ldL + eL];
        uR[v] = pick(a.Uf, tR)[(int64_t(fR) * 5 + v) * ldR + eR];
    }
    // gradients of the sides whose LDG weight is not zero, loaded together
    // with the states (beta = +-1/2, the usual choice, needs one side only:
    // the other term would be an exact zero).  One address per side: formed
    // anew for each of the fifteen loads, a wide multiply shared a register
    // pair with the load before it and waited for every load in flight
    // (order 4, 9,261 hexahedra, FP32 state: 35.9 us, without that wait 33.0)
    const T wl = T(0.5) + a.beta, wr = T(0.5) - a.beta;
    T qL[3][5], qR[3][5];
    if (NS && wl != T(0)) {
        const T *__restrict__ q = pick(a.Qf, tL) + (int64_t(fL) * 15 * ldL + eL);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int v = 0; v < 5; ++v) qL[j][v] = q[(j * 5 + v) * ldL];
    }
    if (NS && wr != T(0)) {
        const T *__restrict__ q = pick(a.Qf, tR) + (int64_t(fR) * 15 * ldR + eR);
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int v = 0; v < 5; ++v) qR[j][v] = q[(j * 5 + v) * ldR];
    }
    T FL[3][5], FR[3][5], pL, pR;
    euler_flux(uL, a.gamma, a.pref, FL, pL);
    euler_flux(uR, a.gamma, a.pref, FR, pR);
    const T vnL = (uL[1] * n[0] + uL[2] * n[1] + uL[3] * n[2]) / uL[0];
    const T vnR = (uR[1] * n[0] + uR[2] * n[1] + uR[3] * n[2]) / uR[0];
    const T cL = sqrt(a.gamma * pL / uL[0]), cR = sqrt(a.gamma * pR / uR[0]);
    const T lam = fmax(fabs(vnL) + cL, fabs(vnR) + cR);
    T f[5];
#pragma unroll
    for (int v = 0; v < 5; ++v)
        f[v] = T(0.5) * (n[0] * (FL[0][v] + FR[0][v]) + n[1] * (FL[1][v] + FR[1][v]) +
                         n[2] * (FL[2][v] + FR[2][v])) -
               T(0.5) * lam * (uR[v] - uL[v]);
    if (NS) {
        T FvL[3][5], FvR[3][5];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int v = 0; v < 5; ++v) FvL[j][v] = FvR[j][v] = T(0);
        if (wl != T(0)) viscous_flux(uL, qL, a.gamma, a.mu, a.prandtl, FvL);
        if (wr != T(0)) viscous_flux(uR, qR, a.gamma, a.mu, a.prandtl, FvR);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            T fv = 0;
#pragma unroll
            for (int j = 0; j < 3; ++j) fv += n[j] * (wl * FvL[j][v] + wr * FvR[j][v]);
            f[v] += -fv + a.tau * (uL[v] - uR[v]);
        }
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        pick(a.Fn, tL)[(int64_t(fL) * 5 + v) * ldL + eL] = sL * f[v];
        pick(a.Fn, tR)[(int64_t(fR) * 5 + v) * ldR + eR] = -sR * f[v];
    }
}

// ---------------------------------------------------------------------------
// Boundary points.  Wall (kind 1): Ub = (rho, 0, 0, 0, rho T_w / (gamma - 1)),
// ghost = (rho, -rho v, rho T_w / (gamma - 1) + rho |v|^2 / 2), the interior
// velocity mirrored at the wall temperature.  Far field (kind 2): the
// outgoing invariant v.n + 2c/(gamma-1) of the interior and the incoming
// v.n - 2c/(gamma-1) of the free stream fix v.n and c; entropy p/rho^gamma
// and tangential velocity come from the interior where the flow leaves the
// domain, else from the free stream; the ghost is Ub.  Temperature is p/rho.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void boundary_states(const T u[5], const T n[3], int kind, const BndArgs<T> &a,
                                                T ub[5], T gh[5]) {
    const T g1 = a.gamma - T(1);
    const T rinv = T(1) / u[0];
    if (kind == 1) {
        const T eint = u[0] * a.t_wall / g1;
        const T ke = T(0.5) * (u[1] * u[1] + u[2] * u[2] + u[3] * u[3]) * rinv;
        ub[0] = u[0];
        ub[1] = ub[2] = ub[3] = T(0);
        ub[4] = eint;
        gh[0] = u[0];
        gh[1] = -u[1];
        gh[2] = -u[2];
        gh[3] = -u[3];
        gh[4] = eint + ke;
        return;
    }
    const T v[3] = {u[1] * rinv, u[2] * rinv, u[3] * rinv};
    const T p = g1 * (u[4] - T(0.5) * (u[1] * v[0] + u[2] * v[1] + u[3] * v[2]));
    const T vnL = v[0] * n[0] + v[1] * n[1] + v[2] * n[2];
    const T vnf = a.free[1] * n[0] + a.free[2] * n[1] + a.free[3] * n[2];
    const T cL = sqrt(a.gamma * p * rinv), cf = sqrt(a.gamma * a.free[4] / a.free[0]);
    const T rp = vnL + T(2) * cL / g1, rm = vnf - T(2) * cf / g1;
    const T vnb = T(0.5) * (rp + rm), cb = T(0.25) * g1 * (rp - rm);
    const bool out = vnb > T(0);
    const T ent = out ? p / pow(u[0], a.gamma) : a.free[4] / pow(a.free[0], a.gamma);
    T vb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) vb[d] = (out ? v[d] - vnL * n[d] : a.free[1 + d] - vnf * n[d]) + vnb * n[d];
    const T rhob = pow(cb * cb / (a.gamma * ent), T(1) / g1);
    const T pb = rhob * cb * cb / a.gamma;
    ub[0] = rhob;
    ub[1] = rhob * vb[0];
    ub[2] = rhob * vb[1];
    ub[3] = rhob * vb[2];
    ub[4] = pb / g1 + T(0.5) * rhob * (vb[0] * vb[0] + vb[1] * vb[1] + vb[2] * vb[2]);
#pragma unroll
    for (int k = 0; k < 5; ++k) gh[k] = ub[k];
}

template <typename T>
__global__ __launch_bounds__(256) void boundary_solution_kernel(BndArgs<T> a) {
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= a.nb) return;
    int64_t e;
    int f, t;
    unpack(a.side[p], e, f, t);
    const int64_t ld = pick(a.ld, t);
    const T n[3] = {a.geo[p], a.geo[a.nb + p], a.geo[2 * a.nb + p]};
    T u[5], ub[5], gh[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) u[v] = pick(a.Uf, t)[(int64_t(f) * 5 + v) * ld + e];
    boundary_states(u, n, int(a.kind[p]), a, ub, gh);
#pragma unroll
    for (int v = 0; v < 5; ++v) pick(a.Cf, t)[(int64_t(f) * 5 + v) * ld + e] = ub[v] - u[v];
}

template <typename T, bool NS>
__global__ __launch_bounds__(256) void boundary_flux_kernel(BndArgs<T> a) {
    const int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (p >= a.nb) return;
    int64_t e;
    int f, t;
    unpack(a.side[p], e, f, t);
    const int64_t ld = pick(a.ld, t);
    const int64_t nb = a.nb;
    const T n[3] = {a.geo[p], a.geo[nb + p], a.geo[2 * nb + p]};
    const T sc = a.geo[3 * nb + p];
    T u[5], ub[5], gh[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) u[v] = pick(a.Uf, t)[(int64_t(f) * 5 + v) * ld + e];
    T q[3][5];
    if (NS) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int v = 0; v < 5; ++v) q[j][v] = pick(a.Qf, t)[(int64_t(f) * 15 + j * 5 + v) * ld + e];
    }
    boundary_states(u, n, int(a.kind[p]), a, ub, gh);
    T FL[3][5], FR[3][5], pL, pR;
    euler_flux(u, a.gamma, a.pref, FL, pL);
    euler_flux(gh, a.gamma, a.pref, FR, pR);
    const T vnL = (u[1] * n[0] + u[2] * n[1] + u[3] * n[2]) / u[0];
    const T vnR = (gh[1] * n[0] + gh[2] * n[1] + gh[3] * n[2]) / gh[0];
    const T lam = fmax(fabs(vnL) + sqrt(a.gamma * pL / u[0]), fabs(vnR) + sqrt(a.gamma * pR / gh[0]));
    T fl[5];
#pragma unroll
    for (int v = 0; v < 5; ++v)
        fl[v] = T(0.5) * (n[0] * (FL[0][v] + FR[0][v]) + n[1] * (FL[1][v] + FR[1][v]) +
                          n[2] * (FL[2][v] + FR[2][v])) -
                T(0.5) * lam * (gh[v] - u[v]);
    if (NS) {
        T Fv[3][5];
        viscous_flux(ub, q, a.gamma, a.mu, a.prandtl, Fv);
#pragma unroll
        for (int v = 0; v < 5; ++v)
            fl[v] += -(n[0] * Fv[0][v] + n[1] * Fv[1][v] + n[2] * Fv[2][v]) + a.tau * (u[v] - ub[v]);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) pick(a.Fn, t)[(int64_t(f) * 5 + v) * ld + e] = sc * fl[v];
}

// R = -Rt / J at each solution point, fused with a Runge-Kutta register update.
template <typename T, int ET>
__global__ __launch_bounds__(256) void negdivconf_kernel(NegArgs<T> a) {
    const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int i = blockIdx.y;
    if (e >= a.nelem) return;
    const int64_t ld = a.ld;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        const int64_t o = (int64_t(i) * 5 + v) * ld + e;
        neg_update(a, i, v, e, o, a.Rt[o]);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void reduce_kernel(RedArgs<T> a) {
    double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t n = int64_t(a.nu) * a.nelem;
    for (int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; idx < n;
         idx += int64_t(gridDim.x) * blockDim.x) {
        const int i = int(idx / a.nelem);
        const int64_t e = idx - int64_t(i) * a.nelem;
        const double wJ = a.wJ[int64_t(i) * a.ld + e];
        double u[5], r[5] = {0, 0, 0, 0, 0};
        for (int v = 0; v < 5; ++v) {
            u[v] = double(a.U[(int64_t(i) * 5 + v) * a.ld + e]);
            if (a.R) r[v] = double(a.R[(int64_t(i) * 5 + v) * a.ld + e]);
        }
        if (a.what == 1) {
            for (int v = 0; v < 5; ++v) s[v] += wJ * u[v];
        } else if (a.what == 2) {
            for (int v = 0; v < 5; ++v) s[v] += wJ * r[v];
        } else if (a.what == 3) {
            for (int v = 0; v < 5; ++v) s[v] += wJ * r[v] * r[v];
        } else if (a.what == 4) {
            const double vx = u[1] / u[0], vy = u[2] / u[0], vz = u[3] / u[0];
            const double v2 = vx * vx + vy * vy + vz * vz;
            s[0] += wJ * 0.5 * u[0] * v2;
            s[1] += wJ * (vx * r[1] + vy * r[2] + vz * r[3] - 0.5 * v2 * r[0]);
        } else if (a.what == 5) {
            for (int v = 0; v < 5; ++v) s[0] += isfinite(u[v]) ? 0.0 : 1.0;
        } else if (a.what == 6) {
            for (int v = 0; v < 5; ++v) {
                const double u0 = double(a.U0[(int64_t(i) * 5 + v) * a.ld + e]);
                const double q = r[v] / (a.atol + a.rtol * fmax(fabs(u0), fabs(u[v])));
                s[0] += q * q;
            }
        }
    }
    __shared__ double sh[8][256];
    for (int q = 0; q < 8; ++q) sh[q][threadIdx.x] = s[q];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w)
            for (int q = 0; q < 8; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 8) a.partial[int64_t(blockIdx.x) * 8 + threadIdx.x] = sh[threadIdx.x][0];
}

// out[q] = sum_b partial[b][q]: block q, fixed summation tree (deterministic)
__global__ __launch_bounds__(256) void reduce_final_kernel(const double *partial, int nblocks, double *out) {
    const int q = blockIdx.x;
    double s = 0;
    for (int b = threadIdx.x; b < nblocks; b += 256) s += partial[int64_t(b) * 8 + q];
    __shared__ double sh[256];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (int(threadIdx.x) < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[q] = sh[0];
}

template <typename T>
__global__ void copy_kernel(T *dst, const T *src, int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x)
        dst[i] = src[i];
}

}  // namespace

template <typename T>
hipError_t launch_opmul(int tag, const Op<T> &A, const T *B1, int64_t ldb1, int K1, const T *B2,
                        int64_t ldb2, int K2, T *C, int64_t ldc, int64_t ncols, hipStream_t s,
                        const NegArgs<T> *ep) {
    if (ncols % 64 || K1 + K2 <= 0 || A.nmg * A.mbw * 16 < A.M) return hipErrorInvalidValue;
    const NegArgs<T> E = ep ? *ep : NegArgs<T>{};
    // the fused store addresses the divergence output layout [nu][5][ld]
    if (E.fuse && (tag % 4 != 3 || E.ld % 64 || ldc != 5 * E.ld || ncols != ldc || A.M != E.nu ||
                   E.nelem > E.ld || !E.jinv))
        return hipErrorInvalidValue;
    const int64_t npanels = ncols / 64;
#define FR_TAG(t) \
    case t: return launch_opmul_tag<T, t>(A, B1, ldb1, K1, B2, ldb2, K2, C, ldc, npanels, s, E);
    switch (tag) {
        FR_TAG(0) FR_TAG(1) FR_TAG(2) FR_TAG(3) FR_TAG(4) FR_TAG(5) FR_TAG(6) FR_TAG(7)
        FR_TAG(8) FR_TAG(9) FR_TAG(10) FR_TAG(11)
        default: return hipErrorInvalidValue;
    }
#undef FR_TAG
}

hipError_t launch_opmul_split(int tag, const OpSplit &A, const float *B1, int64_t ldb1, int K1,
                              const float *B2, int64_t ldb2, int K2, float *C, int64_t ldc,
                              int64_t ncols, hipStream_t s, const NegArgs<float> *ep) {
    if (ncols % 64 || K1 + K2 <= 0 || A.nmg * A.mbw * 16 < A.M || (A.Kb & 1))
        return hipErrorInvalidValue;
    const NegArgs<float> E = ep ? *ep : NegArgs<float>{};
    if (E.fuse && (tag % 4 != 3 || E.ld % 64 || ldc != 5 * E.ld || ncols != ldc || A.M != E.nu ||
                   E.nelem > E.ld || !E.jinv))
        return hipErrorInvalidValue;
    const int64_t np = ncols / 64;
#define FR_TAG(t)                                                                            \
    case t:                                                                                  \
        return A.format == 2 ? launch_split_tag<true, t>(A, B1, ldb1, K1, B2, ldb2, K2, C, ldc, np, s, E) \
                             : launch_split_tag<false, t>(A, B1, ldb1, K1, B2, ldb2, K2, C, ldc, np, s, E);
    switch (tag) {
        FR_TAG(0) FR_TAG(1) FR_TAG(2) FR_TAG(3) FR_TAG(4) FR_TAG(5) FR_TAG(6) FR_TAG(7)
        FR_TAG(8) FR_TAG(9) FR_TAG(10) FR_TAG(11)
        default: return hipErrorInvalidValue;
    }
#undef FR_TAG
}

template <typename T>
hipError_t launch_upts(int etype, bool ns, const UptsArgs<T> &a, hipStream_t s) {
    const dim3 grid(unsigned((a.nelem + 255) / 256), unsigned(a.nu)), block(256);
    if (etype == 0) {
        if (ns) upts_kernel<T, 0, true><<<grid, block, 0, s>>>(a);
        else upts_kernel<T, 0, false><<<grid, block, 0, s>>>(a);
    } else if (etype == 1) {
        if (ns) upts_kernel<T, 1, true><<<grid, block, 0, s>>>(a);
        else upts_kernel<T, 1, false><<<grid, block, 0, s>>>(a);
    } else {
        if (ns) upts_kernel<T, 2, true><<<grid, block, 0, s>>>(a);
        else upts_kernel<T, 2, false><<<grid, block, 0, s>>>(a);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_common_solution(const PairArgs<T> &a, hipStream_t s) {
    if (!a.npairs) return hipSuccess;
    common_solution_kernel<T><<<unsigned((a.npairs + 255) / 256), 256, 0, s>>>(a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_common_flux(bool ns, const PairArgs<T> &a, hipStream_t s) {
    if (!a.npairs) return hipSuccess;
    const unsigned g = unsigned((a.npairs + 255) / 256);
    if (ns) common_flux_kernel<T, true><<<g, 256, 0, s>>>(a);
    else common_flux_kernel<T, false><<<g, 256, 0, s>>>(a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_boundary_solution(const BndArgs<T> &a, hipStream_t s) {
    if (!a.nb) return hipSuccess;
    boundary_solution_kernel<T><<<unsigned((a.nb + 255) / 256), 256, 0, s>>>(a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_boundary_flux(bool ns, const BndArgs<T> &a, hipStream_t s) {
    if (!a.nb) return hipSuccess;
    const unsigned g = unsigned((a.nb + 255) / 256);
    if (ns) boundary_flux_kernel<T, true><<<g, 256, 0, s>>>(a);
    else boundary_flux_kernel<T, false><<<g, 256, 0, s>>>(a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_negdivconf(int etype, const NegArgs<T> &a, hipStream_t s) {
    const dim3 grid(unsigned((a.nelem + 255) / 256), unsigned(a.nu)), block(256);
    if (etype == 0) negdivconf_kernel<T, 0><<<grid, block, 0, s>>>(a);
    else if (etype == 1) negdivconf_kernel<T, 1><<<grid, block, 0, s>>>(a);
    else negdivconf_kernel<T, 2><<<grid, block, 0, s>>>(a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_reduce(const RedArgs<T> &a, hipStream_t s) {
    reduce_kernel<T><<<RED_BLOCKS, 256, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_reduce_final(const double *partial, int nblocks, double *out, hipStream_t s) {
    reduce_final_kernel<<<8, 256, 0, s>>>(partial, nblocks, out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_copy(T *dst, const T *src, int64_t n, hipStream_t s) {
    if (!n) return hipSuccess;
    copy_kernel<T><<<1024, 256, 0, s>>>(dst, src, n);
    return hipGetLastError();
}

#define FR_INSTANTIATE(T)                                                                     \
    template hipError_t launch_opmul<T>(int, const Op<T> &, const T *, int64_t, int,          \
                                        const T *, int64_t, int, T *, int64_t, int64_t,       \
                                        hipStream_t, const NegArgs<T> *);                     \
    template hipError_t launch_upts<T>(int, bool, const UptsArgs<T> &, hipStream_t);          \
    template hipError_t launch_common_solution<T>(const PairArgs<T> &, hipStream_t);          \
    template hipError_t launch_common_flux<T>(bool, const PairArgs<T> &, hipStream_t);        \
    template hipError_t launch_boundary_solution<T>(const BndArgs<T> &, hipStream_t);         \
    template hipError_t launch_boundary_flux<T>(bool, const BndArgs<T> &, hipStream_t);       \
    template hipError_t launch_negdivconf<T>(int, const NegArgs<T> &, hipStream_t);           \
    template hipError_t launch_reduce<T>(const RedArgs<T> &, hipStream_t);                    \
    template hipError_t launch_copy<T>(T *, const T *, int64_t, hipStream_t);

FR_INSTANTIATE(float)
FR_INSTANTIATE(double)

}  // namespace frd
