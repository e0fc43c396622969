// Divergence stage of the right-hand side on tiles of elements (gfx950).
//
// Paper, Section 2.1: the last operator product of an FR step and the
// point-wise work around it.  The separate kernels pass three arrays through
// memory here: the transformed flux Ft at the solution points (Euler: from
// the point-wise kernel), and, between two Runge-Kutta stages, the next
// stage's input, which the interpolation to the flux points reads back.  One
// workgroup takes a tile of NE elements with all five fields:
//   1. B -> LDS: the common normal flux Fn, and for the Euler equations in
//      front of it Ft = adj F(U), evaluated from the state (15 values per
//      point that never reach memory).  For Navier-Stokes the fused gradient
//      stage has left the volume part D = [G'_0 G'_1 G'_2] Ft in memory, five
//      values per point instead of fifteen, and the sums start from it;
//   2. Rt = [G'_k | L] [Ft; Fn] (Navier-Stokes: D + L Fn) on the matrix cores
//      -> LDS;
//   3. -Rt / J and the Runge-Kutta register update on 16-byte rows;
//   4. inside a time step, U_f = M0 r of the state r just written (the next
//      stage's input, still in LDS) -> memory, so the next stage needs no
//      interpolation kernel.
// The operators are walked in the K order of the product kernels (gathered
// layout), and the update is the shared one, so every value has the bits of
// the separate kernels.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fr_device.hpp"
#include "fr_opmul.hpp"
#include "fr_pointwise.hpp"
#include "fr_tile.hpp"

namespace frd {
namespace {

// NE elements per workgroup of NW wavefronts; MI: work items (row block,
// column half) of the divergence product per wavefront, whose accumulators
// stay in registers until every wavefront has read B.  Column block n of half
// h holds field n of elements 16 h .. 16 h + 15, so a lane's accumulators are
// one element's.
template <typename T, int ET, int NE, int NW, int MI, bool EULER>
__global__ __launch_bounds__(64 * NW) void divtile_kernel(DivTileArgs<T> a) {
    using v4 = typename Vec4<T>::type;
    constexpr int W5 = TileShape<NE>::W5, WS = tile_stride<NE>(), NH = W5 / 80, NBI = 5;
    static_assert(W5 == 5 * NE && W5 % 80 == 0, "whole column blocks");
    constexpr int NG = n_geom_coeffs<ET>(), VPR = NE * int(sizeof(T)) / 16;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int nu = a.nu, nf = a.nf, k0 = EULER ? 3 * nu : 0;
    T *Bs = reinterpret_cast<T *>(lds_raw);              // [max(k0 + nf, nu)][WS]
    T *Gs = Bs + size_t(max(k0 + nf, nu)) * WS;          // Euler: [NG][NE] Jacobian coefficients
    T *Xs = Gs + NG * NE;                                // Euler: [nu][3] reference coordinates

    const int64_t e0 = int64_t(xcd_block()) * NE;
    if (e0 >= a.nelem) return;                           // whole workgroup: padding of the grid
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int krow = lane >> 4, c16 = lane & 15;
    const int64_t ld = a.ld;

    // 1. B
    tile_to_lds<T, NE, NW>(a.Fn, ld, e0, nf, Bs + size_t(k0) * WS, w, lane);
    v4 acc[MI][NBI];
    int rrow[MI][4];
#pragma unroll
    for (int m = 0; m < MI; ++m) {
        const int it = w + m * NW, g = it / NH, h = it - NH * g;
        block_rows(a.A, g, krow, rrow[m]);
#pragma unroll
        for (int i = 0; i < NBI; ++i) acc[m][i] = v4{0, 0, 0, 0};
        if constexpr (!EULER) {
            // (rows past the last are read as row 0: their sums are not used)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const T *d = a.D + int64_t(max(rrow[m][r], 0)) * 5 * ld + e0 + 16 * h + c16;
#pragma unroll
                for (int i = 0; i < NBI; ++i) acc[m][i][r] = d[i * ld];
            }
        }
    }
    // what this thread's first PU items of the update read (J and the
    // registers), on its way while the tile is loaded and multiplied
    constexpr int Q = NE / 4, PU = 1;
    UpdateIn<T, v4> up[PU];
#pragma unroll
    for (int m = 0; m < PU; ++m) {
        const int idx = tid + m * 64 * NW, q = idx % Q, iv = idx / Q;
        const int64_t eg = e0 + 4 * q;
        if (idx < nu * 5 * Q && update4_whole(a.ep, eg)) update4_load(a.ep, iv / 5, eg, int64_t(iv) * ld + eg, up[m]);
    }
    // (the first item's operator steps travel with the tile)
    GatherWalk<T> walk(a.A, min(w / NH, a.A.nmg - 1), lane);
    if constexpr (EULER) {
        if (!a.padj)
            for (int base = w * 64; base < NG * VPR; base += NW * 64) {
                const int c = base + lane;
                if (c < NG * VPR)
                    load_lds16(a.geom + int64_t(c / VPR) * ld + e0 + (16 / sizeof(T)) * (c % VPR),
                               Gs + size_t(base) * (16 / sizeof(T)));
            }
        for (int idx = tid; idx < 3 * nu; idx += 64 * NW) Xs[idx] = a.xi[idx];
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        for (int it = tid; it < nu * NE; it += 64 * NW) {
            const int i = it / NE, e = it - i * NE;
            const int64_t eg = e0 + e;
            if (eg >= a.nelem) continue;                 // padding columns mix with no other
            T u[5], adj[3][3], Ft[3][5];
#pragma unroll
            for (int v = 0; v < 5; ++v) u[v] = a.U[(int64_t(i) * 5 + v) * ld + eg];
            if (a.padj) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int j = 0; j < 3; ++j) adj[k][j] = a.padj[(int64_t(3 * k + j) * nu + i) * ld + eg];
            } else {
                metric<T, ET>(Gs, NE, e, Xs + 3 * i, adj);
            }
            upts_flux<T, false>(u, nullptr, adj, a.gamma, T(0), T(1), a.pref, Ft);
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int v = 0; v < 5; ++v) Bs[(k * nu + i) * WS + v * NE + e] = Ft[k][v];
        }
    } else {
        __builtin_amdgcn_s_waitcnt(0);                   // this wavefront's direct loads are in LDS
    }
    __syncthreads();

    // 2. Rt: wavefront w takes items w, w + NW, ...
#pragma unroll
    for (int m = 0; m < MI; ++m) {
        const int it = w + m * NW, g = it / NH, h = it - NH * g;
        if (g < a.A.nmg) {
            if (m > 0) walk = GatherWalk<T>(a.A, g, lane);
            gather_products<NH>(walk, Bs + 16 * h + c16, WS, acc[m]);
        }
    }
    __syncthreads();                                     // every wavefront is done with B
#pragma unroll
    for (int m = 0; m < MI; ++m) {
        const int it = w + m * NW, h = it % NH;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (rrow[m][r] >= 0) {
#pragma unroll
                for (int i = 0; i < NBI; ++i) Bs[rrow[m][r] * WS + 16 * (NH * i + h) + c16] = acc[m][i][r];
            }
    }
    // (the interpolation's first operator steps travel during the update)
    int frow[4];
    block_rows(a.M, w / NH, krow, frow);
    walk = GatherWalk<T>(a.M, min(w / NH, a.M.nmg - 1), lane);
    __syncthreads();

    // 3. the last pipeline step, four elements of one (point, field) at a time
    auto update = [&](int idx, const UpdateIn<T, v4> &x) {
        const int q = idx % Q, iv = idx / Q, v = iv % 5, i = iv / 5;
        v4 *p = reinterpret_cast<v4 *>(Bs + i * WS + v * NE + 4 * q);
        const int64_t eg = e0 + 4 * q, o0 = int64_t(iv) * ld + eg;
        const v4 r = update4_whole(a.ep, eg) ? update4(a.ep, eg, o0, *p, x) : update4_tail(a.ep, i, v, eg, o0, *p);
        if (a.Uf) *p = r;
    };
#pragma unroll
    for (int m = 0; m < PU; ++m) {
        const int idx = tid + m * 64 * NW;
        if (idx < nu * 5 * Q) update(idx, up[m]);
    }
    for (int idx = tid + PU * 64 * NW; idx < nu * 5 * Q; idx += 64 * NW) {
        const int64_t eg = e0 + 4 * (idx % Q);
        UpdateIn<T, v4> x;
        if (update4_whole(a.ep, eg)) update4_load(a.ep, idx / Q / 5, eg, int64_t(idx / Q) * ld + eg, x);
        update(idx, x);
    }
    if (!a.Uf) return;
    __syncthreads();

    // 4. U_f = M0 r: items (row block, column half)
    for (int it = w; it < a.M.nmg * NH; it += NW) {
        const int g = it / NH, h = it - NH * g;
        v4 af[NBI];
#pragma unroll
        for (int i = 0; i < NBI; ++i) af[i] = v4{0, 0, 0, 0};
        if (it != w) {
            block_rows(a.M, g, krow, frow);
            walk = GatherWalk<T>(a.M, g, lane);
        }
        gather_products<NH>(walk, Bs + 16 * h + c16, WS, af);
        const int64_t eg = e0 + 16 * h + c16;
        if (eg >= a.nelem) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (frow[r] < 0) continue;
            T *u = a.Uf + int64_t(frow[r]) * 5 * ld + eg;
#pragma unroll
            for (int i = 0; i < NBI; ++i) u[i * ld] = af[i][r];
        }
    }
}

template <typename T>
size_t divtile_bytes(int etype, const DivTileArgs<T> &a, bool euler, int ne) {
    const int ws = ne == 32 ? 176 : 5 * ne, ng = etype == 0 ? 9 : etype == 1 ? 15 : 21;
    return (size_t(std::max((euler ? 3 * a.nu : 0) + a.nf, a.nu)) * ws + (euler ? size_t(ng) * ne + 3 * size_t(a.nu) : 0)) * sizeof(T);
}

// Elements per workgroup (0: the shape does not fit).  Rows of 32 elements
// (FP32) move 128 bytes per access, but only where two workgroups fit a CU,
// so that one loads while the other multiplies; else 16.
template <typename T>
int divtile_elems(int etype, const DivTileArgs<T> &a, bool euler) {
    if (sizeof(T) == 4 && divtile_bytes(etype, a, euler, 32) <= TILE_LDS_MAX / 2) return 32;
    return divtile_bytes(etype, a, euler, 16) <= TILE_LDS_MAX ? 16 : 0;
}

template <typename T, int ET, int NE, int NW, int MI, bool EULER>
hipError_t launch_dt(const DivTileArgs<T> &a, hipStream_t s) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(divtile_kernel<T, ET, NE, NW, MI, EULER>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(TILE_LDS_MAX));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    divtile_kernel<T, ET, NE, NW, MI, EULER>
        <<<xcd_grid((a.nelem + NE - 1) / NE), 64 * NW, divtile_bytes(ET, a, EULER, NE), s>>>(a);
    return hipGetLastError();
}

// wavefronts per workgroup: four where the divergence product has at most
// four items (row block, column half), else eight, with up to two items each
template <typename T, int ET, int NE, bool EULER>
hipError_t launch_dt_nw(const DivTileArgs<T> &a, hipStream_t s) {
    const int items = a.A.nmg * (5 * NE / 80);
    if (items <= 4) return launch_dt<T, ET, NE, 4, 1, EULER>(a, s);
    if (items <= 8) return launch_dt<T, ET, NE, 8, 1, EULER>(a, s);
    if (items <= 16) return launch_dt<T, ET, NE, 8, 2, EULER>(a, s);
    return hipErrorInvalidValue;
}

template <typename T, int ET>
hipError_t launch_dt_et(bool euler, const DivTileArgs<T> &a, hipStream_t s) {
    const int ne = divtile_elems<T>(ET, a, euler);
    if constexpr (sizeof(T) == 4) {
        if (ne == 32) return euler ? launch_dt_nw<T, ET, 32, true>(a, s) : launch_dt_nw<T, ET, 32, false>(a, s);
    }
    if (ne == 16) return euler ? launch_dt_nw<T, ET, 16, true>(a, s) : launch_dt_nw<T, ET, 16, false>(a, s);
    return hipErrorInvalidValue;
}

bool aligned16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

}  // namespace

template <typename T>
bool divtile_supported(int etype, const DivTileArgs<T> &a, bool euler) {
    return divtile_elems<T>(etype, a, euler) > 0;
}

template <typename T>
hipError_t launch_divtile(int etype, bool euler, const DivTileArgs<T> &a, hipStream_t s) {
    if (!gathered(a.A, a.nu) || !gathered(a.M, a.nf) || a.ld % 64 || a.nelem > a.ld || a.ep.ld != a.ld || a.ep.nelem != a.nelem ||
        a.ep.nu != a.nu || !a.ep.jinv || !a.Fn || (euler ? !a.U : !a.D) || !aligned16(a.Fn) || !aligned16(a.geom))
        return hipErrorInvalidValue;
    if (!a.nelem) return hipSuccess;
    if (etype == 0) return launch_dt_et<T, 0>(euler, a, s);
    if (etype == 1) return launch_dt_et<T, 1>(euler, a, s);
    return launch_dt_et<T, 2>(euler, a, s);
}

template bool divtile_supported<float>(int, const DivTileArgs<float> &, bool);
template bool divtile_supported<double>(int, const DivTileArgs<double> &, bool);
template hipError_t launch_divtile<float>(int, bool, const DivTileArgs<float> &, hipStream_t);
template hipError_t launch_divtile<double>(int, bool, const DivTileArgs<double> &, hipStream_t);

}  // namespace frd
