// Fused gradient stage of the Navier-Stokes right-hand side (gfx950).
//
// Paper, Section 2.1: an FR step is operator products C <- A B with the
// element state as B, separated by point-wise work.  Between the common
// solution and the common flux the separate kernels pass three arrays
// through memory: the reference gradient Qt (corrected gradient product),
// the physical gradient Q and the transformed flux Ft (point-wise kernel),
// and Q again (gradient interpolation).  Here one workgroup takes a tile of
// NE elements with all five fields and keeps Qt and Q in LDS:
//   1. B = [U; Cf] of the tile -> LDS;
//   2. Qt = [G_k | L_k] B on the matrix cores -> LDS;
//   3. per (solution point, element): Q = adj^T Qt / J (in place);
//   4. Qf = M0 Q on the matrix cores -> memory, only on the faces whose
//      gradient the interface and boundary kernels read (with the usual LDG
//      weights one side of each interface);
//   5. Ft = adj (F_inv(U) - F_vis(U, Q)) in Q's place;
//   6. the volume part of the divergence, D = [G'_0 G'_1 G'_2] Ft, on the
//      matrix cores -> memory: five values per point for the divergence
//      stage to read instead of the fifteen of Ft.
// Without the divergence stage on tiles (FR_SEPARATE_UPDATE, a forced
// divergence product, the streaming form, or the autotuner found the
// divergence product faster) Ft goes to memory in step 3 and the kernel ends
// with step 4.  The operators are walked in the K order of the product kernels
// (gathered layout, below), and the point-wise arithmetic is the shared one,
// so every value has the bits of the separate kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "fr_device.hpp"
#include "fr_opmul.hpp"
#include "fr_pointwise.hpp"
#include "fr_tile.hpp"

namespace frd {
namespace {

// acc[j][i] += A_g Q_j[:, column block NH i + h] for the row block of a walk
// and all three gradient directions j: one operator fragment feeds 3 NBI
// matrix instructions.  q points at row 0, column 16 h + lane % 16 of Q_0 in
// LDS, Q_j is jstride values further on.
template <int NBI, int NH, int W5, typename T, int AD, typename V4>
__device__ __forceinline__ void interp3_products(GatherWalk<T, AD> &w, const T *q, int jstride, V4 (&acc)[3][NBI]) {
    BVals<T, 3 * NBI> bb[2];
    w.run(
        bb,
        [&](int row, BVals<T, 3 * NBI> &x) {
            const T *p = q + __umul24(row, W5);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int i = 0; i < NBI; ++i) x.v[NBI * j + i] = p[j * jstride + 16 * NH * i];
        },
        [&](T a, const BVals<T, 3 * NBI> &x) {
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int i = 0; i < NBI; ++i) acc[j][i] = mfma16(a, x.v[NBI * j + i], acc[j][i]);
        });
}

// Elements per tile.  The wider the tile, the more matrix instructions each
// operator fragment feeds and the longer the rows that memory accesses move,
// which the measurements favour over more workgroups per CU: FP32 tets and
// prisms take 32 (at p = 4: 74 KB of LDS, two workgroups per CU for tets;
// 161 KB, one workgroup of 16 wavefronts for prisms; 16 elements measured
// 572 -> 653 us and 497 -> 501 us), hexahedra 16 (123 KB), FP64 half of that.
template <typename T, int ET>
constexpr int tile_elems() { return (ET == 2 ? 16 : 32) * 4 / int(sizeof(T)); }

// One workgroup of NW wavefronts per tile.  Work items of the gradient
// product: (row block, every GH-th column block), MG per wavefront; their
// accumulators stay in registers until every wavefront has finished reading
// B, so that Qt takes B's place in LDS and a tile needs max(B, Qt) of it.
// NBI: column blocks per item of the other two products.
// VD: the volume part D = [G'_0 G'_1 G'_2] Ft of the divergence is written
// instead of Ft: Q stays in LDS until it is interpolated, then Ft takes its
// place (phase 5) and is multiplied there (phase 6).
// What bounds it (p = 4, FP32, 196,608 tets and 110,592 prisms: 571 and 492
// us with the volume part): the matrix cores, busy 44 per cent of the time for
// tets, and the waits between the phases; the interpolation's and phase 6's
// first operator steps and row numbers are loaded one phase ahead (tets 595 ->
// 571 us).  With the divergence stage, inside a step, 571 + 264 and 492 + 294
// us; without the volume part and with the fastest divergence and
// interpolation products 466 + 246 + 90 and 397 + 360 + 111 us: the dense
// operators of tets make the volume part dear, so the autotuner takes the
// products for them there, and tiles for prisms.
template <typename T, int ET, int NE, int GH, int NBI, int NW, int MG, bool VD>
__device__ __forceinline__ void gradflux(const GradFluxArgs<T> a, int64_t e0, unsigned char *lds_raw) {
    using v4 = typename Vec4<T>::type;
    constexpr int W5 = TileShape<NE>::W5, NB = TileShape<NE>::NB, WS = tile_stride<NE>();
    constexpr int NG = n_geom_coeffs<ET>();
    constexpr int V = 16 / int(sizeof(T)), VPR = NE / V;   // values per 16 bytes, 16-byte pieces per (row, field)
    const int nu = a.nu, nf = a.nf;
    // one region: B = [U; Cf] ([nu + nf][WS]) for the gradient product, then Qt
    // and, in place, Q and Ft ([3 nu][WS], row k nu + i)
    T *Bs = reinterpret_cast<T *>(lds_raw);
    T *QT = Bs;
    T *Gs = Bs + size_t(max(nu + nf, 3 * nu)) * WS;      // [NG][NE] Jacobian coefficients
    T *Xs = Gs + NG * NE;                                // [nu][3] reference coordinates

    // the wavefront index is uniform in the wavefront: say so, so that the
    // loops branch on scalars
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int krow = lane >> 4, c16 = lane & 15;
    const int64_t ld = a.ld;

    // 1. B rows: U (k < nu), Cf (nu <= k < nu + nf), straight from memory into
    // LDS (no registers, every load of the tile in flight before the one wait)
    tile_to_lds<T, NE, NW>(a.U, ld, e0, nu, Bs, w, lane);
    tile_to_lds<T, NE, NW>(a.Cf, ld, e0, nf, Bs + size_t(nu) * WS, w, lane);
    if (!a.padj)
        for (int base = w * 64; base < NG * VPR; base += NW * 64) {
            const int c = base + lane;
            if (c < NG * VPR) load_lds16(a.geom + int64_t(c / VPR) * ld + e0 + V * (c % VPR), Gs + size_t(base) * V);
        }
    for (int idx = tid; idx < 3 * nu; idx += 64 * NW) Xs[idx] = a.xi[idx];
    if constexpr (WS == W5 && W5 > 5 * NE)               // unused columns of the last block
        for (int idx = tid; idx < (nu + nf) * (W5 - 5 * NE); idx += 64 * NW)
            Bs[(idx / (W5 - 5 * NE)) * WS + 5 * NE + idx % (W5 - 5 * NE)] = T(0);

    // 2. Qt = [G_k | L_k] B: wavefront w takes items w, w + NW, ... (row block,
    // every GH-th column block)
    constexpr int NBG = NB / GH;
    static_assert(NB % GH == 0 && NB % NBI == 0, "whole column blocks");
    v4 acc[MG][NBG];
    int qrow[MG][4];
#pragma unroll
    for (int m = 0; m < MG; ++m) block_rows(a.G, (w + m * NW) / GH, krow, qrow[m]);
    __builtin_amdgcn_s_waitcnt(0);                       // this wavefront's direct loads are in LDS
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MG; ++m) {
#pragma unroll
        for (int n = 0; n < NBG; ++n) acc[m][n] = v4{0, 0, 0, 0};
        const int g = (w + m * NW) / GH, h = (w + m * NW) % GH;
        if (g < a.G.nmg) {
            GatherWalk<T> gwalk(a.G, g, lane);
            gather_products<GH>(gwalk, Bs + 16 * h + c16, WS, acc[m]);
        }
    }
    // the states of this thread's first PI points of the point-wise phase,
    // from B while it is still in LDS (at p = 4 three cover every point of
    // an FP32 tet or prism tile)
    constexpr int PI = sizeof(T) == 4 && ET < 2 ? 3 : 2;
    T uu[PI][5];
    if constexpr (!VD) {
#pragma unroll
        for (int q = 0; q < PI; ++q) {
            const int it = q * 64 * NW + tid;
            const int i = it / NE, e = it - i * NE;
            if (it < nu * NE) {
#pragma unroll
                for (int v = 0; v < 5; ++v) uu[q][v] = Bs[i * WS + v * NE + e];
            }
        }
    }
    __syncthreads();                                     // every wavefront is done with B
#pragma unroll
    for (int m = 0; m < MG; ++m) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = qrow[m][r];
            if (row >= 0) {
#pragma unroll
                for (int n = 0; n < NBG; ++n)
                    QT[row * WS + 16 * (GH * n + (w + m * NW) % GH) + c16] = acc[m][n][r];
            }
        }
    }
    // the interpolation's work items: (row block g, part h of the column
    // blocks) with the three directions together, so an operator fragment
    // feeds 3 NBI matrix instructions; the first item's operator steps, flux
    // points and faces are on their way during the point-wise phase
    constexpr int NH = NB / NBI;
    const int nit = a.M.nmg * NH;
    int frow[4];
    unsigned fb[4];
    auto item_rows = [&](int it) {
        block_rows(a.M, it / NH, krow, frow);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            fb[r] = a.qmask ? unsigned(a.fbit[16 * min(it / NH, a.M.nmg - 1) + acc_row<T>(krow, r)]) : 1u;
    };
    item_rows(w);
    GatherWalk<T> mwalk(a.M, min(w, nit - 1) / NH, lane);
    __syncthreads();

    // the metric of point i and element e of the tile: the adjugate, returns 1 / J
    auto point_metric = [&](int i, int e, T (&adj)[3][3]) -> T {
        if (!a.padj) return T(1) / metric<T, ET>(Gs, NE, e, Xs + 3 * i, adj);
        // (the metric is waited for inside this branch: left in flight, it
        // would make the straight elements wait at the join, and with it for
        // the previous point's stores)
        const int64_t eg = e0 + e;
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) adj[k][j] = a.padj[(int64_t(3 * k + j) * nu + i) * ld + eg];
        const T Jinv = a.pjinv[int64_t(i) * ld + eg];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < 3; ++j) adj[k][j] = opaque(adj[k][j]);
        return opaque(Jinv);
    };
    // the 15 values of a point in LDS (Qt, Q or Ft)
    auto point_read = [&](int i, int e, T (&x)[3][5]) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) x[k][v] = QT[(k * nu + i) * WS + v * NE + e];
    };
    auto point_write = [&](int i, int e, const T (&x)[3][5]) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int v = 0; v < 5; ++v) QT[(k * nu + i) * WS + v * NE + e] = x[k][v];
    };
    // the states of this thread's points base + q 64 NW + tid, from memory
    // (L2 serves them)
    auto load_states = [&](int base) {
#pragma unroll
        for (int q = 0; q < PI; ++q) {
            const int it = base + q * 64 * NW + tid;
            const int i = it / NE, e = it - i * NE;
            if (it < nu * NE && e0 + e < a.nelem) {
#pragma unroll
                for (int v = 0; v < 5; ++v) uu[q][v] = a.U[(int64_t(i) * 5 + v) * ld + e0 + e];
            }
        }
    };

    // 3. point-wise: one (solution point, element) per thread; Q replaces Qt
    // in place
    if constexpr (VD) {
        for (int it = tid; it < nu * NE; it += 64 * NW) {
            const int i = it / NE, e = it - i * NE;
            if (e0 + e >= a.nelem) continue;
            T adj[3][3], qt[3][5], q3[3][5];
            const T Jinv = point_metric(i, e, adj);
            point_read(i, e, qt);
            upts_gradient(qt, adj, Jinv, q3);
            point_write(i, e, q3);
        }
    } else {
        // and Ft goes to memory.  A thread's first PI states came from B
        // above; further ones (B's place in LDS holds Qt now) come again from
        // memory, PI points at a time, so that no load queues behind the Ft
        // stores of the points before it (memory operations of a wavefront
        // retire in order).
        for (int base = 0; base < nu * NE; base += PI * 64 * NW) {
            if (base > 0) load_states(base);
#pragma unroll
            for (int q = 0; q < PI; ++q) {
                const int it = base + q * 64 * NW + tid;
                const int i = it / NE, e = it - i * NE;
                const int64_t eg = e0 + e;
                if (it >= nu * NE || eg >= a.nelem) continue;
                T adj[3][3], qt[3][5], q3[3][5], Ft[3][5];
                const T Jinv = point_metric(i, e, adj);
                point_read(i, e, qt);
                upts_point<T, true>(uu[q], qt, adj, Jinv, a.gamma, a.mu, a.prandtl, a.pref, q3, Ft);
                point_write(i, e, q3);
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int v = 0; v < 5; ++v) a.Ft[((int64_t(k) * nu + i) * 5 + v) * ld + eg] = Ft[k][v];
            }
        }
    }
    __syncthreads();

    // 4. Qf = M0 Q for the three gradient directions, stored only on the faces
    // of an element whose gradient is read (qm of this lane's elements; none
    // past the last element)
    constexpr int NQ = NE >= 16 ? NE / 16 : 1;
    unsigned qm[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        const int64_t eg = e0 + (16 * n + c16) % NE;
        qm[n] = eg >= a.nelem ? 0u : a.qmask ? unsigned(a.qmask[eg]) : 0xffu;
    }
    v4 acc3[3][NBI];
    auto zero3 = [&]() {
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int i = 0; i < NBI; ++i) acc3[j][i] = v4{0, 0, 0, 0};
    };
    auto store3 = [&](int it) {
        const int h = it % NH;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (frow[r] < 0) continue;
            T *qf = a.Qf + int64_t(frow[r]) * 15 * ld + e0;
            if constexpr (NE >= 16 && NBI == 5) {
                const TileColumn<NE> c(h, c16);
                if (!(qm[h] & fb[r])) continue;
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int i = 0; i < NBI; ++i) qf[(j * 5 + i) * ld + c.e] = acc3[j][i][r];
            } else {
#pragma unroll
                for (int i = 0; i < NBI; ++i) {
                    const TileColumn<NE> c(NH * i + h, c16);
                    if (c.v >= 5 || !(qm[(NH * i + h) % NQ] & fb[r])) continue;
#pragma unroll
                    for (int j = 0; j < 3; ++j) qf[(j * 5 + c.v) * ld + c.e] = acc3[j][i][r];
                }
            }
        }
    };
    int it4 = w;
    zero3();
    if (it4 < nit) {
        interp3_products<NBI, NH, WS>(mwalk, QT + 16 * (it4 % NH) + c16, nu * WS, acc3);
        for (; it4 + NW < nit; it4 += NW) {
            store3(it4);
            zero3();
            item_rows(it4 + NW);
            mwalk = GatherWalk<T>(a.M, (it4 + NW) / NH, lane);
            interp3_products<NBI, NH, WS>(mwalk, QT + 16 * ((it4 + NW) % NH) + c16, nu * WS, acc3);
        }
    }
    if constexpr (!VD) {
        if (it4 < nit) store3(it4);
        return;
    }
    // (phase 6's first operator steps, ahead of the last Qf stores)
    constexpr int ND = NBI, DH = NH;
    const int ndt = a.V.nmg * DH;
    GatherWalk<T> vwalk(a.V, min(w, ndt - 1) / DH, lane);
    if (it4 < nit) store3(it4);
    __syncthreads();                                     // every wavefront is done with Q

    // 5. Ft takes the place of Q
    for (int base = 0; base < nu * NE; base += PI * 64 * NW) {
        load_states(base);
#pragma unroll
        for (int q = 0; q < PI; ++q) {
            const int it = base + q * 64 * NW + tid;
            const int i = it / NE, e = it - i * NE;
            if (it >= nu * NE || e0 + e >= a.nelem) continue;
            T adj[3][3], q3[3][5], Ft[3][5];
            point_metric(i, e, adj);
            point_read(i, e, q3);
            upts_flux<T, true>(uu[q], q3, adj, a.gamma, a.mu, a.prandtl, a.pref, Ft);
            point_write(i, e, Ft);
        }
    }
    __syncthreads();

    // 6. D = [G'_k] Ft: items (row block, part of the column blocks)
    for (int it = w; it < ndt; it += NW) {
        const int g = it / DH, h = it - DH * g;
        int drow[4];
        block_rows(a.V, g, krow, drow);
        v4 accd[ND];
#pragma unroll
        for (int n = 0; n < ND; ++n) accd[n] = v4{0, 0, 0, 0};
        if (it != w) vwalk = GatherWalk<T>(a.V, g, lane);
        gather_products<DH>(vwalk, QT + 16 * h + c16, WS, accd);
#pragma unroll
        for (int n = 0; n < ND; ++n) {
            const TileColumn<NE> c(DH * n + h, c16);
            if (c.v >= 5 || e0 + c.e >= a.nelem) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (drow[r] >= 0) a.D[(int64_t(drow[r]) * 5 + c.v) * ld + e0 + c.e] = accd[n][r];
        }
    }
}

template <typename T, int ET, int NE, int GH, int NBI, int NW, int MG, bool VD>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void gradflux_kernel(GradFluxArgs<T> a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int64_t e0 = int64_t(xcd_block()) * NE;
    if (e0 < a.nelem)                                    // (whole workgroup: padding of the grid)
        gradflux<T, ET, NE, GH, NBI, NW, MG, VD>(a, e0, lds_raw);
}

// Small meshes: one launch for the tiles of every type, one column block per
// item over 16 wavefronts (FP64: 8, whose point-wise work needs more than 128
// registers).
template <typename T>
constexpr int small_waves() { return sizeof(T) == 4 ? 16 : 8; }
template <typename T, int MG>
__global__ __launch_bounds__(64 * small_waves<T>()) void gradflux_small_kernel(PerType<GradFluxArgs<T>> a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    small_tile(a, [&](auto et, const GradFluxArgs<T> &x, int64_t e0) {
        gradflux<T, decltype(et)::value, 16, 5, 1, small_waves<T>(), MG, true>(x, e0, lds_raw);
    });
}

// Streaming form (FP32): a workgroup takes a contiguous run of tiles and,
// while it works on one, the next tile's B = [U; Cf] and Jacobian
// coefficients travel straight from memory into a second LDS buffer
// (global_load_lds: no registers, no wait until the tile starts), so the
// matrix cores do not sit idle on the loads.  LDS: Qt / Q [3 nu][80], B
// [Kp][80], two geometry buffers, reference coordinates.  Same arithmetic,
// same bits as gradflux_kernel.
template <int ET, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(ET == 0 ? 4 : 2))) void gradflux_stream_kernel(GradFluxArgs<float> a, int tiles_per_wg) {
    using v4 = floatx4;
    constexpr int NE = 16, W5 = 80, NB = 5;
    constexpr int NG = n_geom_coeffs<ET>();
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int nu = a.nu, nf = a.nf;
    float *QT = reinterpret_cast<float *>(lds_raw);      // [3 nu][W5]
    float *Bs = QT + size_t(3 * nu) * W5;                // [nu + nf][W5]
    float *Gs = Bs + size_t(nu + nf) * W5;               // [2][NG][NE]
    float *Xs = Gs + 2 * NG * NE;                        // [nu][3]

    const int64_t ntiles = (a.nelem + NE - 1) / NE;
    const int64_t t_begin = int64_t(xcd_block()) * tiles_per_wg;
    const int64_t t_end = min(t_begin + tiles_per_wg, ntiles);
    if (t_begin >= t_end) return;                        // whole workgroup
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int krow = lane >> 4, c16 = lane & 15;
    const int64_t ld = a.ld;

    for (int idx = tid; idx < 3 * nu; idx += 64 * NW) Xs[idx] = a.xi[idx];

    // B and the coefficients of tile `tile` into LDS: chunk c (16 bytes) of
    // B is row k, field v, elements 4 q .. 4 q + 3 with c = 4 (5 k + v) + q;
    // lane l of a wavefront instruction writes chunk base + l
    auto issue = [&](int64_t tile, float *gdst) {
        const int64_t e0 = tile * NE;
        const int nchunk = (nu + nf) * 5 * 4;
        for (int base = w * 64; base < nchunk; base += NW * 64) {
            const int c = base + lane, q = c & 3, kv = c >> 2, v = kv % 5, k = kv / 5;
            if (c < nchunk) {
                const float *src = k < nu ? a.U + (int64_t(k) * 5 + v) * ld + e0 + 4 * q
                                          : a.Cf + (int64_t(k - nu) * 5 + v) * ld + e0 + 4 * q;
                __builtin_amdgcn_global_load_lds(src, Bs + size_t(base) * 4, 16, 0, 0);
            }
        }
        if (!a.padj && w == NW - 1) {
            // NG rows of 16 coefficients: 4 NG chunks, one instruction
            const int c = lane, g = c >> 2, q = c & 3;
            if (c < 4 * NG) __builtin_amdgcn_global_load_lds(a.geom + int64_t(g) * ld + e0 + 4 * q, gdst, 16, 0, 0);
        }
    };
    issue(t_begin, Gs);
    int buf = 0;
    for (int64_t tile = t_begin; tile < t_end; ++tile, buf ^= 1) {
        const int64_t e0 = tile * NE;
        float *G = Gs + buf * NG * NE;
        __builtin_amdgcn_s_waitcnt(0);                   // this wavefront's direct loads (and stores) are done
        __syncthreads();                                 // everyone's: B and G of this tile are in LDS

        // 1. Qt = [G_k | L_k] B -> LDS
        for (int g = w; g < a.G.nmg; g += NW) {
            v4 acc[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[n] = v4{0, 0, 0, 0};
            GatherWalk<float> walk(a.G, g, lane);
            gather_products(walk, Bs + c16, W5, acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = a.G.rowmap[16 * g + acc_row<float>(krow, r)];
                if (row >= 0) {
#pragma unroll
                    for (int n = 0; n < NB; ++n) QT[row * W5 + 16 * n + c16] = acc[n][r];
                }
            }
        }
        __syncthreads();                                 // B is free, Qt complete
        if (tile + 1 < t_end) issue(tile + 1, Gs + (buf ^ 1) * NG * NE);

        // 2. point-wise: Q replaces Qt in place, Ft to memory
        for (int it = tid; it < nu * NE; it += 64 * NW) {
            const int i = it / NE, e = it - i * NE;
            const int64_t eg = e0 + e;
            if (eg >= a.nelem) continue;
            float adj[3][3], Jinv;
            if (a.padj) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int j = 0; j < 3; ++j) adj[k][j] = a.padj[(int64_t(3 * k + j) * nu + i) * ld + eg];
                Jinv = a.pjinv[int64_t(i) * ld + eg];
            } else {
                Jinv = 1.0f / metric<float, ET>(G, NE, e, Xs + 3 * i, adj);
            }
            float u[5], qt[3][5], q[3][5], Ft[3][5];
#pragma unroll
            for (int v = 0; v < 5; ++v) u[v] = a.U[(int64_t(i) * 5 + v) * ld + eg];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int v = 0; v < 5; ++v) qt[k][v] = QT[(k * nu + i) * W5 + v * NE + e];
            upts_point<float, true>(u, qt, adj, Jinv, a.gamma, a.mu, a.prandtl, a.pref, q, Ft);
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int v = 0; v < 5; ++v) QT[(j * nu + i) * W5 + v * NE + e] = q[j][v];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int v = 0; v < 5; ++v) a.Ft[((int64_t(k) * nu + i) * 5 + v) * ld + eg] = Ft[k][v];
        }
        __syncthreads();

        // 3. Qf = M0 Q (the faces whose gradient is read, as above)
        const unsigned qm = a.qmask ? unsigned(a.qmask[e0 + c16]) : 0xffu;
        for (int it = w; it < a.M.nmg * 3; it += NW) {
            const int g = it / 3, j = it - 3 * g;
            const float *Qj = QT + size_t(j) * nu * W5 + c16;
            v4 acc2[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n) acc2[n] = v4{0, 0, 0, 0};
            GatherWalk<float> walk(a.M, g, lane);
            gather_products(walk, Qj, W5, acc2);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int slot = 16 * g + acc_row<float>(krow, r), f = a.M.rowmap[slot];
                if (f < 0 || e0 + c16 >= a.nelem || (a.qmask && !(qm & a.fbit[slot]))) continue;
#pragma unroll
                for (int n = 0; n < NB; ++n) a.Qf[(int64_t(f) * 15 + j * 5 + n) * ld + e0 + c16] = acc2[n][r];
            }
        }
        // the next iteration's barrier keeps Qt of the next tile from
        // overwriting Q while it is read here
    }
}


template <typename T, int ET, int NE>
size_t gradflux_bytes(const GradFluxArgs<T> &a) {
    return (size_t(std::max(a.nu + a.nf, 3 * a.nu)) * tile_stride<NE>() + size_t(n_geom_coeffs<ET>()) * NE +
            size_t(3 * a.nu)) * sizeof(T);
}

template <typename T, int ET, int NE, int GH, int NBI, int NW, int MG, bool VD>
hipError_t launch_gf_mg(const GradFluxArgs<T> &a, hipStream_t s) {
    static LdsLimit limit;
    const auto kernel = gradflux_kernel<T, ET, NE, GH, NBI, NW, MG, VD>;
    if (hipError_t e = limit.raise(kernel); e != hipSuccess) return e;
    const int64_t ntiles = (a.nelem + NE - 1) / NE;
    kernel<<<xcd_grid(ntiles), 64 * NW, gradflux_bytes<T, ET, NE>(a), s>>>(a);
    return hipGetLastError();
}

template <typename T, int ET, bool VD>
hipError_t launch_gf(const GradFluxArgs<T> &a, hipStream_t s) {
    const int nmg = a.G.nmg;
    constexpr int NE = tile_elems<T, ET>(), NB = TileShape<NE>::NB, NBI = NB % 5 == 0 ? 5 : NB;
    // wavefronts per workgroup (row blocks of the gradient operator at p = 4:
    // tets 7, prisms 15, hexahedra 25): FP32 8, 16 and 16; FP64, whose
    // accumulators are twice as large, 4, 8 and 8
    constexpr int NW = (ET == 0 ? 8 : 16) * 4 / int(sizeof(T));
    // (next to the divergence stage on tiles only)
    if constexpr (VD) {
        // Low orders: the gradient operator has few row blocks, so they are also
        // split by column blocks (FP32 in two, FP64 in five), and a workgroup has
        // only as many wavefronts as that gives work to.  Times of this kernel
        // before -> after: order 1, FP32, 82,944 tets 52 -> 34 us, 46,080 prisms
        // 54 -> 29 us; order 2, 79 -> 62 and 85 -> 68 us; 13,824 hexahedra, order
        // 1, 34 -> 16 us, order 2, 47 -> 30 us; FP64, order 1, prisms 103 -> 70
        // us, hexahedra 48 -> 29 us, order 2, prisms 168 -> 146 us (but tets 84
        // -> 88 us and 150 -> 169 us: FP64 tets stay with whole row blocks).
        if constexpr (sizeof(T) == 4) {
            if (ET < 2 || gradflux_bytes<T, ET, 32>(a) <= TILE_LDS_MAX / 2) {
                if (nmg <= 2) return launch_gf_mg<T, ET, 32, 2, 5, 4, 1, VD>(a, s);
                if (nmg <= 4) return launch_gf_mg<T, ET, 32, 2, 5, 8, 1, VD>(a, s);
                if constexpr (ET == 2)
                    if (nmg <= 8) return launch_gf_mg<T, ET, 32, 1, 5, 8, 1, VD>(a, s);
            }
        } else if (ET > 0 && gradflux_bytes<T, ET, 16>(a) <= TILE_LDS_MAX / 2) {
            if (nmg <= 2) return launch_gf_mg<T, ET, 16, 5, 5, 4, 3, VD>(a, s);
            if (nmg <= 4) return launch_gf_mg<T, ET, 16, 5, 5, 4, 5, VD>(a, s);
        }
    }
    const int mg = (nmg + NW - 1) / NW;
    if (mg <= 1) return launch_gf_mg<T, ET, NE, 1, NBI, NW, 1, VD>(a, s);
    if constexpr (sizeof(T) == 8 || ET == 2)
        if (mg <= 2) return launch_gf_mg<T, ET, NE, 1, NBI, NW, 2, VD>(a, s);
    if constexpr (sizeof(T) == 8 && ET == 2)
        if (mg <= 4) return launch_gf_mg<T, ET, NE, 1, NBI, NW, 4, VD>(a, s);
    return hipErrorInvalidValue;
}

template <typename T, int ET>
hipError_t launch_gf_et(const GradFluxArgs<T> &a, hipStream_t s) {
    return a.D ? launch_gf<T, ET, true>(a, s) : launch_gf<T, ET, false>(a, s);
}

size_t gradflux_stream_lds_bytes(int etype, const GradFluxArgs<float> &a) {
    const int ng = etype == 0 ? 9 : 15;
    return (size_t(3 * a.nu) * 80 + size_t(a.nu + a.nf) * 80 + 2 * size_t(ng) * 16 + size_t(3 * a.nu)) * 4;
}

template <int ET, int NW>
hipError_t launch_gf_stream(const GradFluxArgs<float> &a, size_t lds, hipStream_t s) {
    static LdsLimit limit;
    hipError_t e = limit.raise(gradflux_stream_kernel<ET, NW>);
    int dev = 0, ncu = 0;
    if (e == hipSuccess) e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    // as many workgroups as fit at once (LDS-bound), each a contiguous run of tiles
    const int per_cu = std::max(1, int(TILE_LDS_MAX / lds));
    const int64_t ntiles = (a.nelem + 15) / 16;
    int64_t nwg = std::min<int64_t>(ntiles, int64_t(ncu) * per_cu);
    const int tiles_per_wg = int((ntiles + nwg - 1) / nwg);
    nwg = (ntiles + tiles_per_wg - 1) / tiles_per_wg;
    gradflux_stream_kernel<ET, NW><<<xcd_grid(nwg), 64 * NW, lds, s>>>(a, tiles_per_wg);
    return hipGetLastError();
}

}  // namespace

namespace {
template <typename T, int ET>
size_t gradflux_lds_t(const GradFluxArgs<T> &a) {
    const size_t bytes = gradflux_bytes<T, ET, tile_elems<T, ET>()>(a);
    return bytes <= TILE_LDS_MAX ? bytes : 0;
}
}  // namespace

template <typename T>
size_t gradflux_lds(int etype, const GradFluxArgs<T> &a) {
    return etype == 0 ? gradflux_lds_t<T, 0>(a) : etype == 1 ? gradflux_lds_t<T, 1>(a)
                                                : etype == 2 ? gradflux_lds_t<T, 2>(a) : 0;
}

namespace {
template <typename T>
bool valid_args(const GradFluxArgs<T> &a) {
    return gathered(a.G, 3 * a.nu) && gathered(a.M, a.nf) && (!a.D || gathered(a.V, a.nu)) && a.ld % 64 == 0 &&
           a.nelem <= a.ld &&
           (reinterpret_cast<uintptr_t>(a.U) | reinterpret_cast<uintptr_t>(a.Cf) |
            reinterpret_cast<uintptr_t>(a.geom)) % 16 == 0;   // 16-byte direct loads into LDS
}

template <typename T>
size_t gradflux_small_bytes(int etype, const GradFluxArgs<T> &a) {
    return etype == 0 ? gradflux_bytes<T, 0, 16>(a) : etype == 1 ? gradflux_bytes<T, 1, 16>(a)
                                                                 : gradflux_bytes<T, 2, 16>(a);
}

template <typename T, int MG>
hipError_t launch_gf_small(const PerType<GradFluxArgs<T>> &p, int64_t ntiles, size_t lds, hipStream_t s) {
    static LdsLimit limit;
    if (hipError_t e = limit.raise(gradflux_small_kernel<T, MG>); e != hipSuccess) return e;
    gradflux_small_kernel<T, MG><<<unsigned(ntiles), 64 * small_waves<T>(), lds, s>>>(p);
    return hipGetLastError();
}
}  // namespace

// Next to the divergence stage on tiles only.  A right-hand side of 2,058
// tets and 1,176 prisms at order 4: 87 -> 54 us.  Hexahedra with more than
// eight row blocks (orders 3 and 4) keep the tiles of 16 elements and 16
// wavefronts of larger meshes, whose items are full (order 3, 256 tiles: 25
// against 31 us).
template <typename T>
bool gradflux_small(int etype, const GradFluxArgs<T> &a) {
    return a.D && narrow_mesh(a.nelem) && a.G.nmg <= (etype == 2 ? 8 : 16) &&
           gradflux_small_bytes(etype, a) <= TILE_LDS_MAX;
}

template <typename T>
hipError_t launch_gradflux_small(const GradFluxArgs<T> *const a[3], hipStream_t s) {
    PerType<GradFluxArgs<T>> p;
    size_t lds = 0;
    int64_t ntiles = 0;
    int nmg = 1;
    for (int t = 0; t < 3; ++t) {
        if (!a[t]) continue;
        if (!valid_args(*a[t]) || !gradflux_small(t, *a[t])) return hipErrorInvalidValue;
        p.a[t] = *a[t];
        ntiles += (a[t]->nelem + 15) / 16;
        lds = std::max(lds, gradflux_small_bytes(t, *a[t]));
        nmg = std::max(nmg, a[t]->G.nmg);
    }
    if (!ntiles) return hipSuccess;
    constexpr int F = 16 / small_waves<T>();             // five items per row block
    if (nmg <= 3) return launch_gf_small<T, F>(p, ntiles, lds, s);
    if (nmg <= 9) return launch_gf_small<T, 3 * F>(p, ntiles, lds, s);
    return launch_gf_small<T, 5 * F>(p, ntiles, lds, s);
}

template <typename T>
hipError_t launch_gradflux(int etype, const GradFluxArgs<T> &a, hipStream_t s, bool stream) {
    size_t lds = gradflux_lds<T>(etype, a);
    if constexpr (std::is_same<T, float>::value) {
        if (stream) {
            if (etype > 1) return hipErrorInvalidValue;   // the streaming form covers tets and prisms
            lds = gradflux_stream_lds_bytes(etype, a);
            if (lds > TILE_LDS_MAX) return hipErrorInvalidValue;
        }
    } else {
        if (stream) return hipErrorInvalidValue;
    }
    if (!lds || !valid_args(a) || (a.D && stream)) return hipErrorInvalidValue;
    if (!a.nelem) return hipSuccess;
    if (gradflux_small(etype, a) && !stream) {
        const GradFluxArgs<T> *p[3] = {nullptr, nullptr, nullptr};
        p[etype] = &a;
        return launch_gradflux_small(p, s);
    }
    if constexpr (std::is_same<T, float>::value) {
        if (stream) return etype == 0 ? launch_gf_stream<0, 8>(a, lds, s) : launch_gf_stream<1, 8>(a, lds, s);
    }
    if (etype == 0) return launch_gf_et<T, 0>(a, s);
    if (etype == 1) return launch_gf_et<T, 1>(a, s);
    return launch_gf_et<T, 2>(a, s);
}

template size_t gradflux_lds<float>(int, const GradFluxArgs<float> &);
template size_t gradflux_lds<double>(int, const GradFluxArgs<double> &);
template bool gradflux_small<float>(int, const GradFluxArgs<float> &);
template bool gradflux_small<double>(int, const GradFluxArgs<double> &);
template hipError_t launch_gradflux_small<float>(const GradFluxArgs<float> *const[3], hipStream_t);
template hipError_t launch_gradflux_small<double>(const GradFluxArgs<double> *const[3], hipStream_t);
template hipError_t launch_gradflux<float>(int, const GradFluxArgs<float> &, hipStream_t, bool);
template hipError_t launch_gradflux<double>(int, const GradFluxArgs<double> &, hipStream_t, bool);

}  // namespace frd
