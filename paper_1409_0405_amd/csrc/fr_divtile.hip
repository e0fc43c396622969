// Divergence stage of the right-hand side on tiles of elements (gfx950).
//
// Paper, Section 2.1: the last operator product of an FR step and the
// point-wise work around it.  The separate kernels pass three arrays through
// memory here: the transformed flux Ft at the solution points (Euler: from
// the point-wise kernel), and, between two Runge-Kutta stages, the next
// stage's input, which the interpolation to the flux points reads back.  One
// workgroup takes a tile of NE elements with all five fields:
//   1. the volume part [G'_0 G'_1 G'_2] Ft.  Euler: Ft = adj F(U) -> LDS,
//      evaluated from the state (15 values per point that never reach
//      memory), and its product on the matrix cores.  For Navier-Stokes the
//      fused gradient stage has left it in memory as D, five values per point
//      instead of fifteen, and the sums start from it;
//   2. the common normal flux Fn -> LDS, Rt = volume part + L Fn -> LDS;
//   3. -Rt / J and the Runge-Kutta register update on 16-byte rows (element
//      by element where the learned closure adds its correction);
//   4. inside a time step, U_f = M0 r of the state r just written (the next
//      stage's input, still in LDS) -> memory, so the next stage needs no
//      interpolation kernel.
// The operators are walked in the K order of the product kernels (gathered
// layout), and the update is the shared one, so every value has the bits of
// the separate kernels.
//
// What bounds it: memory.  At p = 4, FP32, Navier-Stokes inside a step, 196,608
// tets take 264 us and 110,592 prisms 294 us, about 4 TB/s of the arrays named
// above (the card copies at 4.9); the separate divergence and interpolation
// products take 246 + 90 and 360 + 111 us and have Ft, three times D, to read.
// What the volume part costs in the gradient stage is told there.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fr_device.hpp"
#include "fr_opmul.hpp"
#include "fr_pointwise.hpp"
#include "fr_tile.hpp"

namespace frd {
namespace {

// U_f = M0 U for the tile in LDS: wavefront w takes items w, w + NW, ... (row
// block, every NH-th column block); walk and frow hold the first one's.
template <typename T, int NE, int NBI, int NW>
__device__ __forceinline__ void interp_items(const Op<T> &M, const T *Bs, T *Uf, int64_t ld, int64_t e0, int64_t nelem,
                                             int w, int lane, GatherWalk<T> &walk, int (&frow)[4]) {
    using v4 = typename Vec4<T>::type;
    constexpr int WS = tile_stride<NE>(), NH = TileShape<NE>::NB / NBI;
    const int krow = lane >> 4, c16 = lane & 15;
    for (int it = w; it < M.nmg * NH; it += NW) {
        const int g = it / NH, h = it - NH * g;
        v4 af[NBI];
#pragma unroll
        for (int i = 0; i < NBI; ++i) af[i] = v4{0, 0, 0, 0};
        if (it != w) {
            block_rows(M, g, krow, frow);
            walk = GatherWalk<T>(M, g, lane);
        }
        gather_products<NH>(walk, Bs + 16 * h + c16, WS, af);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (frow[r] < 0) continue;
            T *u = Uf + int64_t(frow[r]) * 5 * ld + e0;
#pragma unroll
            for (int i = 0; i < NBI; ++i) {
                const TileColumn<NE> c(NH * i + h, c16);
                if (e0 + c.e < nelem) u[c.v * ld + c.e] = af[i][r];
            }
        }
    }
}

// A workgroup of NW wavefronts takes NE elements.  NBI column blocks make a
// work item (row block, every (NB / NBI)-th column block); MI: items of the
// divergence product per wavefront, whose accumulators stay in registers
// until every wavefront has read B.
//
// Euler: Ft and Fn take turns in LDS, so a tile needs the larger of the two
// (Fn travels in registers while G' Ft is multiplied): at p = 3 a prism tile
// of 16 elements needs 38 KB instead of 61 KB and four workgroups share a CU.
// Order 3, FP32, 13,824 prisms and 24,576 tets: 92.0 -> 76.2 us for the right-hand side.
// The register bounds keep two workgroups of eight wavefronts (FP32) on a CU.
// (a by value: by reference the compiler reads it again around every store,
// 76.4 -> 82.7 us for the order-3 right-hand side above.)
template <typename T, int ET, int NE, int NBI, int NW, int MI, bool EULER>
__device__ __forceinline__ void divtile(const DivTileArgs<T> a, int64_t e0, unsigned char *lds_raw) {
    using v4 = typename Vec4<T>::type;
    constexpr int W5 = TileShape<NE>::W5, WS = tile_stride<NE>(), NB = W5 / 16, NH = NB / NBI;
    static_assert(W5 == 5 * NE && NB % NBI == 0, "whole column blocks");
    constexpr int NG = n_geom_coeffs<ET>(), V = 16 / int(sizeof(T)), VPR = NE / V;
    const int nu = a.nu, nf = a.nf;
    T *Bs = reinterpret_cast<T *>(lds_raw);              // [divtile_rows][WS]
    T *Gs = Bs + size_t(EULER ? max(3 * nu, nf) : max(nf, nu)) * WS;   // Euler: [NG][NE] Jacobian coefficients
    T *Xs = Gs + NG * NE;                                // Euler: [nu][3] reference coordinates

    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int krow = lane >> 4, c16 = lane & 15;
    const int64_t ld = a.ld;

    // Fn: straight into LDS (Navier-Stokes); the first FR 16-byte pieces per
    // thread into registers (Euler; the piece's row, field and position in it)
    constexpr int FR = NW == 16 ? 2 : NW == 8 ? 5 : 6;
    floatx4 fr[EULER ? FR : 1];
    auto piece = [&](int c, int &dst) -> const T * {
        const int row = c / (5 * VPR), q = c - row * (5 * VPR);
        dst = row * WS + V * q;
        return a.Fn + (int64_t(row) * 5 + q / VPR) * ld + e0 + V * (q % VPR);
    };
    // the first PT solution points of this thread (Euler)
    constexpr int PT = NW == 16 ? 1 : 2;
    T u[EULER ? PT : 1][5];
    auto load_points = [&](int base) {
#pragma unroll
        for (int q = 0; q < PT; ++q) {
            const int it = base + q * 64 * NW + tid, i = it / NE, e = it - i * NE;
            if (it < nu * NE && e0 + e < a.nelem) {
#pragma unroll
                for (int v = 0; v < 5; ++v) u[q][v] = a.U[(int64_t(i) * 5 + v) * ld + e0 + e];
            }
        }
    };
    if constexpr (EULER) {
        if (!a.padj)
            for (int base = w * 64; base < NG * VPR; base += NW * 64) {
                const int c = base + lane;
                if (c < NG * VPR)
                    load_lds16(a.geom + int64_t(c / VPR) * ld + e0 + V * (c % VPR), Gs + size_t(base) * V);
            }
        for (int idx = tid; idx < 3 * nu; idx += 64 * NW) Xs[idx] = a.xi[idx];
        load_points(0);
    } else {
        tile_to_lds<T, NE, NW>(a.Fn, ld, e0, nf, Bs, w, lane);
    }
    v4 acc[MI][NBI];
    int rrow[MI][4];
#pragma unroll
    for (int m = 0; m < MI; ++m) {
        const int it = w + m * NW, g = it / NH, h = it - NH * g;
        block_rows(a.A, g, krow, rrow[m]);
#pragma unroll
        for (int i = 0; i < NBI; ++i) {
            acc[m][i] = v4{0, 0, 0, 0};
            if constexpr (!EULER) {
                // (rows past the last are read as row 0: their sums are not used)
                const TileColumn<NE> c(NH * i + h, c16);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[m][i][r] = a.D[(int64_t(max(rrow[m][r], 0)) * 5 + c.v) * ld + e0 + c.e];
            }
        }
    }
    // what this thread's first item of the update reads (J and the registers)
    // and the first product item's operator steps travel with the tile
    // (Euler: with Fn's product)
    constexpr int Q = NE / 4;
    UpdateIn<T, v4> up;
    auto first_update = [&] {
        const int64_t eg = e0 + 4 * (tid % Q);
        if (tid < nu * 5 * Q && update4_whole(a.ep, eg)) update4_load(a.ep, tid / Q / 5, eg, int64_t(tid / Q) * ld + eg, up);
    };
    if constexpr (!EULER) first_update();
    GatherWalk<T> walk(a.A, (EULER ? 2 : 1) * min(w / NH, a.A.nmg - 1), lane);
    if constexpr (EULER) {
        // 1. Ft = adj F(U) -> LDS
        __builtin_amdgcn_s_waitcnt(0);                   // this wavefront's direct loads are in LDS
        __syncthreads();
#pragma unroll
        for (int m = 0; m < FR; ++m) {
            const int c = tid + m * 64 * NW;
            int dst;
            if (c < nf * 5 * VPR) fr[m] = *reinterpret_cast<const floatx4 *>(piece(c, dst));
        }
        for (int base = 0; base < nu * NE; base += PT * 64 * NW) {
            if (base > 0) load_points(base);
#pragma unroll
            for (int q = 0; q < PT; ++q) {
                const int it = base + q * 64 * NW + tid, i = it / NE, e = it - i * NE;
                const int64_t eg = e0 + e;
                if (it >= nu * NE || eg >= a.nelem) continue;   // padding columns mix with no other
                T adj[3][3], Ft[3][5];
                if (a.padj) {
#pragma unroll
                    for (int k = 0; k < 3; ++k)
#pragma unroll
                        for (int j = 0; j < 3; ++j) adj[k][j] = a.padj[(int64_t(3 * k + j) * nu + i) * ld + eg];
                } else {
                    metric<T, ET>(Gs, NE, e, Xs + 3 * i, adj);
                }
                upts_flux<T, false>(u[q], nullptr, adj, a.gamma, T(0), T(1), a.pref, Ft);
#pragma unroll
                for (int k = 0; k < 3; ++k)
#pragma unroll
                    for (int v = 0; v < 5; ++v) Bs[(k * nu + i) * WS + v * NE + e] = Ft[k][v];
            }
        }
    } else {
        __builtin_amdgcn_s_waitcnt(0);
    }
    __syncthreads();

    // 2. Rt: wavefront w takes items w, w + NW, ... (Euler: first G' Ft, then
    // L Fn on the same accumulators)
    auto product = [&](int part) {
#pragma unroll
        for (int m = 0; m < MI; ++m) {
            const int it = w + m * NW, g = it / NH, h = it - NH * g;
            if (g < a.A.nmg) {
                if (m > 0 || part > 0) walk = GatherWalk<T>(a.A, (EULER ? 2 : 1) * g + part, lane);
                gather_products<NH>(walk, Bs + 16 * h + c16, WS, acc[m]);
            }
        }
    };
    product(0);
    if constexpr (EULER) {
        __syncthreads();                                 // every wavefront is done with Ft
#pragma unroll
        for (int m = 0; m < FR; ++m) {
            const int c = tid + m * 64 * NW;
            int dst;
            piece(c, dst);
            if (c < nf * 5 * VPR) *reinterpret_cast<floatx4 *>(Bs + dst) = fr[m];
        }
        for (int c = tid + FR * 64 * NW; c < nf * 5 * VPR; c += 64 * NW) {
            int dst;
            const T *src = piece(c, dst);
            *reinterpret_cast<floatx4 *>(Bs + dst) = *reinterpret_cast<const floatx4 *>(src);
        }
        first_update();
        __syncthreads();
        product(1);
    }
    __syncthreads();                                     // every wavefront is done with B
#pragma unroll
    for (int m = 0; m < MI; ++m) {
        const int h = (w + m * NW) % NH;
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
    for (int idx = tid; idx < nu * 5 * Q; idx += 64 * NW) {
        const int q = idx % Q, iv = idx / Q, v = iv % 5, i = iv / 5;
        v4 *p = reinterpret_cast<v4 *>(Bs + i * WS + v * NE + 4 * q);
        const int64_t eg = e0 + 4 * q, o0 = int64_t(iv) * ld + eg;
        v4 r;
        if (update4_whole(a.ep, eg)) {
            if (idx != tid) update4_load(a.ep, i, eg, o0, up);
            r = update4(a.ep, eg, o0, *p, up);
        } else {
            r = update4_tail(a.ep, i, v, eg, o0, *p);
        }
        if (a.Uf) *p = r;
    }
    if (!a.Uf) return;
    __syncthreads();

    // 4. U_f = M0 r
    interp_items<T, NE, NBI, NW>(a.M, Bs, a.Uf, ld, e0, a.nelem, w, lane, walk, frow);
}

// U_f = M0 U of a tile: the interpolation of a right-hand side's or a step's
// first stage.
template <typename T, int NE, int NBI, int NW>
__device__ __forceinline__ void interptile(const InterpTileArgs<T> a, int64_t e0, unsigned char *lds_raw) {
    constexpr int NH = TileShape<NE>::NB / NBI;
    T *Bs = reinterpret_cast<T *>(lds_raw);              // [nu][tile_stride]
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    tile_to_lds<T, NE, NW>(a.U, a.ld, e0, a.nu, Bs, w, lane);
    int frow[4];
    block_rows(a.M, w / NH, lane >> 4, frow);
    GatherWalk<T> walk(a.M, min(w / NH, a.M.nmg - 1), lane);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    interp_items<T, NE, NBI, NW>(a.M, Bs, a.Uf, a.ld, e0, a.nelem, w, lane, walk, frow);
}

template <typename T, int ET, int NE, int NBI, int NW, int MI, bool EULER>
__global__ __launch_bounds__(64 * NW, sizeof(T) == 4 ? NW == 4 ? 3 : 4 : 2) void divtile_kernel(DivTileArgs<T> a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int64_t e0 = int64_t(xcd_block()) * NE;
    if (e0 < a.nelem)                                    // (whole workgroup: padding of the grid)
        divtile<T, ET, NE, NBI, NW, MI, EULER>(a, e0, lds_raw);
}
template <typename T, int NE, int NBI, int NW>
__global__ __launch_bounds__(64 * NW) void interptile_kernel(InterpTileArgs<T> a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int64_t e0 = int64_t(xcd_block()) * NE;
    if (e0 < a.nelem) interptile<T, NE, NBI, NW>(a, e0, lds_raw);
}

// Small meshes: one launch for the tiles of every type.
template <typename T, int MI, bool EULER>
__global__ __launch_bounds__(1024, sizeof(T) == 4 ? 4 : 2) void divtile_small_kernel(PerType<DivTileArgs<T>> a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    small_tile(a, [&](auto et, const DivTileArgs<T> &x, int64_t e0) {
        divtile<T, decltype(et)::value, 16, 1, 16, MI, EULER>(x, e0, lds_raw);
    });
}
template <typename T>
__global__ __launch_bounds__(1024) void interptile_small_kernel(PerType<InterpTileArgs<T>> a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    small_tile(a, [&](auto, const InterpTileArgs<T> &x, int64_t e0) { interptile<T, 16, 1, 16>(x, e0, lds_raw); });
}

template <typename T>
size_t tile_bytes(int rows, int ne) {
    return size_t(rows) * (ne == 32 ? 176 : 5 * ne) * sizeof(T);
}

template <typename T>
size_t divtile_bytes(int etype, const DivTileArgs<T> &a, bool euler, int ne) {
    const int ng = etype == 0 ? 9 : etype == 1 ? 15 : 21;
    return tile_bytes<T>(euler ? std::max(3 * a.nu, a.nf) : std::max(a.nf, a.nu), ne) +
           (euler ? size_t(ng) * ne + 3 * size_t(a.nu) : 0) * sizeof(T);
}

// Elements per workgroup (0: the shape does not fit).  Rows of 32 elements
// (FP32) move 128 bytes per access, but only where two workgroups fit a CU,
// so that one loads while the other multiplies; else 16.
template <typename T>
int divtile_elems(int etype, const DivTileArgs<T> &a, bool euler) {
    if (sizeof(T) == 4 && divtile_bytes(etype, a, euler, 32) <= TILE_LDS_MAX / 2) return 32;
    return divtile_bytes(etype, a, euler, 16) <= TILE_LDS_MAX ? 16 : 0;
}

template <typename T, int ET, int NE, int NBI, int NW, int MI, bool EULER>
hipError_t launch_dt(const DivTileArgs<T> &a, hipStream_t s) {
    static LdsLimit limit;
    const auto kernel = divtile_kernel<T, ET, NE, NBI, NW, MI, EULER>;
    if (hipError_t e = limit.raise(kernel); e != hipSuccess) return e;
    kernel<<<xcd_grid((a.nelem + NE - 1) / NE), 64 * NW, divtile_bytes(ET, a, EULER, NE), s>>>(a);
    return hipGetLastError();
}

}  // namespace
// (More than six row blocks, hexahedra of order 4, keep eight wavefronts busy
// without the split by column blocks: 512 of them, 57.3 against 54.9 us for a
// right-hand side.)
template <typename T>
bool divtile_small(const DivTileArgs<T> &a) {
    return narrow_mesh(a.nelem) && a.A.nmg <= 6;
}
namespace {

template <typename T, int ET, bool EULER>
hipError_t launch_dt_et(const DivTileArgs<T> &a, hipStream_t s) {
    const int nmg = a.A.nmg;
    if (divtile_small(a)) {
        if (nmg * 5 <= 16) return launch_dt<T, ET, 16, 1, 16, 1, EULER>(a, s);
        return launch_dt<T, ET, 16, 1, 16, 2, EULER>(a, s);
    }
    // four wavefronts where the divergence product has at most four items
    // (row block, five column blocks), else eight with up to two items each
    const int ne = divtile_elems<T>(ET, a, EULER);
    if constexpr (sizeof(T) == 4) {
        if (ne == 32) {
            if (nmg * 2 <= 4) return launch_dt<T, ET, 32, 5, 4, 1, EULER>(a, s);
            if (nmg * 2 <= 8) return launch_dt<T, ET, 32, 5, 8, 1, EULER>(a, s);
            if (nmg * 2 <= 16) return launch_dt<T, ET, 32, 5, 8, 2, EULER>(a, s);
        }
    }
    if (ne == 16) {
        if (nmg <= 4) return launch_dt<T, ET, 16, 5, 4, 1, EULER>(a, s);
        if (nmg <= 8) return launch_dt<T, ET, 16, 5, 8, 1, EULER>(a, s);
        if (nmg <= 16) return launch_dt<T, ET, 16, 5, 8, 2, EULER>(a, s);
    }
    return hipErrorInvalidValue;
}

template <typename T, int NE, int NBI, int NW>
hipError_t launch_it(const InterpTileArgs<T> &a, hipStream_t s) {
    static LdsLimit limit;
    const auto kernel = interptile_kernel<T, NE, NBI, NW>;
    if (hipError_t e = limit.raise(kernel); e != hipSuccess) return e;
    kernel<<<xcd_grid((a.nelem + NE - 1) / NE), 64 * NW, tile_bytes<T>(a.nu, NE), s>>>(a);
    return hipGetLastError();
}

// Launch of a small-mesh kernel over the tiles of the types present.
template <typename K, typename A, typename Bytes>
hipError_t launch_small(K *kernel, LdsLimit &limit, const A *const a[3], Bytes bytes, hipStream_t s) {
    if (hipError_t e = limit.raise(kernel); e != hipSuccess) return e;
    PerType<A> p;
    size_t lds = 0;
    int64_t ntiles = 0;
    for (int t = 0; t < 3; ++t) {
        if (!a[t]) continue;
        p.a[t] = *a[t];
        ntiles += (a[t]->nelem + 15) / 16;
        lds = std::max(lds, bytes(t));
    }
    if (!ntiles) return hipSuccess;
    kernel<<<unsigned(ntiles), 1024, lds, s>>>(p);
    return hipGetLastError();
}

template <typename T, int MI, bool EULER>
hipError_t launch_dt_small(const DivTileArgs<T> *const a[3], hipStream_t s) {
    static LdsLimit limit;
    return launch_small(divtile_small_kernel<T, MI, EULER>, limit, a,
                        [&](int t) { return divtile_bytes(t, *a[t], EULER, 16); }, s);
}

bool aligned16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

}  // namespace

template <typename T>
bool divtile_supported(int etype, const DivTileArgs<T> &a, bool euler) {
    return divtile_elems<T>(etype, a, euler) > 0;
}

namespace {
template <typename T>
bool valid_args(const DivTileArgs<T> &a, bool euler) {
    return gathered(a.A, a.nu) && a.A.parts == (euler ? 2 : 1) && gathered(a.M, a.nf) && a.M.parts == 1 &&
           a.ld % 64 == 0 && a.nelem <= a.ld && a.ep.ld == a.ld && a.ep.nelem == a.nelem && a.ep.nu == a.nu &&
           a.ep.jinv && a.Fn && (euler ? a.U != nullptr : a.D != nullptr) && aligned16(a.Fn) && aligned16(a.geom);
}
template <typename T>
bool valid_args(const InterpTileArgs<T> &a) {
    return gathered(a.M, a.M.M) && a.M.parts == 1 && a.ld % 64 == 0 && a.nelem <= a.ld && a.U && a.Uf &&
           aligned16(a.U);
}
}  // namespace

template <typename T>
hipError_t launch_divtile_small(bool euler, const DivTileArgs<T> *const a[3], hipStream_t s) {
    int nmg = 1, ntypes = 0, et = 0;
    for (int t = 0; t < 3; ++t) {
        if (!a[t]) continue;
        if (!valid_args(*a[t], euler) || !divtile_small(*a[t]) || divtile_bytes(t, *a[t], euler, 16) > TILE_LDS_MAX)
            return hipErrorInvalidValue;
        nmg = std::max(nmg, a[t]->A.nmg);
        ++ntypes;
        et = t;
    }
    // (one type alone: without the choice of the type, ten RK4 steps of 1,296
    // tets, FP64, took 477 instead of 496 us)
    if (ntypes == 1) return launch_divtile(et, euler, *a[et], s);
    if (nmg * 5 <= 16) return euler ? launch_dt_small<T, 1, true>(a, s) : launch_dt_small<T, 1, false>(a, s);
    return euler ? launch_dt_small<T, 2, true>(a, s) : launch_dt_small<T, 2, false>(a, s);
}

template <typename T>
hipError_t launch_divtile(int etype, bool euler, const DivTileArgs<T> &a, hipStream_t s) {
    if (!valid_args(a, euler)) return hipErrorInvalidValue;
    if (!a.nelem) return hipSuccess;
    if (etype == 0) return euler ? launch_dt_et<T, 0, true>(a, s) : launch_dt_et<T, 0, false>(a, s);
    if (etype == 1) return euler ? launch_dt_et<T, 1, true>(a, s) : launch_dt_et<T, 1, false>(a, s);
    return euler ? launch_dt_et<T, 2, true>(a, s) : launch_dt_et<T, 2, false>(a, s);
}

template <typename T>
bool interptile_small(const InterpTileArgs<T> &a) {
    return narrow_mesh(a.nelem);
}

template <typename T>
hipError_t launch_interptile_small(const InterpTileArgs<T> *const a[3], hipStream_t s) {
    static LdsLimit limit;
    for (int t = 0; t < 3; ++t)
        if (a[t] && (!valid_args(*a[t]) || !interptile_small(*a[t]) || tile_bytes<T>(a[t]->nu, 16) > TILE_LDS_MAX))
            return hipErrorInvalidValue;
    return launch_small(interptile_small_kernel<T>, limit, a, [&](int t) { return tile_bytes<T>(a[t]->nu, 16); }, s);
}

template <typename T>
hipError_t launch_interptile(const InterpTileArgs<T> &a, hipStream_t s) {
    if (interptile_small(a)) {
        const InterpTileArgs<T> *p[3] = {&a, nullptr, nullptr};   // (the type plays no part)
        return launch_interptile_small(p, s);
    }
    if (!valid_args(a)) return hipErrorInvalidValue;
    if constexpr (sizeof(T) == 4) {
        if (tile_bytes<T>(a.nu, 32) <= TILE_LDS_MAX / 2) {
            if (a.M.nmg <= 2) return launch_it<T, 32, 5, 4>(a, s);
            return launch_it<T, 32, 5, 8>(a, s);
        }
    }
    if (tile_bytes<T>(a.nu, 16) > TILE_LDS_MAX) return hipErrorInvalidValue;
    if (a.M.nmg <= 4) return launch_it<T, 16, 5, 4>(a, s);
    return launch_it<T, 16, 5, 8>(a, s);
}

#define FR_DIVTILE_INSTANCES(T)                                                                              \
    template bool divtile_supported<T>(int, const DivTileArgs<T> &, bool);                                   \
    template bool divtile_small<T>(const DivTileArgs<T> &);                                                  \
    template hipError_t launch_divtile<T>(int, bool, const DivTileArgs<T> &, hipStream_t);                   \
    template hipError_t launch_divtile_small<T>(bool, const DivTileArgs<T> *const[3], hipStream_t);          \
    template bool interptile_small<T>(const InterpTileArgs<T> &);                                            \
    template hipError_t launch_interptile<T>(const InterpTileArgs<T> &, hipStream_t);                        \
    template hipError_t launch_interptile_small<T>(const InterpTileArgs<T> *const[3], hipStream_t);
FR_DIVTILE_INSTANCES(float)
FR_DIVTILE_INSTANCES(double)

}  // namespace frd
