// Building blocks of the kernels that keep a tile of elements in LDS (the
// fused gradient stage and the divergence stage): direct loads into LDS and
// products of a step-list operator with a tile.
// Internal header (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>

#include "fr_device.hpp"
#include "fr_opmul.hpp"

namespace frd {
namespace {

template <int ET>
constexpr int n_geom_coeffs() { return ET == 0 ? 9 : ET == 1 ? 15 : 21; }

// Entry i of a read-only list through the scalar data cache: the index is
// uniform in the wavefront, and a constant-space load lets the compiler use a
// scalar load, which the vector-memory counter (the operator fragments in
// flight) does not wait for.
template <typename V>
__device__ __forceinline__ V sload(const V *p, int i) {
    return ((const __attribute__((address_space(4))) V *)p)[i];
}

// 16 (4) bytes from memory straight into LDS (global_load_lds): lane l of
// the wavefront writes dst + 16 l (dst + 4 l), dst uniform in the wavefront.
__device__ __forceinline__ void load_lds16(const void *src, void *dst) {
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
}
__device__ __forceinline__ void load_lds4(const void *src, void *dst) {
    __builtin_amdgcn_global_load_lds(src, dst, 4, 0, 0);
}

// Walk of a gathered operator (Op stage 7) over one row block: the K steps of
// the block, each naming the four rows of B that its fragment multiplies.
// The lists are read through the scalar cache four steps at a time and one
// group ahead (both lists have slack at their end, so the walk reads past a
// block without a test), the fragments travel four steps ahead of their use
// and the B values (LDS) one step.
template <typename T>
struct GatherWalk {
    const uint64_t *kl;
    const T *frag;      // this lane's fragment of step 0
    int ns, sel, sh;    // steps; this lane's row of a step: dword sel, bits sh .. sh + 15
    __device__ __forceinline__ GatherWalk(const Op<T> &A, int g, int lane) {
        const int s0 = sload(A.koff, g);
        ns = sload(A.koff, g + 1) - s0;
        kl = reinterpret_cast<const uint64_t *>(A.klist) + s0;
        frag = A.frag + size_t(s0) * 64 + lane;
        sel = lane >> 5;
        sh = 16 * ((lane >> 4) & 1);
    }
    __device__ __forceinline__ int row(uint64_t q) const {
        const unsigned d = sel ? unsigned(q >> 32) : unsigned(q);
        return int((d >> sh) & 0xffffu);
    }
    // for each step in order: load(row, buffer) fills the next step's B
    // values, mul(fragment, buffer) multiplies the current one's
    template <typename Buf, typename Load, typename Mul>
    __device__ __forceinline__ void run(Buf &b0, Buf &b1, Load load, Mul mul) const {
        T a[4];
        uint64_t q[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            a[d] = frag[size_t(d) * 64];
            q[d] = sload(kl, d + 1);
        }
        load(row(sload(kl, 0)), b0);
        for (int st = 0; st < ns; st += 4) {
            uint64_t qn[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) qn[d] = sload(kl, st + d + 5);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                if (st + d >= ns) break;
                load(row(q[d]), b1);
                __builtin_amdgcn_sched_barrier(0);
                mul(a[d], b0);
                __builtin_amdgcn_sched_barrier(0);
                a[d] = frag[size_t(st + d + 4) * 64];
                b0 = b1;
            }
#pragma unroll
            for (int d = 0; d < 4; ++d) q[d] = qn[d];
        }
    }
};

template <typename T, int N>
struct BVals {
    T v[N];
};

// acc[n] += A_g B[:, 16 ST n .. 16 ST n + 15] for row block g of a gathered
// operator; b points at row 0 of B in LDS (rows ws values apart), column
// lane % 16 of the first column block.  The K order is the operator's column
// order, as in the product kernels, and an accumulator that starts at +0 is
// never -0, so the exact-zero products that a step leaves out or adds change
// no bit.
template <typename T, int NB, int ST = 1, typename V4>
__device__ __forceinline__ void gather_products(const Op<T> &A, int g, int lane, const T *b, int ws, V4 (&acc)[NB]) {
    BVals<T, NB> b0, b1;
    GatherWalk<T>(A, g, lane).run(
        b0, b1,
        [&](int row, BVals<T, NB> &x) {
            const T *p = b + row * ws;
#pragma unroll
            for (int n = 0; n < NB; ++n) x.v[n] = p[16 * ST * n];
        },
        [&](T a, const BVals<T, NB> &x) {
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[n] = mfma16(a, x.v[n], acc[n]);
        });
}

// Whether op is a gathered operator of M rows.
template <typename T>
bool gathered(const Op<T> &op, int M) {
    return op.stage == 7 && op.mbw == 1 && op.M == M && op.nmg > 0 && op.frag && op.klist && op.koff && op.rowmap;
}

// Tile of NE elements with all five fields: row r of a tile in LDS holds W5
// columns, (field v, element e) at v NE + e and zeros up to W5; column block
// n of the matrix instructions is columns 16 n .. 16 n + 15.
template <int NE>
struct TileShape {
    static constexpr int W5 = (5 * NE + 15) / 16 * 16;
    static constexpr int NB = W5 / 16;
};

constexpr size_t TILE_LDS_MAX = 160 * 1024;   // LDS of a CU

}  // namespace
}  // namespace frd
