// Building blocks of the kernels that keep a tile of elements in LDS (the
// fused gradient stage and the divergence stage): direct loads into LDS and
// products of a gathered operator with a tile.
// Internal header (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

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

// f(0), f(1), ..., f(N - 1) with the index as a compile-time constant
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<N, I + 1>(f);
    }
}

// 16 bytes from memory straight into LDS (global_load_lds): lane l of the
// wavefront writes dst + 16 l, dst uniform in the wavefront.
__device__ __forceinline__ void load_lds16(const void *src, void *dst) {
    __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
}

// One lane's share of a step of a gathered operator (Op stage 7): its
// fragment value and the row of B it multiplies, loaded together.
template <typename T>
struct GatherStep {
    T a;
    int row;
};

// Walk of a gathered operator over one row block (with two parts: list 2 g + part).  The first AD steps are
// loaded when the walk is made (before a barrier or a wait that comes
// anyway), later ones AD steps ahead of their use; the B values (LDS) one
// step ahead.  The loop has no exit between its steps, so the compiler counts
// the loads in flight instead of waiting for all of them, and the lane's rows
// come with the fragments: read through the scalar cache, their loads shared
// the counter of the LDS reads and every step waited for both.
template <typename T, int AD = 4>
struct GatherWalk {
    static_assert(AD % 2 == 0, "two B buffers take turns");
    using Step = GatherStep<T>;
    const Step *p;
    int ns;
    Step s[AD];
    __device__ __forceinline__ GatherWalk(const Op<T> &A, int g, int lane) {
        const int s0 = sload(A.koff, g);
        ns = sload(A.koff, g + 1) - s0;
        p = reinterpret_cast<const Step *>(A.frag) + size_t(s0) * 64 + lane;
#pragma unroll
        for (int d = 0; d < AD; ++d) s[d] = p[size_t(d) * 64];
    }
    // load(row, buffer) fills the B values of a step, mul(fragment, buffer)
    // multiplies them; steps in order.  Reads up to AD steps past the block
    // (the lists have slack).
    template <typename Buf, typename Load, typename Mul>
    __device__ __forceinline__ void run(Buf (&b)[2], Load load, Mul mul) {
#pragma unroll
        for (int d = 0; d < AD; ++d) {
            s[d].a = opaque(s[d].a);
            s[d].row = opaque(s[d].row);
        }
        load(s[0].row, b[0]);
        auto step = [&](auto dc, int st) {
            constexpr int d = decltype(dc)::value;
            load(s[(d + 1) % AD].row, b[(d + 1) % 2]);
            __builtin_amdgcn_sched_barrier(0);
            mul(s[d].a, b[d % 2]);
            __builtin_amdgcn_sched_barrier(0);
            s[d] = p[size_t(st + d + AD) * 64];
        };
        int st = 0;
        for (; st + AD <= ns; st += AD) unrolled<AD>([&](auto dc) { step(dc, st); });
        unrolled<AD - 1>([&](auto dc) {
            if (st + decltype(dc)::value < ns) step(dc, st);
        });
    }
};

template <typename T, int N>
struct BVals {
    T v[N];
};

// acc[n] += A_g B[:, 16 ST n .. 16 ST n + 15] for the row block of a walk; b
// points at row 0 of B in LDS (rows ws values apart), column lane % 16 of the
// first column block.  The K order is the operator's column order, as in the
// product kernels, and an accumulator that starts at +0 is never -0, so the
// exact-zero products that a step leaves out or adds change no bit.
template <int ST = 1, typename T, int AD, int NB, typename V4>
__device__ __forceinline__ void gather_products(GatherWalk<T, AD> &w, const T *b, int ws, V4 (&acc)[NB]) {
    BVals<T, NB> bb[2];
    w.run(
        bb,
        [&](int row, BVals<T, NB> &x) {
            const T *p = b + __umul24(row, ws);
#pragma unroll
            for (int n = 0; n < NB; ++n) x.v[n] = p[16 * ST * n];
        },
        [&](T a, const BVals<T, NB> &x) {
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[n] = mfma16(a, x.v[n], acc[n]);
        });
}

// The operator rows of this lane's accumulator elements in row block g (-1:
// none), and -1 for a block past the operator's last.
template <typename T>
__device__ __forceinline__ void block_rows(const Op<T> &A, int g, int krow, int (&row)[4]) {
    const int gc = min(g, A.nmg - 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) row[r] = A.rowmap[16 * gc + acc_row<T>(krow, r)];
#pragma unroll
    for (int r = 0; r < 4; ++r) row[r] = g < A.nmg ? row[r] : -1;
}

// Whether op is a gathered operator of M rows.
template <typename T>
bool gathered(const Op<T> &op, int M) {
    return op.stage == 7 && op.mbw == 1 && op.M == M && op.nmg > 0 && op.parts > 0 && op.frag && op.koff && op.rowmap;
}

// Tile of NE elements with all five fields: row r of a tile in LDS holds W5
// columns, (field v, element e) at v NE + e and zeros up to W5; column block
// n of the matrix instructions is columns 16 n .. 16 n + 15.
template <int NE>
struct TileShape {
    static constexpr int W5 = (5 * NE + 15) / 16 * 16;
    static constexpr int NB = W5 / 16;
};

// Column block n of a tile, lane c16, is field v of element e: with at least
// 16 elements, block NH i + h is field i of elements 16 h .. 16 h + 15.
template <int NE>
struct TileColumn {
    int v, e;
    __device__ __forceinline__ TileColumn(int n, int c16) {
        constexpr int NH = NE >= 16 ? NE / 16 : 1;
        const int flat = 16 * n + c16;
        v = NE >= 16 ? n / NH : flat / NE;
        e = NE >= 16 ? 16 * (n % NH) + c16 : flat - v * NE;
    }
};

// Row stride of a tile in LDS.  A matrix instruction reads B at four
// consecutive rows and 16 columns: with 80 values per row (tiles of 16) the
// four rows fall into different banks, with 160 (tiles of 32) rows two apart
// would share theirs, so those rows are 16 values longer.
template <int NE>
constexpr int tile_stride() { return NE == 32 ? 176 : TileShape<NE>::W5; }

// Rows [0, rows) of a [rows][5][ld] array, elements e0 .. e0 + NE - 1, straight
// into LDS rows of stride WS (no registers; the caller waits).
template <typename T, int NE, int NW>
__device__ __forceinline__ void tile_to_lds(const T *src, int64_t ld, int64_t e0, int rows, T *dst, int w, int lane) {
    constexpr int V = 16 / int(sizeof(T)), VPR = NE / V, W5 = 5 * NE, WS = tile_stride<NE>();
    if constexpr (WS == W5) {
        const int nchunk = rows * 5 * VPR;
        for (int base = w * 64; base < nchunk; base += NW * 64) {
            const int c = base + lane, q = c % VPR, kv = c / VPR;     // kv = 5 row + field
            if (c < nchunk) load_lds16(src + int64_t(kv) * ld + e0 + V * q, dst + size_t(base) * V);
        }
    } else {
        // padded rows: one instruction per row, its 5 VPR 16-byte pieces
        const int q = lane % VPR, v = lane / VPR;
        for (int k = w; k < rows; k += NW)
            if (lane < 5 * VPR) load_lds16(src + (int64_t(k) * 5 + v) * ld + e0 + V * q, dst + size_t(k) * WS);
    }
}

constexpr size_t TILE_LDS_MAX = 160 * 1024;   // LDS of a CU

// Raises a kernel's limit on dynamic LDS to a CU's on its first use on each
// device (the limit belongs to the device; threads that meet here raise it
// twice, which changes nothing).  One static object per kernel.
class LdsLimit {
    std::atomic<uint64_t> raised{0};          // by device, the first 64
public:
    template <typename K>
    hipError_t raise(K *kernel) {
        int dev = 0;
        if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
        const uint64_t bit = dev < 64 ? uint64_t(1) << dev : 0;
        if (raised.load(std::memory_order_relaxed) & bit) return hipSuccess;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(TILE_LDS_MAX));
        if (e == hipSuccess) raised.fetch_or(bit, std::memory_order_relaxed);
        return e;
    }
};

// Small meshes, at most one tile of 16 elements per CU: no second workgroup
// fills a CU's waits, so the tile's own chain of steps is what counts, and
// sixteen wavefronts with one column block each shorten it (608 elements,
// order 2: 54.1 -> 52.6 us for a Navier-Stokes right-hand side with this in
// the divergence stage and the interpolation; 1,296 tets, FP64, order 2: 51.5
// -> 47.8 us for an RK4 step).  With two to four tiles per CU the wider work
// items win (FP64, order 4: 312 against 323 and 332 us; order 3, FP32: 76
// against 92).
constexpr int64_t NARROW_TILES = 256;
inline bool narrow_mesh(int64_t nelem) { return (nelem + 15) / 16 <= NARROW_TILES; }

// Their kernels take the tiles of every element type in one launch: the
// types' own launches run one after the other, each with the chip mostly
// idle and a launch's cost of its own (the 608 elements: 40.6 -> 26.0 us).
// Arguments by type, nelem 0 where a type is absent.
template <typename A>
struct PerType {
    A a[3];
};
// f(type, its arguments, first element) for this workgroup's tile of 16:
// prisms and hexahedra, whose tiles take longer, come first.
template <typename A, typename F>
__device__ __forceinline__ void small_tile(const PerType<A> &p, F &&f) {
    int64_t b = blockIdx.x;
    const int64_t n1 = (p.a[1].nelem + 15) / 16, n2 = (p.a[2].nelem + 15) / 16;
    if (b < n1) return f(std::integral_constant<int, 1>{}, p.a[1], 16 * b);
    b -= n1;
    if (b < n2) return f(std::integral_constant<int, 2>{}, p.a[2], 16 * b);
    b -= n2;
    if (16 * b < p.a[0].nelem) f(std::integral_constant<int, 0>{}, p.a[0], 16 * b);
}

}  // namespace
}  // namespace frd
