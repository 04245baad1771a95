// MFMA arithmetic traits shared by the block-product kernels (gfx950): operand fragment types,
// packed-operator loads, conversion of FP64 data values to the MFMA input type, and the
// multiply-accumulate of one K chunk.
//
// Inside one MFMA the K index each lane group supplies is free as long as A and B agree.  Lane
// group g takes the KPL consecutive indices k = KPL g + t of a chunk, and the operator factors
// are packed in exactly that order (see internal.hpp), so lane (g, r) reads its part of a chunk
// as one contiguous piece.  FP64, whose four values are two 16-byte loads, takes the pairs
// k = 2 g and k = 8 + 2 g instead (koff): the four lane groups of one load then cover 64
// contiguous bytes of a column of the workspace, and a whole packed half chunk is one contiguous
// kilobyte.  With four consecutive indices each load touched every line of both halves for half
// of its bytes, and the vector L1 spent twice the cycles on the same operands.
#pragma once

#include "internal.hpp"

namespace dmrg {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// Global-memory loads (pointers from descriptor tables would otherwise become flat loads).
template <typename T>
__device__ __forceinline__ T ldg(const T* p, int64_t i) {
    return ((const __attribute__((address_space(1))) T*)p)[i];
}
template <typename V>
__device__ __forceinline__ void stgv(void* p, const V& v) {
    *((__attribute__((address_space(1))) V*)p) = v;
}
template <typename V>
__device__ __forceinline__ V ldgv(const void* p) {
    return *((const __attribute__((address_space(1))) V*)p);
}

// ---------------------------------------------------------------------------------------
// arithmetic traits
// ---------------------------------------------------------------------------------------
struct PF64 {
    static constexpr int CK = 16, KPL = 4, PER = 1;   // PER: packed pieces per value
    using op_t = double;          // packed operator element
    using ws_t = double;          // workspace element
    using acc_t = d4;
    using frag_t = d4;            // one lane's operand values of one chunk
    __device__ static frag_t from(const double (&v)[KPL]) { return (d4){v[0], v[1], v[2], v[3]}; }
    static constexpr int KP = 2;  // consecutive K indices per lane group
    __device__ static frag_t load_op(const op_t* p) {
        const d2 lo = ldgv<d2>(p), hi = ldgv<d2>(p + kPanel * 4 * KP);
        return (d4){lo[0], lo[1], hi[0], hi[1]};
    }
    __device__ static acc_t mma(const frag_t& a, const frag_t& b, acc_t c) {
#pragma unroll
        for (int t = 0; t < 4; ++t) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], b[t], c, 0, 0, 0);
        return c;
    }
    __device__ static int row(int g, int v) { return g + 4 * v; }   // result lane layout
};

struct PF32 {
    static constexpr int CK = 16, KPL = 4, PER = 1;
    using op_t = float;
    using ws_t = float;
    using acc_t = f4;
    using frag_t = f4;
    __device__ static frag_t from(const double (&v)[KPL]) {
        return (f4){(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
    }
    static constexpr int KP = KPL;
    __device__ static frag_t load_op(const op_t* p) { return ldgv<f4>(p); }
    __device__ static acc_t mma(const frag_t& a, const frag_t& b, acc_t c) {
#pragma unroll
        for (int t = 0; t < 4; ++t) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b[t], c, 0, 0, 0);
        return c;
    }
    __device__ static int row(int g, int v) { return 4 * g + v; }
};

// Split bf16 operands: NP pieces per value; the products of total order below NP (pieces
// i + j < NP) are accumulated, smallest orders last.
template <int NP>
struct PSplit {
    static constexpr int CK = 32, KPL = 8, PER = NP;
    using op_t = __bf16;          // packed as KPL values of piece 0, then piece 1, ... per lane
    using ws_t = float;
    using acc_t = f4;
    struct frag_t {
        bf8 p[NP];
    };
    __device__ static frag_t from(const double (&v)[KPL]) {
        frag_t f;
#pragma unroll
        for (int t = 0; t < KPL; ++t) {
            float rest = (float)v[t];
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                // the first piece rounds the value itself (one rounding, not through FP32): the
                // compiler took either for the other, by context
                const __bf16 h = q == 0 ? (__bf16)v[t] : (__bf16)rest;
                f.p[q][t] = h;
                rest -= (float)h;
            }
        }
        return f;
    }
    static constexpr int KP = KPL;
    __device__ static frag_t load_op(const op_t* p) {
        frag_t f;
#pragma unroll
        for (int q = 0; q < NP; ++q) f.p[q] = ldgv<bf8>(p + q * KPL);
        return f;
    }
    __device__ static acc_t mma(const frag_t& a, const frag_t& b, acc_t c) {
#pragma unroll
        for (int o = 0; o < NP; ++o)
#pragma unroll
            for (int i = 0; i <= o; ++i)
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[i], b.p[o - i], c, 0, 0, 0);
        return c;
    }
    __device__ static int row(int g, int v) { return 4 * g + v; }
};
using PBF3 = PSplit<2>;
using PBF6 = PSplit<3>;

// Elements of one packed panel chunk per lane (all pieces of a split value) and per chunk.
template <class P>
constexpr int lane_elems() {
    return P::KPL * P::PER;
}
template <class P>
constexpr int chunk_elems() {
    return kPanel * 4 * lane_elems<P>();
}

template <class P>
__device__ __forceinline__ void zero(typename P::acc_t& a) {
#pragma unroll
    for (int v = 0; v < 4; ++v) a[v] = 0;
}

// K index inside a chunk of value t of lane group g
template <class P>
__device__ __forceinline__ int koff(int g, int t) {
    return t / P::KP * (4 * P::KP) + P::KP * g + t % P::KP;
}
// First element of lane (g, r) inside a packed panel chunk
template <class P>
__device__ __forceinline__ int lane_off(int g, int r) {
    return (kPanel * g + r) * (P::KP * P::PER);
}

// Element (k, col) of a plane of the stage-1 workspace (S1Block::T), ld = elements of a panel.
template <typename T>
__device__ __forceinline__ int64_t tpos(int ld, int col, int k) {
    constexpr int U = 16 / sizeof(T);
    return (int64_t)(col >> 4) * ld + k / U * (16 * U) + (col & 15) * U + (k & (U - 1));
}

// FP64: zeros in the padding rows of the columns n0 .. n0 + 63 (< N), by the work group (NT threads)
// whose 64 rows m0 .. hold a plane's last one: stage 2 multiplies them with zero factors, and what the
// K-split family's layout (FP64 only) or a vector of NaN left there need not be finite.  Stage 1
// LDS-tiled and LDS-staged without and with it: 1000-state ladder 38.0 -> 38.6 and 35.1 -> 35.6 us,
// 400-state chain 8.3 -> 8.6 and 7.8 -> 8.2; by the lanes that store a column's last row 40.8
// and 40.5, 9.7 and 9.9.
template <int NT>
__device__ __forceinline__ void pad_rows(double* __restrict__ T, const View& tv, int m0, int n0, int N) {
    const int pad = (kChunk - tv.split % kChunk) % kChunk;
    for (int pl = 0; pl < 2; ++pl) {
        const int last = (pl + 1) * tv.split - 1;
        if (last < m0 || last >= m0 + 64) continue;
        for (int t = threadIdx.x; t < 64 * pad; t += NT) {
            const int n = n0 + (t & 63);
            if (n < N) T[tv.off + pl * tv.poff + tpos<double>(tv.ld, n, tv.split + (t >> 6))] = 0;
        }
    }
}

// The lane's data values k = koff(g, t) of a chunk of the workspace, base at the lane's column in
// the chunk's first unit: 16-byte units, so that 16 lanes read 256 contiguous bytes.  (From a
// column-major intermediate every lane of a load was in a line of its own; the L1's data return
// then took four times the cycles and bounded stage 2, see gemm.hip.)
template <class P, typename T>
__device__ __forceinline__ void load_units(const T* src, int64_t base, int g, T (&v)[P::KPL]) {
    constexpr int U = 16 / sizeof(T);
    typedef T unit_t __attribute__((ext_vector_type(U)));
#pragma unroll
    for (int t = 0; t < P::KPL; t += U) {
        const unit_t u = ldgv<unit_t>(src + base + koff<P>(g, t) / U * (16 * U));
#pragma unroll
        for (int q = 0; q < U; ++q) v[t + q] = u[q];
    }
}
template <class P, typename T>
__device__ __forceinline__ void load_run(const T* src, int64_t base, int g, double (&v)[P::KPL]) {
    T u[P::KPL];
    load_units<P>(src, base, g, u);
#pragma unroll
    for (int t = 0; t < P::KPL; ++t) v[t] = (double)u[t];
}
// The lane's values src[base + min(k0 + koff(g, t), K - 1) * stride] (input vector, clamped)
template <class P>
__device__ __forceinline__ void load_clamped(const double* src, int64_t base, int k0, int g, int K,
                                             int64_t stride, double (&v)[P::KPL]) {
#pragma unroll
    for (int t = 0; t < P::KPL; ++t)
        v[t] = ldg(src, base + (int64_t)min(k0 + koff<P>(g, t), K - 1) * stride);
}
// Two consecutive values as one 16-byte load (8-byte aligned).
__device__ __forceinline__ d2 ldg2(const double* p, int64_t i) {
    typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
    const d2u v = ldgv<d2u>(p + i);
    return (d2){v[0], v[1]};
}
// The lane's values src[base + k0 + koff(g, t)] of a whole chunk (input vector, K contiguous)
template <class P>
__device__ __forceinline__ void load_pairs(const double* src, int64_t base, int k0, int g,
                                           double (&v)[P::KPL]) {
#pragma unroll
    for (int t = 0; t < P::KPL; t += 2) {
        const d2 p = ldg2(src, base + k0 + koff<P>(g, t));
        v[t] = p[0];
        v[t + 1] = p[1];
    }
}

// Rows of a 16-row A operand whose row index is contiguous in memory, loaded two at a time: lane
// (g, r) asks for rows 2 (r mod 8), 2 (r mod 8) + 1 at k = koff(g, t) + r / 8 (t even), 8 lanes per
// column of 128 bytes.  Exchanging the lanes of each half row of 16 (DPP) then leaves lane (g, r)
// with row a_row(r) at koff(g, t) and koff(g, t + 1): the operand with its rows permuted.
__device__ __forceinline__ int a_row(int r) { return r < 8 ? 2 * r : 2 * r - 15; }
__device__ __forceinline__ void half_rows(const d2& p, double& v0, double& v1) {
    union {
        double d;
        int u[2];
    } a, b, x, y;
    a.d = p[0];
    b.d = p[1];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        // lanes 8..15 of v0 from lanes 0..7 of the second row, lanes 0..7 of v1 from lanes 8..15 of
        // the first
        x.u[w] = __builtin_amdgcn_update_dpp(a.u[w], b.u[w], 0x118, 0xf, 0xc, false);   // row_shr:8
        y.u[w] = __builtin_amdgcn_update_dpp(b.u[w], a.u[w], 0x108, 0xf, 0x3, false);   // row_shl:8
    }
    v0 = x.d;
    v1 = y.d;
}

}  // namespace dmrg
