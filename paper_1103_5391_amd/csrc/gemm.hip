// Grouped block products of H_sb.psi on gfx950 MFMA, in four arithmetics:
//   FP64    v_mfma_f64_16x16x4f64, FP64 workspace
//   FP32    v_mfma_f32_16x16x4f32, FP32 operands and workspace
//   BF16x3  v_mfma_f32_16x16x32_bf16 on split operands a = a0 + a1 (bf16 pieces, each the
//           rounding of what the previous leave): a0 b0 + a0 b1 + a1 b0 accumulated in FP32
//           (relative error about 2^-16), FP32 workspace
//   BF16x6  three pieces a = a0 + a1 + a2, the six products of total order <= 2
//           (about 2^-24, FP32-like), FP32 workspace
// The result of the second stage is always written in FP64.
//
// The Hamiltonian connections (Sec. IV) are applied as psi' = A psi B^T over (N_up, N_dn)
// symmetry blocks in two stages, each one launch over a list of output tiles:
//   stage 1  T_b  = X_b R_b        right products, X_b = [Re; Im] planes of the source block
//   stage 2  Y_b' = T0 + Acat Bcat left products summed over all terms entering the block
// Stage 1 gives each tile of 16 rows of both planes x 64 columns (or x 32: twice the tiles, for better
// balance on small problems) to a work group of one wavefront (single-wave work groups let the
// dispatcher balance the compute units at the end of the launch).  In stage 2 a work group of four
// wavefronts owns one 32 x 32 tile (or 32 x 16, narrow) and deals its K chunks round-robin to the
// waves; the four partial tiles are summed in LDS in a fixed order (deterministic, no atomics).
//
// The operator factors are packed in MFMA lane order (mfma.hpp) and zero-padded so no operator
// load needs a bounds check.  The input vector is read in place, out-of-range K indices clamped to
// a valid element, whose product with the padded zeros vanishes.  Stage 1 writes its intermediate
// in the order stage 2's lanes read it (S1Block::T, zero-padded to whole chunks): a load of 16
// lanes is then 256 contiguous bytes.  From a column-major intermediate each lane of such a load
// was in a line of its own, which costs the L1 64 cycles instead of 14, and its tiles stored
// pieces of 32 bytes, whose write-back held up the loads of the tiles that follow.  Stage 1 / 2
// of the 2x16 ladder at m = 1000: 34.4 / 36.4 us column-major, 29.8 / 32.2 in units; 2x32 at
// m = 2000: 186 / 187 -> 161 / 166; BF16x3 at m = 1000: 21.8 / 26.7 -> 21.6 / 23.4.
#include "mfma.hpp"

#include <type_traits>

namespace dmrg {

// Whether the problem's work is skipped (after a breakdown): a scalar load, tested after the first
// operand loads have been issued.
__device__ __forceinline__ int skip_of(const ProbPtrs& pp) {
    return pp.skip ? *(const __attribute__((address_space(4))) int*)pp.skip : 0;
}

// ---------------------------------------------------------------------------------------
// stage 1: one tile of 16 rows of both planes x 16 NJ columns (NJ = 4 wide, 2 narrow) per
// single-wavefront work group
// ---------------------------------------------------------------------------------------
// One 16 x 16 fragment of T (the lane's values: rows a_row(row(g, v)) of column r) into a chunk of
// the workspace, contiguous kilobytes of 16-byte units.  In FP64 a lane holds the two rows of two
// units; in FP32 swapping two pairs of values between the wave's halves gives it the four of one.
__device__ __forceinline__ void store_frag(double* t, const d4& c, int g, int r) {
    stgv(t + 32 * g + 2 * r, (d2){c[0], c[2]});
    stgv(t + 128 + 32 * g + 2 * r, (d2){c[1], c[3]});
}
__device__ __forceinline__ void store_frag(float* t, const f4& c, int g, int r) {
    union {
        f4 f;
        unsigned u[4];
    } a, b;
    a.f = c;
    const auto p = __builtin_amdgcn_permlane32_swap(a.u[0], a.u[2], false, false);
    const auto q = __builtin_amdgcn_permlane32_swap(a.u[1], a.u[3], false, false);
    b.u[0] = p[0];
    b.u[1] = p[1];
    b.u[2] = q[0];
    b.u[3] = q[1];
    const int unit = ((g & 1) << 1) | (g >> 1);     // lane groups 0..3 hold units 0, 2, 1, 3
    stgv(t + 64 * unit + 4 * r, b.f);
}

template <class P, int NJ>
__device__ __forceinline__ void stage1_tile(const Tile& tl, const S1Block& B, const ProbPtrs& P_) {
    using op_t = typename P::op_t;
    using ws_t = typename P::ws_t;
    using acc_t = typename P::acc_t;
    using frag_t = typename P::frag_t;
    const int skip = skip_of(P_);
    const int lane = threadIdx.x;
    const int g = lane >> 4, r = lane & 15;
    const double* __restrict__ X = P_.x;
    const int K = B.K;
    const int nch = (K + P::CK - 1) / P::CK;

    // The operand's rows are permuted (a_row).  A whole tile loads two rows per lane: a load of
    // one row costs the L1 the same 14 cycles for half the bytes (stage 1 at m = 1000: 29.8 ->
    // 28.3 us).  At the block's end rows past it are its last one, in padding rows of T.
    const bool whole = tl.m0 + 16 <= B.X.split;       // the same in every lane
    int64_t arow[2];
    arow[0] = B.X.off + (whole ? tl.m0 + 2 * (r & 7) : min(tl.m0 + a_row(r), B.X.split - 1));
    arow[1] = arow[0] + B.X.poff;
    const op_t* pb = static_cast<const op_t*>(P_.Rops) + B.Roff * P::PER +
                     (int64_t)(tl.n0 / kPanel) * nch * chunk_elems<P>() + lane_off<P>(g, r);
    const int64_t panel = (int64_t)nch * chunk_elems<P>();
    const int64_t ldx = B.X.ld;
    acc_t acc[2][NJ];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj) zero<P>(acc[mi][nj]);
    auto run = [&](auto pairs) {
        constexpr bool kPairs = decltype(pairs)::value;
        struct Chunk {
            double x[2][P::KPL];      // as loaded: exchanged and converted when it is multiplied
                                      // (a conversion beside the load waits for it there: FP32
                                      // 24.7 -> 21.2 us, BF16x3 21.6 -> 19.9)
            frag_t b[NJ];
        };
        auto load = [&](int c, Chunk& k) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if constexpr (kPairs) {
#pragma unroll
                    for (int t = 0; t < P::KPL; t += 2) {
                        const int kk = min(c * P::CK + koff<P>(g, t) + (r >> 3), K - 1);
                        const d2 p = ldg2(X, arow[i] + kk * ldx);
                        k.x[i][t] = p[0];
                        k.x[i][t + 1] = p[1];
                    }
                } else {
                    load_clamped<P>(X, arow[i], c * P::CK, g, K, ldx, k.x[i]);
                }
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                k.b[j] = P::load_op(pb + j * panel + (int64_t)c * chunk_elems<P>());
        };
        auto mma = [&](const Chunk& k) {
#pragma unroll
            for (int mi = 0; mi < 2; ++mi) {
                double v[P::KPL];
#pragma unroll
                for (int t = 0; t < P::KPL; t += 2) {
                    v[t] = k.x[mi][t];
                    v[t + 1] = k.x[mi][t + 1];
                    if constexpr (kPairs) half_rows((d2){k.x[mi][t], k.x[mi][t + 1]}, v[t], v[t + 1]);
                }
                const frag_t fa = P::from(v);
#pragma unroll
                for (int nj = 0; nj < NJ; ++nj) acc[mi][nj] = P::mma(fa, k.b[nj], acc[mi][nj]);
            }
        };
        // two register buffers, the next chunk always in flight (as in the stage-2 loop)
        Chunk k0, k1;
        load(0, k0);
        if (skip) return false;
        int c = 0;
        for (; c + 1 < nch; c += 2) {
            load(c + 1, k1);
            __builtin_amdgcn_sched_barrier(0);
            mma(k0);
            load(min(c + 2, nch - 1), k0);
            __builtin_amdgcn_sched_barrier(0);
            mma(k1);
        }
        if (c < nch) mma(k0);
        return true;
    };
    if (!(whole ? run(std::true_type{}) : run(std::false_type{}))) return;
    // whole fragments, padding columns (never read) and rows (zero) included
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (tl.m0 + a_row(P::row(g, v)) >= B.X.split)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int nj = 0; nj < NJ; ++nj) acc[mi][nj][v] = 0;
    ws_t* __restrict__ T = static_cast<ws_t*>(P_.T) + B.T.off + tpos<ws_t>(B.T.ld, tl.n0, tl.m0);
#pragma unroll
    for (int nj = 0; nj < NJ; ++nj)
        if (tl.n0 + 16 * nj < B.N)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
                store_frag(T + mi * B.T.poff + (int64_t)nj * B.T.ld, acc[mi][nj], g, r);
}

// Wide tiles take two wavefronts per SIMD: at three they spilled (FP64 at m = 2000: 174 -> 154 us,
// BF16x6 at m = 1000: 48.7 -> 20.7).
template <class P, int NJ>
__global__ __launch_bounds__(64, NJ > 2 ? 2 : 3) void stage1(const S1Block* __restrict__ blks,
                                                 const Tile* __restrict__ tiles, int ntiles,
                                                 const ProbPtrs* __restrict__ probs,
                                                 ProbPtrs single) {
    const int ti = blockIdx.x;
    if (ti >= ntiles) return;
    const Tile tl = tiles[ti];
    if (tl.blk < 0) return;   // padding of the XCD-ordered list
    const S1Block B = blks[tl.blk];
    const ProbPtrs P_ = probs ? probs[B.prob] : single;
    stage1_tile<P, NJ>(tl, B, P_);
}

// ---------------------------------------------------------------------------------------
// stage 2: one 32 x 32 (or 32 x 16) tile per work group, K chunks dealt round-robin to its waves
// ---------------------------------------------------------------------------------------
constexpr int kChunkTab = 64 * kWaves;   // entries of the chunk table in LDS (one per thread)
// D: element type of the data operand as it is loaded; it is converted to the MFMA input type when
// it is multiplied (a conversion beside the load would wait for it there).
template <class P, int MI, int NJ, typename D>
struct Chunk2 {
    typename P::frag_t a[MI];
    D b[NJ][P::KPL];
    __device__ __forceinline__ typename P::frag_t right(int j) const {
        double v[P::KPL];
#pragma unroll
        for (int t = 0; t < P::KPL; ++t) v[t] = (double)b[j][t];
        return P::from(v);
    }
};
// Chunks c0, c0 + step, ... below nch.  mid() runs once, after the first chunk's load where
// `early` (that load does not depend on it), else before it; false from it ends the tile.
template <class P, int MI, int NJ, typename D, class Load, class Mid>
__device__ __forceinline__ bool kloop(typename P::acc_t (&acc)[MI][NJ], int c0, int step, int nch,
                                      Load load, bool early, Mid mid) {
    const int last = c0 + (nch - 1 - c0) / step * step;
    Chunk2<P, MI, NJ, D> k0, k1;
    if (early && c0 < nch) load(c0, k0);
    if (!mid()) return false;
    if (c0 >= nch) return true;
    if (!early) load(c0, k0);
    auto mma = [&](const Chunk2<P, MI, NJ, D>& k) {
        typename P::frag_t fb[NJ];
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj) fb[nj] = k.right(nj);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int nj = 0; nj < NJ; ++nj) acc[mi][nj] = P::mma(k.a[mi], fb[nj], acc[mi][nj]);
    };
    // Two register buffers, one exit test per pair of chunks: the chunk after the one being
    // multiplied is always in flight (the last prefetch is clamped and unused).  The
    // scheduling barriers keep each prefetch ahead of the products it overlaps; without them
    // the compiler moved the loads down to their products and waited for them there.
    int c = c0;
    for (; c + step <= last; c += 2 * step) {
        load(c + step, k1);
        __builtin_amdgcn_sched_barrier(0);
        mma(k0);
        load(min(c + 2 * step, last), k0);
        __builtin_amdgcn_sched_barrier(0);
        mma(k1);
    }
    if (c <= last) mma(k0);   // odd count: chunk c is in k0
    return true;
}

// One 16 MI x 16 NJ output tile (MI = 2, or 1 for a half-height tile) per work group of NW
// wavefronts (K chunks dealt round-robin); ctab and red live in the kernel's LDS.
template <class P, int MI, int NJ, int NW>
__device__ __forceinline__ void stage2_tile(const Tile& tl, const S2Block& B,
                                            const XChunk* __restrict__ xch, const ProbPtrs& P_,
                                            int64_t (&ctab)[kChunkTab][3],
                                            double (&red)[NW][16 * NJ][kTile + 1]) {
    using op_t = typename P::op_t;
    using ws_t = typename P::ws_t;
    using acc_t = typename P::acc_t;
    using frag_t = typename P::frag_t;
    constexpr int TN = 16 * NJ;
    const int skip = skip_of(P_);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
    const int g = lane >> 4, r = lane & 15;
    const int split = B.Y.split;   // columns per plane of the output and of every source
    const ws_t* __restrict__ Tws = static_cast<const ws_t*>(P_.T);

    const op_t* pa[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int pnl = tl.m0 / kPanel + i;
        pa[i] = static_cast<const op_t*>(P_.Lops) + B.Aoff * P::PER +
                (int64_t)pnl * B.nch * chunk_elems<P>() + lane_off<P>(g, r);
    }
    int pl[NJ], col[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int n = min(tl.n0 + 16 * j + r, B.N - 1);
        pl[j] = n >= split;
        col[j] = n - pl[j] * split;
    }
    acc_t acc[MI][NJ];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj) zero<P>(acc[mi][nj]);
    // segment 0, the diagonal H_S term, reads the block itself from the input vector; the other
    // chunks read the workspace, their sources from the block's chunk table, kept in LDS (the
    // first kChunkTab entries, the next ones when those are done)
    const int K0 = B.M, nch0 = (K0 + P::CK - 1) / P::CK;
    const int nT = B.nch - nch0;
    const XChunk* __restrict__ tab = xch + B.ctab0 + nch0;
    XChunk e{};
    if ((int)threadIdx.x < min(nT, kChunkTab)) e = tab[threadIdx.x];
    auto fill = [&] {
        if (skip) return false;          // the same in every wave
        ctab[threadIdx.x][0] = e.off;
        ctab[threadIdx.x][1] = e.poff;
        ctab[threadIdx.x][2] = ((int64_t)e.col0 << 32) | (uint32_t)e.ld;
        __syncthreads();
        return true;
    };
    int64_t bcol[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
        bcol[j] = B.Y.off + pl[j] * B.Y.poff + (int64_t)col[j] * B.Y.ld;
    auto load_a = [&](int c, auto& k) {
        const int64_t ga = (int64_t)c * chunk_elems<P>();
#pragma unroll
        for (int i = 0; i < MI; ++i) k.a[i] = P::load_op(pa[i] + ga);
    };
    auto load_x = [&](int c, Chunk2<P, MI, NJ, double>& k) {
        load_a(c, k);
        // a lane's values lie in a line of its own: half the loads where the chunk is whole
        if ((c + 1) * P::CK <= K0) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) load_pairs<P>(P_.x, bcol[j], c * P::CK, g, k.b[j]);
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                load_clamped<P>(P_.x, bcol[j], c * P::CK, g, K0, 1, k.b[j]);
        }
    };
    int tc = nch0;      // chunk of the table's first entry
    auto load_t = [&](int c, Chunk2<P, MI, NJ, ws_t>& k) {
        load_a(c, k);
        const int64_t* q = ctab[c - tc];
        const int ld = (int)q[2], col0 = (int)(q[2] >> 32);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            load_units<P>(Tws, q[0] + (pl[j] ? q[1] : 0) + tpos<ws_t>(ld, col0 + col[j], 0), g,
                          k.b[j]);
    };
    const int end0 = min(B.nch, nch0 + kChunkTab);
    if constexpr (std::is_same<ws_t, double>::value) {
        // one stream of both kinds
        auto load = [&](int c, Chunk2<P, MI, NJ, double>& k) {
            if (c < nch0)
                load_x(c, k);
            else
                load_t(c, k);
        };
        if (!kloop<P, MI, NJ, double>(acc, wave, NW, end0, load, wave < nch0, fill)) return;
    } else {
        if (!kloop<P, MI, NJ, double>(acc, wave, NW, nch0, load_x, true, fill)) return;
        kloop<P, MI, NJ, ws_t>(acc, nch0 + ((wave - nch0) % NW + NW) % NW, NW, end0, load_t, true,
                               [] { return true; });
    }
    for (int c1 = end0; c1 < B.nch; c1 += kChunkTab) {
        __syncthreads();                 // every wave is done with the table
        tc = c1;
        if ((int)threadIdx.x < B.nch - c1) e = tab[c1 - nch0 + threadIdx.x];
        fill();
        kloop<P, MI, NJ, ws_t>(acc, c1 + ((wave - c1) % NW + NW) % NW, NW,
                               min(B.nch, c1 + kChunkTab), load_t, true,
                               [] { return true; });
    }

#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                red[wave][16 * nj + r][16 * mi + P::row(g, v)] = (double)acc[mi][nj][v];
    __syncthreads();
    double* __restrict__ Y = P_.y;
    const View t0 = B.T0, yv = B.Y;
    const int m = threadIdx.x & 31;
    constexpr int kCols = 2 * NW;   // columns handled per pass of the work group
#pragma unroll
    for (int q = 0; q < TN / kCols; ++q) {
        const int n = (threadIdx.x >> 5) + kCols * q;
        const int gm = tl.m0 + m, gn = tl.n0 + n;
        if (gm < B.M && gn < B.N) {
            double v = red[0][n][m];
#pragma unroll
            for (int w = 1; w < NW; ++w) v += red[w][n][m];
            const int p = gn >= split;
            const int c = gn - p * split;
            const double init = (double)Tws[t0.off + p * t0.poff + tpos<ws_t>(t0.ld, c, gm)];
            Y[yv.off + p * yv.poff + (int64_t)c * yv.ld + gm] = init + v;
        }
    }
}

template <class P, int NJ, int NW>
__global__ __launch_bounds__(64 * NW, 3) void stage2(const S2Block* __restrict__ blks,
                                                     const XChunk* __restrict__ xch,
                                                     const Tile* __restrict__ tiles,
                                                     const ProbPtrs* __restrict__ probs,
                                                     ProbPtrs single) {
    const Tile tl = tiles[blockIdx.x];
    if (tl.blk < 0) return;   // padding of the XCD-ordered list
    const S2Block B = blks[tl.blk];
    const ProbPtrs P_ = probs ? probs[B.prob] : single;
    __shared__ int64_t ctab[kChunkTab][3];
    __shared__ double red[NW][16 * NJ][kTile + 1];
    if (tl.half)
        stage2_tile<P, 1, NJ, NW>(tl, B, xch, P_, ctab, red);
    else
        stage2_tile<P, 2, NJ, NW>(tl, B, xch, P_, ctab, red);
}

// ---------------------------------------------------------------------------------------
// stage 2 for several right-hand sides that share the operators (the chains of the 4-RHS
// mode): the tile list of the owners' plans, chain c of problem p at probs[NR p + c].  Each
// chunk's left-factor fragments are loaded once for all NR chains.  Every chain's products run
// in the order of the single-vector kernel above, so its results have the same bits.  A chain
// whose skip flag is set is computed (its buffers are allocated) but not stored.  (Stage 1
// stays per chain: four chains' accumulators and fragments there exceed the registers.)
// ---------------------------------------------------------------------------------------
// The problem pointers of chains c0 .. c0 + NR - 1 of a tile and which of them are live.
template <int NR>
__device__ __forceinline__ bool chain_ptrs(const ProbPtrs* __restrict__ probs, int prob, int c0,
                                           ProbPtrs (&PP)[NR], bool (&act)[NR]) {
    bool any = false;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        PP[q] = probs[kMultiRhs * prob + c0 + q];
        act[q] = !(PP[q].skip && *PP[q].skip);
        any |= act[q];
    }
    return any;
}

// kloop for NR chains sharing the A fragments.
template <class P, int MI, int NJ, int NR, class Load>
__device__ __forceinline__ void kloop_mr(typename P::acc_t (&acc)[NR][MI][NJ], int c0, int step,
                                         int nch, Load load) {
    using frag_t = typename P::frag_t;
    if (c0 >= nch) return;
    const int last = c0 + (nch - 1 - c0) / step * step;
    frag_t a0[MI], b0[NR][NJ], a1[MI], b1[NR][NJ];
    auto mma = [&](const frag_t (&fa)[MI], const frag_t (&fb)[NR][NJ]) {
#pragma unroll
        for (int q = 0; q < NR; ++q)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int nj = 0; nj < NJ; ++nj) acc[q][mi][nj] = P::mma(fa[mi], fb[q][nj], acc[q][mi][nj]);
    };
    load(c0, a0, b0);
    int c = c0;
    for (; c + step <= last; c += 2 * step) {
        load(c + step, a1, b1);
        __builtin_amdgcn_sched_barrier(0);
        mma(a0, b0);
        load(min(c + 2 * step, last), a0, b0);
        __builtin_amdgcn_sched_barrier(0);
        mma(a1, b1);
    }
    if (c <= last) mma(a0, b0);
}

template <class P, int MI, int NJ, int NW, int NR>
__device__ __forceinline__ void stage2_tile_mr(const Tile& tl, const S2Block& B,
                                               const XChunk* __restrict__ xch,
                                               const ProbPtrs (&PP)[NR], const bool (&act)[NR],
                                               int64_t (&ctab)[kChunkTab][3],
                                               double (&red)[NW][16 * NJ][kTile + 1]) {
    using op_t = typename P::op_t;
    using ws_t = typename P::ws_t;
    using acc_t = typename P::acc_t;
    using frag_t = typename P::frag_t;
    constexpr int TN = 16 * NJ;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
    const int g = lane >> 4, r = lane & 15;
    const int split = B.Y.split;
    const op_t* pa[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int pnl = tl.m0 / kPanel + i;
        pa[i] = static_cast<const op_t*>(PP[0].Lops) + B.Aoff * P::PER +
                (int64_t)pnl * B.nch * chunk_elems<P>() + lane_off<P>(g, r);
    }
    int pl[NJ], col[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int n = min(tl.n0 + 16 * j + r, B.N - 1);
        pl[j] = n >= split;
        col[j] = n - pl[j] * split;
    }
    acc_t acc[NR][MI][NJ];
#pragma unroll
    for (int q = 0; q < NR; ++q)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int nj = 0; nj < NJ; ++nj) zero<P>(acc[q][mi][nj]);
    // segment 0 (H_S) from each chain's input vector, then the workspace chunks from each chain's
    // stage-1 intermediate (sources in the chunk table, as in the single-vector kernel)
    const int K0 = B.M, nch0 = (K0 + P::CK - 1) / P::CK;
    const XChunk* __restrict__ tab = xch + B.ctab0 + nch0;
    auto fill = [&](int c1) {
        if ((int)threadIdx.x < min(B.nch - c1, kChunkTab)) {
            const XChunk e = tab[c1 - nch0 + threadIdx.x];
            ctab[threadIdx.x][0] = e.off;
            ctab[threadIdx.x][1] = e.poff;
            ctab[threadIdx.x][2] = ((int64_t)e.col0 << 32) | (uint32_t)e.ld;
        }
        __syncthreads();
    };
    {
        int64_t bcol[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            bcol[j] = B.Y.off + pl[j] * B.Y.poff + (int64_t)col[j] * B.Y.ld;
        auto load = [&](int c, frag_t (&fa)[MI], frag_t (&fb)[NR][NJ]) {
            const int64_t ga = (int64_t)c * chunk_elems<P>();
#pragma unroll
            for (int i = 0; i < MI; ++i) fa[i] = P::load_op(pa[i] + ga);
#pragma unroll
            for (int q = 0; q < NR; ++q)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    double v[P::KPL];
                    load_clamped<P>(PP[q].x, bcol[j], c * P::CK, g, K0, 1, v);
                    fb[q][j] = P::from(v);
                }
        };
        kloop_mr<P, MI, NJ, NR>(acc, wave, NW, nch0, load);
    }
    for (int c1 = nch0; c1 < B.nch; c1 += kChunkTab) {
        if (c1 > nch0) __syncthreads();
        fill(c1);
        auto load = [&](int c, frag_t (&fa)[MI], frag_t (&fb)[NR][NJ]) {
            const int64_t ga = (int64_t)c * chunk_elems<P>();
#pragma unroll
            for (int i = 0; i < MI; ++i) fa[i] = P::load_op(pa[i] + ga);
            const int64_t* e = ctab[c - c1];
            const int ld = (int)e[2], col0 = (int)(e[2] >> 32);
#pragma unroll
            for (int q = 0; q < NR; ++q)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    double v[P::KPL];
                    load_run<P>(static_cast<const ws_t*>(PP[q].T),
                                e[0] + (pl[j] ? e[1] : 0) + tpos<ws_t>(ld, col0 + col[j], 0), g, v);
                    fb[q][j] = P::from(v);
                }
        };
        kloop_mr<P, MI, NJ, NR>(acc, c1 + ((wave - c1) % NW + NW) % NW, NW,
                                min(B.nch, c1 + kChunkTab), load);
    }
    // the waves' partial tiles summed in LDS in a fixed order, one chain after another
    const View t0 = B.T0, yv = B.Y;
    const int m = threadIdx.x & 31;
    constexpr int kCols = 2 * NW;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
        if (!act[q]) continue;                          // the same in every thread
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    red[wave][16 * nj + r][16 * mi + P::row(g, v)] = (double)acc[q][mi][nj][v];
        __syncthreads();
        const ws_t* __restrict__ Tws = static_cast<const ws_t*>(PP[q].T);
        double* __restrict__ Y = PP[q].y;
#pragma unroll
        for (int qq = 0; qq < TN / kCols; ++qq) {
            const int n = (threadIdx.x >> 5) + kCols * qq;
            const int gm = tl.m0 + m, gn = tl.n0 + n;
            if (gm < B.M && gn < B.N) {
                double v = red[0][n][m];
#pragma unroll
                for (int w = 1; w < NW; ++w) v += red[w][n][m];
                const int p = gn >= split;
                const int c = gn - p * split;
                const double init = (double)Tws[t0.off + p * t0.poff + tpos<ws_t>(t0.ld, c, gm)];
                Y[yv.off + p * yv.poff + (int64_t)c * yv.ld + gm] = init + v;
            }
        }
        __syncthreads();                                // red is written again for the next chain
    }
}

template <class P, int NJ, int NW, int NR>
__global__ __launch_bounds__(64 * NW, 2) void stage2_mr(const S2Block* __restrict__ blks,
                                                        const XChunk* __restrict__ xch,
                                                        const Tile* __restrict__ tiles,
                                                        const ProbPtrs* __restrict__ probs) {
    const Tile tl = tiles[blockIdx.x];
    if (tl.blk < 0) return;   // padding of the XCD-ordered list
    const S2Block B = blks[tl.blk];
    ProbPtrs PP[NR];
    bool act[NR];
    if (!chain_ptrs<NR>(probs, B.prob, NR * (int)blockIdx.y, PP, act)) return;
    __shared__ int64_t ctab[kChunkTab][3];
    __shared__ double red[NW][16 * NJ][kTile + 1];
    if (tl.half)
        stage2_tile_mr<P, 1, NJ, NW, NR>(tl, B, xch, PP, act, ctab, red);
    else
        stage2_tile_mr<P, 2, NJ, NW, NR>(tl, B, xch, PP, act, ctab, red);
}

// ---------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------
namespace {

template <class P>
hipError_t launch1(int narrow, const S1Block* blks, const Tile* tiles, int ntiles,
                   const ProbPtrs* probs, ProbPtrs single, hipStream_t st) {
    if (ntiles == 0) return hipSuccess;
    if (narrow)
        hipLaunchKernelGGL((stage1<P, kTile1NN / 16>), dim3(ntiles), dim3(64), 0, st, blks, tiles,
                           ntiles, probs, single);
    else
        hipLaunchKernelGGL((stage1<P, kTile1N / 16>), dim3(ntiles), dim3(64), 0, st, blks, tiles,
                           ntiles, probs, single);
    return hipGetLastError();
}

template <class P>
hipError_t launch2(int narrow, const S2Block* blks, const XChunk* xch, const Tile* tiles,
                   int ntiles, const ProbPtrs* probs, ProbPtrs single, hipStream_t st) {
    if (ntiles == 0) return hipSuccess;
    if (narrow)
        hipLaunchKernelGGL((stage2<P, kTile2NN / 16, kWaves>), dim3(ntiles), dim3(64 * kWaves), 0,
                           st, blks, xch, tiles, probs, single);
    else
        hipLaunchKernelGGL((stage2<P, kTile / 16, kWaves>), dim3(ntiles), dim3(64 * kWaves), 0, st,
                           blks, xch, tiles, probs, single);
    return hipGetLastError();
}

}  // namespace

// Stage 2 of the chains of the 4-RHS mode in one launch (FP64, narrow tiles): the owners' tile
// list, chain c of problem p at probs[kMultiRhs p + c].
hipError_t launch_stage2_mr(const S2Block* blks, const XChunk* xch, const Tile* tiles,
                            int ntiles, const ProbPtrs* probs, hipStream_t st) {
    if (ntiles == 0) return hipSuccess;
    // all chains in one work group (two per work group, with a second grid row for the other
    // two, measured the same)
    constexpr int NR = kMultiRhs;
    hipLaunchKernelGGL((stage2_mr<PF64, kTile2NN / 16, kWaves, NR>), dim3(ntiles, kMultiRhs / NR),
                       dim3(64 * kWaves), 0, st, blks, xch, tiles, probs);
    return hipGetLastError();
}

// prec: 0 FP64, 1 FP32, 2 BF16x3, 3 BF16x6 (the operator buffers and workspace must match);
// narrow: the tiles have kTile1NN columns (else kTile1N)
hipError_t launch_stage1(int prec, int narrow, const S1Block* blks, const Tile* tiles, int ntiles,
                         const ProbPtrs* probs, ProbPtrs single, hipStream_t st) {
    switch (prec) {
        case 0: return launch1<PF64>(narrow, blks, tiles, ntiles, probs, single, st);
        case 1: return launch1<PF32>(narrow, blks, tiles, ntiles, probs, single, st);
        case 2: return launch1<PBF3>(narrow, blks, tiles, ntiles, probs, single, st);
        default: return launch1<PBF6>(narrow, blks, tiles, ntiles, probs, single, st);
    }
}

// narrow: the tiles are kTile x kTile2NN (else kTile x kTile)
hipError_t launch_stage2(int prec, int narrow, const S2Block* blks, const XChunk* xch,
                         const Tile* tiles, int ntiles, const ProbPtrs* probs, ProbPtrs single,
                         hipStream_t st) {
    switch (prec) {
        case 0: return launch2<PF64>(narrow, blks, xch, tiles, ntiles, probs, single, st);
        case 1: return launch2<PF32>(narrow, blks, xch, tiles, ntiles, probs, single, st);
        case 2: return launch2<PBF3>(narrow, blks, xch, tiles, ntiles, probs, single, st);
        default: return launch2<PBF6>(narrow, blks, xch, tiles, ntiles, probs, single, st);
    }
}

}  // namespace dmrg
