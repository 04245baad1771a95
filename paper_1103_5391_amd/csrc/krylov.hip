// Lanczos vector kernels, tridiagonal exponential and Krylov combination (FP64, gfx950).
//
// Sec. II.A: the Lanczos recursion is started from phi itself, H ~ V^T T V, and
//   phi(t) ~ beta0 V^T S exp(-i D t) S^T e_1,     T = S D S^T.
// Storage: slot j of the basis buffer holds u_j = beta_j v_j (the vector before
// normalisation) and the state keeps scale[j] = 1/beta_j, so no separate normalisation pass
// is needed; every consumer multiplies by scale[j] on load.
//
// Orthogonalisation: full reorthogonalisation by two classical Gram-Schmidt sweeps against
// the whole basis, with the second sweep of each new vector delayed into the next iteration so
// that one iteration is one reduction pass, a small totals kernel where there are many partial
// rows (kDirectRows) and one update pass.  Slot j
// holds u1, the new vector after its first sweep, when iteration j starts; the block products
// are applied to that slot as it is (w_raw = H u1).  Then
//   reduce    a = V^H u1, b = V^H w_raw (slots c < j), c = u1^H w_raw, d = ||u1||^2,
//             e = ||w_raw||^2                                             (one pass)
//   algebra   (O(j) work, repeated by every block of the update pass)
//             second sweep of u1: u = u1 - V a, beta_j^2 = d - |a|^2, v_j = u / beta_j;
//             H u = w_raw - H V a, where H V a = V T a up to second order in the loss of
//             orthogonality (T: the Lanczos matrix so far), so w = H v_j is known in the basis:
//             h_c = v_c^H w = (b_c - t_c) / beta_j (c < j), t = T a,
//             h_j = (c - a^H b) / beta_j^2 - t_j / beta_j, alpha_j = Re h_j
//   update    slot j <- u; slot j+1 <- w - sum_c h_c v_c (first sweep of the next vector;
//             it contains the three-term recurrence, whose coefficients are h_j and h_{j-1})
//                                                                          (one pass)
// In exact arithmetic this is the two-sweep recurrence; the dropped terms are products of two
// quantities of the order of the loss of orthogonality.
//
// Every kernel runs over a table of problems (one entry for a single superblock, many for a
// batch): block b of a pass works on problem bmap[b] (problem 0 when there is no map), as block
// b - b0 of that problem's nb blocks; the small kernels run one block (or a few) per problem.
// The three kernels of a Lanczos iteration have a second instance for a lone problem, which
// takes its descriptor by value instead of from the table.
// Grid-wide sums are deterministic: every block writes its partial sums and a later kernel adds
// them in a fixed order (the kernel boundary orders the two; no device-wide fences or atomics:
// on this chip a device-scope release writes back the XCD's L2 and costs more than a launch).
#include <array>
#include <type_traits>
#include <utility>

#include "internal.hpp"
#include "tridiag.hpp"

namespace dmrg {

static_assert(kDVals % (kVecThreads / 64) == 0, "k_dsum: whole blocks of values");

namespace {

typedef const double __attribute__((address_space(1)))* gcptr;

typedef double d2v __attribute__((ext_vector_type(2)));
// Elements i, i + 1 (i even, p 16-byte aligned) of the slot starting at p.
__device__ __forceinline__ d2v ld2(const double* p, int64_t i) {
    return *((const d2v __attribute__((address_space(1)))*)(p + i));
}
__device__ __forceinline__ void st2(double* p, int64_t i, d2v v) {
    *((d2v __attribute__((address_space(1)))*)(p + i)) = v;
}

// Load of element i of the basis slot starting at p (global address space: the uniform slot
// base can live in scalar registers, the lane offset in one vector register).
__device__ __forceinline__ double ldv(const double* p, int64_t i) { return ((gcptr)p)[i]; }

// DPP move of a double (both 32-bit halves) with the given data-parallel-primitive control.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double lane_read(double v, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes of a wavefront, returned in every lane: butterflies inside each row of
// 16 lanes with DPP (quad swaps, half-row and row mirrors), then the four row sums read out
// with readlane.  Fixed order, no LDS traffic.
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp<0x141>(v);   // row_half_mirror: lane i <-> 7 - i within each half row
    v += dpp<0x140>(v);   // row_mirror: lane i <-> 15 - i within the row
    return (lane_read(v, 0) + lane_read(v, 16)) + (lane_read(v, 32) + lane_read(v, 48));
}

// The largest of the 64 lanes' values, returned in every lane.
__device__ __forceinline__ double wave_fmax(double v) {
    v = fmax(v, dpp<0xB1>(v));
    v = fmax(v, dpp<0x4E>(v));
    v = fmax(v, dpp<0x141>(v));
    v = fmax(v, dpp<0x140>(v));
    return fmax(fmax(lane_read(v, 0), lane_read(v, 16)), fmax(lane_read(v, 32), lane_read(v, 48)));
}

// Where block blockIdx.x of a pass works: problem bmap[blockIdx.x / mult] (0 without a map),
// block lb of the nbt = nb * mult blocks that pass gives that problem.
struct Where {
    VecProb p;
    int prob, lb, nbt;
};
__device__ __forceinline__ Where locate(const VecProb* vp, const int* bmap, int mult) {
    Where w;
    w.prob = bmap ? bmap[blockIdx.x / mult] : 0;
    w.p = vp[w.prob];
    w.lb = (int)blockIdx.x - w.p.b0 * mult;
    w.nbt = w.p.nb * mult;
    return w;
}

// The per-iteration passes are instantiated twice: ONE for a lone problem, whose descriptor
// comes by value with the kernel arguments (`one`), so the first data loads wait for no global
// load of a table entry; otherwise the table vp and the block map.  (A run-time choice between
// the two would read the descriptor through a generic pointer.)
template <bool ONE>
__device__ __forceinline__ Where locate1(const VecProb* vp, const int* bmap, const VecProb& one) {
    Where w;
    if constexpr (ONE) {
        w.prob = 0;
        w.p = one;
    } else {
        w.prob = bmap[blockIdx.x];
        w.p = vp[w.prob];
    }
    w.lb = (int)blockIdx.x - w.p.b0;
    w.nbt = w.p.nb;
    return w;
}

// The same for the reduction pass, which has its own block decomposition (nbr blocks per problem,
// several elements per thread, so that the per-block sums of its many values are amortised).
template <bool ONE>
__device__ __forceinline__ Where locate_red(const VecProb* vp, const int* bmapr,
                                            const VecProb& one) {
    Where w;
    if constexpr (ONE) {
        w.prob = 0;
        w.p = one;
    } else {
        w.prob = bmapr[blockIdx.x];
        w.p = vp[w.prob];
    }
    w.lb = (int)blockIdx.x - w.p.b0r;
    w.nbt = w.p.nbr;
    return w;
}

// Block-level sums of NV per-thread values; writes the block partials value-major,
// part[v * kVecMaxBlocks + lb], so that the finalise block reads each value's rows contiguously.
template <int NV>
__device__ __forceinline__ void block_partials(const double (&vals)[NV], double* part, int lb) {
    __shared__ double red[NV][kVecThreads / 64];
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int v = 0; v < NV; ++v) red[v][wave] = wave_sum(vals[v]);   // every lane holds the sum
    __syncthreads();
    for (int v = threadIdx.x; v < NV; v += blockDim.x) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kVecThreads / 64; ++w) s += red[v][w];
        part[(int64_t)v * kVecMaxBlocks + lb] = s;
    }
}

// Exchange partner for the reduce-scatter step on lane bit B: lane ^ B for the bits that cross
// rows of 16 (through the LDS permute network), otherwise a DPP move within the row whose
// partner differs in bit B (and possibly lower bits, which are not yet reduced).
template <int B>
__device__ __forceinline__ double partner(double v) {
    if constexpr (B >= 16) return __shfl_xor(v, B, 64);
    else if constexpr (B == 8) return dpp<0x140>(v);   // row_mirror: lane i <-> 15 - i
    else if constexpr (B == 4) return dpp<0x141>(v);   // row_half_mirror: i <-> 7 - i
    else if constexpr (B == 2) return dpp<0x4E>(v);    // quad_perm [2,3,0,1]
    else return dpp<0xB1>(v);                          // quad_perm [1,0,3,2]
}

// Reduce-scatter of P (a power of two, <= 64) per-lane values over the wavefront by recursive
// halving: at the step on lane bit B a lane keeps the half of its remaining values selected by
// that bit and adds its partner's copy of the same half; after log2 P steps each lane holds one
// value, the wavefront sum of value index lane >> (6 - log2 P), and the remaining lane bits are
// summed by plain butterflies.  P - 1 + 6 - log2 P exchanges instead of 6 P for P wave sums.
template <int P, int B = 32>
__device__ __forceinline__ void halve(double (&v)[P], int lane) {
    if constexpr (P > 1) {
        constexpr int H = P / 2;
        const bool upper = lane & B;
        double keep[H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const double give = upper ? v[i] : v[i + H];
            const double mine = upper ? v[i + H] : v[i];
            keep[i] = mine + partner<B>(give);
        }
        double (&w)[H] = *reinterpret_cast<double(*)[H]>(v);
#pragma unroll
        for (int i = 0; i < H; ++i) w[i] = keep[i];
        halve<H, B / 2>(w, lane);
    } else if constexpr (B >= 1) {
        v[0] += partner<B>(v[0]);
        halve<1, B / 2>(v, lane);
    }
}

// Finalise kernels run one block of FT threads per problem: totals[v] = sum_b part[v][b] for
// v < NV in a fixed order (thread t adds rows t, t + FT, ... in turn, then the block reduction
// of block_partials; nb <= kVecMaxBlocks, value-major layout as written by block_partials).
template <int NV, int FT = kVecThreads>
__device__ void final_sums(const double* part, int nb, double* totals_lds) {
    __shared__ double red[NV][FT / 64];
    const int wave = threadIdx.x >> 6;
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    // global-address-space loads: all NV of a row group are requested before the first use
    const gcptr gp = (gcptr)part;
#pragma unroll 1
    for (int q = 0; q < kVecMaxBlocks / FT; ++q) {
        const int b0 = q * FT + threadIdx.x;
        const int b = b0 < nb ? b0 : nb - 1;
        const double keep = b0 < nb ? 1.0 : 0.0;
        double x[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) x[v] = gp[(int64_t)v * kVecMaxBlocks + b];
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] += x[v] * keep;
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) red[v][wave] = wave_sum(acc[v]);   // every lane holds the sum
    __syncthreads();
    for (int v = threadIdx.x; v < NV; v += FT) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < FT / 64; ++w) t += red[v][w];
        totals_lds[v] = t;
    }
    __syncthreads();
}

// Starts a Krylov step from ||x||^2: beta0, scale0, per-step flags.
__device__ void begin_step(KState* st, double norm2, int kdim) {
    double b0 = sqrt(norm2);
    if (!isfinite(b0)) {          // NaN or infinity in the vector: flagged, run as zero
        st->nonfinite = 1;
        b0 = 0.0;
    }
    st->beta[0] = b0;
    st->kdim = kdim;
    if (b0 > 0.0) {
        st->scale[0] = 1.0 / b0;
        st->keff = kdim;
        st->broken = 0;
    } else {
        st->scale[0] = 0.0;
        st->keff = 0;
        st->broken = 1;
    }
}

}  // namespace

// ---------------------------------------------------------------------------------------
// start: slot 0 <- x, partial ||x||^2.  x is x1 (one problem) or xt[problem] (a batch).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kVecThreads) void k_start(const VecProb* vp, const int* bmap,
                                                       const double* x1,
                                                       const double* const* xt) {
    const Where W = locate(vp, bmap, 1);
    const double* __restrict__ x = xt ? xt[W.prob] : x1;
    double* __restrict__ u0 = W.p.V;
    const int64_t n = W.p.n;
    double acc[1] = {0.0};
    const int64_t stride = (int64_t)W.nbt * blockDim.x;
    for (int64_t i = (int64_t)W.lb * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double re = x[i], im = x[n + i];
        u0[i] = re;
        u0[n + i] = im;
        acc[0] += re * re + im * im;
    }
    block_partials<1>(acc, W.p.part, W.lb);
}

__global__ __launch_bounds__(kVecThreads) void k_fin_start(const VecProb* vp, int kdim, int first) {
    const VecProb P = vp[blockIdx.x];
    KState* st = P.st;
    __shared__ double tot[1];
    final_sums<1>(P.part, P.nb, tot);
    if (threadIdx.x == 0) {
        if (first) st->nonfinite = 0;
        begin_step(st, tot[0], kdim);
        st->err_est = 0.0;
        st->exp_fail = 0;
        if (first) {
            st->keff_min = kMaxKrylov + 1;
            st->any_break = 0;
            st->beta0_first = st->beta[0];
        }
    }
}

// ---------------------------------------------------------------------------------------
// Lanczos iteration j: reduction pass.  Launch q covers slots c0 .. c0+NC-1 (NC <= kDSlots);
// the first launch also accumulates u1^H w_raw, ||u1||^2 and ||w_raw||^2.  Partial rows of
// launch q: kDVals values (a_c, b_c per slot, then c, d, e), unused values zero.
// ---------------------------------------------------------------------------------------
// The inner products are one small matrix product, rows (Re v_c, Im v_c) of the slots by columns
// (Re u1, Im u1, Re w, Im w), summed over the elements: v_mfma_f64_4x4x4 takes two slots' rows by the
// four columns (no row or column unused) over 16 elements, lane (i, b, k) = (l mod 4, l div 4 mod 4,
// l div 16) row or column i of element (b, k), and D[i][j] of block b in lane j + 4 b + 16 i.  A wave
// reads 32 elements at a time (two per lane: 256 consecutive bytes of every row).
// Bound by memory traffic where there is much (16 slots of the 1000-state ladder: 77 MB, 18.6 us before,
// 16.2 now, 4.8 TB/s; twice or half as many groups in flight measured the same), by latency where there
// is little: with a lane's own sums (60 values, 300 registers) and their reduction over 64 lanes
// 15 slots of 48600 states took 7.5 us, with these 5.8.
typedef double d2m __attribute__((ext_vector_type(2), aligned(8)));    // any element
template <int NC, bool FIRST, bool ONE>
__global__ __launch_bounds__(kRedThreads) void k_dreduce(const VecProb* vp, const int* bmap, int j,
                                                         int c0, int q, VecProb one) {
    constexpr int NV = 4 * NC + (FIRST ? 4 : 0), NW = kRedThreads / 64;
    constexpr int T = (NC + 1) / 2, TT = T + (FIRST ? 1 : 0);          // tiles; the last: u1, w alone
    constexpr int S = 2;                                   // groups of 32 elements in flight
    const Where W = locate_red<ONE>(vp, bmap, one);
    // No breakdown test: the pass writes only its partial rows, which the totals kernel ignores
    // after a breakdown (the slots stay allocated, so every load is in bounds); a test here
    // would put the flag's load before the first data load.
    const int64_t n = W.p.n, vstride = W.p.vstride;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 3, e = 2 * (lane >> 2);
    // row i of tile t: slot c0 + 2 t + i / 2, plane i mod 2 (an odd NC's last rows are those of a
    // slot <= j, whose products are not used); column i: u1, then w
    typedef const d2m __attribute__((address_space(1)))* pairs;
    const gcptr pv = (gcptr)W.p.V + (int64_t)(c0 + (i >> 1)) * vstride + (i & 1) * n;
    const gcptr pb = (i < 2 ? (gcptr)W.p.V + (int64_t)j * vstride : (gcptr)W.p.w) + (i & 1) * n;
    double acc[TT > 0 ? TT : 1];
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[t] = 0.0;
    auto products = [&](double (&a)[T > 0 ? T : 1], double b) {
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[t], b, acc[t], 0, 0, 0);
        if (FIRST) acc[TT - 1] = __builtin_amdgcn_mfma_f64_4x4x4f64(b, b, acc[TT - 1], 0, 0, 0);
    };
    auto groups = [&](auto count, int64_t g, int64_t nw) {      // whole groups g, g + nw, ..
        constexpr int N = decltype(count)::value;
        d2m a[N][T > 0 ? T : 1], b[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int64_t at = 32 * (g + k * nw) + e;
            b[k] = *(pairs)(pb + at);
#pragma unroll
            for (int t = 0; t < T; ++t) a[k][t] = *(pairs)(pv + 2 * t * vstride + at);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                double x[T > 0 ? T : 1];
#pragma unroll
                for (int t = 0; t < T; ++t) x[t] = a[k][t][h];
                products(x, b[k][h]);
            }
    };
    const int64_t nfull = n / 32, nw = (int64_t)W.nbt * NW;
    int64_t g = (int64_t)W.lb * NW + wave;
    for (; g + (S - 1) * nw < nfull; g += S * nw) groups(std::integral_constant<int, S>{}, g, nw);
    for (; g < nfull; g += nw) groups(std::integral_constant<int, 1>{}, g, nw);
    if (g == nfull && n % 32 != 0) {                            // the rest: zeros beyond n
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t at = 32 * nfull + e + h, to = at < n ? at : n - 1;
            double x[T > 0 ? T : 1];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const double v = pv[2 * t * vstride + to];
                x[t] = at < n ? v : 0.0;
            }
            const double v = pb[to];
            products(x, at < n ? v : 0.0);
        }
    }
    // the four blocks of a tile, then the wavefronts
    __shared__ double red[NW][TT > 0 ? TT : 1][16];
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        double v = acc[t];
        v += dpp<0x128>(v);                                     // row_ror:8
        v += dpp<0x124>(v);                                     // row_ror:4
        if ((lane & 12) == 0) red[wave][t][4 * (lane >> 4) + i] = v;
    }
    __syncthreads();
    double* part = W.p.part + (int64_t)q * kRedStride * kDVals;
    for (int v = threadIdx.x; v < kDVals; v += kRedThreads) {
        double sum = 0.0;
        if (v < NV) {
            // entries (row, column) of the tile that make up value v: + first, +- second
            const int c = v >> 2, m = v & 3;
            int t = c >> 1, p, r;
            double sg;
            if (c < NC) {                                       // conj(v_c) u1, conj(v_c) w
                const int row = 8 * (c & 1), col = m & 2;
                p = row + col + (m & 1);
                r = row + 4 + col + 1 - (m & 1);
                sg = (m & 1) ? -1.0 : 1.0;
            } else {                                            // conj(u1) w, |u1|^2, |w|^2
                t = TT - 1;
                p = m == 0 ? 2 : m == 1 ? 3 : m == 2 ? 0 : 10;
                r = m == 0 ? 7 : m == 1 ? 6 : m == 2 ? 5 : 15;
                sg = m == 1 ? -1.0 : 1.0;
            }
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += red[w][t][p] + sg * red[w][t][r];
        }
        part[(int64_t)v * kRedStride + W.lb] = sum;
    }
}

// Totals of the reduction launches: every total is summed in the same order whichever kernel forms
// it.  Lane l adds partial rows l, l + 64, ... in turn, then the lanes are added in the order of
// the recursive halving (halve; tree_sum for one value).
__device__ __forceinline__ double tree_sum(double v) {
    v += partner<32>(v);
    v += partner<16>(v);
    v += partner<8>(v);
    v += partner<4>(v);
    v += partner<2>(v);
    v += partner<1>(v);
    return v;
}

// Lanczos iteration j: totals of the reduction launches in a launch of their own, for problems of
// many partial rows (launch_lanczos_iter).  Wave w of block (x, problem) sums value v = 4 x + w of
// the nq * kDVals values into the state; many blocks, so the partial rows are read in parallel
// across the chip rather than through one compute unit.
template <bool ONE>
__global__ __launch_bounds__(kVecThreads) void k_dsum(const VecProb* vp, VecProb one) {
    const VecProb P = ONE ? one : vp[blockIdx.y];
    KState* st = P.st;
    const int broken = ((const int __attribute__((address_space(1)))*)&st->broken)[0];
    const int lane = threadIdx.x & 63;
    const int v = blockIdx.x * (kVecThreads / 64) + (threadIdx.x >> 6);
    const gcptr row = (gcptr)(P.part + (int64_t)v * kRedStride);
    const int nbr = P.nbr;
    double x[kRedRows / 64];
#pragma unroll
    for (int k = 0; k < kRedRows / 64; ++k) {
        const int b = lane + 64 * k;
        x[k] = row[b < nbr ? b : nbr - 1] * (b < nbr ? 1.0 : 0.0);
    }
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kRedRows / 64; ++k) acc += x[k];
    acc = tree_sum(acc);
    if (lane == 0 && !broken) st->red[v] = acc;
}

// The same totals formed by every block of the update pass itself (kDVals values of each of nq
// launches into LDS): each wavefront takes a quarter of a launch's values, one per register.
__device__ __forceinline__ void sum_rows(const double* part, int nbr, int nq, double* tot) {
    constexpr int P = kDVals / (kVecThreads / 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int q = 0; q < nq; ++q) {
        const gcptr p = (gcptr)(part + (int64_t)q * kRedStride * kDVals) +
                        (int64_t)wave * P * kRedStride;
        double v[P];
#pragma unroll
        for (int i = 0; i < P; ++i) v[i] = 0.0;
        for (int b0 = 0; b0 < nbr; b0 += 64) {
            const int b = b0 + lane;
            const double keep = b < nbr ? 1.0 : 0.0;
            double x[P];
#pragma unroll
            for (int i = 0; i < P; ++i) x[i] = p[(int64_t)i * kRedStride + (b < nbr ? b : nbr - 1)];
#pragma unroll
            for (int i = 0; i < P; ++i) v[i] += x[i] * keep;
        }
        halve<P>(v, lane);
        constexpr int SPAN = 64 / P;
        if ((lane & (SPAN - 1)) == 0) tot[q * kDVals + wave * P + lane / SPAN] = v[0];
    }
}

// Coefficients of one update pass: co[x][c] (LDS, the wavefront's own) = {a_c, t_c, h_c} scale_c for
// x = 0, 1, 2 (c < j, zero up to j8), and slot j's in registers.
struct SlotJ {
    double s, tr, ti, hr, hi;     // scale_j, t_j scale_j, h_j scale_j
};

// Lanczos iteration j: the small algebra of the iteration (see the top of this file), run by
// every wavefront of the update pass from the totals of the reduction launches (row layout as
// above; the first launch has nc0 = min(j, kDSlots) slots) and the Lanczos matrix so far, so
// that no one-block launch sits between the reduction and the update.  Lane c holds slot c and
// neighbours come by DPP, so a wavefront needs no barrier and no other's results (with the steps
// split over a block between four barriers the pass of a 4900-state chain took 0.8 us longer).
// Every wavefront computes the same values in the same order; the first of block 0 of the problem
// (`writer`) stores alpha_j, beta_j, scale_j, the breakdown flag and, on the last iteration,
// beta_{j+1} from ||w||^2 - |h|^2 for the error estimate.  The others read only entries < j of the
// state, which nothing writes here.  Returns false (the same everywhere) when the basis has broken
// down.  total(i): total i of the launches.
template <class Total>
__device__ __forceinline__ bool iteration_coefficients(KState* st, int j, int kdim, int nc0,
                                                       bool writer, int j8, int broken, Total total,
                                                       double (&co)[3][2 * kMaxKrylov], SlotJ& cj) {
    const int lane = threadIdx.x & 63;
    const bool in = lane < j;
    const int c = in ? lane : 0;
    const int base = (c / kDSlots) * kDVals + 4 * (c % kDSlots);
    const double sc = in ? ((gcptr)st->scale)[c] : 0.0, al = in ? ((gcptr)st->alpha)[c] : 0.0;
    double be = in ? ((gcptr)st->beta)[c] : 0.0;
    const double beta0 = ((gcptr)st->beta)[0];
    double cde[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) cde[k] = total(4 * nc0 + k);
    const double Ar = in ? sc * total(base) : 0.0, Ai = in ? sc * total(base + 1) : 0.0;
    const double Br = in ? sc * total(base + 2) : 0.0, Bi = in ? sc * total(base + 3) : 0.0;
    if (broken) return false;   // an earlier iteration broke down: nothing is written
    // second sweep of u1: beta_j^2 = ||u1||^2 - |a|^2 (beta_0 = ||x|| from the start); breakdown
    // against the scale max(1, |alpha_c|, beta_c) over the iterations before j
    const double a2 = wave_sum(Ar * Ar + Ai * Ai);
    const double m = wave_fmax(fmax(fabs(al), lane >= 1 ? be : 0.0));
    double bj = beta0;
    if (j > 0) {
        bj = sqrt(fmax(cde[2] - a2, 0.0));
        const bool good = bj > 1e-12 * fmax(1.0, m);
        if (writer && lane == 0) {
            st->beta[j] = bj;
            if (good) {
                st->scale[j] = 1.0 / bj;
            } else {
                st->broken = 1;
                st->keff = j;
            }
        }
        if (!good) return false;
    }
    const double ib = 1.0 / bj;
    // u^H w_raw = c - a^H b
    const double ur = cde[0] - wave_sum(Ar * Br + Ai * Bi), ui = cde[1] - wave_sum(Ar * Bi - Ai * Br);
    // t = T a (lanes 0 .. j): T[m][m] = alpha_m, T[m][m-1] = beta_m, T[m][m+1] = beta_{m+1}
    if (lane == j) be = bj;
    const double bup = dpp<0x130>(be);                          // wave_shl: from lane + 1
    const double lo = lane >= 1 && lane <= j ? be : 0.0;
    const double Tr = al * Ar + lo * dpp<0x138>(Ar) + bup * dpp<0x130>(Ar);   // wave_shr: lane - 1
    const double Ti = al * Ai + lo * dpp<0x138>(Ai) + bup * dpp<0x130>(Ai);
    const double xr = (Br - Tr) * ib, xi = (Bi - Ti) * ib;      // h_c for c < j
    if (lane < j8) {
        co[0][2 * lane] = Ar * sc;
        co[0][2 * lane + 1] = Ai * sc;
        co[1][2 * lane] = Tr * sc;
        co[1][2 * lane + 1] = Ti * sc;
        co[2][2 * lane] = xr * sc;
        co[2][2 * lane + 1] = xi * sc;
    }
    const double tjr = lane_read(Tr, j), tji = lane_read(Ti, j);
    const double hr = ur * ib * ib - tjr * ib, hi = ui * ib * ib - tji * ib;
    if (writer && lane == 0) st->alpha[j] = hr;
    if (writer && j == kdim - 1) {
        // ||w||^2 = (e - 2 Re(t^H V^H w_raw) + |t|^2) / beta_j^2, V^H w_raw = (b, (u^H w_raw) / beta_j)
        const double tr = in ? Tr : 0.0, ti = in ? Ti : 0.0;
        const double yr = in ? xr : 0.0, yi = in ? xi : 0.0;
        const double tw = wave_sum(tr * Br + ti * Bi) + tjr * ur * ib + tji * ui * ib;
        const double t2 = wave_sum(tr * tr + ti * ti) + tjr * tjr + tji * tji;
        const double h2 = wave_sum(yr * yr + yi * yi) + hr * hr + hi * hi;
        const double w2 = (cde[3] - 2.0 * tw + t2) * ib * ib;
        if (lane == 0) {
            st->beta[j + 1] = sqrt(fmax(w2 - h2, 0.0));
            st->keff = kdim;
        }
    }
    cj = SlotJ{ib, tjr * ib, tji * ib, hr * ib, hi * ib};
    return true;
}

// Lanczos iteration j: update pass.  slot j <- u = u1 - sum_c a_c v_c; with v_j = u scale_j and
// w = (w_raw - sum_{c<j} t_c v_c - t_j v_j) scale_j: slot j+1 <- w - sum_{c<j} h_c v_c - h_j v_j
// (skipped after the last iteration).
template <bool ONE>
__global__ __launch_bounds__(kVecThreads) void k_dupdate(const VecProb* vp, const int* bmap, int j,
                                                         int kdim, int nc0, int nq_direct,
                                                         VecProb one) {
    const Where W = locate1<ONE>(vp, bmap, one);
    KState* st = W.p.st;
    const int broken = ((const int __attribute__((address_space(1)))*)&st->broken)[0];
    // basis slots loaded per round trip; a last group is padded with loads of slot j - 1, and eight at a
    // time padded more than they hid: 30-vector bases of the 8-site chain 2421 us and four chains of the
    // 1000-state ladder 4585 us with eight, 2365 and 4537 with four, 2370 and 4532 with two (a
    // 40-vector basis of 48600 states 4071, 4044 and 4197)
    constexpr int G = 4;
    const int j8 = (j + G - 1) / G * G;
    __shared__ double cos[kVecThreads / 64][3][2 * kMaxKrylov];
    double (&co)[3][2 * kMaxKrylov] = cos[threadIdx.x >> 6];
    SlotJ cj;
    double* __restrict__ uj = W.p.V + (int64_t)j * W.p.vstride;
    double* __restrict__ un = W.p.V + (int64_t)(j + 1) * W.p.vstride;
    const double* __restrict__ V = W.p.V;
    const double* __restrict__ w = W.p.w;
    const int64_t n = W.p.n, vstride = W.p.vstride;
    const int64_t stride = (int64_t)W.nbt * blockDim.x;
    const bool even = (n & 1) == 0;
    // even length: every element pair's loads of the first G basis slots are issued ahead of
    // its arithmetic, for the first pair before the coefficients, so that their latency
    // overlaps the small algebra; the slots are allocated whatever the state, and nothing is
    // stored after a breakdown
    const int64_t i0 = 2 * ((int64_t)W.lb * blockDim.x + threadIdx.x);
    d2v vr[G], vi[G];
    auto head = [&](int64_t i) {
        if (j > 0) {
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const double* v = V + (int64_t)min(k, j - 1) * vstride;
                vr[k] = ld2(v, i);
                vi[k] = ld2(v, n + i);
            }
        }
    };
    if (even && i0 < n) head(i0);
    __shared__ double tot[kDMaxQ * kDVals];
    const bool writer = W.lb == 0 && threadIdx.x < 64;
    if (nq_direct > 0) {
        sum_rows(W.p.part, W.p.nbr, nq_direct, tot);
        __syncthreads();
        if (!iteration_coefficients(st, j, kdim, nc0, writer, j8, broken,
                                    [&](int i) { return tot[i]; }, co, cj))
            return;
    } else if (!iteration_coefficients(st, j, kdim, nc0, writer, j8, broken,
                                       [&](int i) { return ((gcptr)st->red)[i]; }, co, cj)) {
        return;
    }
    // the lanes' coefficients before the others' reads of them: within a wavefront LDS accesses are
    // in order, so this holds the compiler only (no wait for the loads in flight)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const bool last = j == kdim - 1;
    const double sj = cj.s, tjr = cj.tr, tji = cj.ti, hjr = cj.hr, hji = cj.hi;
    if (even) {
        for (int64_t i = i0; i < n; i += 2 * stride) {
            if (i != i0) head(i);
            const d2v u0r = ld2(uj, i), u0i = ld2(uj, n + i), w0r = ld2(w, i), w0i = ld2(w, n + i);
            d2v ar = 0.0, ai = 0.0, tr = 0.0, ti = 0.0, hr = 0.0, hi = 0.0;
            for (int c0 = 0; c0 < j; c0 += G) {
                if (c0 > 0) {
#pragma unroll
                    for (int k = 0; k < G; ++k) {
                        const double* v = V + (int64_t)min(c0 + k, j - 1) * vstride;
                        vr[k] = ld2(v, i);
                        vi[k] = ld2(v, n + i);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    const int c = c0 + k;
                    ar += co[0][2 * c] * vr[k] - co[0][2 * c + 1] * vi[k];
                    ai += co[0][2 * c] * vi[k] + co[0][2 * c + 1] * vr[k];
                    tr += co[1][2 * c] * vr[k] - co[1][2 * c + 1] * vi[k];
                    ti += co[1][2 * c] * vi[k] + co[1][2 * c + 1] * vr[k];
                    hr += co[2][2 * c] * vr[k] - co[2][2 * c + 1] * vi[k];
                    hi += co[2][2 * c] * vi[k] + co[2][2 * c + 1] * vr[k];
                }
            }
            const d2v ur = u0r - ar, ui = u0i - ai;
            const d2v wr = (w0r - tr - (tjr * ur - tji * ui)) * sj;
            const d2v wi = (w0i - ti - (tjr * ui + tji * ur)) * sj;
            st2(uj, i, ur);
            st2(uj, n + i, ui);
            if (!last) {
                st2(un, i, wr - hr - (hjr * ur - hji * ui));
                st2(un, n + i, wi - hi - (hjr * ui + hji * ur));
            }
        }
        return;
    }
    for (int64_t i = (int64_t)W.lb * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double u0r = ldv(uj, i), u0i = ldv(uj, n + i), w0r = ldv(w, i), w0i = ldv(w, n + i);
        double ar = 0.0, ai = 0.0, tr = 0.0, ti = 0.0, hr = 0.0, hi = 0.0;
        for (int c0 = 0; c0 < j; c0 += G) {
            // G slots per round trip (slots past j - 1 re-read slot j - 1, zero coefficients)
            double vr[G], vi[G];
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const double* v = V + (int64_t)min(c0 + k, j - 1) * vstride;
                vr[k] = ldv(v, i);
                vi[k] = ldv(v, n + i);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const int c = c0 + k;
                ar += co[0][2 * c] * vr[k] - co[0][2 * c + 1] * vi[k];
                ai += co[0][2 * c] * vi[k] + co[0][2 * c + 1] * vr[k];
                tr += co[1][2 * c] * vr[k] - co[1][2 * c + 1] * vi[k];
                ti += co[1][2 * c] * vi[k] + co[1][2 * c + 1] * vr[k];
                hr += co[2][2 * c] * vr[k] - co[2][2 * c + 1] * vi[k];
                hi += co[2][2 * c] * vi[k] + co[2][2 * c + 1] * vr[k];
            }
        }
        const double ur = u0r - ar, ui = u0i - ai;
        const double wr = (w0r - tr - (tjr * ur - tji * ui)) * sj;
        const double wi = (w0i - ti - (tjr * ui + tji * ur)) * sj;
        uj[i] = ur;
        uj[n + i] = ui;
        if (!last) {
            un[i] = wr - hr - (hjr * ur - hji * ui);
            un[n + i] = wi - hi - (hjr * ui + hji * ur);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Small exponential: c(t_x) = beta0 exp(-i T t_x) e_1 for the k x k Lanczos matrix T
// (diagonal alpha, off-diagonal beta_1..beta_{k-1}), one wavefront per time and problem, lane r
// holding component r.  This is the quantity Sec. II.A obtains from T = S D S^T; on the device it is
// evaluated without the eigen-decomposition (a serial QL chase keeps one wavefront busy for
// ~1e5 cycles): T is shifted by the centre sigma of its Gershgorin interval (radius rho bounds
// ||T - sigma||_2), the vector is advanced to the target time in s substeps of length h with
// rho |h| <= 2, each by the Taylor series of exp(-i h (T - sigma)) to order 30, or fewer where rho |h| is
// smaller (first left-out term below 2^31 / 31! ~ 3e-25 relative; the largest term is at most 2,
// so no cancellation), and the phase exp(-i sigma t_x) is applied to the output.  Every term costs
// one tridiagonal product: two neighbour exchanges and three multiply-adds per lane.
// Bound by that dependent chain.  The four times of a step one after another, each from the last, with
// the neighbours through LDS and a division per term, took 23.8 us for the 400-state chain; 12.9.
// Also the error estimate beta_k |c_{k-1}(t_last)|.
// ---------------------------------------------------------------------------------------
namespace {

constexpr int kTaylorOrder = 30;
constexpr double kTaylorRadius = 2.0;
constexpr double kTaylorTail = 2.6e-25;     // 2^31 / 31!

}  // namespace

__global__ __launch_bounds__(64 * kMaxTimes) void k_tridiag_expm(const VecProb* vp, double t0,
                                                                 double t1, double t2, double t3,
                                                                 int ntimes, int* klog, int step) {
    KState* st = vp[blockIdx.x].st;
    const int r = threadIdx.x & 63;
    const int x = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);     // this wavefront's time
    const int k = st->keff;
    if (klog && threadIdx.x == 0) klog[step] = k > 0 ? k : 0;   // Lanczos vectors of this step
    if (k <= 0) {
        st->coef[x][2 * r] = 0.0;
        st->coef[x][2 * r + 1] = 0.0;
        if (threadIdx.x == 0) {
            st->err_est = 0.0;
            st->keff_min = 0;
            st->any_break = 1;
        }
        return;
    }
    __shared__ int s_bad;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    const bool in = r < k;
    const double a = in ? st->alpha[r] : 0.0;
    const double bl = (in && r >= 1) ? st->beta[r] : 0.0;     // couples r-1 and r
    const double bu = (r + 1 < k) ? st->beta[r + 1] : 0.0;    // couples r and r+1
    const double beta0 = st->beta[0], bk = st->beta[k];
    const double reach = fabs(bl) + fabs(bu);
    const double hi = wave_fmax(in ? a + reach : -INFINITY);
    const double lo = -wave_fmax(in ? reach - a : -INFINITY);
    const double sigma = 0.5 * (hi + lo), rho = 0.5 * (hi - lo);
    const double d = in ? a - sigma : 0.0;
    const double t = x == 0 ? t0 : x == 1 ? t1 : x == 2 ? t2 : t3;
    const double need = rho * fabs(t) / kTaylorRadius;
    const int64_t nsub = t == 0.0 ? 0 : (need <= 1.0 ? 1 : (int64_t)ceil(need));
    const double h = nsub ? t / (double)nsub : 0.0;
    const double hm = h / (double)max(r, 1);        // h / m in lane m
    // the order whose first left-out term is at most 2^31 / 31! for this radius too
    int order = 0;
    for (double term = 1.0; order < kTaylorOrder && !(term <= kTaylorTail);)
        term *= rho * fabs(lane_read(hm, ++order));
    double vr = (r == 0) ? beta0 : 0.0, vi = 0.0;
    for (int64_t sub = 0; sub < nsub; ++sub) {
        // sum_m (-i h (T - sigma))^m v / m!
        double sr = vr, si = vi, tr = vr, ti = vi;
#pragma unroll 2
        for (int m = 1; m <= order; ++m) {
            const double ur = d * tr + bl * dpp<0x138>(tr) + bu * dpp<0x130>(tr);
            const double ui = d * ti + bl * dpp<0x138>(ti) + bu * dpp<0x130>(ti);
            const double f = lane_read(hm, m);
            tr = f * ui;        // -i f (ur + i ui)
            ti = -f * ur;
            sr += tr;
            si += ti;
        }
        vr = sr;
        vi = si;
    }
    double sn, cs;
    sincos(sigma * t, &sn, &cs);                    // exp(-i sigma t) = cs - i sn
    const double cr = vr * cs + vi * sn, ci = vi * cs - vr * sn;
    st->coef[x][2 * r] = in ? cr : 0.0;
    st->coef[x][2 * r + 1] = in ? ci : 0.0;
    if (__any(!isfinite(cr) || !isfinite(ci)) && r == 0) atomicOr(&s_bad, 1);
    __syncthreads();
    if (x != ntimes - 1) return;
    const double er = lane_read(cr, k - 1), ei = lane_read(ci, k - 1);
    if (r == 0) {
        st->err_est = st->broken ? 0.0 : bk * sqrt(er * er + ei * ei);
        st->exp_fail = s_bad;
        st->keff_min = min(st->keff_min, k);
        st->any_break = st->any_break | st->broken;
    }
}

// ---------------------------------------------------------------------------------------
// Ground-state targeting (the same Lanczos basis, with the lowest eigenpair of T in place of
// the exponential): one wavefront per problem.  The lowest eigenvalue lambda of the k x k
// tridiagonal T is found by multisection of its Gershgorin interval: each round, lane l counts
// the eigenvalues below the l-th of 64 interior points (signs of the leading minors) and
// the interval shrinks to the first gap that holds lambda, 65 times narrower.  Its eigenvector z
// then comes from three steps of inverse iteration on T - lambda, solved by Gaussian
// elimination with partial pivoting (every lane the same, rows loaded in runs; tiny pivots replaced by
// a floor).
// Output: coef[0] = z (real, unit norm; the combination gives the unit Ritz vector V z),
// eig = lambda, err_est = beta_k |z_{k-1}| (the residual norm ||H V z - lambda V z||).
// Bound by dependent arithmetic: 25 us for 40 vectors.  With a division per pivot of the counts, and the
// solves on one lane that waited for LDS at every step, it was 78 us.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_tridiag_lowest(const VecProb* vp, int* klog, int step) {
    KState* st = vp[blockIdx.x].st;
    const int r = threadIdx.x;
    const int k = st->keff;
    if (klog && r == 0) klog[step] = k > 0 ? k : 0;     // Lanczos vectors of this basis
    if (k <= 0) {
        st->coef[0][2 * r] = 0.0;
        st->coef[0][2 * r + 1] = 0.0;
        if (r == 0) {
            st->err_est = 0.0;
            st->eig = 0.0;
            st->keff_min = 0;
            st->any_break = 1;
        }
        return;
    }
    __shared__ double al[kMaxKrylov], bt[kMaxKrylov];   // alpha_i; beta_{i+1}, between i and i + 1
    __shared__ double rec[2 * kMaxKrylov];              // T scaled, in runs (sturm_count)
    __shared__ __align__(16) double inv[6 * kMaxKrylov];
    static_assert(kMaxKrylov == 64 && kMaxKrylov % kSturmRun == 0, "a lane per row, whole runs");
    const bool in = r < k;
    const double a = in ? st->alpha[r] : 0.0;
    const double bl = (in && r >= 1) ? st->beta[r] : 0.0;
    const double bu = (r + 1 < k) ? st->beta[r + 1] : 0.0;
    al[r] = a;
    bt[r] = bu;
    const double reach = fabs(bl) + fabs(bu);
    double hi = wave_fmax(in ? a + reach : -INFINITY);
    double lo = -wave_fmax(in ? reach - a : -INFINITY);
    const double tnorm = fmax(fabs(hi), fabs(lo));
    const double pivmin = 1e-290 * fmax(1.0, tnorm * tnorm);
    // the counts run on the matrix scaled by a power of two to |T| in [0.5, 1)
    const int ex = __builtin_amdgcn_frexp_exp(fmax(tnorm, 1e-300));
    const double bs = __builtin_amdgcn_ldexp(bl, -ex);
    rec[2 * kSturmRun * (r / kSturmRun) + r % kSturmRun] = in ? __builtin_amdgcn_ldexp(a, -ex) : 4.0;
    rec[2 * kSturmRun * (r / kSturmRun) + kSturmRun + r % kSturmRun] = bs * bs;
    __syncthreads();
    // multisection: count(x) = number of eigenvalues below x
    for (int it = 0; it < 16; ++it) {
        const double x = lo + (hi - lo) * (double)(r + 1) / 65.0;
        const int cnt = sturm_count((k + kSturmRun - 1) / kSturmRun, rec, __builtin_amdgcn_ldexp(x, -ex));
        const unsigned long long m = __ballot(cnt >= 1);
        const int f = m ? __ffsll(m) - 1 : 64;     // first point above lambda (64: the top end)
        const double nlo = f == 0 ? lo : lo + (hi - lo) * (double)f / 65.0;
        const double nhi = f == 64 ? hi : lo + (hi - lo) * (double)(f + 1) / 65.0;
        lo = nlo;
        hi = nhi;
        if (hi - lo <= 4.0 * 2.220446049250313e-16 * fmax(fabs(lo), fabs(hi)) + pivmin) break;
    }
    const double lam = 0.5 * (lo + hi);
    // inverse iteration from a vector of ones; every lane runs the same solves
    const InvLds m{inv, 1, 6};
    tri_factor<true>(m, k, 0, al, bt, lam, fmax(pivmin, 2.220446049250313e-16 * tnorm),
                     [] { return 1.0; });
    double z = 0.0, nrm = tri_backward(m, k, 0);
    for (int it = 1; it < 3; ++it) nrm = tri_solve(m, k, 0, 1.0 / sqrt(nrm));
    // unit norm, the first of the largest entries positive
    z = in ? m.z(m.at(r, 0)) : 0.0;
    const double big = wave_fmax(fabs(z));
    const unsigned long long at = __ballot(in && fabs(z) == big);
    const double sign = at && lane_read(z, __ffsll(at) - 1) < 0.0 ? -1.0 : 1.0;
    z *= sign / sqrt(nrm);
    const double zk = lane_read(z, k - 1);
    if (r == 0) {
        st->eig = lam;
        st->err_est = st->broken ? 0.0 : fabs(st->beta[k] * zk);
        st->exp_fail = !isfinite(lam) || !isfinite(zk);
        st->keff_min = min(st->keff_min, k);
        st->any_break = st->any_break | st->broken;
    }
    st->coef[0][2 * r] = in ? z : 0.0;
    st->coef[0][2 * r + 1] = 0.0;
}

// ---------------------------------------------------------------------------------------
// combine: y_x = sum_{c < keff} coef_x[c] scale_c u_c for x < ntimes.  With chain != 0 the
// single output is slot 0 itself (in place) and its norm seeds the next step.  Outputs of a
// batch come from the table yst[problem * kMaxTimes + x].  Without chaining a pass may give
// each problem mult blocks per block of the other passes (no partial sums to collect).
// ---------------------------------------------------------------------------------------
// X: the times of the launch (1, or up to kMaxTimes).  G slots' loads are in flight at once, the first
// ones before the coefficients are there: with four at a time, after the coefficients, 30 slots of 4900
// states took 11.5 us, now 6.2; 40 slots of 48600 states 27.4, now 11.2; many states are bound by
// memory traffic either way (the 1000-state ladder 19.8, now 19.1; four chains of it 57.6 and 57.4, with
// 16 slots at a time, whose registers leave fewer wavefronts, 67).
template <int X>
__global__ __launch_bounds__(kVecThreads) void k_combine(const VecProb* vp, const int* bmap,
                                                         int mult, double* y0, double* y1,
                                                         double* y2, double* y3,
                                                         double* const* yst, int ntimes,
                                                         int chain) {
    constexpr int G = X == 1 ? 8 : 4;
    const Where W = locate(vp, bmap, mult);
    const KState* st = W.p.st;
    __shared__ double cs[X][2 * kMaxKrylov];
    static_assert(kMaxKrylov % G == 0, "whole groups of slots");
    const int k = st->keff, kg = (k + G - 1) / G * G;
    const double* V = W.p.V;
    const int64_t n = W.p.n, vstride = W.p.vstride;
    const int64_t first = (int64_t)W.lb * blockDim.x + threadIdx.x;
    double vr[G], vi[G];
    auto load = [&](int64_t i, int c0) {                // slots from k on re-read slot k - 1
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const double* u = V + (int64_t)min(c0 + g, k - 1) * vstride;
            vr[g] = ldv(u, i);
            vi[g] = ldv(u, n + i);
        }
    };
    if (k > 0 && first < n) load(first, 0);
    for (int idx = threadIdx.x; idx < X * kg; idx += blockDim.x) {
        const int x = idx / kg, c = idx % kg;
        const bool ok = x < ntimes && c < k;            // the rest of a group: zero
        const double s = ok ? st->scale[c] : 0.0;
        cs[x][2 * c] = ok ? st->coef[x][2 * c] * s : 0.0;
        cs[x][2 * c + 1] = ok ? st->coef[x][2 * c + 1] * s : 0.0;
    }
    __syncthreads();
    double* ys[kMaxTimes];
    if (chain) {
        ys[0] = W.p.V;
        ys[1] = ys[2] = ys[3] = nullptr;
    } else if (yst) {
#pragma unroll
        for (int x = 0; x < kMaxTimes; ++x) ys[x] = yst[W.prob * kMaxTimes + x];
    } else {
        ys[0] = y0;
        ys[1] = y1;
        ys[2] = y2;
        ys[3] = y3;
    }
    double acc[1] = {0.0};
    const int64_t stride = (int64_t)W.nbt * blockDim.x;
    for (int64_t i = first; i < n; i += stride) {
        double yr[X], yi[X];
#pragma unroll
        for (int x = 0; x < X; ++x) {
            yr[x] = 0.0;
            yi[x] = 0.0;
        }
        for (int c0 = 0; c0 < k; c0 += G) {
            if (c0 > 0 || i != first) load(i, c0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int c = c0 + g;
#pragma unroll
                for (int x = 0; x < X; ++x) {
                    const double cr = cs[x][2 * c], ci = cs[x][2 * c + 1];
                    yr[x] += cr * vr[g] - ci * vi[g];
                    yi[x] += cr * vi[g] + ci * vr[g];
                }
            }
        }
#pragma unroll
        for (int x = 0; x < X; ++x) {
            if (x < ntimes) {
                ys[x][i] = yr[x];
                ys[x][n + i] = yi[x];
            }
        }
        acc[0] += yr[0] * yr[0] + yi[0] * yi[0];
    }
    if (chain) block_partials<1>(acc, W.p.part, W.lb);
}

__global__ __launch_bounds__(kVecThreads) void k_fin_chain(const VecProb* vp) {
    const VecProb P = vp[blockIdx.x];
    __shared__ double tot[1];
    final_sums<1>(P.part, P.nb, tot);
    if (threadIdx.x == 0) begin_step(P.st, tot[0], P.st->kdim);
}

// ---------------------------------------------------------------------------------------
// launchers.  vp: device table of nprob problems; bmap: block -> problem map of the nblk
// blocks of a pass (nullptr for a single problem).
// ---------------------------------------------------------------------------------------
// Blocks of a vector pass for one problem: about one element per thread (enough waves in flight
// to cover the memory latency of these streaming passes), at most kVecMaxBlocks rows of partial
// sums.
int vec_blocks(int64_t n) {
    int64_t nb = (n / 2 + kVecThreads - 1) / kVecThreads;
    if (nb < 1) nb = 1;
    if (nb > kVecMaxBlocks) nb = kVecMaxBlocks;
    return (int)nb;
}

// Blocks (partial rows) of the Lanczos reduction pass: a group of 32 elements per wavefront, or as many
// groups each as keep the rows at most kRedRows, one block of 16 wavefronts per CU.  Blocks of four
// wavefronts with 512 elements each (587 rows for 300000 states) took 1289 us for the targets of the
// 1000-state ladder and 8329 for a 2000-state basis, these 1236 and 8251; with up to 128 rows 1272 and
// 8605, with 512 1284 and 8276.  Four chains or 16 problems in common launches measure the same (4537
// and 4545 us, 5862 and 5878), small ones less rounds per wavefront (10 bases of the 8-site chain
// 2365 and 2331 us, a 400-state chain's ground state 4044 and 3950).
int red_blocks(int64_t n) {
    constexpr int64_t waves = kRedThreads / 64;
    const int64_t groups = n > 32 ? (n + 31) / 32 : 1;
    const int64_t rounds = (groups + waves * kRedRows - 1) / (waves * kRedRows);
    return (int)((groups + waves * rounds - 1) / (waves * rounds));
}
static_assert(kRedRows <= kVecMaxBlocks, "rows of partial sums");

hipError_t launch_start(const VecGroup& g, const double* x1, const double* const* xt, int kdim,
                        int first, hipStream_t s) {
    hipLaunchKernelGGL(k_start, dim3(g.nblk), dim3(kVecThreads), 0, s, g.vp, g.bmap, x1, xt);
    hipLaunchKernelGGL(k_fin_start, dim3(g.nprob), dim3(kVecThreads), 0, s, g.vp, kdim, first);
    return hipGetLastError();
}

namespace {

typedef void (*RedFn)(const VecProb*, const int*, int, int, int, VecProb);

template <bool FIRST, bool ONE, int... I>
constexpr auto red_table(std::integer_sequence<int, I...>) {
    return std::array<RedFn, sizeof...(I)>{&k_dreduce<I, FIRST, ONE>...};
}

// [one problem][slots of the launch]
const std::array<RedFn, kDSlots + 1> kRedFirst[2] = {
    red_table<true, false>(std::make_integer_sequence<int, kDSlots + 1>{}),
    red_table<true, true>(std::make_integer_sequence<int, kDSlots + 1>{})};
const std::array<RedFn, kDSlots + 1> kRedMore[2] = {
    red_table<false, false>(std::make_integer_sequence<int, kDSlots + 1>{}),
    red_table<false, true>(std::make_integer_sequence<int, kDSlots + 1>{})};

}  // namespace

// Runs Lanczos iteration j (after the block products of slot j) on every problem of the group.
hipError_t launch_lanczos_iter(const VecGroup& g, int j, int kdim, hipStream_t s) {
    const dim3 grid(g.nblk), gridr(g.nblkr), blk(kVecThreads), blkr(kRedThreads);
    const int nq = j > kDSlots ? (j + kDSlots - 1) / kDSlots : 1;
    const int nc0 = min(j, kDSlots);
    // one problem (no block map): its descriptor travels by value
    const int one = g.nprob == 1 && g.bmap == nullptr && g.bmapr == nullptr;
    const VecProb* vp = g.vp;
    hipLaunchKernelGGL(kRedFirst[one][nc0], gridr, blkr, 0, s, vp, g.bmapr, j, 0, 0, g.one);
    for (int q = 1; q < nq; ++q) {
        const int nc = min(kDSlots, j - q * kDSlots);
        hipLaunchKernelGGL(kRedMore[one][nc], gridr, blkr, 0, s, vp, g.bmapr, j, q * kDSlots, q,
                           g.one);
    }
    // few partial rows: every block of the update pass sums them itself
    const int direct = nq * g.max_nbr <= kDirectRows ? nq : 0;
    const dim3 grids(nq * kDVals / (kVecThreads / 64), g.nprob);
    if (one) {
        if (!direct) hipLaunchKernelGGL(k_dsum<true>, grids, blk, 0, s, vp, g.one);
        hipLaunchKernelGGL(k_dupdate<true>, grid, blk, 0, s, vp, g.bmap, j, kdim, nc0, direct, g.one);
    } else {
        if (!direct) hipLaunchKernelGGL(k_dsum<false>, grids, blk, 0, s, vp, g.one);
        hipLaunchKernelGGL(k_dupdate<false>, grid, blk, 0, s, vp, g.bmap, j, kdim, nc0, direct, g.one);
    }
    return hipGetLastError();
}

// klog (one problem only, else nullptr): device array receiving the Lanczos vectors of the
// basis at index step.
hipError_t launch_lowest(const VecGroup& g, int* klog, int step, hipStream_t s) {
    hipLaunchKernelGGL(k_tridiag_lowest, dim3(g.nprob), dim3(64), 0, s, g.vp, klog, step);
    return hipGetLastError();
}

hipError_t launch_tridiag(const VecGroup& g, const double* times, int ntimes, int* klog, int step,
                          hipStream_t s) {
    double t[kMaxTimes] = {0, 0, 0, 0};
    for (int i = 0; i < ntimes; ++i) t[i] = times[i];
    hipLaunchKernelGGL(k_tridiag_expm, dim3(g.nprob), dim3(64 * ntimes), 0, s, g.vp, t[0], t[1], t[2],
                       t[3], ntimes, klog, step);
    return hipGetLastError();
}

// Number of non-finite values among x[0 .. m) added to *count (which the caller zeroes):
// integer atomics, one per thread that found any (their sum does not depend on the order).
__global__ __launch_bounds__(kVecThreads) void k_count_nonfinite(const double* __restrict__ x,
                                                                 int64_t m, int* count) {
    int c = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride)
        c += !isfinite(x[i]);
    if (c) atomicAdd(count, c);       // only where non-finite values were found
}

hipError_t launch_count_nonfinite(const double* x, int64_t m, int* count, hipStream_t s) {
    int64_t nb = (m + kVecThreads - 1) / kVecThreads;
    if (nb > 1024) nb = 1024;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_count_nonfinite, dim3((unsigned)nb), dim3(kVecThreads), 0, s, x, m, count);
    return hipGetLastError();
}

// ys: ntimes output pointers of a single problem, or nullptr with yst, the batch table
// [nprob][kMaxTimes].  chain: write slot 0 in place and start the next step from it.
hipError_t launch_combine(const VecGroup& g, double* const* ys, double* const* yst, int ntimes,
                          int chain, hipStream_t s) {
    double* y[kMaxTimes] = {nullptr, nullptr, nullptr, nullptr};
    if (ys)
        for (int i = 0; i < ntimes; ++i) y[i] = ys[i];
    const int mult = chain ? 1 : g.combine_mult;
    auto* const kern = ntimes == 1 ? &k_combine<1> : &k_combine<kMaxTimes>;
    hipLaunchKernelGGL(kern, dim3(g.nblk * mult), dim3(kVecThreads), 0, s, g.vp, g.bmap, mult, y[0],
                       y[1], y[2], y[3], yst, ntimes, chain);
    if (chain) hipLaunchKernelGGL(k_fin_chain, dim3(g.nprob), dim3(kVecThreads), 0, s, g.vp);
    return hipGetLastError();
}

}  // namespace dmrg
