// Wave-function transformation (FP64, gfx950): products of complex matrices on the FP64 MFMA.
//
// Sec. II.B: when the centre moves one site to the right, a target psi on
// (A x s1) x (s2 x R) is carried to (A' x s2) x (s3 x R'') by
//   stage A   Phi[(alpha', a), beta] = sum_alpha conj(U[alpha, alpha']) psi[alpha, (a, beta)]
//             (U: the kept eigenvectors of the system's density matrix; one product per
//             sub-block (kept sector, site state a, R sector), written into the rows of the new
//             system sector that the sub-block occupies: the regrouping of s2 is the write
//             address, with no sign since the bases are normal-ordered)
//   stage B   psi'[(alpha', a), gamma] = sum_beta Phi[(alpha', a), beta] W[gamma, beta]
//             (W_r: the states of R sector r in the product basis of s3 x R'')
// Both stages are one launch over a list of 16 x 16 output tiles for every vector of the call, one
// wavefront per tile and vector, with two accumulators: Re C += Re A Re B - Im A Im B and
// Im C += Re A Im B + Im A Re B.
#include <algorithm>
#include <cstdint>

#include "internal.hpp"

namespace dmrg {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));   // 8-byte aligned
typedef const double __attribute__((address_space(1)))* gcptr;

// The K index of MFMA u of a chunk of 16 in lane group g: pairs, so that a row's four lane groups
// read 64 consecutive bytes with one 16-byte load each.
__device__ __forceinline__ int koff(int g, int u) { return 8 * (u >> 1) + 2 * g + (u & 1); }
// The four values of one lane from a row that starts at p and runs along K (8-byte aligned).
__device__ __forceinline__ d4 ld4u(gcptr p, int g) {
    const d2u a = *((const __attribute__((address_space(1))) d2u*)(p + 2 * g));
    const d2u b = *((const __attribute__((address_space(1))) d2u*)(p + 8 + 2 * g));
    return (d4){a[0], a[1], b[0], b[1]};
}

// Offset of operand element (i, k) of A, (k, j) of B, and its step along K (modes of the planner;
// the identity has no elements).
template <int AM>
__device__ __forceinline__ int64_t at_a(const ZTile& t, int i, int k) {
    return t.aoff + (AM == ZM_COL || AM == ZM_RCOL ? (int64_t)k * t.lda + i : (int64_t)i * t.lda + k);
}
template <int BM>
__device__ __forceinline__ int64_t at_b(const ZTile& t, int k, int j) {
    return t.boff + (BM == ZM_COL || BM == ZM_RCOL ? (int64_t)j * t.ldb + k : (int64_t)k * t.ldb + j);
}

__device__ __forceinline__ d4 mma4(const double (&a)[4], const double (&b)[4], d4 c) {
#pragma unroll
    for (int u = 0; u < 4; ++u) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], c, 0, 0, 0);
    return c;
}

}  // namespace

constexpr int kZWaves = 4;          // tiles (wavefronts) of a work group
constexpr int kZBuf = 2;            // chunks held by a wavefront
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// One wavefront per 16 x 16 output tile, four neighbours of the list in a work group, work groups
// tile-major over the vectors.  Lane (g, r) = (lane / 16, lane % 16) supplies rows (columns) r and
// the K indices koff(g, u) of a chunk of 16; B goes in as the MFMA's first operand, so that result
// element (row r, column g + 4 q) is accumulator component q and 16 lanes store consecutive rows.
// Rows and columns outside the matrix read the last one (they only enter results that are not
// stored); K indices beyond K are zero in both operands.
// Bound by load latency: five vectors of the 1000-state ladder's move are 0.6 GFLOP (13 us of
// padded MFMAs if spread evenly) and 60 MB, but the longest tiles run 10 chunks in turn.  So the
// tiles are small (they end sooner, and 3800 of them fill 1024 SIMDs more evenly than 2300 of
// 32 x 32, whose operands also left no room beside the accumulators: the compiler moved these to
// accumulation registers and back around every chunk), the planner lists the longest K first, and
// a tile's neighbours share its part of the vector in the CU's L1.  Stage A 47.0 -> 21.0 us, stage
// B 25.5 -> 17.3 us; three or four chunks in flight measured the same.
template <int AM, int BM>
__global__ __launch_bounds__(64 * kZWaves, 3) void k_zgemm(const ZTile* __restrict__ tiles, int n,
                                                           ZPtrs ptr, int nvec) {
    const int ti = (int)(blockIdx.x / nvec) * kZWaves + wave_id();
    if (ti >= n) return;
    const ZTile t = tiles[ti];
    const int v = blockIdx.x % nvec;
    const gcptr A = (gcptr)ptr.a[v];
    const gcptr B = (gcptr)ptr.b[v];
    double* __restrict__ C = ptr.c[v];
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    const int i = min(t.m0 + r, t.M - 1), j = min(t.n0 + r, t.N - 1);
    d4 cre = (d4){0.0, 0.0, 0.0, 0.0}, cim = cre;
    double ar[kZBuf + 1][4], ai[kZBuf + 1][4], br[kZBuf + 1][4], bi[kZBuf + 1][4];   // [buffer][u]; last: the tail
    auto load = [&](int buf, int k0) {
        if (buf < kZBuf) {                     // a whole chunk: no tests
            if constexpr (AM == ZM_CT) {               // four consecutive values per plane
                const gcptr p = A + at_a<AM>(t, i, k0);
                const d4 re = ld4u(p, g), im = ld4u(p + t.aim, g);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    ar[buf][u] = re[u];
                    ai[buf][u] = -im[u];               // conjugate transpose
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int k = k0 + koff(g, u);
                    const int64_t at = at_a<AM>(t, i, k);
                    ar[buf][u] = AM == ZM_ID ? (t.m0 + r == k ? 1.0 : 0.0) : A[at];
                    ai[buf][u] = AM == ZM_COL ? A[at + t.aim] : 0.0;
                }
            }
            if constexpr (BM == ZM_COL) {
                const gcptr p = B + at_b<BM>(t, k0, j);
                const d4 re = ld4u(p, g), im = ld4u(p + t.bim, g);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    br[buf][u] = re[u];
                    bi[buf][u] = im[u];
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t at = at_b<BM>(t, k0 + koff(g, u), j);
                    br[buf][u] = B[at];
                    bi[buf][u] = BM == ZM_CT ? B[at + t.bim] : 0.0;   // transpose only
                }
            }
            return;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ku = k0 + koff(g, u), k = min(ku, t.K - 1);
            const bool ok = ku < t.K;
            double xr, xi = 0.0;
            if constexpr (AM == ZM_ID) {
                xr = t.m0 + r == ku ? 1.0 : 0.0;
            } else {
                const int64_t at = at_a<AM>(t, i, k);
                xr = A[at];
                if constexpr (AM == ZM_COL || AM == ZM_CT) xi = A[at + t.aim];
            }
            const int64_t bt = at_b<BM>(t, k, j);
            const double yr = B[bt], yi = BM == ZM_COL || BM == ZM_CT ? B[bt + t.bim] : 0.0;
            ar[buf][u] = ok ? xr : 0.0;
            ai[buf][u] = ok ? (AM == ZM_CT ? -xi : xi) : 0.0;
            br[buf][u] = ok ? yr : 0.0;
            bi[buf][u] = ok ? yi : 0.0;
        }
    };
    auto mma = [&](int buf) {
        double an[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) an[u] = -ai[buf][u];
        // B first: the result block then has its rows along the lanes
        cre = mma4(br[buf], ar[buf], cre);
        cim = mma4(bi[buf], ar[buf], cim);
        cre = mma4(bi[buf], an, cre);
        cim = mma4(br[buf], ai[buf], cim);
    };
    // The rest of K first, then whole chunks, chunks c + 1 .. c + kZBuf - 1 on their way while chunk c
    // is multiplied.  The loads in the loop are unconditional (the last ones repeat the last
    // chunk): a load that may be left out would make every wait one for all loads in flight.
    const int nfull = t.K >> 4;
    const bool tail = (t.K & 15) != 0;
    if (tail) load(kZBuf, 16 * nfull);
    if (nfull > 0) {
#pragma unroll
        for (int b = 0; b + 1 < kZBuf; ++b) load(b, 16 * min(b, nfull - 1));
        int c = 0;
        for (; c + kZBuf <= nfull; c += kZBuf) {
#pragma unroll
            for (int b = 0; b < kZBuf; ++b) {
                load((b + kZBuf - 1) % kZBuf, 16 * min(c + b + kZBuf - 1, nfull - 1));
                mma(b);
            }
        }
#pragma unroll
        for (int b = 0; b + 1 < kZBuf; ++b)
            if (c + b < nfull) mma(b);
    }
    if (tail) mma(kZBuf);
    const int ic = t.m0 + r;
    if (ic >= t.M) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int jc = t.n0 + g + 4 * q;
        if (jc >= t.N) continue;
        const int64_t at = t.coff + (int64_t)jc * t.ldc + ic;
        double vr = t.alpha * cre[q], vi = t.alpha * cim[q];
        if (t.acc) {
            vr += C[at];
            vi += C[at + t.cim];
        }
        C[at] = vr;
        C[at + t.cim] = vi;
    }
}

// Launch of one tile list whose tiles share the operand modes (am, bm).
hipError_t launch_zgemm_modes(const ZTile* t, int n, const ZPtrs& p, int nvec, int am, int bm,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const dim3 grid((unsigned)((n + kZWaves - 1) / kZWaves) * nvec);
#define DMRG_ZGEMM_CASE(A_, B_)                                                            \
    if (am == A_ && bm == B_) {                                                            \
        hipLaunchKernelGGL((k_zgemm<A_, B_>), grid, dim3(64 * kZWaves), 0, s, t, n, p, nvec);                \
        return hipGetLastError();                                                          \
    }
    DMRG_ZGEMM_CASE(ZM_CT, ZM_COL)        // wave-function transformation, stage A
    DMRG_ZGEMM_CASE(ZM_COL, ZM_CT)        // wave-function transformation, stage B
    DMRG_ZGEMM_CASE(ZM_COL, ZM_RT)        // local operators: right products
    DMRG_ZGEMM_CASE(ZM_COL, ZM_RCOL)
    DMRG_ZGEMM_CASE(ZM_RCOL, ZM_COL)      // local operators: left products
    DMRG_ZGEMM_CASE(ZM_RT, ZM_COL)
    DMRG_ZGEMM_CASE(ZM_ID, ZM_COL)
#undef DMRG_ZGEMM_CASE
    return hipErrorInvalidValue;
}

__global__ __launch_bounds__(256) void k_zero(double* __restrict__ x, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        x[i] = 0.0;
}

// Stage A then stage B for nvec vectors; zero_n > 0 first clears the intermediate (nvec
// consecutive pieces of zero_n doubles from pA.c[0]), for moves whose sub-blocks leave rows of
// it unwritten.
hipError_t launch_wft(const ZTile* tA, int nA, const ZPtrs& pA, const ZTile* tB, int nB,
                      const ZPtrs& pB, int nvec, int64_t zero_n, hipStream_t s) {
    if (nvec < 1 || nvec > kWftMaxVec) return hipErrorInvalidValue;
    if (zero_n > 0) {
        const int64_t tot = zero_n * nvec;
        const int blocks = (int)std::min<int64_t>((tot + 255) / 256, 4096);
        hipLaunchKernelGGL(k_zero, dim3(blocks), dim3(256), 0, s, pA.c[0], tot);
    }
    hipError_t e = launch_zgemm_modes(tA, nA, pA, nvec, ZM_CT, ZM_COL, s);
    if (e == hipSuccess) e = launch_zgemm_modes(tB, nB, pB, nvec, ZM_COL, ZM_CT, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

// One list of product tiles for nvec vectors (local operators, Sec. II.B: B|psi> and the
// measured operators).
hipError_t launch_zgemm(const ZTile* t, int n, const ZPtrs& p, int nvec, int am, int bm,
                        hipStream_t s) {
    if (nvec < 1 || nvec > kWftMaxVec) return hipErrorInvalidValue;
    return launch_zgemm_modes(t, n, p, nvec, am, bm, s);
}

// Sum of (ar, ai) over the work group's four wavefronts into part[0], part[1].
__device__ __forceinline__ void store_group_sum(double ar, double ai, double* __restrict__ part) {
    __shared__ double sr[4], si[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        ar += __shfl_xor(ar, o, 64);
        ai += __shfl_xor(ai, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sr[threadIdx.x >> 6] = ar;
        si[threadIdx.x >> 6] = ai;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        part[0] = (sr[0] + sr[1]) + (sr[2] + sr[3]);
        part[1] = (si[0] + si[1]) + (si[2] + si[3]);
    }
}

// Local terms with monomial factors, by destination: every element of y is the sum over the terms
// of alpha times the two factor values times one element of x (0 where no term reaches it), in the
// order of the terms.  DOT: nothing is stored; <x|y> goes to the work group's partial sums instead
// (source and destination then share their layout).  Real and imaginary planes at +nx / +ny.
// Bound by memory traffic (x and y once; 9.6 MB, 2 us for the 1000-state ladder) and, per term, the
// chain source, map, element, of which a thread has two elements in flight: 4.7 us for a pair of
// operators, 6.6 us for the expectation of two densities.  By source block the same work was a
// clearing pass (3 us), a pass per term that read and wrote y (10 us each, with 64-bit divisions)
// and for an expectation a pass over x and y (5 us).
template <bool DOT>
__global__ __launch_bounds__(256) void k_local_mono(const LocalItem* __restrict__ items, int nitems,
                                                    const LocalSrc* __restrict__ srcs,
                                                    const int* __restrict__ mapS,
                                                    const double* __restrict__ valS,
                                                    const int* __restrict__ mapE,
                                                    const double* __restrict__ valE,
                                                    const double* __restrict__ x, int64_t nx,
                                                    double* __restrict__ y, int64_t ny) {
    constexpr int kPer = kLocalChunk / 256;
    double ar = 0.0, ai = 0.0;
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const LocalItem I = items[it];
        // a thread's elements together, term by term: their loads are in flight at once
        int i[kPer], j[kPer];
        double zr[kPer], zi[kPer];
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int o = min((int)threadIdx.x + 256 * e, I.m - 1);
            const unsigned u = (unsigned)I.i0 + (unsigned)o, dj = u / (unsigned)I.d;
            i[e] = (int)(u - dj * (unsigned)I.d);
            j[e] = I.j0 + (int)dj;
            zr[e] = 0.0;
            zi[e] = 0.0;
        }
        for (int k = I.t0; k < I.t0 + I.nt; ++k) {
            const LocalSrc S = srcs[k];
            int is[kPer], js[kPer];
            double sc[kPer];
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                is[e] = S.amap < 0 ? i[e] : mapS[S.amap + i[e]];
                js[e] = S.bmap < 0 ? j[e] : mapE[S.bmap + j[e]];
                sc[e] = S.alpha * (S.amap < 0 ? 1.0 : valS[S.amap + i[e]]) *
                        (S.bmap < 0 ? 1.0 : valE[S.bmap + j[e]]);
            }
            double xr[kPer], xi[kPer];
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                const int64_t at = S.off + (int64_t)max(js[e], 0) * S.d + max(is[e], 0);
                xr[e] = x[at];
                xi[e] = x[nx + at];
            }
#pragma unroll
            for (int e = 0; e < kPer; ++e) {
                const bool ok = is[e] >= 0 && js[e] >= 0;
                zr[e] = ok ? fma(sc[e], xr[e], zr[e]) : zr[e];
                zi[e] = ok ? fma(sc[e], xi[e], zi[e]) : zi[e];
            }
        }
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int o = (int)threadIdx.x + 256 * e;
            if (o >= I.m) break;
            const int64_t to = I.to + o;
            if constexpr (DOT) {
                const double xr = x[to], xi = x[nx + to];
                ar += xr * zr[e] + xi * zi[e];
                ai += xr * zi[e] - xi * zr[e];
            } else {
                y[to] = zr[e];
                y[ny + to] = zi[e];
            }
        }
    }
    if constexpr (DOT) store_group_sum(ar, ai, y + 2 * blockIdx.x);
}

// part != nullptr: <x|y> in nblocks partial sums instead of y.
hipError_t launch_local_mono(const LocalItem* items, int nitems, const LocalSrc* srcs,
                             const int* mapS, const double* valS, const int* mapE,
                             const double* valE, const double* x, int64_t nx, double* y, int64_t ny,
                             double* part, int nblocks, hipStream_t s) {
    if (part)
        hipLaunchKernelGGL((k_local_mono<true>), dim3(nblocks), dim3(256), 0, s, items, nitems, srcs,
                           mapS, valS, mapE, valE, x, nx, part, ny);
    else if (nitems > 0)
        hipLaunchKernelGGL((k_local_mono<false>), dim3(nitems), dim3(256), 0, s, items, nitems, srcs,
                           mapS, valS, mapE, valE, x, nx, y, ny);
    return hipGetLastError();
}

hipError_t launch_zero(double* x, int64_t n, hipStream_t s) {
    if (n > 0) {
        const int blocks = (int)std::min<int64_t>((n + 255) / 256, 4096);
        hipLaunchKernelGGL(k_zero, dim3(blocks), dim3(256), 0, s, x, n);
    }
    return hipGetLastError();
}

// Partial sums of <x|z> = sum conj(x) z over n complex elements (planes at +n): block b writes
// (Re, Im) of its grid-stride share to part[2 b], part[2 b + 1]; the caller adds the partials
// in order.
__global__ __launch_bounds__(256) void k_zdot(const double* __restrict__ x, const double* __restrict__ z,
                                              int64_t n, double* __restrict__ part) {
    double ar = 0.0, ai = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const double xr = x[i], xi = x[n + i], zr = z[i], zi = z[n + i];
        ar += xr * zr + xi * zi;
        ai += xr * zi - xi * zr;
    }
    store_group_sum(ar, ai, part + 2 * blockIdx.x);
}

hipError_t launch_zdot(const double* x, const double* z, int64_t n, double* part, int nblocks,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_zdot, dim3(nblocks), dim3(256), 0, s, x, z, n, part);
    return hipGetLastError();
}

}  // namespace dmrg
