// Real symmetric tridiagonal matrices (diagonal, subdiagonal) on the device: Sturm counts, and the
// solves of inverse iteration, shared by the density matrices and the ground state of a Lanczos
// basis.
#pragma once

#include "internal.hpp"

namespace dmrg {
namespace {

// 1 / x: the hardware reciprocal and one Newton step (within a few ulp)
__device__ __forceinline__ double recip(double x) {
    const double r0 = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r0, 1.0), r0, r0);
}

// 1 / x with two Newton steps (to about an ulp; the reflector's scalars)
__device__ __forceinline__ double recip2(double x) {
    const double r0 = __builtin_amdgcn_rcp(x);
    const double r1 = fma(fma(-x, r0, 1.0), r0, r0);
    return fma(fma(-x, r1, 1.0), r1, r1);
}

// The Sturm count of T - x I (the number of its eigenvalues below 0) by the signs of its leading
// principal minors, p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2} (Givens): a step is one dependent
// fused multiply-add, where the ratios p_i / p_{i-1} cost a reciprocal and three (88 cycles a step).
// Each step is exact for entries changed by an ulp or two, so the counts place every
// eigenvalue within a few eps |T|.  |T| is scaled to [0.5, 1) by the caller, so a run of kSturmRun steps
// grows by less than 2^24 and the two minors carried on are scaled between runs.  A zero counts by
// its sign bit, whichever it is, as its neighbours have opposite signs; two zeros in turn (a
// diagonal entry equal to x beside a zero e) would stay zeros, so a run that ends in them is taken
// again with -kTinyMinor times the minor before it in place of a zero: the exact minor of an entry
// changed by that much (whatever couples to it, the ratio has to be tiny, not the minor alone).  A
// zero carried in from the run before has been counted by its sign bit there, so its replacement
// takes that sign.
// The entries are the same in every lane; from global memory they come by scalar loads, a run ahead
// (many wavefronts' broadcast reads from LDS bound the pass: two per step and wavefront).  rec: per run of kSturmRun rows the diagonal entries
// and the squares of the subdiagonal entries above them (the first 0), nrun runs, the last one
// padded with rows that change no sign (diagonal 4, above every x; subdiagonal 0).
constexpr double kTinyMinor = 1e-30;    // eight in turn stay far above the smallest double
__device__ __forceinline__ int sturm_count(int nrun, const double* __restrict__ rec, double x) {
    static_assert(kSturmRun < 32, "the signs of a run in one word");
    double p2 = 0.0, p1 = 1.0;
    unsigned sg = 0;                                    // signs of the minors, the latest lowest
    int cnt = 0;
    double cur[2 * kSturmRun], nxt[2 * kSturmRun];
#pragma unroll
    for (int t = 0; t < 2 * kSturmRun; ++t) cur[t] = rec[t];
    for (int k = 0; k < nrun; ++k) {
        // this run's entries are here before the next one's loads go out (scalar loads return in any
        // order, so a wait is one for all of them)
        __builtin_amdgcn_s_waitcnt(0xc07f);             // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        const double* __restrict__ rn = rec + 2 * kSturmRun * min(k + 1, nrun - 1);
#pragma unroll
        for (int t = 0; t < 2 * kSturmRun; ++t) nxt[t] = rn[t];
        auto run = [&](bool guard) {
#pragma unroll
            for (int t = 0; t < kSturmRun; ++t) {
                double p = fma(cur[t] - x, p1, -(cur[kSturmRun + t] * p2));
                if (guard && p == 0.0) p = -kTinyMinor * p1;
                sg = __builtin_amdgcn_alignbit(sg, (unsigned)__double2hiint(p), 31);
                p2 = p1;
                p1 = p;
            }
        };
        const double p10 = p1, p20 = p2;
        const unsigned s0 = sg;
        run(false);
        if (p1 == 0.0 && p2 == 0.0) {
            p1 = p10 != 0.0 ? p10 : (s0 & 1 ? -kTinyMinor : kTinyMinor);
            p2 = p20;
            sg = s0;
            run(true);
        }
        cnt += __popc((sg ^ (sg >> 1)) & ((1u << kSturmRun) - 1));
        const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
        p1 = __builtin_amdgcn_ldexp(p1, -ex);
        p2 = __builtin_amdgcn_ldexp(p2, -ex);
#pragma unroll
        for (int t = 0; t < 2 * kSturmRun; ++t) cur[t] = nxt[t];
    }
    return cnt;
}
// Factors and vectors of an inverse iteration: row i of column l at offset at(i, l), the next row
// `row` further on.  In LDS a record of six values (z, U: 1 / pivot, superdiagonals 1 and 2, L:
// multiplier, swap flag: 1 where rows i, i + 1 were exchanged), so that a row needs one address and few
// wide accesses.
typedef double dv2u __attribute__((ext_vector_type(2), aligned(16)));
struct InvLds {
    double* p;                                          // 16-byte aligned
    int nc, row;
    __device__ __forceinline__ int at(int i, int l) const { return 6 * (i * nc + l); }
    __device__ __forceinline__ double& z(int o) const { return p[o]; }
    __device__ __forceinline__ void put_u(int o, double a, double b, double c) const {
        p[o + 1] = a;
        *reinterpret_cast<dv2u*>(p + o + 2) = (dv2u){b, c};
    }
    __device__ __forceinline__ void get_zu(int o, double& z, double& a, double& b, double& c) const {
        const dv2u x = *reinterpret_cast<const dv2u*>(p + o), y = *reinterpret_cast<const dv2u*>(p + o + 2);
        z = x[0];
        a = x[1];
        b = y[0];
        c = y[1];
    }
    __device__ __forceinline__ void put_l(int o, double m, double s) const {
        *reinterpret_cast<dv2u*>(p + o + 4) = (dv2u){m, s};
    }
    __device__ __forceinline__ void get_l(int o, double& m, double& s) const {
        const dv2u x = *reinterpret_cast<const dv2u*>(p + o + 4);
        m = x[0];
        s = x[1];
    }
};
constexpr int kInvRun = 8;          // rows a solve loads before storing

// T - x I = P L U of column l (partial pivoting, pivots floored at tiny), row by row ((dd, du) = the
// current row's diagonal and superdiagonal), with the forward substitution P, L^-1 of a start vector
// whose entries start() gives in turn.  EXACT: correctly rounded reciprocals.
template <bool EXACT, class M, class Start>
__device__ __forceinline__ void tri_factor(const M& m, int d, int l, const double* __restrict__ dg,
                                           const double* __restrict__ e, double x, double tiny,
                                           Start start) {
    double dd = dg[0] - x, du = d > 1 ? e[0] : 0.0;
    double cur = start();
    int o = m.at(0, l);
    auto row = [&](double sub, double di, double nu) {
        const double nd = di - x, nxt = start();
        // without a swap: U row (1 / dd, du, 0); with one: (1 / sub, nd, nu)
        const bool keep = fabs(dd) >= fabs(sub);
        const double piv = fabs(dd) >= tiny ? dd : (dd < 0.0 ? -tiny : tiny);
        const double by = keep ? piv : sub;
        const double ip = EXACT ? 1.0 / by : recip(by);
        const double mu = (keep ? sub : dd) * ip;
        m.put_u(o, ip, keep ? du : nd, keep ? 0.0 : nu);
        m.put_l(o, mu, keep ? 0.0 : 1.0);
        const double dn = keep ? nd - mu * du : du - mu * nd;
        du = keep ? nu : -mu * nu;
        dd = dn;
        const double a = keep ? cur : nxt, b = keep ? nxt : cur;
        m.z(o) = a;
        cur = b - mu * a;
        o += m.row;
    };
    int i = 0;
    for (; i + kInvRun < d - 1; i += kInvRun) {
        double er[kInvRun + 1], dr[kInvRun];
#pragma unroll
        for (int t = 0; t <= kInvRun; ++t) er[t] = e[i + t];
#pragma unroll
        for (int t = 0; t < kInvRun; ++t) dr[t] = dg[i + 1 + t];
#pragma unroll
        for (int t = 0; t < kInvRun; ++t) row(er[t], dr[t], er[t + 1]);
    }
    for (; i + 1 < d; ++i) row(e[i], dg[i + 1], i + 2 < d ? e[i + 1] : 0.0);
    const double piv = fabs(dd) >= tiny ? dd : (dd < 0.0 ? -tiny : tiny);
    m.put_u(o, 1.0 / piv, 0.0, 0.0);
    m.z(o) = cur;
}

// Backward substitution U^-1 of column l, rows loaded a run of kInvRun ahead of the arithmetic (the
// first d mod kInvRun rows one by one); returns |z|^2.
template <class M>
__device__ __forceinline__ double tri_backward(const M& m, int d, int l) {
    double y1 = 0.0, y2 = 0.0, nrm = 0.0;
    int o = m.at(d - 1, l);
    auto row = [&](int at, double zv, double a0, double a1, double a2) {
        const double y = ((zv - a2 * y2) - a1 * y1) * a0;
        m.z(at) = y;
        nrm += y * y;
        y2 = y1;
        y1 = y;
    };
    int left = d;
    for (; left % kInvRun != 0; --left, o -= m.row) {
        double zv, a0, a1, a2;
        m.get_zu(o, zv, a0, a1, a2);
        row(o, zv, a0, a1, a2);
    }
    for (; left > 0; left -= kInvRun, o -= kInvRun * m.row) {
        double zv[kInvRun], a0[kInvRun], a1[kInvRun], a2[kInvRun];
#pragma unroll
        for (int t = 0; t < kInvRun; ++t) m.get_zu(o - t * m.row, zv[t], a0[t], a1[t], a2[t]);
#pragma unroll
        for (int t = 0; t < kInvRun; ++t) row(o - t * m.row, zv[t], a0[t], a1[t], a2[t]);
    }
    return nrm;
}

// One solve of column l from Z (times scale): P and L^-1 (the current entry carried in a register; row
// i is stored only after row i + 1 is read), then U^-1; returns |z|^2.
template <class M>
__device__ __forceinline__ double tri_solve(const M& m, int d, int l, double scale) {
    int o = m.at(0, l);
    double cur = scale * m.z(o);
    auto row = [&](int at, double zn, double lw, double pw) {
        const double nxt = scale * zn;
        const bool swap = pw != 0.0;
        const double a = swap ? nxt : cur, b = swap ? cur : nxt;
        m.z(at) = a;
        cur = b - lw * a;
    };
    int left = d - 1;
    for (; left % kInvRun != 0; --left, o += m.row) {
        double lw, pw;
        m.get_l(o, lw, pw);
        row(o, m.z(o + m.row), lw, pw);
    }
    for (; left > 0; left -= kInvRun, o += kInvRun * m.row) {
        double zn[kInvRun], pw[kInvRun], lw[kInvRun];
#pragma unroll
        for (int t = 0; t < kInvRun; ++t) {
            zn[t] = m.z(o + (t + 1) * m.row);
            m.get_l(o + t * m.row, lw[t], pw[t]);
        }
#pragma unroll
        for (int t = 0; t < kInvRun; ++t) row(o + t * m.row, zn[t], lw[t], pw[t]);
    }
    m.z(o) = cur;
    return tri_backward(m, d, l);
}

}  // namespace
}  // namespace dmrg
