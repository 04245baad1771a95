"""The Sturm count of the tridiagonal eigensolvers (csrc/tridiag.hpp), compiled for the host with the
GPU's builtins written out, against the eigenvalues themselves."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_1103_5391_amd import build as B

RUN = 8                             # rows of a run (kSturmRun)
SOURCE = r"""
#include "internal.hpp"
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
using std::min;
static void none(int) {}
static unsigned alignbit(unsigned a, unsigned b, int s) {
    return (unsigned)((((uint64_t)a << 32) | b) >> s);
}
static int hiint(double p) {
    int64_t u;
    std::memcpy(&u, &p, 8);
    return (int)(u >> 32);
}
static int frexp_exp(double p) {
    int e = 0;
    std::frexp(p, &e);
    return e;
}
#define __builtin_amdgcn_s_waitcnt none
#define __builtin_amdgcn_sched_barrier none
#define __builtin_amdgcn_alignbit alignbit
#define __builtin_amdgcn_frexp_exp frexp_exp
#define __builtin_amdgcn_ldexp std::ldexp
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __popc __builtin_popcount
#define __double2hiint hiint
#include "tridiag.hpp"
extern "C" int sturm(int nrun, const double* rec, double x) { return dmrg::sturm_count(nrun, rec, x); }
"""


@pytest.fixture(scope="module")
def count(tmp_path_factory):
    d = tmp_path_factory.mktemp("sturm")
    (d / "sturm.cpp").write_text(SOURCE)
    rocm = os.path.dirname(os.path.dirname(B._hipcc()))
    subprocess.run([os.path.join(rocm, "bin", "amdclang++"), "-std=c++17", "-O1", "-ffp-contract=off",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(B.HERE, "csrc"), "-shared", "-fPIC", "-o", str(d / "sturm.so"),
                    str(d / "sturm.cpp")], check=True, capture_output=True)
    lib = C.CDLL(str(d / "sturm.so"))
    lib.sturm.argtypes = [C.c_int, C.c_void_p, C.c_double]

    def f(diag, e, x):
        n, nrun = len(diag), -(-len(diag) // RUN)
        rec = np.zeros((nrun, 2, RUN))
        rec[:, 0] = 4.0
        for i in range(n):
            rec[i // RUN, 0, i % RUN] = diag[i]
            rec[i // RUN, 1, i % RUN] = e[i - 1] ** 2 if i else 0.0
        rec = np.ascontiguousarray(rec.ravel())
        return lib.sturm(nrun, rec.ctypes.data, float(x))

    return f


def test_decoupled_entry_on_the_last_row_of_a_run(count):
    """A minor that vanishes in the last row of a run, with nothing coupled behind it: the count at
    the entry lies between those on either side."""
    diag = [0.9] * 7 + [0.5] + [0.1] * 8
    zero = np.zeros(15)
    assert [count(diag, zero, x) for x in (0.4999999, 0.5000001)] == [8, 9]
    assert count(diag, zero, 0.5) in (8, 9)


@pytest.mark.parametrize("seed", range(4))
def test_decoupled_counts_are_exact(count, seed):
    """Matrices of 1 to 40 rows with exact entries of either sign, some repeated, diagonal (even
    seeds: the signs of the minors are exact, no tolerance) or with some neighbours coupled (odd
    seeds): at every diagonal entry and between any two the count is that of the smaller
    eigenvalues, or of them and the equal ones."""
    rng = np.random.default_rng(1100 + seed)
    for _ in range(150):
        n = int(rng.integers(1, 41))
        diag = rng.integers(-20, 21, n) / 64.0
        e = np.where(rng.random(n) < 0.4, 0.125, 0.0) if seed % 2 else np.zeros(n)
        lam = np.linalg.eigvalsh(np.diag(diag) + np.diag(e[:n - 1], 1) + np.diag(e[:n - 1], -1)) \
            if seed % 2 else np.sort(diag)
        near = 1e-13 if seed % 2 else 0.0              # rounding of the reference
        for x in sorted(set(diag) | set(diag + 1 / 128)):
            assert np.sum(lam < x - near) <= count(diag, e, x) <= np.sum(lam <= x + near), (diag, e, x)


def test_coupled_counts(count):
    """Coupled matrices: the count at the middle of every gap wider than rounding."""
    rng = np.random.default_rng(1110)
    for n in (1, 2, 7, 8, 9, 16, 33, 150):
        diag = rng.uniform(-0.3, 0.3, n)
        e = rng.uniform(-0.1, 0.1, n)
        lam = np.linalg.eigvalsh(np.diag(diag) + np.diag(e[:n - 1], 1) + np.diag(e[:n - 1], -1))
        for j in range(n - 1):
            if lam[j + 1] - lam[j] > 1e-12:
                assert count(diag, e, 0.5 * (lam[j] + lam[j + 1])) == j + 1
        assert count(diag, e, lam[0] - 0.01) == 0 and count(diag, e, lam[-1] + 0.01) == n
