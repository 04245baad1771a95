"""Inputs whose results depend on a rare branch or on what an earlier call left behind (needs an
MI355X)."""
import numpy as np
import pytest

from oracle import matvec as M
from oracle import observables as Ob
from paper_1103_5391_amd import inputs as I
from tests.test_gpu_block_edges import BOUND, DIMS, _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1103_5391_amd import lib as L
    return torch, L


@pytest.mark.parametrize("d,seed", [(16, 0), (40, 1), (64, 2), (170, 3)])
def test_density_of_diagonal_matrices(env, d, seed):
    """Diagonal density matrices with the entries 0 .. 33, the values in the last rows of the Sturm
    counts' runs among the points of the first section (its 32 points lie at 1, 2, .. but for
    rounding, which leaves those around the middle exact).  The entries are exact sums of the
    weights 1, 2, 4, .. of six targets; eigenvalues within 1e-12 of the largest, orthonormality and
    residuals within 1e-11 d, as in the parity tests."""
    torch, L = env
    pb = _problem(((d,) * 4, (d,) * 4))
    rng = np.random.default_rng(seed)
    vals = []
    for _ in I.psi_blocks(pb):
        a = rng.integers(0, 34, d)
        a[0], a[1] = 33, 0
        for r in range(7, d, 8):
            a[r] = rng.integers(13, 22)
        vals.append(a)
    vecs = []
    for bit in range(6):
        re = [np.diag(((a >> bit) & 1).astype(float)).ravel() for a in vals]
        vecs.append(torch.from_numpy(np.concatenate(re + [np.zeros(4 * d * d)])).to("cuda"))
    h = L.dmrg_create(pb)
    ev = torch.zeros(4 * d, dtype=torch.float64, device="cuda")
    vc = torch.zeros(8 * d * d, dtype=torch.float64, device="cuda")
    h.density_truncate(vecs, 2.0 ** np.arange(6), 4 * d, ev, vc)
    ev, vc = ev.cpu().numpy().reshape(4, d), vc.cpu().numpy().reshape(4, 2, d, d)
    for b, a in enumerate(vals):
        assert np.max(np.abs(ev[b] - np.sort(a)[::-1])) <= 1e-12 * 33
        U = (vc[b, 0] + 1j * vc[b, 1]).T
        assert np.linalg.norm(U.conj().T @ U - np.eye(d)) <= 1e-11 * d
        assert np.linalg.norm(a[:, None] * U - U * ev[b]) <= 1e-11 * 33 * d
    h.destroy()


def test_noalloc_with_an_array_of_its_own(env):
    """A problem within the limit of dmrg_matvec_noalloc (66.8 of 67.1 MB by its columns) whose column
    panels take more (87.3 MB): the bits of dmrg_matvec in every family and arithmetic that clears or
    does not clear the array, also after a call of another handle and from a vector of NaN."""
    from tests.test_noalloc_memory import panel_problem
    torch, L = env
    h, small = L.dmrg_create(panel_problem()), L.dmrg_create(_problem(((17, 5, 3, 9), (4, 8, 7, 6))))
    rng = np.random.default_rng(I.SEED_BASE + 21)
    x = torch.from_numpy(I.random_psi(h.n, rng)).to("cuda")
    xs = torch.from_numpy(I.random_psi(small.n, rng)).to("cuda")
    bad, y, z = torch.full_like(x, float("nan")), torch.empty_like(x), torch.empty_like(x)
    ys, zs = torch.empty_like(xs), torch.empty_like(xs)
    small.matvec(xs, ys)
    for prec, variants in ((0, (0, 12, 3, 16)), (1, (0, 3)), (2, (0, 3))):
        h.set_precision(prec)
        for v in variants:
            h.set_gemm(v)
            h.matvec_noalloc(bad, z)
            h.matvec_noalloc(x, z)
            small.matvec_noalloc(xs, zs)
            h.matvec(x, y)
            assert torch.equal(y, z), (prec, v)
            assert torch.equal(ys, zs), (prec, v)
    h.destroy()
    small.destroy()


@pytest.mark.parametrize("dims", DIMS[:4], ids=["1", "16", "32", "64"])
def test_families_after_nan_in_the_k_split_layout(env, dims):
    """The K-split family lays the handle's workspace out in its own way: after it has run on a vector of
    NaN, no value that another family reads may come from what it left (bounds: FP64 products at the
    tile edges)."""
    torch, L = env
    pb = _problem(dims)
    h = L.dmrg_create(pb)
    x = I.random_psi(h.n, np.random.default_rng(I.SEED_BASE + 22))
    ref = M.matvec_sector(pb, x)
    xd = torch.from_numpy(x).to("cuda")
    bad, y = torch.full_like(xd, float("nan")), torch.empty_like(xd)
    for v in (0, 1, 2, 3, 12, 16, 32):
        h.set_gemm(32)
        h.matvec(bad, y)
        h.set_gemm(v)
        h.matvec(xd, y)
        assert np.linalg.norm(y.cpu().numpy() - ref) < BOUND[0] * np.linalg.norm(ref), v
    h.destroy()


def _local_problem():
    """A superblock with an operator per half that has one value per row and column, and the lists of
    a pair of them with the coefficient c (for the library and for the oracle)."""
    pb = _problem(DIMS[2])
    ops = []
    for space in (pb.S.space, pb.E.space):
        o = I.BlockOp((0, 0))
        for p, d in enumerate(space.dim):
            o.blocks[p] = np.diag(1.0 + np.arange(d))[::-1].copy()
        ops.append(o)
    pbx, iS, iE = I.with_ops(pb, [ops[0]], [ops[1]])
    return pbx, (lambda c: [(c, iS[0], 0, iE[0], 0, 0)]), (lambda c: [(c, ops[0], ops[1], 0)])


def _capped(L, pb, cap):
    import os
    os.environ["DMRG_MAX_WORKSPACE"] = str(cap)
    try:
        return L.dmrg_create(pb)
    finally:
        del os.environ["DMRG_MAX_WORKSPACE"]


def test_local_terms_below_and_above_a_memory_cap(env):
    """Caps on the handle's memory from far below what the local operators take to all of it, in steps
    smaller than their last buffers: a call that does not fit fails, and fails again, and the first
    that fits is right."""
    torch, L = env
    pb, terms, oterms = _local_problem()
    base = L.plan_stats(pb)["create_bytes"]
    x = I.random_psi(L.plan_stats(pb)["n"], np.random.default_rng(I.SEED_BASE + 23))
    ref = Ob.apply_terms(pb, pb, oterms(1.0), x)
    xd = torch.from_numpy(x).to("cuda")

    def fits(extra):
        h = _capped(L, pb, base + extra)
        done = []
        for _ in range(2):
            y = torch.full_like(xd, float("nan"))
            try:
                h.apply_local(h, terms(1.0), xd, y)
                assert np.max(np.abs(y.cpu().numpy() - ref)) <= 1e-13 * np.max(np.abs(ref))
                done.append(True)
            except L.DmrgError as e:
                assert e.status == L.STATUS_CODE["DMRG_ENOMEM"]
                done.append(False)
        h.destroy()
        assert done[0] == done[1], extra
        return done[0]

    lo, hi = 8, 1 << 24
    assert not fits(lo) and fits(hi)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if fits(mid) else (mid, hi)
    for below in list(range(1, 12000, 120)) + [hi - hi // 2, hi - hi // 8]:
        if below < hi:
            assert not fits(hi - below)


def test_kept_lists_give_way_to_other_buffers(env):
    """A memory cap that holds the tables of one list of local terms and a Krylov workspace holds them
    after eight lists too: the lists a handle keeps are no reason to refuse another call."""
    torch, L = env
    pb, terms, oterms = _local_problem()
    base = L.plan_stats(pb)["create_bytes"]
    x = torch.from_numpy(I.random_psi(L.plan_stats(pb)["n"], np.random.default_rng(I.SEED_BASE + 24))).to("cuda")
    y, z = torch.empty_like(x), torch.empty_like(x)

    def fits(extra, lists):
        h = _capped(L, pb, base + extra)
        try:
            for c in range(lists):
                h.apply_local(h, terms(1.0 + c), x, y)
            h.krylov_expm(x, z, 0.01, 4, 1)
            h.apply_local(h, terms(1.0), x, z)
            return True
        except L.DmrgError as e:
            assert e.status == L.STATUS_CODE["DMRG_ENOMEM"]
            return False
        finally:
            h.destroy()

    lo, hi = 8, 1 << 24
    assert not fits(lo, 1) and fits(hi, 1)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if fits(mid, 1) else (mid, hi)
    assert fits(hi, 8)
    assert np.max(np.abs((y - 8.0 * z).cpu().numpy())) <= 1e-13 * float(y.abs().max())


@pytest.mark.parametrize("first", ["density", "expectation"])
def test_density_and_expectation_share_their_results_area(env, first):
    """Truncations and expectations in turn on one handle, either of them first: the weights add up and
    the expectation is the oracle's (1e-12), every time."""
    torch, L = env
    pb, terms, oterms = _local_problem()
    h = L.dmrg_create(pb)
    x = I.random_psi(h.n, np.random.default_rng(I.SEED_BASE + 25))
    xd = torch.from_numpy(x).to("cuda")
    rows = [r for (_, _, r, _) in I.psi_blocks(pb)]
    ev = torch.zeros(sum(rows), dtype=torch.float64, device="cuda")
    U = torch.zeros(2 * sum(r * r for r in rows), dtype=torch.float64, device="cuda")
    want = Ob.expect(pb, oterms(1.0), x)
    for k in range(6):
        if (k % 2 == 0) == (first == "density"):
            kept, err = h.density_truncate([xd], np.array([1.0]), 10, ev, U)
            assert sum(kept) == 10
            top = np.sort(ev.cpu().numpy())[::-1]
            assert abs(float(top.sum()) - float(x @ x)) <= 1e-12 * float(x @ x)
            assert abs(err - float(top[10:].sum())) <= 1e-12 * float(x @ x)
        else:
            assert abs(h.expect_local(terms(1.0), xd) - want) <= 1e-12 * max(1.0, abs(want))
    h.destroy()


def _truncate(torch, L, h, mats, weights, keep):
    """density_truncate of the targets whose blocks are mats[l][b] (complex): per block the
    eigenvalues and eigenvectors, and the states kept."""
    planes = lambda M: np.concatenate([m.real.ravel(order="F") for m in M] + [m.imag.ravel(order="F") for m in M])
    rows = [len(m) for m in mats[0]]
    ev = torch.zeros(sum(rows), dtype=torch.float64, device="cuda")
    vc = torch.zeros(sum(2 * r * r for r in rows), dtype=torch.float64, device="cuda")
    vecs = [torch.from_numpy(planes(M)).to("cuda") for M in mats]
    kept, err = h.density_truncate(vecs, np.array(weights), keep, ev, vc)
    ev, vc, out, eo, vo = ev.cpu().numpy(), vc.cpu().numpy(), [], 0, 0
    for r in rows:
        out.append((ev[eo:eo + r], (vc[vo:vo + r * r] + 1j * vc[vo + r * r:vo + 2 * r * r]).reshape(r, r).T))
        eo += r
        vo += 2 * r * r
    return out, kept, err


def test_density_with_nan(env):
    """NaN in one sector of a target, whose own results mean nothing: the other sectors' are right (1e-12
    of their largest eigenvalue) and every state kept is counted once."""
    torch, L = env
    dims = (12, 40, 30, 170)
    h = L.dmrg_create(_problem((dims, dims[::-1])))
    rng = np.random.default_rng(I.SEED_BASE + 30)
    mats = [rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)) for d in dims]
    for nan in (0, 1, 3):
        M = [m.copy() for m in mats]
        M[nan][-1, 0] = np.nan
        keep = 100 if nan == 3 else 200
        out, kept, _ = _truncate(torch, L, h, [M], [1.0], keep)
        assert sum(kept) == keep and all(0 <= k <= d for k, d in zip(kept, dims))
        for b, (w, U) in enumerate(out):
            if b == nan:
                continue
            lam = np.linalg.eigvalsh(mats[b] @ mats[b].conj().T)[::-1]
            assert np.max(np.abs(w - lam)) <= 1e-12 * lam[0]
            assert np.linalg.norm(U.conj().T @ U - np.eye(len(w))) <= 1e-11 * len(w)
    h.destroy()


def _check_spectrum(out, rho):
    """Eigenvalues (1e-12 of the largest), orthonormality and residuals (1e-11 d) of one block against
    its density matrix, as in the parity tests."""
    w, U = out
    d, lam = len(w), np.linalg.eigvalsh(rho)[::-1]
    top = max(abs(lam[0]), 1e-300)
    assert np.max(np.abs(w - lam)) <= 1e-12 * top
    assert np.linalg.norm(U.conj().T @ U - np.eye(d)) <= 1e-11 * d
    assert np.linalg.norm(rho / top @ U - U * (w / top)) <= 1e-11 * d


@pytest.mark.parametrize("dims", [(1, 2, 3, 8), (5, 4, 9, 30), (7, 6, 40, 170)])
def test_density_with_empty_sectors(env, dims):
    """Targets with no weight in some sectors: eigenvalues 0 with orthonormal vectors there."""
    torch, L = env
    h = L.dmrg_create(_problem((dims, dims[::-1])))
    rng = np.random.default_rng(I.SEED_BASE + 31)
    for empty in ((0,), (0, 1), (2,), (0, 1, 2, 3)):
        M = [np.zeros((d, d), complex) if b in empty else rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
             for b, d in enumerate(dims)]
        out, kept, err = _truncate(torch, L, h, [M], [1.0], sum(dims))
        assert list(kept) == list(dims)
        for b, m in enumerate(M):
            _check_spectrum(out[b], m @ m.conj().T)
    h.destroy()


@pytest.mark.parametrize("size", [1, 4])
@pytest.mark.parametrize("exponent", [-480, -430, 400])
def test_density_scaled_by_powers_of_two(env, exponent, size):
    """Density matrices of norm 2^exponent (isolated eigenvalues, and clusters of four): the eigenvectors'
    squares and reciprocals stay in range."""
    torch, L = env
    dims = (3, 20, 60, 165)
    h = L.dmrg_create(_problem((dims, dims[::-1])))
    rng = np.random.default_rng(I.SEED_BASE + 32)
    M = []
    for d in dims:
        q = [np.linalg.qr(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))[0] for _ in range(2)]
        lam = (1.0 + np.arange(d) // size + 1e-8 * (np.arange(d) % size)) / d
        M.append((q[0] * np.sqrt(lam)) @ q[1] * 2.0 ** (exponent // 2))
    out, _, _ = _truncate(torch, L, h, [M], [1.0], 50)
    for b, m in enumerate(M):
        w, U = out[b]
        s = 2.0 ** -(exponent // 2)
        _check_spectrum((w * s * s, U), (m * s) @ (m * s).conj().T)
    h.destroy()


@pytest.mark.parametrize("exponent", [-560, -500, 0])
def test_density_of_tiny_norm(env, exponent):
    """Density matrices of norm 2^exponent: the squares of a column leave the range of doubles (isolated
    eigenvalues; sectors that the reduction holds in registers, and a larger one)."""
    torch, L = env
    dims = (2, 20, 60, 165)
    h = L.dmrg_create(_problem((dims, dims[::-1])))
    rng = np.random.default_rng(I.SEED_BASE + 33)
    s = 2.0 ** (exponent // 2)
    M = [(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))) * s for d in dims]
    out, _, _ = _truncate(torch, L, h, [M], [1.0], 50)
    for b, m in enumerate(M):
        w, U = out[b]
        _check_spectrum((w / s / s, U), (m / s) @ (m / s).conj().T)
    h.destroy()


@pytest.mark.parametrize("scale", [1.0, 1e-30, 3e-45])
def test_density_of_equal_amplitudes(env, scale):
    """Rank one with equal amplitudes: every column of the reduction after the first is rounding of
    the one before it."""
    torch, L = env
    rng = np.random.default_rng(I.SEED_BASE + 34)
    for dims in ((9, 14, 34, 21), (3, 8, 29, 45), (137, 12, 89, 20), (7, 170, 16, 60)):
        h = L.dmrg_create(_problem((dims, dims[::-1])))
        for phase in (1.0, np.exp(0.7j)):
            M = [np.full((d, d), scale * phase * rng.uniform(0.1, 1.0)) for d in dims]
            out, _, _ = _truncate(torch, L, h, [M, M], [0.5, 0.25], 50)
            for b, m in enumerate(M):
                rho = 0.75 * (m / scale) @ (m / scale).conj().T
                w, U = out[b]
                _check_spectrum((w / scale / scale, U), rho)
        h.destroy()


@pytest.mark.parametrize("decades", [3, 14, 30])
def test_density_of_decaying_weights(env, decades):
    """Weights that fall by that many decades over a sector, as those of a sweep's targets do, alone and
    beside low-rank blocks; and norms from 2^-560 on."""
    torch, L = env
    rng = np.random.default_rng(I.SEED_BASE + 35)
    cplx = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    for dims in ((12, 40, 85, 170), (59, 20, 150, 9)):
        h = L.dmrg_create(_problem((dims, dims[::-1])))
        for exponent in (0, -40, -560):
            s = 2.0 ** (exponent // 2)
            M = []
            for b, d in enumerate(dims):
                if (b + exponent) % 3 == 2:
                    M.append(cplx(d, 2) @ cplx(2, d))
                    continue
                q, p = np.linalg.qr(cplx(d, d))[0], np.linalg.qr(cplx(d, d))[0]
                M.append((q * 10.0 ** (-decades / 2 * np.arange(d) / (d - 1))) @ p)
            out, _, _ = _truncate(torch, L, h, [[m * s for m in M]], [1.0], 50)
            for b, m in enumerate(M):
                w, U = out[b]
                _check_spectrum((w / s / s, U), m @ m.conj().T)
        h.destroy()


@pytest.mark.parametrize("copies", [2, 3, 5, 8])
def test_density_of_equal_blocks(env, copies):
    """Density matrices made of equal blocks along the diagonal: every eigenvalue `copies` times, its
    eigenvectors without common rows."""
    torch, L = env
    sizes = (3, 5, 8, 25)
    dims = tuple(copies * s for s in sizes)
    h = L.dmrg_create(_problem((dims, dims[::-1])))
    for seed in range(4):
        rng = np.random.default_rng([I.SEED_BASE, seed])
        M = []
        for s in sizes:
            c = rng.standard_normal((s, s)) + 1j * rng.standard_normal((s, s))
            M.append(np.kron(np.eye(copies), c))
        out, _, _ = _truncate(torch, L, h, [M], [1.0], 50)
        for b, m in enumerate(M):
            _check_spectrum(out[b], m @ m.conj().T)
    h.destroy()
