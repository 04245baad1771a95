"""Block products at the sizes where a tile, a K chunk or a column panel ends: superblocks with
hand-picked sector dimensions, every kernel family and arithmetic, against the oracle."""
import numpy as np
import pytest

from oracle import krylov as K
from oracle import matvec as M
from paper_1103_5391_amd import inputs as I

pytestmark = pytest.mark.gpu

QN = np.array([[0, 0], [0, 1], [1, 0], [1, 1]], dtype=np.int32)
# sector dimensions of the two halves: 16 rows and columns make a panel and an FP64 chunk, 32 a
# tile and a bf16 chunk, 64 the widest tile
DIMS = [((1, 1, 1, 1), (1, 1, 1, 1)), ((15, 16, 17, 2), (17, 15, 1, 16)),
        ((31, 32, 33, 48), (3, 33, 32, 31)), ((64, 65, 1, 47), (49, 1, 64, 65)),
        # K = 7 x about 700 in stage 2: more chunks than its table in LDS holds at once
        ((700, 650, 720, 680), (3, 5, 2, 4))]
VARIANTS = [0, 1, 2, 3, 4, 6, 8, 9, 12, 16, 32]
# relative 2-norm bounds: K <= 5000 terms of relative error 2^-53, 2^-24 (twice: the intermediate
# is rounded too), and 2^-16 for two bf16 pieces
BOUND = {0: 1e-13, 1: 2e-6, 2: 1e-4, 3: 2e-6}


def _half(dims, rng):
    sp = I.Space(QN.copy(), np.array(dims, dtype=np.int32))
    H = []
    for d in dims:
        a = rng.standard_normal((d, d))
        H.append(a + a.T)
    ops = []
    for dq in I.E_SIGMA:
        op = I.BlockOp(dq)
        for p in range(4):
            p2 = sp.shift(p, dq)
            if p2 is not None:
                op.blocks[p] = rng.standard_normal((dims[p2], dims[p]))
        ops.append(op)
    return I.Half(sp, H, ops, [(0, 0), (0, 1)], [0])


def _problem(dims, seed=5):
    rng = np.random.default_rng(I.SEED_BASE + seed)
    S, E = _half(dims[0], rng), _half(dims[1], rng)
    bonds = [I.Bond((0, 1), (0, 1), t, (0, 1)) for t in ((1.0, 0.5, 0.25) if max(dims[0]) > 500 else (1.0,))]
    return I.Problem(S, E, (1, 1), bonds)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1103_5391_amd import lib as L
    return torch, L


@pytest.mark.parametrize("prec", [0, 1, 2, 3], ids=["fp64", "fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("dims", DIMS, ids=["1", "16", "32", "64", "long"])
def test_products_at_tile_edges(env, dims, prec):
    torch, L = env
    pb = _problem(dims)
    h = L.dmrg_create(pb)
    h.set_precision(prec)
    x = I.random_psi(h.n, np.random.default_rng(I.SEED_BASE + 6))
    ref = M.matvec_sector(pb, x)
    xd = torch.from_numpy(x).to("cuda")
    bad = torch.full_like(xd, float("nan"))
    y = torch.empty_like(xd)
    for v in VARIANTS:
        h.set_gemm(v)
        h.matvec(bad, y)          # nothing of a vector of NaN may stay behind in the workspace
        for w in (v, 0) if v != 32 else (v,):
            h.set_gemm(w)
            y.fill_(0.0)
            h.matvec(xd, y)
            err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
            assert err < BOUND[prec], (v, w, err)
    for v in (0, 12, 3):
        h.set_gemm(v)
        y.fill_(0.0)
        h.matvec_noalloc(xd, y)
        err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err < BOUND[prec], ("noalloc", v, err)
    h.destroy()


@pytest.mark.parametrize("d,extra,rows", [(5, 0, 1), (64, 0, 32), (64, 1, 33), (128, 0, 128), (128, 1, 129),
                                          (181, 0, 256), (181, 2, 257)])
def test_lanczos_totals_at_row_limits(env, d, extra, rows):
    """64 Lanczos vectors (1 to 5 reduction launches) on either side of 128 partial rows, up to
    which the update pass sums them itself, and 256, the most there are; `rows` counts 512 states
    each (16 wavefronts of 32)."""
    torch, L = env
    pb = _problem(((d,) * 4, (d, d, d, d + extra)))
    h = L.dmrg_create(pb)
    assert -(-h.n // 512) == rows
    x = I.random_psi(h.n, np.random.default_rng(I.SEED_BASE + 9))
    xd = torch.from_numpy(x).to("cuda")
    y = torch.empty_like(xd)
    tau = 0.2 / d                       # of the order of 1 / ||H||: converged with 64 vectors
    info = h.krylov_expm(xd, y, tau, 64, 1)
    yref, oinfo = K.krylov_expm(lambda v: M.matvec_sector(pb, v), x, tau, 64, 1)
    assert info["k_eff"] == oinfo.k_eff[-1]
    assert np.linalg.norm(y.cpu().numpy() - yref) <= 1e-10 * np.linalg.norm(yref)
    h.destroy()


@pytest.mark.parametrize("m", [100, 400])
def test_move_at_tile_edges(env, m):
    """Moves of the centre that keep 1, 15, 16, 17, 31, 32, 33 ... states of sectors of 1 to 60 (rows,
    columns and inner dimensions around the 16 of a tile and a chunk), against the oracle: sums of
    at most 60 products in each of two stages."""
    from oracle import wft as Wo
    torch, L = env
    pb = I.synthetic_problem(24, m, 4.0, I.chain_bonds(24), I.SEED_BASE + 11)
    rng = np.random.default_rng(I.SEED_BASE + 12)
    blk = I.psi_blocks(pb)
    kept = [min((1, 15, 16, 17, 31, 32, 33, 60)[b % 8], r) for b, (_, _, r, _) in enumerate(blk)]
    mv = I.wft_move(pb, kept, seed=3)
    evecs = [rng.standard_normal((r, r)) + 1j * rng.standard_normal((r, r)) for (_, _, r, _) in blk]
    planes = lambda a: np.concatenate([a.real.ravel(order="F"), a.imag.ravel(order="F")])
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    h = L.dmrg_create(pb)
    w = h.wft_create(mv, [cuda(planes(m)) for m in mv.W])
    xs = [I.random_psi(h.n, rng) for _ in range(3)]
    ys = [torch.full((2 * w.n_new,), float("nan"), dtype=torch.float64, device="cuda") for _ in xs]
    w.apply(cuda(np.concatenate([planes(u) for u in evecs])), [cuda(x) for x in xs], ys)
    for x, y in zip(xs, ys):
        ref = Wo.wft_right(pb, mv, evecs, x)
        assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-13 * np.linalg.norm(ref)
    w.destroy()
    h.destroy()


def test_local_terms_mixed_and_many(env):
    """Lists of terms with monomial factors (gathered), dense factors (products) and both, more lists
    than a handle keeps, each called twice in turn, into the same sector; and their expectations.
    Sums of at most 33 products per element: 1e-13 of the largest."""
    from oracle import observables as Ob
    torch, L = env
    pb = _problem(DIMS[2])
    rng = np.random.default_rng(I.SEED_BASE + 14)

    def op(space, mono):
        o = I.BlockOp((0, 0))
        for p, d in enumerate(space.dim):
            a = rng.standard_normal((d, d))
            if mono:                                    # a permutation with values, some rows empty
                a = np.where(np.eye(d)[rng.permutation(d)] > 0, a, 0.0)
                a[rng.random(d) < 0.2] = 0.0
            o.blocks[p] = a
        return o

    sS = [op(pb.S.space, m) for m in (True, False)]
    sE = [op(pb.E.space, m) for m in (True, False)]
    pbx, iS, iE = I.with_ops(pb, sS, sE)
    h = L.dmrg_create(pbx)
    x = I.random_psi(h.n, rng)
    xd = torch.from_numpy(x).to("cuda")
    none = -1
    lists = []
    for k in range(4):
        c = 0.5 + k
        lists += [([(c, iS[0], 0, iE[0], 0, 1), (1.0, none, 0, iE[0], 1, 0)],
                   [(c, sS[0], sE[0], 1), (1.0, None, I._transpose(sE[0], pb.E.space), 0)]),
                  ([(c, iS[1], 0, none, 0, 0), (2.0, iS[0], 1, none, 0, 1)],
                   [(c, sS[1], None, 0), (2.0, I._transpose(sS[0], pb.S.space), None, 1)]),
                  ([(c, iS[0], 0, iE[1], 0, 0)], [(c, sS[0], sE[1], 0)])]
    for g, o in lists + lists:
        y = torch.full((2 * h.n,), float("nan"), dtype=torch.float64, device="cuda")
        for _ in range(2):
            h.apply_local(h, g, xd, y)
        ref = Ob.apply_terms(pbx, pbx, o, x)
        assert np.max(np.abs(y.cpu().numpy() - ref)) <= 1e-13 * np.max(np.abs(ref)) * 33
        e, want = h.expect_local(g, xd), Ob.expect(pbx, o, x)
        assert abs(e - want) <= 1e-12 * max(1.0, abs(want))
    h.destroy()


@pytest.mark.parametrize("dims", [(1, 15, 17, 33), (64, 84, 90, 161), (9, 160, 230, 341)],
                         ids=["33", "161", "341"])
@pytest.mark.parametrize("size", [1, 2, 5, 8, 9])
def test_density_clusters(env, dims, size):
    """Spectra in clusters of `size` eigenvalues 1e-8 apart (from 9 on QL takes the sector), with the
    columns of a cluster on either side of a work group's range, in sectors whose columns fit in
    LDS and in larger ones: eigenvalues, residuals and orthonormality, with the bounds of the
    parity test (1e-12 of the largest eigenvalue; 1e-11 d)."""
    torch, L = env
    pb = _problem((dims, dims[::-1]))       # square blocks
    rng = np.random.default_rng(I.SEED_BASE + 16)
    blk = I.psi_blocks(pb)
    re, im, rhos = [], [], []
    for (_, _, r, c) in blk:
        assert r == c
        q = [np.linalg.qr(rng.standard_normal((r, r)) + 1j * rng.standard_normal((r, r)))[0] for _ in range(2)]
        lam = (1.0 + np.arange(r) // size + 1e-8 * (np.arange(r) % size)) / r
        m = (q[0] * np.sqrt(lam)) @ q[1]
        re.append(m.real.ravel(order="F"))
        im.append(m.imag.ravel(order="F"))
        rhos.append((m @ m.conj().T, lam[::-1]))
    x = np.concatenate(re + im)
    h = L.dmrg_create(pb)
    total = sum(r for (_, _, r, _) in blk)
    ev = torch.zeros(total, dtype=torch.float64, device="cuda")
    vc = torch.zeros(sum(2 * r * r for (_, _, r, _) in blk), dtype=torch.float64, device="cuda")
    h.density_truncate([torch.from_numpy(x).to("cuda")], np.array([1.0]), total, ev, vc)
    ev, vc = ev.cpu().numpy(), vc.cpu().numpy()
    eo = vo = 0
    for (rho, lam) in rhos:
        d = len(lam)
        w = ev[eo:eo + d]
        U = (vc[vo:vo + d * d] + 1j * vc[vo + d * d:vo + 2 * d * d]).reshape(d, d).T
        assert np.max(np.abs(w - lam)) <= 1e-12 * lam[0]
        assert np.linalg.norm(U.conj().T @ U - np.eye(d)) <= 1e-11 * d
        assert np.linalg.norm(rho @ U - U * w) <= 1e-11 * lam[0] * d
        eo += d
        vo += 2 * d * d
    h.destroy()


@pytest.mark.parametrize("dims,kdim", [(((1, 1, 1, 1), (1, 1, 1, 1)), 4), (((3, 2, 1, 3), (1, 3, 5, 2)), 15),
                                       (((3, 2, 1, 3), (2, 3, 5, 5)), 18), (((5, 4, 3, 3), (5, 4, 3, 5)), 33),
                                       (((9, 8, 7, 11), (7, 9, 8, 9)), 48)])
@pytest.mark.parametrize("tau", [1e-7, 0.03, 2.0])
def test_lanczos_small_and_odd(env, dims, kdim, tau):
    """Spaces of 4 to some 290 states (odd numbers, less than one group of 32 and a few more), bases around
    the 15 slots of a reduction launch, and times from far below to far above 1 / ||H||."""
    torch, L = env
    pb = _problem(dims)
    h = L.dmrg_create(pb)
    x = I.random_psi(h.n, np.random.default_rng(I.SEED_BASE + 17))
    xd = torch.from_numpy(x).to("cuda")
    y = torch.empty_like(xd)
    kdim = min(kdim, h.n)
    tau = tau / max(max(d) for d in dims)
    info = h.krylov_expm(xd, y, tau, kdim, 2)
    yref, oinfo = K.krylov_expm(lambda v: M.matvec_sector(pb, v), x, tau, kdim, 2)
    assert info["k_eff"] == oinfo.k_eff[-1]
    assert np.linalg.norm(y.cpu().numpy() - yref) <= 1e-10 * np.linalg.norm(yref)
    h.destroy()
