"""Device memory that dmrg_create plans for the allocation-free product (host only)."""
import numpy as np

from paper_1103_5391_amd import inputs as I
from paper_1103_5391_amd import lib as L

D, E = 64, 49                       # rows and columns of every block
GRID = (36, 37)                     # sectors (N_up, N_dn)


def panel_problem(grid=GRID):
    """No connection terms: every block's intermediate has E columns."""
    rng = np.random.default_rng(I.SEED_BASE + 20)
    qn = np.array([[a, b] for a in range(grid[0]) for b in range(grid[1])], dtype=np.int32)

    def half(d):
        h = rng.standard_normal((d, d))
        return I.Half(I.Space(qn.copy(), np.full(len(qn), d, dtype=np.int32)), [h + h.T] * len(qn), [],
                      [(0, 0), (0, 1)], [])

    return I.Problem(half(D), half(E), (grid[0] - 1, grid[1] - 1), [])


def test_panels_above_the_scratch_have_an_array_of_their_own():
    """Blocks whose intermediate is within the limit by their columns and above it in panels of 16: the
    handle holds dmrg_matvec's workspace and an array for dmrg_matvec_noalloc, not one for both.
    Everything else grows with the number of blocks, so the array shows against a problem of fewer
    blocks whose panels fit the library's (to a tenth: work lists are padded)."""
    scratch, small = 64 << 20, (28, 35)
    nb, ns = GRID[0] * GRID[1], small[0] * small[1]
    panels = 16 * D * 64                # bytes of one block's
    assert 16 * D * E * nb <= scratch < panels * nb and panels * ns <= scratch
    per_block = lambda grid: L.plan_stats(panel_problem(grid))["create_bytes"] / (grid[0] * grid[1])
    assert abs(per_block(GRID) - per_block(small) - panels) < 0.1 * panels
