"""P2G's search for a round's particles (16 a wave): crowded columns of cells, whose rounds lie in a few runs of
the cell-sorted order, next to sparse ones, with cell sizes on both sides of a round, runs that end with a
slab, and rounds cut short by a pass of four slabs.  The grid is compared with the oracle's element by element at
1e-12 of its max (FP64 sums in different orders)."""
import numpy as np
import pytest

from oracle import spectral as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("P,m", [(4, 3.0), (12, 5.8), (16, 6.6)])
@pytest.mark.parametrize("grid", [(8, 16, 16), (64, 32, 16)])
@pytest.mark.parametrize("n_max", [6000, 200_000])
def test_crowded_columns_match_oracle(grid, n_max, P, m):
    import paper_2606_19059_amd as E

    box = tuple(g / 64.0 for g in grid)
    rng = np.random.default_rng(71)
    cells = []
    # the columns of five slabs, with the cells' sizes in turn, and single particles all over the box
    sizes = [1, 15, 16, 17, 0, 64, 3, 200, 33, 1, 1, 5]
    for i, (cx, cy) in enumerate([(1, 2), (2, 2), (3, 9), (6, 2), (7, 15), (2, 3), (1, 12)]):
        cells += [((cx, cy, cz), sizes[(cz + 5 * i) % len(sizes)]) for cz in range(grid[2])]
    x = np.concatenate([(np.array(c)[:, None] + rng.random((3, k))) / 64.0 for c, k in cells] +
                       [rng.random((3, 300)) * np.array(box)[:, None]], axis=1)
    f = rng.standard_normal(x.shape)
    pl = E.Plan(box, 1e-11, xi=12.0, r_c=0.12, grid=grid, P=P, window_shape=m, n_max=max(n_max, x.shape[1]))
    g = pl.spread(torch.from_numpy(x).to("cuda"), torch.from_numpy(f).to("cuda")).cpu().numpy()
    ref = S.p2g(x, f, box, grid, P, m)
    assert np.max(np.abs(g - ref)) < 1e-12 * np.max(np.abs(ref))
