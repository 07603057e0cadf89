"""P2G's sweep where it can go wrong: grids shorter than the stencil in x (points added modulo
M1), run tables that shrink the sweep's window (small tiles), segments of several windows, and
clusters that make all waves of a block share the same slabs.  The grid is compared with the
oracle's element by element at 1e-12 of its max (FP64 sums in different orders)."""
import numpy as np
import pytest

from oracle import spectral as S
from paper_2606_19059_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# name: box, grid, P, window shape, particles, share of them clustered into 1.5 cells along x
CASES = {
    "fold_P10": ((0.5, 1.0, 0.5), (8, 16, 8), 10, 5.3, 500, 0.0),
    "fold_P12": ((0.5, 1.0, 0.5), (8, 16, 8), 12, 5.8, 500, 0.5),
    "fold_P14": ((0.5, 0.5, 1.0), (8, 8, 16), 14, 6.2, 333, 0.0),
    "fold_small_tiles_P16": ((1.0, 1.0, 1.0), (8, 8, 8), 16, 6.6, 9000, 0.0),
    "small_tiles_P14": ((1.0, 0.5, 0.5), (16, 8, 8), 14, 6.2, 17000, 0.0),
    "one_window_P8": ((1.0, 0.25, 0.25), (64, 16, 16), 8, 4.8, 3001, 0.9),
    "two_windows_P16": ((1.0, 0.25, 0.25), (64, 16, 16), 16, 6.6, 2000, 0.95),
    "two_windows_even_P16": ((1.0, 0.25, 0.25), (64, 16, 16), 16, 6.6, 2000, 0.0),
    "one_slab_P4": ((2.0, 0.25, 0.25), (128, 16, 16), 4, 3.0, 2500, 1.0),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_p2g_sweep_matches_oracle(name):
    import paper_2606_19059_amd as E

    box, grid, P, m, n, share = CASES[name]
    x, f = W.particles(n, box, seed=17)
    k = int(share * n)
    h = box[0] / grid[0]
    x[0, :k] = np.mod(0.45 * box[0] + 1.5 * h * x[0, :k] / box[0], box[0])
    pl = E.Plan(box, 1e-11, xi=1.5 / h / 4, r_c=0.2, grid=grid, P=P, window_shape=m, n_max=n)
    g = pl.spread(torch.from_numpy(x).to("cuda"), torch.from_numpy(f).to("cuda")).cpu().numpy()
    ref = S.p2g(x, f, box, grid, P, m)
    assert np.max(np.abs(g - ref)) < 1e-12 * np.max(np.abs(ref))
