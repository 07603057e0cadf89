"""G2P's two forms on FP64 grids (a wave per 16 targets, and four waves sharing them) at every tile
edge: the far field of few particles, with plans made for sizes on both sides of the rule, against
the oracle's spectral far field at 1e-12 of its max (FP64 sums in different orders)."""
import numpy as np
import pytest

from oracle import spectral as S
from paper_2606_19059_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# grid, plan sizes of the two forms (a wave per group, split), tile edge of the former
CASES = [((16, 16, 16), 200_000, 100_000, 2), ((32, 32, 32), 200_000, 60_000, 4),
         ((64, 64, 32), 200_000, 100_000, 8), ((128, 128, 64), 140_000, 50_000, 16)]


@pytest.mark.parametrize("precision,tol,P,m", [("fp64", 1e-11, 16, 6.6), ("fp64", 1e-11, 6, 4.1),
                                               ("fp32", 5e-7, 10, 5.3)])
@pytest.mark.parametrize("grid,n_wave,n_split,tile", CASES)
def test_g2p_forms_match_oracle(grid, n_wave, n_split, tile, precision, tol, P, m):
    import paper_2606_19059_amd as E

    box = tuple(g / 64.0 for g in grid)
    n, xi = 333, 0.2 * 64
    x, f = W.particles(n, box, seed=29)
    ref = S.far_field(x, f, box, grid, xi, P, m)
    bound = 1e-12 if precision == "fp64" else 3e-6  # FP32 weights: each product rounded
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    for n_max in (n_wave, n_split):
        pl = E.Plan(box, tol, xi=xi, r_c=0.2, grid=grid, P=P, window_shape=m, n_max=n_max, precision=precision)
        assert n_max != n_wave or pl.info["tile"] == tile
        uf = pl.eval_parts(d(x), d(f))[1].cpu().numpy()
        assert np.max(np.abs(uf - ref)) < bound * np.max(np.abs(ref))


@pytest.mark.parametrize("grid,tile", [((16, 16, 16), 2), ((32, 32, 32), 4), ((64, 64, 32), 8), ((128, 128, 64), 16)])
def test_target_order_of_dense_tiles_matches_oracle(grid, tile):
    """Tiles on both sides of the density from which G2P keeps the sort's order (8 targets per column of a
    tile): each target still gets its own far field."""
    import paper_2606_19059_amd as E

    box = tuple(g / 64.0 for g in grid)
    n, xi = 700 + 9 * tile * tile, 0.2 * 64
    x, f = W.particles(n, box, seed=43)
    x[:, 700:] = (tile + tile * (x[:, 700:] / np.array(box)[:, None])) / 64.0  # one tile's cells
    ref = S.far_field(x, f, box, grid, xi, 6, 4.1)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    pl = E.Plan(box, 1e-11, xi=xi, r_c=0.2, grid=grid, P=6, window_shape=4.1, n_max=140_000)
    uf = pl.eval_parts(d(x), d(f))[1].cpu().numpy()
    assert np.max(np.abs(uf - ref)) < 1e-12 * np.max(np.abs(ref))
