"""The waves that share a P2P target chunk: inputs with fewer source batches than waves, all sources
in the targets' own tile, and plans of every size class of the deterministic kernel.  The near field is compared with the oracle's real-space sum at 1e-12 of its max
(full-precision pair formula, FP64 sums in different orders)."""
import numpy as np
import pytest

import oracle
from paper_2606_19059_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOX = (1.0, 1.0, 1.0)


def near_error(x, f, n_max, deterministic):
    import paper_2606_19059_amd as E

    pl = E.Plan(BOX, 1e-11, xi=10.0, r_c=0.45, grid=(32, 32, 32), P=8, window_shape=4.8, n_max=n_max,
                deterministic=deterministic)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    un = pl.eval_parts(d(x), d(f))[0].cpu().numpy()
    ref = oracle.real_space(x, f, BOX, 10.0, 0.45)
    return np.max(np.abs(un - ref)) / max(np.max(np.abs(ref)), 1e-300)


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("n,n_max", [(2, 2), (65, 65), (700, 700), (700, 20_000), (1500, 200_000), (1500, 600_000)])
@pytest.mark.parametrize("one_tile", [False, True])
def test_split_chunks_match_oracle(n, n_max, one_tile, deterministic):
    x, f = W.particles(n, BOX, seed=23)
    if one_tile:
        x = 0.51 + 0.03 * x  # inside one cell of the 32^3 grid's coarsest and finest tiles
    assert near_error(x, f, n_max, deterministic) < 1e-12


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("tol,bound", [(1e-11, 1e-12), (1e-9, 1e-10), (1e-7, 1e-9)])
def test_largest_queue_excess_matches_oracle(tol, bound, deterministic):
    """Chunks whose first half accepts every source of a neighbouring tile and whose second half
    none: 32 pairs for half the lanes, the largest excess a batch can have (512 pairs)."""
    import paper_2606_19059_amd as E

    rng = np.random.default_rng(31)
    parts = []
    # per tile of 0.5: clusters of 32 near one corner and 32 near the opposite one (farther apart than
    # r_c), and in the next tile along z 96 sources within r_c of the first cluster only
    for corner, n in (((0.03, 0.03, 0.42), 32), ((0.45, 0.45, 0.02), 32), ((0.05, 0.05, 0.53), 96)):
        parts.append(np.array(corner)[:, None] + 0.02 * rng.random((3, n)))
    x = np.concatenate(parts, axis=1)
    f = rng.standard_normal(x.shape)
    pl = E.Plan(BOX, tol, xi=10.0, r_c=0.4, grid=(32, 32, 32), P=8, window_shape=4.8, n_max=x.shape[1],
                deterministic=deterministic)
    assert pl.info["tile"] == 16
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    un = pl.eval_parts(d(x), d(f))[0].cpu().numpy()
    ref = oracle.real_space(x, f, BOX, 10.0, 0.4)
    assert np.max(np.abs(un - ref)) < bound * np.max(np.abs(ref))


@pytest.mark.parametrize("precision,tol,bound", [("fp64", 1e-11, 1e-12), ("fp64", 1e-9, 1e-10), ("fp64", 1e-7, 1e-9),
                                                 ("fp32", 1e-6, 5e-6)])
@pytest.mark.parametrize("n_max", [3000, 400_000])
@pytest.mark.parametrize("box,grid", [((0.5, 1.0, 2.0), (16, 32, 64)), ((2.0, 1.0, 0.5), (64, 32, 16))])
def test_deterministic_rows_of_tiles_match_oracle(box, grid, n_max, precision, tol, bound):
    """Rows of tiles that wrap around the box once and several times (r_c of nearly the short edge), sparse
    and crowded tiles."""
    import paper_2606_19059_amd as E

    x, f = W.particles(1500, box, seed=37)
    x[:, :400] = 0.2 + 0.1 * x[:, :400] / np.array(box)[:, None]
    pl = E.Plan(box, tol, xi=10.0, r_c=0.45, grid=grid, P=8, window_shape=4.8, n_max=n_max, precision=precision,
                deterministic=True)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    un = pl.eval_parts(d(x), d(f))[0].cpu().numpy()
    ref = oracle.real_space(x, f, box, 10.0, 0.45)
    assert np.max(np.abs(un - ref)) < bound * np.max(np.abs(ref))
