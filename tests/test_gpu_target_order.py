"""Batches on plans that give G2P's targets an order of their own (FP64 grids, made for 32768 particles or
more): every system's result is the one it has alone, bit for bit (deterministic plans), and the far
field is the oracle's.  The last plan has 131072 tiles, so that 64 systems have 2^23: one block a tile
would be more threads than a launch can have."""
import numpy as np
import pytest

from oracle import spectral as S
from paper_2606_19059_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid,n_max,tile,sizes", [
    ((32, 32, 32), 600_000, 2, [300, 1, 0, 700, 65]),
    ((32, 32, 32), 100_000, 4, [300, 1, 0, 700, 65]),
    ((64, 64, 64), 40_000, 16, [1500, 1, 0, 700, 65]),
    ((128, 128, 64), 1 << 24, 2, [20 + k for k in range(64)]),
])
def test_batch_with_target_order_equals_systems_alone(grid, n_max, tile, sizes):
    import paper_2606_19059_amd as E

    box = tuple(g / 64.0 for g in grid)
    x, f = W.particles(sum(sizes), box, seed=61)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    pl = E.Plan(box, 1e-11, xi=0.2 * 64, r_c=0.2, grid=grid, P=4, window_shape=3.3, n_max=n_max, deterministic=True)
    assert pl.info["tile"] == tile
    u = pl.eval_batch(d(x), d(f), sizes).cpu()
    at = 0
    for k, n in enumerate(sizes):
        s = slice(at, at + n)
        at += n
        if n == 0 or 4 <= k < len(sizes) - 1:
            continue
        assert torch.equal(u[:, s], pl.eval(d(x[:, s]), d(f[:, s])).cpu())
        if k in (0, 3):
            uf = pl.eval_parts(d(x[:, s]), d(f[:, s]))[1].cpu().numpy()
            ref = S.far_field(x[:, s], f[:, s], box, grid, 0.2 * 64, 4, 3.3)
            assert np.max(np.abs(uf - ref)) < 1e-12 * np.max(np.abs(ref))
