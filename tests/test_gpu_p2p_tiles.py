"""The symmetric P2P kernel's other dealing rule: launches of 8192 chunks and more (tiles plus chunks of the
plan's grid; here by a plan made for many particles, with tiles of two cells) deal whole neighbour tiles to
the three waves of a chunk instead of units of eight sources.  Repeated positions, crowded and empty tiles
and boxes that wrap, with the bounds of the sweep over small launches: 1e-12 of the max for the full FP64
pair formula, 1e-10 and 1e-9 for the reduced-cost levels, 2e-6 for FP32 pairs."""
import numpy as np
import pytest
from test_gpu_p2p_sweep import dev, host, maxrel, positions

import oracle
from paper_2606_19059_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (n, box, grid, xi, r_c, distribution)
CASES = [
    (777, (1.0, 1.0, 1.0), (64, 64, 64), 14.0, 0.25, "sparse"),
    (1024, (1.0, 1.0, 1.0), (64, 64, 64), 14.0, 0.15, "repeats"),
    (1500, (1.0, 1.0, 1.0), (64, 64, 64), 14.0, 0.3, "dense"),
    (1100, (0.25, 1.0, 1.0), (16, 64, 128), 14.0, 0.24, "uniform"),  # r_c of nearly the short edge: wraps
]
LEVELS = [("fp64", 1e-11, 1e-12), ("fp64", 1e-9, 1e-10), ("fp64", 1e-7, 1e-9), ("fp32", 1e-5, 2e-6)]


def _plan(E, case, precision, tol, **kw):
    n, box, grid, xi, rc, _ = CASES[case]
    cells = grid[0] * grid[1] * grid[2]
    pl = E.Plan(box, tol, xi=xi, r_c=rc, grid=grid, P=8, n_max=16 * cells, precision=precision, **kw)
    assert pl.info["tile"] == 2 and cells // 8 >= 8192
    return pl


def _particles(case):
    n, box, _, _, _, kind = CASES[case]
    rng = np.random.default_rng(700 + case)
    return positions(kind, n, box, rng), W.mean_free_forces(rng, n), rng


@pytest.mark.parametrize("precision,tol,bound", LEVELS)
@pytest.mark.parametrize("case", range(len(CASES)))
def test_tile_dealing_matches_oracle(case, precision, tol, bound):
    import paper_2606_19059_amd as E

    _, box, _, xi, rc, _ = CASES[case]
    x, f, _ = _particles(case)
    un, _ = _plan(E, case, precision, tol).eval_parts(dev(x), dev(f))
    assert maxrel(host(un), oracle.real_space(x, f, box, xi, rc)) < bound


@pytest.mark.parametrize("precision,tol,bound", [LEVELS[0], LEVELS[3]])
@pytest.mark.parametrize("case", [1, 2])
def test_tile_dealing_stresslet_matches_oracle(case, precision, tol, bound):
    import paper_2606_19059_amd as E

    n, box, _, xi, rc, _ = CASES[case]
    x, f, rng = _particles(case)
    q, nr = rng.standard_normal((3, n)), rng.standard_normal((3, n))
    un, _ = _plan(E, case, precision, tol, stresslet=True).eval_combined_parts(dev(x), dev(f), dev(q), dev(nr))
    ref = oracle.real_space(x, f, box, xi, rc) + oracle.real_space_st(x, oracle.stresslet_tensor(q, nr), box, xi, rc)
    assert maxrel(host(un), ref) < bound
