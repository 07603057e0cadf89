"""Nearly touching particles: the near field of pairs 1e-10 (FP32, deterministic: 1e-12) apart, dominated by each particle's partner,
against the oracle's real-space sum, particle by particle.  The difference of two such positions is
exact in FP64, and has to reach the pair formula so.

The symmetric kernel takes positions relative to the centre of a chunk's targets, which rounds few of
them (those near a face of the box): the median error is that of the pair formula (full FP64 1e-13;
reduced-cost levels 1e-11 and 5e-10, the screening polynomial's and the exponential's error at
r = 0; FP32 2e-6).  The deterministic kernel takes the particles' own positions: the same bounds hold for
every particle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOX = (1.0, 1.0, 1.0)
VARIANTS = [("fp64", 1e-11, 1e-13), ("fp64", 1e-9, 1e-11), ("fp64", 1e-7, 5e-10), ("fp32", 1e-5, 2e-6)]


def pair_errors(sep, n, n_max, xi, deterministic, precision, tol):
    import paper_2606_19059_amd as E

    rng = np.random.default_rng(53)
    a = rng.random((3, n // 2))
    d = rng.standard_normal(a.shape)
    x = np.concatenate([a, a + sep * d / np.linalg.norm(d, axis=0)], axis=1)
    x = np.minimum(x, np.nextafter(1.0, 0.0))
    f = rng.standard_normal(x.shape)
    pl = E.Plan(BOX, tol, xi=xi, r_c=0.25, grid=(32, 32, 32), P=8, n_max=n_max, precision=precision,
                deterministic=deterministic)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda")
    un = pl.eval_parts(dev(x), dev(f))[0].cpu().numpy()
    ref = oracle.real_space(x, f, BOX, xi, 0.25)
    return np.linalg.norm(un - ref, axis=0) / np.linalg.norm(ref, axis=0)


@pytest.mark.parametrize("precision,tol,bound", VARIANTS)
@pytest.mark.parametrize("xi,n_max", [(9.0, 1500), (14.0, 1500), (18.0, 200_000)])
def test_close_pairs_match_oracle(xi, n_max, precision, tol, bound):
    assert np.median(pair_errors(1e-10, 1500, n_max, xi, False, precision, tol)) < bound


@pytest.mark.parametrize("precision,tol,bound", VARIANTS)
@pytest.mark.parametrize("xi,n_max", [(9.0, 1500), (14.0, 200_000)])
def test_close_pairs_deterministic_match_oracle(xi, n_max, precision, tol, bound):
    sep = 1e-12 if precision == "fp32" else 1e-10
    assert np.max(pair_errors(sep, 1500, n_max, xi, True, precision, tol)) < bound


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("tol,bound", [(1e-9, 1e-10), (1e-7, 1e-9)])
@pytest.mark.parametrize("side", [3e-9, 1e-3, 7e8])
def test_power_of_two_scale_of_any_box(side, tol, bound, deterministic):
    """The reduced-cost levels scale positions by a power of two near xi (log2 e)^1/2: boxes of any size, with
    the bounds of the sweep over unit boxes."""
    import paper_2606_19059_amd as E

    rng = np.random.default_rng(59)
    box, xi, rc = (side, side, side), 11.0 / side, 0.35 * side
    x, f = rng.random((3, 700)) * side, rng.standard_normal((3, 700))
    pl = E.Plan(box, tol, xi=xi, r_c=rc, grid=(32, 32, 32), P=8, window_shape=4.8, n_max=700,
                deterministic=deterministic)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda")
    un = pl.eval_parts(dev(x), dev(f))[0].cpu().numpy()
    ref = oracle.real_space(x, f, box, xi, rc)
    assert np.max(np.abs(un - ref)) < bound * np.max(np.abs(ref))
