"""The error of the reduced-cost FP64 pair formulas (screening polynomial and exponential together),
against that of the rational-variable forms with the same exponentials (csrc/screening.h, 64s and
64f): no larger at its maximum, for x > 1, where most pairs within the cutoff lie, and as
(integral of dC^2 dx)^1/2, which enters a sum over uniform pairs."""
import math
import os
import re

import numpy as np
import pytest
from test_screening import HDR, _c_ref, _consts


def _exp2(z, lead, m):
    n = np.rint(z)
    s = z - n
    p = s + m[-1]
    for a in m[-2::-1]:
        p = p * s + a
    return np.ldexp(lead * p, n.astype(int))


def _kernel_tables():
    """The tables that the kernels' arguments are filled from, for levels 1 and 2."""
    src = open(os.path.join(os.path.dirname(HDR), "p2p.hip")).read()
    two, one = re.search(r"mw = lv == 2 \? kScreen(\w+) : kScreen(\w+);", src).groups()
    return {1: one, 2: two}


@pytest.mark.parametrize("lv,rational", [(1, "64s"), (2, "64f")])
def test_error_of_the_pair_formula_is_no_larger_than_the_rational_form(lv, rational):
    s, arrs = _consts()
    x = np.linspace(0.0, s["kScreenXmax"], 6501)[1:]
    ref = _c_ref(x)
    X = x * math.sqrt(1.0 / math.log(2.0))
    e = _exp2(-X * X, s["kExpLead%d" % lv], arrs["kExpM%d" % lv])

    def horner(v, m):
        q = v + m[-1]
        for a in m[-2::-1]:
            q = q * v + a
        return q

    tag = _kernel_tables()[lv]
    err = np.abs(e * s["kScreenLead" + tag] * horner(X, arrs["kScreen" + tag]) - ref)
    t = 1.0 - 2.0 * s["kScreenK"] / (x + s["kScreenK"])
    q = s["kScreenLead" + rational] * horner(t, arrs["kScreenM" + rational]) + 2.0 / math.sqrt(math.pi) * x
    base = np.abs(e * q - ref)
    assert err.max() <= base.max()
    assert err[x > 1].max() <= base[x > 1].max()
    assert np.sum(err**2) <= np.sum(base**2)
