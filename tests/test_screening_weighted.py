"""The weighted near-field screening polynomials (csrc/screening.h, kScreenW*) against mpmath: C(x) =
e^{-x^2} times a polynomial in X = x sqrt(log2 e), evaluated in FP64 by Horner as the reduced-cost
FP64 pairs do.  Bounds on |dC| over 0 <= x <= 6.5: the minimax errors of degrees 18 and 15
(2.72e-12, 1.53e-10) with 3% for the 3001-point exchange grid."""
import math

import numpy as np
from test_screening import _c_ref, _consts


def test_weighted_screening_polynomials_meet_their_bounds():
    s, arrs = _consts()
    x = np.linspace(0.0, s["kScreenXmax"], 5201)
    ref = _c_ref(x)
    X = x * math.sqrt(1.0 / math.log(2.0))
    for tag, deg, bound in (("W1", 18, 2.8e-12), ("W2", 15, 1.58e-10)):
        m = arrs["kScreen" + tag]
        assert len(m) == deg
        q = X + m[-1]
        for a in m[-2::-1]:
            q = q * X + a
        err = np.max(np.abs(np.exp2(-X * X) * (s["kScreenLead" + tag] * q) - ref))
        assert err < bound, (tag, err)
