"""|M_h|^2 of opposite helicity combinations, the identity by which the FP64 kernels evaluate one
combination of each pair: equal in the oracle, which evaluates every combination."""
import numpy as np
import oracle
import pytest
from tests import workloads as W


# the rounding of |M_h|^2 grows with the cancellation between its diagrams: bounded for these few
# ordinary points by 1e-12 of the largest combination (typically 1e-15)
@pytest.mark.parametrize("name", ["ee_mumu", "gg_tt", "gg_ttg", "gg_ttgg"])
def test_opposite_helicities_have_equal_squares(name):
    p = oracle.rambo(11, W.sqrt_s(name), W.final_masses(name), 4)
    for e in range(len(p)):
        _, h = oracle.me(name, p[e], params=W.PARAMS, per_helicity=True)
        h = np.asarray(h)
        assert np.abs(h - h[::-1]).max() <= 1e-12 * h.max()
