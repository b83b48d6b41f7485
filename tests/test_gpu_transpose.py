"""Transposed interaction lists over the widths of their sort (one digit of 8,
9 and 10 bits, two of 8, 9 and 10, more than two digits, no far pairs at all),
through two identities of the reverse pass that hold for any cotangent and tie
the sink side of every pair to its source side: accelerations do not change
under translation, so sum_j xbar_j = 0, and they are homogeneous of degree one
in the masses, so sum_j m_j mbar_j = <abar, a>.  Both to 1e-11 of the sum of
the absolute terms (rounding of sums of up to 1e5 terms of 1e-16)."""
import numpy as np
import pytest

from paper_2502_01496_amd import workloads as W
from tests.gpu_util import gpu_vjp, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf,theta", [(5, 8, 0.5), (100, 1, 0.5), (200, 1, 0.5), (400, 1, 0.5),
                                          (600, 1, 0.5), (30001, 8, 0.5), (40000, 1, 0.7),
                                          (140000, 1, 0.9), (530000, 1, 1.0)])
def test_sink_and_source_sides_agree(n, leaf, theta):
    x, m, h = W.plummer(n, 80)
    abar = W.cotangent(n, 81)
    say(f"[gpu transpose] plummer {n}, leaf {leaf}, theta {theta}")
    a, [(xb, mb)] = gpu_vjp(x, m, h, abar, theta=theta, leaf=leaf)
    assert (np.abs(xb.sum(0)) <= 1e-11 * np.abs(xb).sum(0)).all()
    lhs, rhs = (m * mb).sum(), (abar * a).sum()
    assert abs(lhs - rhs) <= 1e-11 * (np.abs(m * mb).sum() + np.abs(abar * a).sum())
