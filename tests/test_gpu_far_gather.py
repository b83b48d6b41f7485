"""The FP64 far field of the leaf <- cell lists over short and ragged lists (a
unit of 8 lanes reads the records of its sources four lanes together, so the
ends of the lists are where lanes have no source of their own), forces against
the oracle and the reverse pass through the identities sum_j xbar_j = 0 and
sum_j m_j mbar_j = <abar, a> (bars as in the other parity tests; 1e-11 of the
sums of the absolute terms)."""
import numpy as np
import pytest

from paper_2502_01496_amd import workloads as W
from tests.gpu_util import force_err, gpu_run, gpu_vjp, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("theta", [0.4, 1.0])
@pytest.mark.parametrize("n,leaf", [(30, 1), (47, 1), (90, 2), (200, 8), (333, 3), (1501, 8)])
def test_short_far_lists(orc, n, leaf, theta):
    x, m, h = W.plummer(n, 90)
    say(f"[gpu far gather] plummer {n}, leaf {leaf}, theta {theta}")
    ref = orc.fmm(x, m, h, theta=theta, leaf_size=leaf)
    a, _, _ = gpu_run(x, m, h, theta=theta, leaf=leaf, export=False)
    assert force_err(a, ref.a) <= 1e-12
    abar = W.cotangent(n, 91)
    a, [(xb, mb)] = gpu_vjp(x, m, h, abar, theta=theta, leaf=leaf)
    assert (np.abs(xb.sum(0)) <= 1e-11 * np.abs(xb).sum(0)).all()
    lhs, rhs = (m * mb).sum(), (abar * a).sum()
    assert abs(lhs - rhs) <= 1e-11 * (np.abs(m * mb).sum() + np.abs(abar * a).sum())
