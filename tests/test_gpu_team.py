"""The near field of few leaves, whose blocks a team of wavefronts shares:
lists shorter than a share of eight blocks, of one share and of several, leaves
of several blocks, and the last tree that takes a team with the next one, in
both directions.  Forces against the oracle (1e-12), the reverse pass at theta
= 0 (no far field) against the direct-sum adjoint, both as in the other tests."""
import numpy as np
import pytest

from paper_2502_01496_amd import workloads as W
from tests.gpu_util import force_err, gpu_run, gpu_vjp, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(5, 8), (9, 8), (65, 8), (257, 1), (600, 64), (1024, 1), (1025, 1),
                                    (2100, 20)])
def test_reverse_pass(orc, n, leaf):
    x, m, h = W.plummer(n, 95)
    h = h * 5.0
    abar = W.cotangent(n, 96)
    say(f"[gpu team] plummer {n}, leaf {leaf}")
    a, [(xb, mb), (xb2, mb2)] = gpu_vjp(x, m, h, abar, theta=0.0, leaf=leaf, repeat=2)
    assert np.array_equal(xb, xb2) and np.array_equal(mb, mb2)
    assert force_err(a, orc.direct(x, m, h)) <= 1e-12
    xr, mr = orc.direct_vjp(x, m, h, abar)
    assert np.abs(xb - xr).max() <= 1e-12 * np.abs(xr).max()
    assert np.abs(mb - mr).max() <= 1e-12 * np.abs(mr).max()


@pytest.mark.parametrize("n", [4096, 4097])
def test_last_team(orc, n):
    x, m, h = W.clumpy_cube(n, 97, n_clumps=3, cache=False)
    say(f"[gpu team] clumpy {n}, leaf 1")
    a, _, _ = gpu_run(x, m, h, leaf=1, export=False)
    assert force_err(a, orc.fmm(x, m, h, leaf_size=1).a) <= 1e-12
