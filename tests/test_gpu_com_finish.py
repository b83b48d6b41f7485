"""The centre-of-mass tree around the size from which a cell is finished by one
workgroup in LDS (2048): one such cell, cells above it, leaves of one particle
to the largest, particles that share a grid point, cuts that split off a few
particles at a time, and strongly unequal weights.  Tree, numbering and levels
must be the oracle's."""
import numpy as np
import pytest

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import gpu_run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["plain", "clones", "nested", "weights"])
@pytest.mark.parametrize("leaf", [1, 10, 64])
@pytest.mark.parametrize("n", [1, 11, 65, 2048, 2049, 4500, 9001])
def test_tree_is_the_oracles(orc, n, leaf, kind):
    x, m, h = W.clumpy_cube(max(n, 70), 75, n_clumps=3, cache=False)
    x, m, h = x[:n].copy(), m[:n].copy(), h[:n].copy()
    if kind == "clones":
        x[n // 2:] = x[: n - n // 2]
        x[: n // 3] = x[0]
    elif kind == "nested":
        x *= 2.0 ** -(np.arange(n) % 23)[:, None]
    elif kind == "weights":
        m *= 10.0 ** (8.0 * np.sin(np.arange(n)))
    say(f"[gpu com finish] n {n} leaf {leaf} {kind}")
    t = orc.build_tree_com(x, m, leaf_size=leaf)
    _, exp, info = gpu_run(x, m, h, theta=1.0, leaf=leaf, tree_shape=F.FMM_TREE_COM)
    for k in ("perm", "first", "count", "left", "right", "axis"):
        np.testing.assert_array_equal(exp[k], getattr(t, k))
    assert info["nodes"] == t.nnodes
