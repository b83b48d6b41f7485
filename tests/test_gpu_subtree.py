"""The workgroup that finishes a cell in LDS, at the sizes where its layout
changes: cells within one wavefront, within one and two positions per thread,
around the largest, leaves of one particle to the largest leaf, a cell that is
a leaf, and coordinates with many ties.  The tree must be the oracle's."""
import numpy as np
import pytest

from paper_2502_01496_amd import workloads as W
from tests.gpu_util import gpu_run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf", [1, 8, 64])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129, 1023, 1024, 1025, 2047, 2048, 2049, 4097,
                               6000])
def test_tree_is_the_oracles(orc, n, leaf):
    x, m, h = W.plummer(n, 60 + n % 7)
    if n % 2:
        x[::3, 0] = x[0, 0]  # ties on one axis
    say(f"[gpu subtree] n {n} leaf {leaf}")
    t = orc.build_tree(x, leaf_size=leaf)
    _, exp, _ = gpu_run(x, m, h, leaf=leaf)
    for k in ("perm", "first", "count", "left", "right", "axis"):
        np.testing.assert_array_equal(exp[k], getattr(t, k))
