"""Trees of few particles, whose orders are found by counting: one element to
several wavefronts of keys, the largest such tree and the next one, equal keys
over many positions (Morton cells and coordinates), and distant outliers.  The
tree must be the oracle's, and the centre-of-mass tree's, which takes the same
Morton order."""
import numpy as np
import pytest

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import gpu_run, say

pytestmark = pytest.mark.gpu


def same_tree(exp, t):
    for k in ("perm", "first", "count", "left", "right", "axis"):
        np.testing.assert_array_equal(exp[k], getattr(t, k))


@pytest.mark.parametrize("kind", ["plain", "ties", "one_point", "outlier"])
@pytest.mark.parametrize("n", [1, 17, 64, 130, 3001, 12288, 12289])
def test_order_by_counting(orc, n, kind):
    x, m, h = W.plummer(n, 70)
    if kind == "ties":
        x = np.round(x * 4.0) / 4.0
    elif kind == "one_point":
        x[n // 3:] = x[0]
    elif kind == "outlier":
        x[-1] = 1e9
    say(f"[gpu few] n {n}, {kind}")
    _, exp, _ = gpu_run(x, m, h, theta=1.0)
    same_tree(exp, orc.build_tree(x, leaf_size=8))
    if n <= 3001 and kind != "one_point":
        _, exp, _ = gpu_run(x, m, h, theta=1.0, tree_shape=F.FMM_TREE_COM)
        same_tree(exp, orc.build_tree_com(x, m, leaf_size=8))
