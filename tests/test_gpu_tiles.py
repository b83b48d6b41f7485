"""The radix sorts of the build at the edges of their tiles of 4096 keys: the
first tree that takes them, whole and ragged last tiles, and both sides of the
tile count up to which a pass has no scan of its own (64).  The tree must be the
oracle's."""
import numpy as np
import pytest
import torch

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [12289, 16384, 16385, 20479, 262144, 262145])
def test_tree_is_the_oracles(orc, n):
    x, m, h = W.plummer(n, 65)
    x[::5, 1] = x[0, 1]  # ties on one axis
    say(f"[gpu tiles] n {n}")
    ref = orc.build_tree(x, leaf_size=64)
    t = F.fmm_build_tree(torch.from_numpy(x).to("cuda"), F.default_params(leaf_size=64))
    try:
        torch.cuda.synchronize()
        exp = F.fmm_debug_export(t, lists=False)
    finally:
        F.fmm_tree_free(t)
    for k in ("perm", "first", "count", "left", "right", "axis"):
        np.testing.assert_array_equal(exp[k], getattr(ref, k))
