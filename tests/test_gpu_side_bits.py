"""The level split on both sides of the size from which the sides by rank are
looked up as bits (2^21 particles), with a ragged last word.  The tree must be
the oracle's."""
import numpy as np
import pytest
import torch

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1, (1 << 21) + 4103])
def test_tree_is_the_oracles(orc, n):
    x, m, h = W.plummer(n, 95)
    say(f"[gpu side bits] n {n}")
    ref = orc.build_tree(x, leaf_size=64)
    t = F.fmm_build_tree(torch.from_numpy(x).to("cuda"), F.default_params(leaf_size=64))
    try:
        torch.cuda.synchronize()
        exp = F.fmm_debug_export(t, lists=False)
    finally:
        F.fmm_tree_free(t)
    for k in ("perm", "first", "count", "left", "right", "axis"):
        np.testing.assert_array_equal(exp[k], getattr(ref, k))
