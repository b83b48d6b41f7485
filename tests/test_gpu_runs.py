"""Runs of coordinates that share the high half of their sort key, at the
lengths where their treatment changes (one entry, up to 64, more) and at every
place against the blocks of 256 and the words of 64 entries; low halves differ,
repeat or are equal.  The tree must be the oracle's."""
import numpy as np
import pytest
import torch

from paper_2502_01496_amd import fmm as F
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [(1,), (2, 3), (63,), (64,), (65,), (66, 1), (1, 64, 65, 2, 130),
                                  (300, 7)])
@pytest.mark.parametrize("low", ["distinct", "repeated", "equal"])
def test_tree_is_the_oracles(orc, lens, low):
    rng = np.random.default_rng(90)
    n = 13001
    x = np.empty((n, 3))
    for d in range(3):
        # 1 + k 2^-20 has its own high half for each k; the low half adds less
        run = np.repeat(np.arange(n), np.resize(lens, n))[:n]
        lo = rng.integers(0, {"distinct": 2 ** 31, "repeated": 5, "equal": 1}[low], n)
        x[:, d] = rng.permutation(1.0 + run * 2.0 ** -20 + lo * 2.0 ** -52)
    say(f"[gpu runs] lengths {lens}, low halves {low}")
    ref = orc.build_tree(x, leaf_size=64)
    t = F.fmm_build_tree(torch.from_numpy(x).to("cuda"), F.default_params(leaf_size=64))
    try:
        torch.cuda.synchronize()
        exp = F.fmm_debug_export(t, lists=False)
    finally:
        F.fmm_tree_free(t)
    for k in ("perm", "first", "count", "left", "right", "axis"):
        np.testing.assert_array_equal(exp[k], getattr(ref, k))
