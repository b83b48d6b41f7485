"""The exact cell extents s (the largest distance of a cell's particle from its
centre) where the evaluation splits: wavefronts that end inside a cell, cells of
64 particles, and more than eight levels of cells that hold a whole wavefront.
The maximum does not depend on the order in which it is taken, so s must equal,
bit for bit, the one formed from the exported centres."""
import numpy as np
import pytest
import torch

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(1, 8), (63, 1), (64, 1), (64, 64), (65, 8), (127, 64),
                                    (128, 64), (129, 1), (4096, 8), (4097, 64), (16384, 64),
                                    (16385, 8), (40000, 3), (65536, 1)])
def test_extents(n, leaf):
    x, m, h = W.plummer(n, 71)
    X, M, H = to_dev(x, m, h)
    say(f"[gpu extents] n {n} leaf {leaf}")
    t = F.fmm_build_tree(X, F.default_params(leaf_size=leaf))
    try:
        F.fmm_moments(t, X, M, H)
        torch.cuda.synchronize()
        e = F.fmm_debug_export(t, lists=False)
    finally:
        F.fmm_tree_free(t)
    xt, rec = x[e["perm"]], e["rec"]
    for v in range(len(e["first"])):
        f, c = e["first"][v], e["count"][v]
        d = xt[f:f + c] - rec[v, 1:4]
        d2 = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]
        assert rec[v, 4] == np.sqrt(d2.max()), v
