"""A reused tree whose last walk found short lists evaluates the next walk's
long ones whole, and in pieces on the next call: the same bits, and those of a
fresh tree, whose first walk splits at once.  Pieces of 64 near blocks, so that a
team's wavefronts all have a share of one, and of 100 far entries; leaf counts
at the last tree that takes a team (4096 leaves forward, 1024 in the reverse
pass), which the pieces exceed."""
import numpy as np
import pytest
import torch

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

BLOCKS, ENTRIES = 64, 100


@pytest.mark.parametrize("nleaves", [1024, 4096])
def test_same_bits(monkeypatch, nleaves):
    n = 8 * nleaves
    x0 = np.random.default_rng(61).random((n, 3))  # no list longer than a piece
    x1, m, h = W.clumpy_cube(n, 61, n_clumps=3, cache=False)
    monkeypatch.setenv("FMM_MI355_PIECE", f"{BLOCKS},{ENTRIES}")
    X0, X1, Mt, H = to_dev(x0, x1, m, np.full(n, 1e-4))
    AB = torch.from_numpy(W.cotangent(n, 62)).cuda()
    p = F.default_params(theta=0.3)

    def evaluate(tree, flags=0):
        A, XB, MB = torch.empty_like(X1), torch.empty_like(X1), torch.empty_like(Mt)
        F.fmm_forces(tree, A, flags)
        F.fmm_forces_vjp(tree, AB, XB, MB)
        torch.cuda.synchronize()
        return [v.cpu().numpy() for v in (A, XB, MB)]

    t = F.fmm_build_tree(X0, F.default_params(theta=1.0))
    fresh = F.fmm_build_tree(X1, p)
    try:
        F.fmm_moments(t, X0, Mt, H)
        evaluate(t)
        assert F.fmm_tree_info(t)["leaves"] == nleaves
        ex = F.fmm_debug_export(t, lists="offsets")
        assert np.diff(ex["near_off"]).max() <= BLOCKS and np.diff(ex["far_off"]).max() <= ENTRIES
        t = F.fmm_build_tree(X1, p, tree=t)
        F.fmm_moments(t, X1, Mt, H)
        whole = evaluate(t)
        ex = F.fmm_debug_export(t, lists="offsets")
        cnt, far = np.diff(ex["near_off"]), np.diff(ex["far_off"])
        pieces = int((-(-cnt // BLOCKS)).sum())
        say(f"[gpu whole/split] {nleaves} leaves, longest near list {cnt.max()}")
        assert cnt.max() > BLOCKS and pieces > nleaves and far.max() > ENTRIES
        split = evaluate(t)
        F.fmm_moments(fresh, X1, Mt, H)
        first = evaluate(fresh)
    finally:
        F.fmm_tree_free(t)
        F.fmm_tree_free(fresh)
    for a, b, c in zip(whole, split, first):
        np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(a, c)
