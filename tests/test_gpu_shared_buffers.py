"""Buffers that two forms of the evaluation share, and workspace that a call
can do without: a tree rebuilt from one form to the other gives the bits of a
fresh tree, and a byte limit that leaves out the pieces of a mutual walk's near
lists, or the order of the reverse pass's pieces, gives the bits of a tree
without a limit (neither changes a sum)."""
import pytest
import torch

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def _run(x, m, h, abar, params, tree=None, vjp=True):
    dt = torch.float32 if params.precision == F.FMM_FP32 else torch.float64
    tree = F.fmm_build_tree(x, params, tree=tree, m=m)
    F.fmm_moments(tree, x, m, h)
    a = torch.empty((x.shape[0], 3), dtype=dt, device=x.device)
    F.fmm_forces(tree, a, F.FMM_REWALK)
    out = [a]
    if vjp:
        xb, mb = torch.empty_like(a), torch.empty(x.shape[0], dtype=dt, device=x.device)
        F.fmm_forces_vjp(tree, abar.to(dt), xb, mb)
        out += [xb, mb]
    torch.cuda.synchronize()
    return tree, out


def _same(a, b):
    return all(torch.equal(p, q) for p, q in zip(a, b))


@pytest.mark.parametrize("shape", [F.FMM_TREE_MEDIAN, F.FMM_TREE_COM])
@pytest.mark.parametrize("leaf", [1, 8])
def test_forms_in_turn(shape, leaf):
    n = 3001
    x, m, h = to_dev(*W.plummer(n, 51))
    abar = torch.from_numpy(W.cotangent(n, 52)).cuda()
    forms = [(F.FMM_FP64, F.FMM_WALK_PHANTOM), (F.FMM_FP32, F.FMM_WALK_PHANTOM),
             (F.FMM_FP64, F.FMM_WALK_PHANTOM), (F.FMM_FP64, F.FMM_WALK_MUTUAL),
             (F.FMM_FP32, F.FMM_WALK_MUTUAL), (F.FMM_FP64, F.FMM_WALK_PHANTOM)]
    tree = None
    try:
        for prec, walk in forms:
            p = F.default_params(precision=prec, walk=walk, tree=shape, leaf_size=leaf)
            tree, got = _run(x, m, h, abar, p, tree)
            fresh, ref = _run(x, m, h, abar, p)
            F.fmm_tree_free(fresh)
            say(f"[gpu shared buffers] shape {shape} leaf {leaf} precision {prec} walk {walk}")
            assert _same(got, ref)
    finally:
        F.fmm_tree_free(tree)


@pytest.mark.parametrize("n,leaf,walk,vjp", [(4096, 10, F.FMM_WALK_MUTUAL, False),
                                             (23832, 1, F.FMM_WALK_PHANTOM, True)])
def test_limit_below_optional_workspace(n, leaf, walk, vjp):
    x, m, h = to_dev(*W.plummer(n, 53))
    abar = torch.from_numpy(W.cotangent(n, 54)).cuda()
    tree, ref = _run(x, m, h, abar, F.default_params(walk=walk, leaf_size=leaf), vjp=vjp)
    held = F.fmm_tree_device_bytes(tree)
    F.fmm_tree_free(tree)
    tree, got = _run(x, m, h, abar, F.default_params(walk=walk, leaf_size=leaf,
                                                     device_bytes_limit=held - 1), vjp=vjp)
    less = F.fmm_tree_device_bytes(tree)
    F.fmm_tree_free(tree)
    say(f"[gpu shared buffers] {held} B without a limit, {less} B under {held - 1} B")
    assert less < held
    assert _same(got, ref)
