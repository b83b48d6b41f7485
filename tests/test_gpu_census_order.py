"""The asymmetry estimates transpose the far lists alone, the reverse pass both
lists: each after the other on the same lists gives the bits it gives by itself."""
import numpy as np
import pytest
import torch

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def run(x, m, h, abar, order, **kw):
    X, Mt, H = to_dev(x, m, h)
    AB = torch.from_numpy(abar).to("cuda")
    t = F.fmm_build_tree(X, F.default_params(**kw), m=Mt)
    out = {}
    try:
        F.fmm_moments(t, X, Mt, H)
        F.fmm_forces(t, torch.empty((len(m), 3), dtype=torch.float64, device="cuda"))
        for op in order:
            if op == "census":
                out[op] = F.fmm_asymmetry_estimate(t)
            else:
                XB = torch.empty((len(m), 3), dtype=torch.float64, device="cuda")
                MB = torch.empty(len(m), dtype=torch.float64, device="cuda")
                F.fmm_forces_vjp(t, AB, XB, MB)
                torch.cuda.synchronize()
                out[op] = (XB.cpu().numpy(), MB.cpu().numpy())
    finally:
        F.fmm_tree_free(t)
    return out


@pytest.mark.parametrize("n,leaf", [(9, 8), (150, 8), (3001, 8), (3001, 1)])
def test_either_order(n, leaf):
    x, m, h = W.plummer(n, 85)
    abar = W.cotangent(n, 86)
    say(f"[gpu census order] plummer {n} leaf {leaf}")
    kw = dict(theta=0.7, leaf_size=leaf)
    c = run(x, m, h, abar, ["census"], **kw)["census"]
    v = run(x, m, h, abar, ["vjp"], **kw)["vjp"]
    for order in (["census", "vjp"], ["vjp", "census"]):
        o = run(x, m, h, abar, order, **kw)
        assert o["census"] == c
        assert np.array_equal(o["vjp"][0], v[0]) and np.array_equal(o["vjp"][1], v[1])
