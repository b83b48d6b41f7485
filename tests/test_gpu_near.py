"""The near field over leaf sizes: a leaf's sinks are laid over the lanes two
by two, so every count from one to the largest leaf is another layout (idle
lanes from three pairs of sinks on, two passes from 17 sinks on), and near
leaves of more than eight particles give several blocks.  Against the oracle
FMM, with the bars of the other parity tests (1e-12 FP64; the FP32 form's
normalised error 1e-5)."""
import numpy as np
import pytest

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import workloads as W
from tests.gpu_util import force_err, gpu_run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf", [1, 2, 4, 5, 6, 9, 12, 14, 16, 17, 33, 64])
def test_leaf_counts(orc, leaf):
    x, m, h = W.clumpy_cube(3001, 90 + leaf, n_clumps=3, cache=False)
    say(f"[gpu near] clumpy 3001, leaf {leaf}, both precisions")
    ref = orc.fmm(x, m, h, leaf_size=leaf)
    a, _, _ = gpu_run(x, m, h, leaf=leaf, export=False)
    assert force_err(a, ref.a) <= 1e-12
    a32, _, _ = gpu_run(x, m, h, leaf=leaf, precision=F.FMM_FP32, export=False)
    d = a32.astype(np.float64) - ref.a
    assert np.sqrt((d * d).sum() / (ref.a ** 2).sum()) <= 1e-5


@pytest.mark.parametrize("h", [1e-6, 0.02, 3.0])
def test_support_radii(orc, h):
    # supports far smaller than the leaves, of their size, and larger than the
    # system: no source, some, and every source of the second ring is softened
    x, m, _ = W.plummer(777, 5)
    hh = np.full(len(m), h)
    hh[::3] *= 0.25
    say(f"[gpu near] plummer 777, h {h}")
    a, _, _ = gpu_run(x, m, hh, export=False)
    assert force_err(a, orc.fmm(x, m, hh).a) <= 1e-12


def test_coincident_particles(orc):
    # pairs at one point (softened, no direction) beside ordinary ones
    x, m, h = W.plummer(500, 6)
    x[100:140] = x[200:240]
    say("[gpu near] 40 coincident pairs")
    a, _, _ = gpu_run(x, m, h, export=False)
    assert force_err(a, orc.fmm(x, m, h).a) <= 1e-12


@pytest.mark.parametrize("precision", [F.FMM_FP64, F.FMM_FP32])
@pytest.mark.parametrize("piece", [1, 7, None])
def test_mutual_near_lists_in_pieces(orc, monkeypatch, piece, precision):
    # two stars and one particle more: the leaf that holds particles of both
    # has every leaf in its near list (longer than a piece of 512 blocks).
    # Forces against the oracle, total force zero to rounding, the reverse pass
    # as with whole lists; forces on kept lists as after the walk
    import torch

    from tests.gpu_util import to_dev

    n = 1501 if piece else 9001
    x, m, h = W.polytrope_binary(n, 8, cache=False)
    x, m, h = x[:-1], m[:-1], h[:-1]
    say(f"[gpu near] mutual binary {len(m)}, pieces of {piece}, precision {precision}")
    dt = torch.float32 if precision == F.FMM_FP32 else torch.float64
    X, Mt, H = to_dev(x, m, h)
    AB = torch.from_numpy(W.cotangent(len(m), 5)).cuda().to(dt)

    def run(hook):
        if hook:
            monkeypatch.setenv("FMM_MI355_PIECE", str(hook))
        t = F.fmm_build_tree(X, F.default_params(walk=F.FMM_WALK_MUTUAL, precision=precision))
        monkeypatch.delenv("FMM_MI355_PIECE", raising=False)
        try:
            F.fmm_moments(t, X, Mt, H)
            out = []
            for flags in (0, 0, F.FMM_REWALK):
                A = torch.empty((len(m), 3), dtype=dt, device="cuda")
                F.fmm_forces(t, A, flags)
                out.append(A)
            XB, MB = torch.empty_like(A), torch.empty(len(m), dtype=dt, device="cuda")
            F.fmm_forces_vjp(t, AB, XB, MB)
            torch.cuda.synchronize()
            st = F.fmm_momentum_stats(X, None, Mt, out[0])
        finally:
            F.fmm_tree_free(t)
        return [a.cpu().numpy() for a in out], XB.cpu().numpy(), MB.cpu().numpy(), st

    a, xb, mb, st = run(piece)
    np.testing.assert_array_equal(a[0], a[1])
    np.testing.assert_array_equal(a[0], a[2])
    ref = orc.fmm(x, m, h, policy=1).a
    if precision == F.FMM_FP64:
        assert force_err(a[0], ref) <= 1e-12
        assert st["ratio"] <= 1e-13
    else:
        d = a[0].astype(np.float64) - ref
        assert np.sqrt((d * d).sum() / (ref ** 2).sum()) <= 1e-5
    # pieces of a million blocks: whole lists
    _, xw, mw, _ = run(1000000)
    tol = 1e-12 if precision == F.FMM_FP64 else 1e-5
    assert np.abs(xb - xw).max() <= tol * np.abs(xw).max()
    assert np.abs(mb - mw).max() <= tol * np.abs(mw).max()
