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
