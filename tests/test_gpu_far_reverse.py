"""The reverse pass of the far field on both sides of the size from which the
pieces of the transposed lists are evaluated in the order of their sinks (leaf
records of more than 4 MiB: 23832 leaves of 176 bytes), at leaf size one.
Against central differences of the oracle's frozen-tree FMM, with the bar of
the other reverse-pass tests."""
import numpy as np
import pytest

from paper_2502_01496_amd import workloads as W
from tests.gpu_util import gpu_vjp, say
from tests.test_gpu_vjp import fd_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [23831, 23832])
def test_order_of_pieces(orc, n):
    x, m, h = W.plummer(n, 41)
    abar = W.cotangent(n, 42)
    say(f"[gpu far reverse] plummer {n}, leaf 1")
    _, [(xb, mb), (xb2, mb2)] = gpu_vjp(x, m, h, abar, leaf=1, repeat=2)
    assert np.array_equal(xb, xb2) and np.array_equal(mb, mb2)
    assert fd_check(orc, x, m, h, abar, xb, mb, 0.5, 1, ndir=1) <= 1e-6
