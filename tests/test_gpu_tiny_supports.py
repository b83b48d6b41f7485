"""The near field where supports are smaller than the rounding of a leaf's
bounding box: a particle that lies in its leaf, or coincides with one that
does, stays softened (no direction at r = 0, the M4 kernel inside 2 h), however
the box rounds.  Supports of 1e-20 at the origin, of a tenth of the coordinates'
spacing away from it, coincident particles, and pairs one spacing apart inside
each other's support; leaves of a team of wavefronts and of one wavefront.
Against the oracle FMM with the bar of the other parity tests (1e-12)."""
import numpy as np
import pytest

from paper_2502_01496_amd import workloads as W
from tests.gpu_util import force_err, gpu_run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3000, 40000])
@pytest.mark.parametrize("case", ["unsoftened", "offset_1e3", "offset_1e8", "coincident",
                                  "one_spacing"])
def test_against_oracle(orc, case, n):
    x, m, _ = W.clumpy_cube(n, 71, n_clumps=3, cache=False)
    h = 1e-20
    if case == "offset_1e3":
        x, h = x + 1e3, 1e-14
    elif case == "offset_1e8":
        x, h = x + 1e8, 1e-9
    elif case == "coincident":
        x[100:140] = x[200:240]
    elif case == "one_spacing":
        x = x + 1.0
        x[100:140] = np.nextafter(x[200:240], 9.0)
        h = 2.5e-16
    hh = np.full(n, h)
    say(f"[gpu tiny supports] clumpy {n}, {case}, h {h}")
    a, _, _ = gpu_run(x, m, hh, export=False)
    assert np.isfinite(a).all()
    assert force_err(a, orc.fmm(x, m, hh).a) <= 1e-12
