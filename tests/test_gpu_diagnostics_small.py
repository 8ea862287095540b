"""The diagnostics' sort of runs that are not whole: particles at and beside the
powers of two, in the first run and in a last one, against the oracle.

Radii agree within 1e-12: both sides pick the same particle, so only the order
of summation of the centre of mass (about 1e-15 of the distances) separates them.
"""
import numpy as np
import pytest

import oracle
from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from synth_inputs.plummer import plummer_imf
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 4, 5, 31, 32, 33, 64, 65, 127, 512, 513, 1026, 1028, 1029, 1537, 2047])
def test_diagnostics_of_part_of_a_run(n):
    m, x, v = (plummer_imf if n % 2 else plummer)(n, 14)
    cl = g.Cluster(m, x, v, device=DEV)
    fr = [k / 32 for k in range(1, 33)]
    d = g.gd_diagnostics(cl.ctx, fr)
    np.testing.assert_allclose(d["radii"], oracle.lagrange_radii(m, x, fr), rtol=1e-12)
    assert d["r_half"] == d["radii"][15]
    cl.close()
