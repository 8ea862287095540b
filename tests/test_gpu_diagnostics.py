"""The diagnostics' sort and cumulative sums at their edges, against the oracle.

Radii agree within 1e-12: both sides pick the same particle (the cumulative
masses decide alike), so only the order of summation of the centre of mass
(about 1e-15 of the distances) separates them.
"""
import numpy as np
import pytest

import oracle
from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from synth_inputs.plummer import plummer_imf
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,imf", [(1023, False), (1024, True), (1025, False), (2500, False), (16384, False),
                                   (16385, True), (16400, False)])
def test_diagnostics_runs_merges_and_sums(n, imf):
    """One run of 1024 keys, one and two merge passes; thresholds that fall on
    a particle (equal masses: exact sums at powers of two, the serial chains
    elsewhere) and between particles (a mass spectrum)."""
    m, x, v = (plummer_imf if imf else plummer)(n, 12)
    cl = g.Cluster(m, x, v, device=DEV)
    fr = [0.9, 0.01, 0.2, 0.5, 0.25, 1.0, 1.0 / n, 0.125]
    d = g.gd_diagnostics(cl.ctx, fr)
    np.testing.assert_allclose(d["radii"], oracle.lagrange_radii(m, x, fr), rtol=1e-12)
    assert d["r_half"] == d["radii"][3]
    cl.close()
