"""A list force without outputs marks nothing: two massless particles that meet
at t = 1 have a force of 0 / 0 there, and the context still steps on from t = 0.
"""
import numpy as np
import pytest
import torch

from paper_1702_00440_amd import gravidy as g
from tests.gpu_util import DEV, dev

pytestmark = pytest.mark.gpu


# one slice per particle, and several
@pytest.mark.parametrize("n", [2, 600])
def test_list_force_without_outputs_marks_nothing(n):
    x, v = np.zeros((n, 3)), np.zeros((n, 3))
    x[:, 1] = np.arange(n)
    x[:2], v[:2] = [[-1, 0, 0], [1, 0, 0]], [[1, 0, 0], [-1, 0, 0]]
    cl = g.Cluster(np.zeros(n), x, v, eps=0.0, device=DEV)
    g.gd_predict(cl.ctx, 1.0)
    idx = dev(np.array([0, 1]), torch.int32)
    g.gd_force(cl.ctx, idx)
    assert g.gd_step_to(cl.ctx, 0.125)["t"] == 0.125
    # with an output the non-finite row is seen, and marked
    acc = torch.zeros(2, 3, dtype=torch.float64, device=DEV)
    g.gd_predict(cl.ctx, 1.0)
    g.gd_force(cl.ctx, idx, acc)
    assert not torch.isfinite(acc).any()
    with pytest.raises(g.GdError) as e:
        g.gd_step_to(cl.ctx, 0.25)
    assert e.value.status == g.GD_ENONFINITE
    cl.close()
