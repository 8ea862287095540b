"""Forces of index lists: one slice per particle (the force kernel writes the
outputs) and several (a reduction does), with and without a context.

Tolerance against the oracle's compensated sums: 1e-12 relative per particle.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from tests.gpu_util import DEV, dev, host, rel_err_rows

pytestmark = pytest.mark.gpu

EPS = 1e-4


def _noalloc(m, x, v, idx, acc, jerk, **kw):
    g.gd_force_noalloc(g.make_params(eps=EPS, **kw), m, x, v, idx, acc, jerk)
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,n_act", [(2, 1), (200, 200), (256, 7), (256, 256), (257, 257), (600, 33), (513, 513)])
def test_list_force_edges_of_one_slice(n, n_act):
    m, x, v = plummer(n, 51)
    idx = np.random.default_rng(5).permutation(n)[:n_act].astype(np.int32)
    ra, rj = oracle.force(m, x, v, EPS, idx=idx, compensated=True)
    out = [torch.full((n_act, 3), float("nan"), dtype=torch.float64, device=DEV) for _ in range(4)]
    _noalloc(dev(m), dev(x), dev(v), dev(idx, torch.int32), out[0], out[1])
    cl = g.Cluster(m, x, v, eps=EPS, device=DEV)
    g.gd_predict(cl.ctx, 0.0)
    g.gd_force(cl.ctx, dev(idx, torch.int32), out[2], out[3])
    for a, j in (out[:2], out[2:]):
        assert rel_err_rows(host(a), ra).max() <= 1e-12
        assert rel_err_rows(host(j), rj).max() <= 1e-12
    assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])
    # either output alone
    one = torch.empty_like(out[0])
    _noalloc(dev(m), dev(x), dev(v), dev(idx, torch.int32), None, one)
    assert torch.equal(one, out[1])
    cl.close()


@pytest.mark.parametrize("n", [200, 2000])
def test_noalloc_outputs_may_overlap_inputs(n):
    """The outputs in place of the positions and velocities."""
    m, x, v = plummer(n, 52)
    idx = dev(np.arange(n, dtype=np.int32), torch.int32)
    acc, jerk = (torch.empty(n, 3, dtype=torch.float64, device=DEV) for _ in range(2))
    _noalloc(dev(m), dev(x), dev(v), idx, acc, jerk)
    xi, vi = dev(x), dev(v)
    _noalloc(dev(m), xi, vi, idx, xi, vi)
    assert torch.equal(xi, acc) and torch.equal(vi, jerk)


@pytest.mark.parametrize("n", [200, 2000])
def test_bad_index_is_reported_and_forgotten(n):
    m, x, v = plummer(n, 53)
    cl = g.Cluster(m, x, v, eps=EPS, device=DEV)
    g.gd_predict(cl.ctx, 0.0)
    acc = torch.empty(3, 3, dtype=torch.float64, device=DEV)
    for bad in (n, -1):
        with pytest.raises(g.GdError) as e:
            g.gd_force(cl.ctx, dev(np.array([0, bad, 1], np.int32), torch.int32), acc, None)
        assert e.value.status == g.GD_EINVAL
    g.gd_force(cl.ctx, dev(np.array([0, 5, 1], np.int32), torch.int32), acc, None)
    ra, _ = oracle.force(m, x, v, EPS, idx=[0, 5, 1], compensated=True)
    assert rel_err_rows(host(acc), ra).max() <= 1e-12
    st = g.gd_step_to(cl.ctx, 0.125)
    assert st["t"] == 0.125
    cl.close()
