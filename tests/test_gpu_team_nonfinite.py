"""A force that turns non-finite inside a team of resident workgroups, after
steps that were fine: the error is reported, and the block steps that the
replay still takes have whole lists.

All masses are zero and eps = 0, so every force is exactly 0 and every
position is exact, until two particles meet: 0 / 0. Times are in units of
dt_max / 64. A context is set to time 31 with two particles at a step of 1
(they meet at 36) and a block of too many particles for a team at a step of 32
or 64. With 64 the first launch of the team (parity 0) takes the particles to
where they meet; with 32 the block is due at 32, and the second launch
(parity 1) does. The workspace is filled with zeros beforehand: entries of a
list that nobody has written name particle 0.
"""
import numpy as np
import pytest
import torch

from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from tests.gpu_util import DEV, dev, host

pytestmark = pytest.mark.gpu

DT_MAX = 0.125
UNIT = DT_MAX / 64


# One owner of all particles (up to 1024), two and more with an exchange.
@pytest.mark.parametrize("block", [600, 1100, 4096])
@pytest.mark.parametrize("step", [64, 32])
def test_nonfinite_step_of_a_team_leaves_whole_lists(block, step):
    n = block + 2
    rng = np.random.default_rng(9)
    x = rng.integers(16, 4096, (n, 3)).astype(np.float64)
    x[:, 0] += 8192.0 * np.arange(n)  # apart from one another
    v = np.zeros((n, 3))
    x[:2] = 0.0
    x[0, 0], x[1, 0] = -5 * UNIT, 5 * UNIT
    v[0, 0], v[1, 0] = 1.0, -1.0
    p = g.make_params(eps=0.0, dt_max=DT_MAX)
    ws = torch.zeros(g.gd_workspace_bytes(n, p), dtype=torch.uint8, device=DEV)
    ctx = g.gd_init(p, dev(np.zeros(n)), dev(x), dev(v), ws)
    zero = dev(np.zeros((n, 3)))
    t_i, dt_i = np.zeros(n), np.full(n, step * UNIT)
    t_i[:2], dt_i[:2] = 31 * UNIT, UNIT
    g.gd_set_state(ctx, dev(x), dev(v), zero, zero, dev(t_i), dev(dt_i), 31 * UNIT)
    with pytest.raises(g.GdError) as e:
        g.gd_step_to(ctx, DT_MAX)
    assert e.value.status == g.GD_ENONFINITE
    # Every particle has the time and step that its record has; the next block
    # has as many particles as are due then.
    out = [torch.empty(n, dtype=torch.float64, device=DEV) for _ in range(2)]
    now = g.gd_get_state(ctx, t_i=out[0], dt_i=out[1])
    t, dt = host(out[0]), host(out[1])
    assert (t % dt == 0).all() and (t <= now).all() and (now < t + dt).all()
    g.gd_predict(ctx)
    assert g.gd_active(ctx) == int((t + dt == (t + dt).min()).sum())
    # From new particles the context is as a new one.
    m, x, v = plummer(n, 23)
    g.gd_reinit(ctx, dev(m), dev(x), dev(v))
    st = g.gd_step_to(ctx, DT_MAX)
    xs, vs = (torch.empty(n, 3, dtype=torch.float64, device=DEV) for _ in range(2))
    g.gd_get_state(ctx, xs, vs)
    g.gd_destroy(ctx)
    cl = g.Cluster(m, x, v, eps=0.0, dt_max=DT_MAX, device=DEV)
    assert g.gd_step_to(cl.ctx, DT_MAX)["block_steps"] == st["block_steps"]
    new = cl.state()
    np.testing.assert_array_equal(host(xs), host(new[0]))
    np.testing.assert_array_equal(host(vs), host(new[1]))
    cl.close()
