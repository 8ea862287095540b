"""Replays with and without a team's launches, as the block sizes make one or
the other the faster: bitwise the steps of separate calls either way.

Plummer spheres of 8192. With a softening of 1e-4 nearly all steps that a team
can take (up to 256 active) are a team's; with 0.02 there are as many larger
blocks as small ones, and most replays go without it. The schedule record tells:
a team counts the steps it exchanged in its epoch.
"""
import pytest

from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from tests.gpu_util import DEV, dev
from tests.test_gpu_team_off import _read, _same, _state

pytestmark = pytest.mark.gpu

T_END = 0.125


@pytest.mark.parametrize("eps,flags,least,most", [(1e-4, 0, 0.95, 1.0), (0.02, 0, 0.0, 0.5),
                                                  (0.02, g.GD_FLAG_MIXED, 0.0, 0.5)])
def test_replays_by_block_sizes(eps, flags, least, most):
    m, x, v = plummer(8192, 3)
    a, b = (g.Cluster(m, x, v, eps=eps, flags=flags, device=DEV) for _ in range(2))
    st = g.gd_step_to(a.ctx, T_END)
    rec = _read(a.workspace)
    sized = sum(rec.nact_hist[:8])
    assert least * sized <= rec.team_epoch <= most * sized
    for _ in range(st["block_steps"]):
        g.gd_predict(b.ctx)
        g.gd_force(b.ctx)
        g.gd_correct(b.ctx)
    _same(_state(a), _state(b))
    assert g.gd_nact_histogram(a.ctx) == g.gd_nact_histogram(b.ctx)
    # on from there, and from the start again
    assert g.gd_step_to(a.ctx, 2 * T_END)["t"] == 2 * T_END
    far = _state(a)
    g.gd_reinit(a.ctx, *(dev(q) for q in (m, x, v)))
    g.gd_step_to(a.ctx, 2 * T_END)
    _same(_state(a), far)
    a.close()
    b.close()

