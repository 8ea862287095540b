"""Small block steps taken by a team of resident workgroups.

A run by gd_step_to is compared bitwise with the same steps taken one call at
a time (gd_predict, gd_force, gd_correct), which never use a team: the sums
and the correction have the same operations in the same order, so the
tolerance is zero.
"""
import threading

import numpy as np
import pytest
import torch

from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from synth_inputs.plummer import plummer_with_bh
from tests.gpu_util import DEV, host

pytestmark = pytest.mark.gpu

T_END = 2.0 ** -5


def _state(cl):
    x, v, a, j, t_i, dt_i, t = cl.state()
    return [host(b) for b in (x, v, a, j, t_i, dt_i)] + [np.array(t)]


# One workgroup with one tile, the edges of a tile and of a slice count, two
# tiles per slice, two slices per owner, the largest team (32512: 64 slices of
# two tiles) and the first size without one; each kernel variant.
CASES = [(2, 1e-4, 0, False), (255, 1e-4, 0, False), (257, 1e-4, 0, False), (600, 0.0, 0, False),
         (1025, 1e-4, 1, False), (2049, 1e-4, 0, True), (2049, 1e-4, 1, True), (4096, 1e-4, 0, False),
         (5003, 0.0, 1, False), (12000, 1e-4, 0, False), (16384, 1e-4, 1, False), (16385, 1e-4, 0, True),
         (32512, 1e-4, 0, False), (32513, 1e-4, 0, False)]


@pytest.mark.parametrize("n,eps,flags,central", CASES)
def test_team_steps_equal_separate_calls_bitwise(n, eps, flags, central):
    m, x, v = plummer_with_bh(n - 1, 31) if central else plummer(n, 31)
    kw = dict(eps=eps, dt_max=T_END, flags=flags, device=DEV)
    if central:
        kw.update(eps_bh=1e-6, bh_index=n - 1)
    a, b = g.Cluster(m, x, v, **kw), g.Cluster(m, x, v, **kw)
    st = g.gd_step_to(a.ctx, T_END)
    for _ in range(st["block_steps"]):
        g.gd_predict(b.ctx)
        g.gd_force(b.ctx)
        g.gd_correct(b.ctx)
    sb = g.gd_stats_get(b.ctx)
    for k in ("t", "block_steps", "particle_steps", "pair_interactions", "dtmin_clamps"):
        assert st[k] == sb[k], k
    assert g.gd_nact_histogram(a.ctx) == g.gd_nact_histogram(b.ctx)
    for p, q in zip(_state(a), _state(b)):
        np.testing.assert_array_equal(p, q)
    # on from there, and again from the start: the exchange lines are used anew
    g.gd_step_to(a.ctx, 2 * T_END)
    far = _state(a)
    g.gd_reinit(a.ctx, a.m, torch.from_numpy(x).to(DEV), torch.from_numpy(v).to(DEV))
    g.gd_step_to(a.ctx, 2 * T_END)
    for p, q in zip(_state(a), far):
        np.testing.assert_array_equal(p, q)
    a.close()
    b.close()


def test_teams_on_several_streams_at_once():
    """Contexts stepped by threads of their own on streams of their own: a team
    that does not find room for all of its workgroups leaves its steps to the
    other kernels. Each result is bitwise that of the context alone."""
    sizes = [256, 1024, 4096, 8192, 16384, 16384]
    ics = [plummer(n, 40 + k) for k, n in enumerate(sizes)]
    want = []
    for m, x, v in ics:
        cl = g.Cluster(m, x, v, dt_max=T_END, device=DEV)
        g.gd_step_to(cl.ctx, T_END)
        want.append(_state(cl))
        cl.close()
    cls = []
    for m, x, v in ics:
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        cls.append(g.Cluster(m, x, v, dt_max=T_END, device=DEV, stream=s))
    errors = []

    def go(cl):
        try:
            g.gd_step_to(cl.ctx, T_END)
        except Exception as e:  # reported below
            errors.append(e)

    threads = [threading.Thread(target=go, args=(cl,)) for cl in cls]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for cl, w in zip(cls, want):
        for p, q in zip(_state(cl), w):
            np.testing.assert_array_equal(p, q)
        cl.close()
