"""Pools whose teams have one, two, four and eight groups (as many as the
resident clusters leave room for), and groups that change as clusters finish:
bitwise the results of plain contexts. Clusters are equal-mass Plummer spheres
(eps 1e-4, eta 0.01, dt_max 1/32).
"""
import numpy as np
import pytest
import torch

from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from tests.gpu_util import DEV, dev, host

pytestmark = pytest.mark.gpu

T = 2.0 ** -5


def _params(flags):
    return g.make_params(eta=0.01, eps=1e-4, dt_max=T, dt_min=2.0 ** -22, flags=flags)


@pytest.mark.parametrize("sizes,flags", [([300, 256], 0), ([513], 0), ([1024, 700], g.GD_FLAG_MIXED),
                                         ([300, 600, 5003], 0), ([8192] * 3, 0), ([2500] * 20, g.GD_FLAG_MIXED),
                                         ([4097] * 9 + [1000] * 9, 0)])
def test_pool_groups_equal_contexts_bitwise(sizes, flags):
    p = _params(flags)
    ics = [[dev(a) for a in plummer(n, 70 + k)] for k, n in enumerate(sizes)]
    ends = [(1 + k % 2) * T for k in range(len(sizes))]
    arena = torch.empty(g.gd_pool_arena_bytes(len(sizes), sizes), dtype=torch.uint8, device=DEV)
    pool = g.gd_pool_create(p, len(sizes), arena)
    slots = [g.gd_pool_admit(pool, *ic, end) for ic, end in zip(ics, ends)]
    for _ in range(10000):
        g.gd_pool_run(pool)
        if g.gd_pool_resident(pool) == 0:
            break
    for (m, x, v), sl, end in zip(ics, slots, ends):
        px, pv = torch.empty_like(x), torch.empty_like(v)
        pst = g.gd_pool_result(pool, sl, px, pv)
        ws = torch.empty(g.gd_workspace_bytes(len(m), p), dtype=torch.uint8, device=DEV)
        ctx = g.gd_init(p, m, x, v, ws)
        st = g.gd_step_to(ctx, end)
        cx, cv = torch.empty_like(x), torch.empty_like(v)
        g.gd_get_state(ctx, cx, cv)
        g.gd_destroy(ctx)
        np.testing.assert_array_equal(host(px), host(cx))
        np.testing.assert_array_equal(host(pv), host(cv))
        for k in ("t", "block_steps", "particle_steps", "pair_interactions", "dtmin_clamps", "e0", "e"):
            assert pst[k] == st[k], k
    g.gd_pool_destroy(pool)
