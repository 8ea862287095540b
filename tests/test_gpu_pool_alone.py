"""Pools whose runs go with and without teams in turn, since the clusters' blocks
are mostly too large for them (strong softening): bitwise the results of plain
contexts, with clusters that end at different times.
"""
import numpy as np
import pytest
import torch

from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from tests.gpu_util import DEV, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,flags", [([2000] * 24, 0), ([2000, 700] * 12, g.GD_FLAG_MIXED)])
def test_pool_of_large_blocks_equals_contexts_bitwise(sizes, flags):
    p = g.make_params(eps=0.05, dt_max=0.125, flags=flags)
    ics = [[dev(a) for a in plummer(n, 900 + k)] for k, n in enumerate(sizes)]
    ends = [0.125 * (1 + k % 2) for k in range(len(sizes))]
    arena = torch.empty(g.gd_pool_arena_bytes(len(sizes), sizes), dtype=torch.uint8, device=DEV)
    pool = g.gd_pool_create(p, len(sizes), arena)
    slots = [g.gd_pool_admit(pool, *ic, end) for ic, end in zip(ics, ends)]
    for _ in range(10000):
        g.gd_pool_run(pool)
        if g.gd_pool_resident(pool) == 0:
            break
    for k in range(0, len(sizes), 3):
        m, x, v = ics[k]
        px, pv = torch.empty_like(x), torch.empty_like(v)
        pst = g.gd_pool_result(pool, slots[k], px, pv)
        cl = g.Cluster(m, x, v, eps=0.05, flags=flags, device=DEV)
        st = g.gd_step_to(cl.ctx, ends[k])
        state = cl.state()
        np.testing.assert_array_equal(host(px), host(state[0]))
        np.testing.assert_array_equal(host(pv), host(state[1]))
        for q in ("t", "block_steps", "particle_steps", "pair_interactions", "dtmin_clamps", "e0", "e"):
            assert pst[q] == st[q], q
        cl.close()
    g.gd_pool_destroy(pool)
