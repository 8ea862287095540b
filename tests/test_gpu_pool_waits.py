"""Pool calls that synchronise leave nothing under way on the pool's stream:
the caller's arena and stream are free when the call returns. A busy kernel
queued before the call makes work that it leaves behind visible.
"""
import pytest
import torch

from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from tests.gpu_util import DEV, dev

pytestmark = pytest.mark.gpu

T = 2.0 ** -5


def test_pool_calls_wait_for_their_work():
    sizes = [300, 700]
    p = g.make_params(dt_max=T)
    ics = [[dev(a) for a in plummer(n, 90 + k)] for k, n in enumerate(sizes)]
    arena = torch.zeros(g.gd_pool_arena_bytes(2, sizes), dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()

    def busy():
        with torch.cuda.stream(s):
            torch.cuda._sleep(20_000_000)

    busy()
    pool = g.gd_pool_create(p, 2, arena, s)
    assert s.query()
    for ic in ics:
        busy()
        assert g.gd_pool_admit(pool, *ic, T) is not None
        assert s.query()
    finished = []
    for _ in range(1000):
        busy()
        finished += g.gd_pool_run(pool)
        assert s.query()
        if finished:
            break
    for sl in finished:
        busy()
        g.gd_pool_result(pool, sl, *(torch.empty_like(a) for a in ics[sl][1:]))
        assert s.query()
    # Released (one of them may be running) and destroyed: the arena is the caller's again.
    for sl in range(2):
        g.gd_pool_release(pool, sl)
    g.gd_pool_destroy(pool)
    arena.fill_(0xA5)
    torch.cuda.synchronize()
    assert bool((arena == 0xA5).all())


def test_clusters_released_and_admitted_between_runs():
    """A running cluster is dropped and another takes its slot before the next
    run: the table that the run uploads is that of the clusters then resident."""
    p = g.make_params(dt_max=T)
    ics = [[dev(a) for a in plummer(n, 95 + k)] for k, n in enumerate([2000, 500, 900])]
    arena = torch.zeros(g.gd_pool_arena_bytes(2, [2000, 2000]), dtype=torch.uint8, device=DEV)
    pool = g.gd_pool_create(p, 2, arena)
    first, kept = (g.gd_pool_admit(pool, *ic, 4 * T) for ic in ics[:2])
    g.gd_pool_run(pool)
    g.gd_pool_release(pool, first)
    again = g.gd_pool_admit(pool, *ics[2], T)
    assert again == first and g.gd_pool_resident(pool) == 2
    for _ in range(10000):
        if g.gd_pool_resident(pool) == 0:
            break
        g.gd_pool_run(pool)
    for sl, (m, x, v), end in ((kept, ics[1], 4 * T), (again, ics[2], T)):
        px = torch.empty_like(x)
        st = g.gd_pool_result(pool, sl, px)
        cl = g.Cluster(m, x, v, dt_max=T, device=DEV)
        assert g.gd_step_to(cl.ctx, end)["block_steps"] == st["block_steps"]
        assert torch.equal(cl.state()[0], px)
        cl.close()
    g.gd_pool_destroy(pool)
