"""Team launches that are called off: the block steps are left to the other
kernels, bit by bit the steps of separate calls, and the next launches end at
once (joining) or use no exchange epoch again (the vote).

A launch is called off from the host: the flag is set, before the replay, in
the word that counts the workgroups, at the place in the workspace (or in a
pool's arena) where the schedule record lies. Every wait then ends with its
first look.
"""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from synth_inputs.plummer import plummer_with_bh
from tests.gpu_util import DEV, dev, host

pytestmark = pytest.mark.gpu

T_END = 2.0 ** -5
OFF, SKIP, STEPS = 1 << 30, 64, 1024  # kTeamOff, kTeamSkip, kTeamSteps


class Sched(C.Structure):
    """The schedule record (struct Sched) at the head of a cluster's workspace."""
    _fields_ = ([(k, C.c_longlong) for k in ("t_now", "t_next", "t_end", "spec")] +
                [(k, C.c_int) for k in ("n_act", "kthr", "done")] + [("lcnt", C.c_int * 2)] +
                [(k, C.c_int) for k in ("nonfinite", "bad_input", "refill", "fine")] +
                [(k, C.c_longlong) for k in ("block_steps", "particle_steps", "pairs", "clamps", "refills")] +
                [("nact_hist", C.c_longlong * 32), ("plan", C.c_int * 6), ("hist", C.c_int * 42)] +
                [(k, C.c_int) for k in ("team_join", "team_vote", "team_skip")] + [("team_epoch", C.c_uint)])


def _read(mem, at=0):
    torch.cuda.synchronize()
    return Sched.from_buffer_copy(host(mem[at:at + C.sizeof(Sched)]).tobytes())


def _write(mem, field, value, at=0):
    o = at + getattr(Sched, field).offset
    mem[o:o + 4] = torch.from_numpy(np.array([value], np.int32).view(np.uint8).copy()).to(DEV)
    torch.cuda.synchronize()


def _state(cl):
    x, v, a, j, t_i, dt_i, t = cl.state()
    return [host(b) for b in (x, v, a, j, t_i, dt_i)] + [np.array(t)]


def _same(a, b):
    for p, q in zip(a, b):
        np.testing.assert_array_equal(p, q)


# Owners of all particles, one slice per owner, two (with a central particle).
@pytest.mark.parametrize("n,central", [(700, False), (2500, False), (16385, True)])
@pytest.mark.parametrize("word", ["team_join", "team_vote"])
def test_called_off_launch_of_a_context(n, central, word):
    m, x, v = plummer_with_bh(n - 1, 31) if central else plummer(n, 31)
    kw = dict(eps_bh=1e-6, bh_index=n - 1) if central else {}
    a, b = (g.Cluster(m, x, v, dt_max=T_END, device=DEV, **kw) for _ in range(2))
    _write(a.workspace, word, OFF)
    st = g.gd_step_to(a.ctx, T_END)
    rec = _read(a.workspace)
    assert (rec.block_steps, rec.particle_steps) == (st["block_steps"], st["particle_steps"])  # the layout
    assert rec.refills == g.gd_refills(a.ctx) and rec.team_join == 0 and rec.team_vote == 0
    for _ in range(st["block_steps"]):
        g.gd_predict(b.ctx)
        g.gd_force(b.ctx)
        g.gd_correct(b.ctx)
    _same(_state(a), _state(b))
    assert g.gd_nact_histogram(a.ctx) == g.gd_nact_histogram(b.ctx)
    if word == "team_vote":
        assert rec.team_epoch > STEPS
    a.close()
    b.close()


def test_launches_after_one_that_did_not_find_room_are_left_out():
    """Particles at rest, all due once: the first of a replay's 16 rounds takes
    the step and the others nothing. Called off, the step is the first
    round's other kernels', and the 15 rounds after it count down from 64."""
    m, x, v = np.full(100, 1e-9), np.zeros((100, 3)), np.zeros((100, 3))
    x[:, 0] = np.arange(100)
    cl = g.Cluster(m, x, v, dt_max=T_END, device=DEV)
    want = g.Cluster(m, x, v, dt_max=T_END, device=DEV)
    assert g.gd_step_to(want.ctx, T_END)["block_steps"] == 1
    _write(cl.workspace, "team_join", OFF)
    assert g.gd_step_to(cl.ctx, T_END)["block_steps"] == 1
    assert _read(cl.workspace).team_skip == SKIP - 15
    _same(_state(cl), _state(want))
    cl.close()
    want.close()


@pytest.mark.parametrize("word", ["team_join", "team_vote"])
def test_called_off_launches_of_a_pool(word):
    """One cluster's team of three is called off: its steps are the packed
    launches', and all three end bitwise as in contexts of their own."""
    sizes = [700, 2500, 300]
    p = g.make_params(dt_max=T_END)
    ics = [[dev(a) for a in plummer(n, 80 + k)] for k, n in enumerate(sizes)]
    arena = torch.zeros(g.gd_pool_arena_bytes(3, sizes), dtype=torch.uint8, device=DEV)
    pool = g.gd_pool_create(p, 3, arena)
    slots = [g.gd_pool_admit(pool, *ic, T_END) for ic in ics]
    # the blocks lie one after the other behind the tables
    at = g.gd_pool_arena_bytes(3, []) + g.gd_workspace_bytes(sizes[0], p)
    _write(arena, word, OFF, at)
    g.gd_pool_run(pool)
    rec = _read(arena, at)
    assert rec.block_steps > 0 and rec.team_join == 0 and rec.team_vote == 0
    assert rec.team_skip > 0 if word == "team_join" else rec.team_epoch > STEPS
    for _ in range(10000):
        if g.gd_pool_resident(pool) == 0:
            break
        g.gd_pool_run(pool)
    for (m, x, v), sl in zip(ics, slots):
        px, pv = torch.empty_like(x), torch.empty_like(v)
        st = g.gd_pool_result(pool, sl, px, pv)
        cl = g.Cluster(m, x, v, dt_max=T_END, device=DEV)
        sc = g.gd_step_to(cl.ctx, T_END)
        _same([host(px), host(pv)], _state(cl)[:2])
        for k in ("t", "block_steps", "particle_steps", "dtmin_clamps", "e"):
            assert st[k] == sc[k], k
        cl.close()
    g.gd_pool_destroy(pool)
