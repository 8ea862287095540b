"""Initial forces of large contexts: each pair once (k_sym_force), with the
energy from the same pairs, against the force of an index list.

Tolerance: a sum of n terms in any order, with chains of at most 8192 terms on
either side and a few roundings per term, differs from another by at most
2 * 8200 * 2^-53 = 1.8e-12 of the sum of the terms' sizes. Terms: |a_ij| =
m_j s^(-3/2) r and |jerk_ij| <= 4 m_j s^(-3/2) w.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1702_00440_amd import gravidy as g
from synth_inputs import plummer
from tests.gpu_util import DEV, dev, host

pytestmark = pytest.mark.gpu

TOL = 2 * 8200 * 2.0 ** -53


def _sizes(m, x, v, eps):
    a, j = (torch.empty(len(m), dtype=torch.float64, device=DEV) for _ in range(2))
    for k in range(0, len(m), 1024):
        r2 = torch.zeros(min(1024, len(m) - k), len(m), dtype=torch.float64, device=DEV)
        w2 = torch.zeros_like(r2)
        for q in range(3):
            r2 += (x[None, :, q] - x[k:k + 1024, None, q]) ** 2
            w2 += (v[None, :, q] - v[k:k + 1024, None, q]) ** 2
        s = r2 + eps * eps
        s[torch.arange(len(r2)), k + torch.arange(len(r2))] = float("inf")
        f = m[None, :] * s ** -1.5
        a[k:k + 1024] = (f * r2.sqrt()).sum(1)
        j[k:k + 1024] = 4 * (f * w2.sqrt()).sum(1)
    return a, j


# 64 blocks of 512 (even), 65 (odd, a ragged last), 129 of 1024 (one particle in the last)
@pytest.mark.parametrize("n,eps", [(32768, 1e-4), (33001, 0.0), (131073, 1e-4)])
def test_initial_force_and_energy(n, eps):
    m, x, v = plummer(n, 61)
    cl = g.Cluster(m, x, v, eps=eps, device=DEV)
    a, j = (torch.empty(n, 3, dtype=torch.float64, device=DEV) for _ in range(2))
    g.gd_get_state(cl.ctx, a=a, jerk=j)
    st = g.gd_stats_get(cl.ctx)
    ek, ep = g.gd_energy(cl.ctx)
    assert abs(st["e0"] - (ek + ep)) <= TOL * (ek - ep)
    # The same again, on the buffers of the first.
    g.gd_reinit(cl.ctx, dev(m), dev(x), dev(v))
    a2, j2 = torch.empty_like(a), torch.empty_like(j)
    g.gd_get_state(cl.ctx, a=a2, jerk=j2)
    assert torch.equal(a, a2) and torch.equal(j, j2) and g.gd_stats_get(cl.ctx)["e0"] == st["e0"]
    ra, rj = torch.empty_like(a), torch.empty_like(j)
    g.gd_predict(cl.ctx, 0.0)
    g.gd_force(cl.ctx, dev(np.arange(n), torch.int32), ra, rj)
    sa, sj = _sizes(dev(m), dev(x), dev(v), eps)
    for got, ref, size in ((a, ra, sa), (j, rj, sj)):
        assert bool(((got - ref).abs().amax(1) <= TOL * size).all())
    idx = np.array([0, 1, 511, 512, n // 2, n - 2, n - 1], dtype=np.int32)
    oa, oj = oracle.force(m, x, v, eps, idx=idx, compensated=True)
    size = host(sa)[idx], host(sj)[idx]
    assert (np.abs(host(a)[idx] - oa).max(1) <= TOL * size[0]).all()
    assert (np.abs(host(j)[idx] - oj).max(1) <= TOL * size[1]).all()
    cl.close()
