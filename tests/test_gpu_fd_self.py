"""Euler FD4 + KO6 steps of small patches that are their own neighbours (one
launch per step): partly filled groups, more groups than work-groups fit the
chip, widths that differ, both Runge-Kutta forms, CFL and fixed dt, eager and
graph replays.  Within 1e-12 of the oracle, the bound of the other Euler FD
tests."""
import numpy as np
import pytest

import oracle
import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,p", [(1, 3), (1, 6), (10, 3), (7, 4), (3, 5), (5, 6), (7001, 3), (3100, 4), (1541, 5),
                                 (800, 6)])
def test_self_step(K, p):
    announce(f"fd self step K={K} p={p}")
    torch = need_gpu()
    b = I.independent_euler_patches_smooth(seed=80 + K, K=K, p=p, halo=3)
    b.dx = b.dx * (1.0 + 0.2 * (np.arange(K) % 5))
    B = pb.PatchBatch(b)
    dts = []
    for steps, graph in ((2, False), (1, True), (1, True), (1, True)):
        dts.append(B.fd_ko_step(cfl=0.5, sigma_ko=0.1, n_steps=steps, use_graph=graph, want_dt=True))
        torch.randn(4096, device="cuda").sum()
    B.fd_ko_step(dt_fixed=1e-3, sigma_ko=0.05, rk_stages=1, n_steps=2)
    B.fd_ko_step(dt_fixed=1e-3, sigma_ko=0.05, n_steps=1)
    g = B.download()
    assert B.stats()["nonfinite_units"] == 0
    B.close()
    o, od = oracle.fd_step(b, cfl=0.5, sigma=0.1, n_steps=5)
    assert np.allclose(dts, od[1:], rtol=1e-12, atol=0)
    b2 = b.copy()
    b2.state = o
    b2.state, _ = oracle.fd_step(b2, dt_fixed=1e-3, sigma=0.05, rk_stages=1, n_steps=2)
    o, _ = oracle.fd_step(b2, dt_fixed=1e-3, sigma=0.05, n_steps=1)
    assert np.all(rel_err(b, g, o) <= 1e-12)


def test_nonfinite_group_counted():
    announce("fd self step, non-finite count")
    need_gpu()
    b = I.independent_euler_patches_smooth(seed=5, K=5, p=6, halo=3)
    b.state[-1] = np.nan
    B = pb.PatchBatch(b)
    B.fd_ko_step(dt_fixed=1e-4, n_steps=2)
    assert B.stats()["nonfinite_units"] == 2
    B.close()
