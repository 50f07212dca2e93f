"""The dt of an FV call's steps at the edges of the hand-over between them:
few patches (two hand-over lines), from four patches on eight, and more
patches than the first kernel has work-groups (1024); calls of one step, of
several and graph replays.  Within 1e-12 of the oracle, the bound of the other
FV tests."""
import numpy as np
import pytest

import oracle
import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,p", [(1, 3), (1, 9), (3, 7), (4, 7), (5, 2), (9, 16), (1024, 3), (1025, 2), (1030, 7)])
def test_dt_hand_over(K, p):
    announce(f"fv hand-over K={K} p={p}")
    torch = need_gpu()
    b = I.independent_euler_patches(seed=40 + K, K=K, p=p)
    o, dts, _ = oracle.fv_step(b, cfl=0.4, n_steps=8)
    B = pb.PatchBatch(b)
    n = 0
    for steps, graph in ((1, False), (4, False), (1, True), (1, True), (1, True)):
        dt = B.fv_rusanov_step(cfl=0.4, n_steps=steps, use_graph=graph, want_dt=True)
        torch.randn(4096, device="cuda").sum()
        n += steps
        assert abs(dt - dts[n - 1]) <= 1e-12 * dts[n - 1]
    assert np.all(rel_err(b, B.download(), o) <= 1e-12)
    assert B.stats()["nonfinite_units"] == 0
    B.close()


@pytest.mark.parametrize("K,p", [(3, 4), (40, 4), (6, 9)])
def test_nonfinite_units_counted(K, p):
    """one cell holding a NaN marks its work-group, in every step that follows"""
    announce(f"fv non-finite count K={K} p={p}")
    need_gpu()
    b = I.independent_euler_patches(seed=7, K=K, p=p)
    B = pb.PatchBatch(b)
    B.fv_rusanov_step(cfl=0.4, n_steps=2)
    assert B.stats()["nonfinite_units"] == 0
    s = b.state.copy()
    s[-1] = np.nan
    B.reset(s)
    B.fv_rusanov_step(dt_fixed=1e-4, n_steps=1)
    assert B.stats()["nonfinite_units"] == 1
    B.fv_rusanov_step(dt_fixed=1e-4, n_steps=2)
    assert B.stats()["nonfinite_units"] == 3
    B.close()
