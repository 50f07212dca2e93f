"""The con2prim pass of the SRHD step where its work-groups' shares have edges:
one work-group, cells that do not fill the last chunk of 256, chunks that span
several patches, more chunks than work-groups (2048), and mixed patch sizes
(chunks of one patch each; more of them than 2039 work-groups); dt and the
con2prim counts with CFL and fixed steps and in graph replays.  Within 1e-12
of the oracle, the bound of the other SRHD tests."""
import numpy as np
import pytest

import oracle
import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu, rel_err

pytestmark = pytest.mark.gpu


def batch(ps, seed):
    b = I.independent_euler_patches(seed=seed, K=len(ps), p=max(ps))
    if len(set(ps)) > 1:
        b.p = np.asarray(ps, dtype=b.p.dtype)
    b.pde, b.params = "srhd", np.array([5.0 / 3.0, 1e-12, 50.0])
    n = sum(p**3 for p in ps)
    cons, _ = I.srhd_prim_to_cons(*I.srhd_primitives(seed, n), 5.0 / 3.0)
    o, parts = 0, []
    for p in ps:
        parts.append(cons[:, o:o + p**3].ravel())
        o += p**3
    b.state = np.concatenate(parts)
    return b


@pytest.mark.parametrize("name,ps", [
    ("one chunk", [5]), ("two, the last partly filled", [7]), ("spans patches", [2] * 70), ("p 3", [3] * 40),
    ("p 9", [9] * 11), ("more chunks than units", [16] * 131), ("mixed", [16, 2, 9, 5] * 3),
    ("mixed, more chunks than units", [16, 3, 4, 8] * 33)])
def test_c2p_shares(name, ps):
    announce(f"con2prim shares: {name}")
    torch = need_gpu()
    b = batch(ps, 60 + len(ps))
    o, dts, ost = oracle.fv_step(b, cfl=0.4, n_steps=4)
    B = pb.PatchBatch(b)
    n = 0
    for steps, graph in ((1, False), (1, True), (1, True), (1, True)):
        dt = B.fv_rusanov_step(cfl=0.4, n_steps=steps, use_graph=graph, want_dt=True)
        torch.randn(4096, device="cuda").sum()
        n += steps
        assert abs(dt - dts[n - 1]) <= 1e-12 * dts[n - 1]
    st = B.stats()
    assert np.all(rel_err(b, B.download(), o) <= 1e-12)
    assert st["c2p_cells"] == 4 * b.total_cells and st["c2p_failures"] == ost.c2p_fail
    B.reset(b.state)
    B.fv_rusanov_step(dt_fixed=dts[0], n_steps=1)
    one = B.stats()
    assert one["c2p_cells"] == b.total_cells and 0 < one["c2p_iterations"] < st["c2p_iterations"]
    assert 0 < one["c2p_max_iterations"] <= 50
    B.close()
