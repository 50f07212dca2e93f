"""pb_autotune can keep the library's own split: it is among the candidates
wherever its runs differ from those of another candidate (patches whose
work-groups have fewer than four waves; 16^3 chains whose share of the runs
does not divide evenly), it is applied when it is the fastest, and a cached
choice of it is applied again."""
import numpy as np
import pytest

import oracle
import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu, rel_err

pytestmark = pytest.mark.gpu

OWN = dict(fv_slab=0, fv_persist=0, fv_column=0, fv_dma=0)


@pytest.mark.parametrize("pde,grid,p", [("euler", (7, 7, 8), 7), ("euler", (7, 7, 6), 8), ("euler", (6, 6, 6), 11),
                                        ("euler", (5, 5, 5), 13), ("euler", (5, 5, 5), 16), ("srhd", (5, 5, 5), 16)])
def test_own_split_is_a_candidate(pde, grid, p):
    announce(f"autotune own split {pde} {grid} p={p}")
    need_gpu()
    pb.pb_autotune_cache_clear()
    b = I.config3(grid=grid, p=p, seed=4) if pde == "srhd" else I.config1(grid=grid, p=p, seed=4)
    B = pb.PatchBatch(b)
    st0 = B.stats()
    r = B.autotune("fv", cfl=0.4, trials=2)
    cand = [c for c, _ in r["candidates"]]
    assert len(cand) <= pb.PB_TUNE_MAX
    assert len({tuple(sorted(c.items())) for c in cand}) == len(cand)
    own = [c for c in cand if all(c[k] == v for k, v in OWN.items())]
    assert {c["fv_xcd_remap"] for c in own} == {0, 1}
    assert r["best_us"] == min(t for _, t in r["candidates"]) and B.get_tuning() == r["best"]
    np.testing.assert_array_equal(B.download(), b.state)
    assert B.stats() == st0
    r2 = B.autotune("fv", cfl=0.4, trials=2)
    assert r2["from_cache"] and r2["best"] == r["best"] == B.get_tuning()
    B.fv_rusanov_step(cfl=0.4, n_steps=2)
    g = B.download()
    B.close()
    o, _, _ = oracle.fv_step(b, cfl=0.4, n_steps=2)
    assert np.all(rel_err(b, g, o) <= 1e-12)
    pb.pb_autotune_cache_clear()
