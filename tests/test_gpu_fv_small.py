"""The small-patch FV kernel where its work-groups go from group to group:
more groups than work-groups fit the chip, a partly filled last group, patches
that are their own neighbours (with widths that differ) and patches of a grid.
Within 1e-12 (binary32 storage 1e-5) of the oracle, the bounds of the other FV
tests."""
import numpy as np
import pytest

import oracle
import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("K,p", [(2, 6), (1100, 6), (2053, 5), (4201, 4), (8203, 3)])
def test_own_neighbours(K, p, storage):
    announce(f"fv small patches, own neighbours K={K} p={p} {storage}")
    need_gpu()
    b = I.independent_euler_patches(seed=60 + K, K=K, p=p)
    b.dx = b.dx * (1.0 + 0.2 * (np.arange(K) % 7))
    B = pb.PatchBatch(b, storage=storage)
    B.fv_rusanov_step(cfl=0.4, n_steps=3)
    g = B.download()
    B.close()
    s0 = b.state if storage == "fp64" else b.state.astype(np.float32).astype(np.float64)
    b.state = s0
    o, _, _ = oracle.fv_step(b, cfl=0.4, n_steps=3, round_fp32=storage == "fp32")
    assert np.all(rel_err(b, g, o) <= (1e-12 if storage == "fp64" else 1e-5))


@pytest.mark.parametrize("grid,p", [((10, 10, 9), 6), ((13, 11, 12), 5), ((17, 16, 13), 4), ((21, 20, 17), 3),
                                    ((20, 20, 43), 2), ((44, 44, 34), 1)])
def test_grid_neighbours(grid, p):
    announce(f"fv small patches, grid {grid} p={p}")
    need_gpu()
    b = I.config1(grid=grid, p=p, seed=71)
    B = pb.PatchBatch(b)
    B.fv_rusanov_step(cfl=0.4, n_steps=3)
    g = B.download()
    B.close()
    o, _, _ = oracle.fv_step(b, cfl=0.4, n_steps=3)
    assert np.all(rel_err(b, g, o) <= 1e-12)
