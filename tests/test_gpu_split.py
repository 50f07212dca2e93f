"""The library's own split of the plane kernels' work (no tuning set): batches
from one patch on, patch sizes and grids whose planes do not divide evenly,
several sizes in one batch, against one work-group per patch and the oracle."""
import numpy as np
import pytest

import oracle
import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu, rel_err

pytestmark = pytest.mark.gpu

GRIDS = [((1, 1, 1), 16), ((1, 1, 1), 7), ((2, 1, 1), 9), ((3, 2, 2), 13), ((2, 2, 5), 8), ((4, 4, 3), 16),
         ((7, 5, 3), 11), ((11, 9, 2), 7)]


def mixed(halo, sizes=(16, 7, 3, 12, 5, 16, 9, 4)):
    """independent patches of several sizes"""
    parts = [I.independent_euler_patches_smooth(seed=9 + i, K=1, p=p, halo=halo) for i, p in enumerate(sizes)]
    return I.Batch(dim=3, p=np.array(sizes, np.int32), dx=np.concatenate([b.dx for b in parts]),
                   nbr=I.self_periodic(len(sizes), 3), halo=halo, pde="euler", params=parts[0].params, n_unknowns=5,
                   state=np.concatenate([b.state for b in parts]))


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("grid,p", GRIDS + [(None, 0)])
def test_fv_own_split(grid, p, storage):
    announce(f"fv own split {grid} p={p} {storage}")
    need_gpu()
    b = I.config1(grid=grid, p=p, seed=5) if grid else mixed(1)
    out = []
    for slab in (0, 16):
        B = pb.PatchBatch(b, storage=storage)
        if slab:
            B.set_tuning(fv_slab=slab)
        B.fv_rusanov_step(cfl=0.4, n_steps=3)
        out.append(B.download())
        B.close()
    # a run that starts inside a patch adds the lower z flux in another order:
    # a few roundings of values of order one per step (binary32: of the stored value)
    assert np.all(rel_err(b, out[0], out[1]) <= (1e-14 if storage == "fp64" else 1e-6))
    if storage == "fp64":
        o, _, _ = oracle.fv_step(b, cfl=0.4, n_steps=3)
        assert np.all(rel_err(b, out[0], o) <= 1e-12)


@pytest.mark.parametrize("grid,p", GRIDS + [(None, 0)])
def test_fd_own_split(grid, p):
    announce(f"fd own split {grid} p={p}")
    need_gpu()
    b = I.config1(grid=grid, p=p, halo=3, seed=6) if grid else mixed(3)
    out = []
    for column in (2, 0):
        B = pb.PatchBatch(b)
        B.set_tuning(fd_column=column)
        B.fd_ko_step(cfl=0.5, sigma_ko=0.1, n_steps=2)
        out.append(B.download())
        B.close()
    np.testing.assert_array_equal(out[0], out[1])
    o, _ = oracle.fd_step(b, cfl=0.5, sigma=0.1, n_steps=2)
    assert np.all(rel_err(b, out[0], o) <= 1e-12)


@pytest.mark.parametrize("grid,p", [((1, 1, 1), 16), ((3, 2, 2), 7), ((4, 4, 2), 13)])
def test_srhd_own_split(grid, p):
    announce(f"srhd own split {grid} p={p}")
    need_gpu()
    b = I.config3(grid=grid, p=p, seed=8)
    B = pb.PatchBatch(b)
    B.fv_rusanov_step(cfl=0.4, n_steps=2)
    g = B.download()
    B.close()
    o, _, _ = oracle.fv_step(b, cfl=0.4, n_steps=2)
    assert np.all(rel_err(b, g, o) <= 1e-12)
