"""The results of the FV plane kernel do not depend on how the planes are dealt
to work-groups, nor on what else is in the batch: the lower z face of a run's
first plane is evaluated with the operations of a face inside a run.  Bitwise,
for each PDE and storage."""
import numpy as np
import pytest

import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu

pytestmark = pytest.mark.gpu

SPLITS = [dict(), dict(fv_slab=1), dict(fv_slab=2), dict(fv_slab=3), dict(fv_slab=5), dict(fv_persist=2),
          dict(fv_persist=7), dict(fv_column=1), dict(fv_column=3), dict(fv_column=8)]


def batch(pde, grid, p):
    if pde == "srhd":
        return I.config3(grid=grid, p=p, seed=20 + p)
    if pde == "euler":
        b = I.config1(grid=grid, p=p, seed=20 + p)
        b.state = b.state * I.uniform(p, b.state.size, 0.98, 1.02)
        return b
    if pde == "adv_var":
        return I.adv_var_batch(grid, p, kappa=0.1, field="random", seed=20 + p)
    b = I.make_uniform_batch(grid, p, 1, pde, [0.7, -0.4, 0.3, 0.8], 1, 1.0 / (3 * p))
    b.state = I.uniform(4, b.total_cells, -1, 1)
    return b


def run(b, storage="fp64", tuning=None, **kw):
    need_gpu()
    B = pb.PatchBatch(b, storage=storage)
    if tuning:
        B.set_tuning(**tuning)
    B.fv_rusanov_step(**kw)
    g = B.download()
    B.close()
    return g


@pytest.mark.parametrize("pde,p,storage", [(pde, p, "fp64") for pde in ("euler", "srhd", "adv_f", "adv_b", "adv_var")
                                           for p in (7, 9, 13, 16)] + [("euler", p, "fp32") for p in (8, 11, 13, 16)])
def test_split_does_not_change_bits(pde, p, storage):
    announce(f"split bits {pde} p={p} {storage}")
    b = batch(pde, (3, 2, 3), p)
    ref = run(b, storage, dict(fv_slab=16), cfl=0.4, n_steps=3)
    assert np.all(np.isfinite(ref))
    for t in SPLITS:
        np.testing.assert_array_equal(run(b, storage, t, cfl=0.4, n_steps=3), ref, err_msg=str(t))


@pytest.mark.parametrize("pde,p,storage", [("euler", 8, "fp64"), ("euler", 11, "fp32"), ("euler", 16, "fp64"),
                                           ("euler", 16, "fp32"), ("srhd", 9, "fp64"), ("srhd", 16, "fp64")])
def test_batch_does_not_change_a_patch(pde, p, storage):
    """one patch, periodic on itself, alone, repeated, and beside 16^3 patches"""
    announce(f"batch bits {pde} p={p} {storage}")
    N = 5
    one = batch(pde, (1, 1, 1), p)

    def of(copies, extra):
        e = batch(pde, (1, 1, 1), 16)
        ps = np.array([p] * copies + [16] * extra, np.int32)
        return I.Batch(dim=3, p=ps, dx=1.0 / ps, nbr=I.self_periodic(len(ps), 3), halo=1, pde=one.pde,
                       params=one.params, n_unknowns=N, state=np.concatenate([one.state] * copies + [e.state] * extra))

    n = one.state.size
    dt = 1e-3
    ref = run(of(1, 0), storage, dt_fixed=dt, n_steps=3)
    assert np.all(np.isfinite(ref)) and np.any(ref != one.state)
    for copies, extra in ((3, 0), (300, 0), (900, 0), (3, 2)):
        g = run(of(copies, extra), storage, dt_fixed=dt, n_steps=3)[:copies * n].reshape(copies, n)
        np.testing.assert_array_equal(g, np.broadcast_to(ref, g.shape), err_msg=f"{copies} copies, {extra} others")
