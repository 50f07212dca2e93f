"""Patches larger than the step kernels take (p > 16): the batch is created,
set up and read back as any other, and only the step refuses it."""
import numpy as np
import pytest

import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,p", [(1, 17), (2, 19), (1, 27), (1, 40)])
@pytest.mark.parametrize("pde", ["euler", "euler_fd", "srhd", "adv_f"])
def test_large_patches_are_created(pde, K, p):
    announce(f"create {pde} K={K} p={p}")
    need_gpu()
    b = I.independent_euler_patches(seed=1, K=K, p=p, halo=3 if pde == "euler_fd" else 1)
    if pde == "srhd":
        b.pde, b.params = "srhd", np.array([5.0 / 3.0, 1e-12, 50.0])
    if pde == "adv_f":
        b.pde, b.params, b.n_unknowns = "adv_f", np.array([0.7, -0.4, 0.3, 0.8]), 1
        b.state = b.state[:b.total_cells]
    B = pb.PatchBatch(b)
    B.set_tuning()
    np.testing.assert_array_equal(B.download(), b.state)
    steps = [lambda: B.fv_rusanov_step(cfl=0.4)]
    if pde == "euler_fd":
        steps.append(lambda: B.fd_ko_step(cfl=0.4))
    for step in steps:
        with pytest.raises(pb.PbError) as e:
            step()
        assert e.value.status == pb.PB_EUNSUPPORTED and "p > 16" in str(e.value)
    np.testing.assert_array_equal(B.download(), b.state)
    B.close()
