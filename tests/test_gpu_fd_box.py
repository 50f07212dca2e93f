"""The box stage kernel of the linear system (the default from more 4^3 tiles
than the chip has CUs): bitwise equal to the kernel in which every wave does
every phase, and within 1e-12 of the oracle (the bound of the other stage
kernels: a few hundred roundings per value and step)."""
import numpy as np
import pytest

import oracle
import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu, rel_err

pytestmark = pytest.mark.gpu


# unknowns at the edges of the row tiles (16) and of the chunks of four, odd
# and even chunk counts; patches that leave boxes partly filled (three 8^3,
# five 4^3) and widths that differ from patch to patch inside a box
@pytest.mark.parametrize("N", [1, 3, 4, 5, 8, 9, 16, 17, 20, 21, 32, 33, 36, 48, 49, 52, 53, 56, 57, 58, 60])
def test_box_kernel_matches(N):
    announce(f"fd box kernel N={N}")
    need_gpu()
    sizes = np.array([8, 16, 4, 16, 4, 16, 8, 4, 16, 4, 8, 4, 16], np.int32)   # 349 tiles
    b = I.config2(n_patches=len(sizes), N=N, sizes=sizes)
    b.dx = b.dx * (1.0 + 0.03 * np.arange(len(sizes)))
    out = {}
    for ws, remap in ((1, 1), (1, 0), (0, 1)):
        B = pb.PatchBatch(b)
        B.set_tuning(fd_ws=ws, fd_xcd_remap=remap)
        B.fd_ko_step(cfl=0.5, sigma_ko=0.1, n_steps=2)
        B.fd_ko_step(cfl=0.5, dt_fixed=1e-3, sigma_ko=0.05, rk_stages=1, n_steps=1)
        out[(ws, remap)] = B.download()
        B.close()
    np.testing.assert_array_equal(out[(1, 1)], out[(0, 1)])
    np.testing.assert_array_equal(out[(1, 0)], out[(0, 1)])
    o, _ = oracle.fd_step(b, cfl=0.5, sigma=0.1, n_steps=2)
    b2 = b.copy()
    b2.state = o
    o2, _ = oracle.fd_step(b2, dt_fixed=1e-3, sigma=0.05, rk_stages=1, n_steps=1)
    assert np.all(rel_err(b, out[(1, 1)], o2) <= 1e-12)


def test_box_kernel_several_boxes_per_work_group():
    """More boxes than two work-groups per CU hold, so that work-groups go
    from box to box: bitwise equal to the all-phases kernel over graph
    replays, with eager work between them."""
    announce("fd box kernel, many boxes")
    torch = need_gpu()
    sizes = np.array([16] * 40 + [8] * 5 + [4] * 3, np.int32)   # 640 + 12 + 1 boxes of 128 cells and more
    b = I.config2(n_patches=len(sizes), N=10, sizes=sizes)
    box, ref = pb.PatchBatch(b), pb.PatchBatch(b)
    ref.set_tuning(fd_ws=0)
    for rep in range(3):
        box.fd_ko_step(cfl=0.5, sigma_ko=0.1, n_steps=2, use_graph=True)
        ref.fd_ko_step(cfl=0.5, sigma_ko=0.1, n_steps=2)
        torch.randn(4096, device="cuda").sum()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(box.download(), ref.download())
    box.close()
    ref.close()
