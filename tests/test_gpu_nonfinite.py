"""The count of patches that hold a NaN or infinity does not depend on how the
library deals their planes to work-groups: its own split (runs shorter and
longer than a patch) against one work-group per patch, step by step, over
several calls, FV and FD steps in turn, a change of tuning and graph replays."""
import numpy as np
import pytest

import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,grid,p", [("fv", (1, 1, 1), 16), ("fv", (3, 2, 2), 9), ("fv", (11, 9, 10), 7),
                                         ("srhd", (3, 2, 3), 8), ("fd", (1, 1, 2), 16), ("fd", (3, 2, 2), 9)])
def test_patches_counted_once(kind, grid, p):
    announce(f"non-finite patches {kind} {grid} p={p}")
    need_gpu()
    b = I.config3(grid=grid, p=p, seed=3) if kind == "srhd" else I.config1(grid=grid, p=p, halo=3, seed=3)
    n = p**3
    for k in {0, b.K // 2, b.K - 1}:   # first and last cell of a patch
        b.state[k * 5 * n + (n - 1 if k else 0)] = np.nan
    counts = []
    for one in (False, True):
        B = pb.PatchBatch(b)
        if one:
            B.set_tuning(fv_slab=p, fd_column=0)
        got = []

        def fv(steps, graph=False):
            B.fv_rusanov_step(dt_fixed=1e-5, n_steps=steps, use_graph=graph)
            got.append(B.stats()["nonfinite_units"])

        def fd(steps):
            if kind == "fd":
                B.fd_ko_step(dt_fixed=1e-5, sigma_ko=0.1, n_steps=steps)
                got.append(B.stats()["nonfinite_units"])

        fd(1)
        fv(1)
        fd(2)
        fv(1, True)
        fv(1, True)
        if not one:
            B.set_tuning(fv_slab=4)
            B.set_tuning(fv_slab=0)
        fv(2)
        B.reset(b.state)
        fv(1)
        fd(1)
        counts.append(got)
        B.close()
    assert counts[0] == counts[1]
    assert 0 < counts[1][0] <= b.K
