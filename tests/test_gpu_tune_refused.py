"""pb_autotune times launches of the step kernels, so it refuses the batches of
the linear system whose state those kernels would read beyond its end (binary32
storage, two dimensions), before any launch, as it does for Euler."""
import numpy as np
import pytest

import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,storage", [(3, "fp32"), (2, "fp64"), (2, "fp32")])
def test_linear_system_autotune_refused(dim, storage):
    announce(f"autotune refused linsym {dim}D {storage}")
    need_gpu()
    N, p, K = 4, 8, 3
    Bs, rad = I.linsym_matrices(1, N)
    b = I.Batch(dim=dim, p=np.full(K, p, np.int32), dx=np.full(K, 1.0 / p), nbr=I.self_periodic(K, dim), halo=3,
                pde="linsym", params=I.linsym_params(Bs, rad), n_unknowns=N, state=I.uniform(2, K * N * p**dim, -1, 1))
    B = pb.PatchBatch(b, storage=storage)
    before = B.download()
    with pytest.raises(pb.PbError) as e:
        B.autotune("fd", cfl=0.5, trials=1, use_cache=False)
    assert e.value.status == pb.PB_EUNSUPPORTED and "linear system" in str(e.value)
    np.testing.assert_array_equal(B.download(), before)
    B.close()
