"""The gradient kernel at the edges of its split: a partly filled chunk of 64
rows, one chunk per group of four waves (up to 256), two groups per
work-group, several rounds.  Ragged sizes against the oracle with the bounds of
the other gradient test; powers of two also against the sum of the gradients of
their 64-row slices (a factor of two in n scales every rounded value exactly, so
only the order of binary32 sums differs: at most 64 additions in a chain)."""
import numpy as np
import pytest

from oracle import mlp as M
import paper_2608_19273_amd as pb
from paper_2608_19273_amd import inputs as I

from gpu_helpers import announce, need_gpu
from test_gpu_mlp import random_net

pytestmark = pytest.mark.gpu


def data(n, norm, seed):
    x = (I.normal(seed, n * 5).reshape(n, 5) * 0.8 + norm[:5]).astype(np.float32)
    return x, I.normal(seed + 1, n).astype(np.float32)


@pytest.mark.parametrize("n", [1, 17, 63, 65, 16383, 16385, 32769, 70001])
def test_ragged_rows(n):
    announce(f"mlp gradient split n={n}")
    torch = need_gpu()
    p, norm = random_net(31)
    net = pb.Mlp(p, norm)
    x, t = data(n, norm, 32)
    g, loss = net.grad(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
    g = g.cpu().numpy().astype(np.float64)
    lo, go = M.loss_and_grad(p, norm, x, t)
    assert abs(loss.item() - lo) <= 1e-4 * lo
    offs = [0, 320, 384, 4480, 4544, 4608, 4609]
    for a, b in zip(offs[:-1], offs[1:]):
        assert np.linalg.norm(g[a:b] - go[a:b]) <= 1e-2 * np.linalg.norm(go[a:b]) + 1e-7, a
    net.close()


@pytest.mark.parametrize("chunks", [2, 256, 512, 1024])
def test_sum_of_slices(chunks):
    announce(f"mlp gradient of {chunks} chunks")
    torch = need_gpu()
    p, norm = random_net(41)
    net = pb.Mlp(p, norm)
    x, t = (torch.from_numpy(a).cuda() for a in data(64 * chunks, norm, 42))
    g, loss = net.grad(x, t)
    parts = [net.grad(x[64 * i:64 * (i + 1)].contiguous(), t[64 * i:64 * (i + 1)].contiguous()) for i in range(chunks)]
    s = np.stack([q.cpu().numpy() for q, _ in parts]).astype(np.float64)
    ls = np.array([q.item() for _, q in parts])
    bound = 64 * 2.0**-24
    assert np.all(np.abs(g.cpu().numpy() - s.mean(0)) <= bound * np.abs(s).mean(0) + 1e-30)
    assert abs(loss.item() - ls.mean()) <= bound * ls.mean()
    net.close()
