"""Both sides of the line scores' launch rule (a workgroup per experiment, or a
wave): each experiment repeats one of a few, so every record must repeat those of
a small batch (which the other tests compare with the oracle).
"""

import numpy as np
import pytest

import paper_2511_05958_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx(dev):
    c = P.Context(0)
    yield c
    c.close()


def _tiled(desc, n):
    """n descriptors that repeat `desc`, on the GPU (24 bytes each)."""
    import torch

    d = P.to_device(desc).view(torch.uint8).view(len(desc), 24)
    return d.repeat((n + len(desc) - 1) // len(desc), 1)[:n].contiguous().view(-1)


def _repeats(big, small, n, size):
    import torch

    k = small.numel() // size
    b, s = big[:n * size].view(n, size), small.view(k, size)
    m = n // k * k
    assert torch.equal(b[:m].view(m // k, k * size), s.view(1, -1).expand(m // k, -1))
    assert torch.equal(b[m:], s[:n - m])


# a workgroup per experiment or a wave each; with more than 128 sizes, fewer, and
# experiments whose steps do not divide
@pytest.mark.parametrize("n,J", [(1024, 2), (1025, 2), (1027, 3), (1025, 4), (32768, 16), (32771, 16), (32769, 5), ((1 << 24) + 2, 17)])
def test_line_scores_of_many_experiments(ctx, n, J):
    import torch

    rng = np.random.default_rng(J)
    A = [1, 2, 64, 128, 129, 256, 255, 3, 100, 130, 257]
    ks = np.array([J * a for a in A if J * a <= 2048] + [J * 3 + 1])
    aux = np.concatenate([[0], np.cumsum(ks)])
    d = P.make_desc(np.zeros(len(ks), np.int64), ks, np.ones(len(ks), np.int64), aux[:-1])
    stats = torch.from_numpy(rng.integers(100, 4000, (int(aux[-1]), 8), dtype=np.int32)).cuda().view(torch.uint8).view(-1)
    strides = torch.arange(16, 16 * (J + 1), 16, dtype=torch.int32, device="cuda")
    small = torch.zeros(len(ks) * 24, dtype=torch.uint8, device="cuda")
    big = torch.zeros(n * 24, dtype=torch.uint8, device="cuda")
    P.ks_line_batch(ctx.handle, P.to_device(d), len(ks), stats, J, strides, small)
    P.ks_line_batch(ctx.handle, _tiled(d, n), n, stats, J, strides, big)
    torch.cuda.synchronize()
    _repeats(big, small, n, 24)
