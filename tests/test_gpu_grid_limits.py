"""Batches of more series than one grid of 2^32 - 1 threads holds at the kernels'
usual workgroup sizes: each series repeats one of a few, so every record must
repeat those of a small batch (which the other tests compare with the oracle).
"""

import numpy as np
import pytest

import paper_2511_05958_amd as P

from test_gpu_line_launches import _repeats, _tiled

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx(dev):
    c = P.Context(0)
    yield c
    c.close()


def _series(rng, num=29):
    ks, ns = rng.integers(2, 4, num), rng.integers(1, 4, num)
    off = np.concatenate([[0], np.cumsum(ks * ns)])
    x = rng.integers(100, 900, off[-1], dtype=np.uint32)
    d = P.make_desc(off[:-1], ks, ns)
    d["K"][5] = 1  # one flagged series
    return x, d


def test_scan_of_more_series_than_a_grid_of_512_thread_workgroups(ctx):
    import torch

    x, d = _series(np.random.default_rng(1))
    n = (1 << 23) + 5
    prm, xd = P.ks_params_init(0.05), P.to_device(x)
    small, big = P.empty_results(len(d)), P.empty_results(n)
    P.ks_scan_batch(ctx.handle, xd, P.to_device(d), len(d), prm, small)
    P.ks_scan_batch(ctx.handle, xd, _tiled(d, n), n, prm, big)
    torch.cuda.synchronize()
    _repeats(big.view(torch.uint8).view(-1), small.view(torch.uint8).view(-1), n, 48)


def test_segmentation_of_more_series_than_a_grid_of_1024_thread_workgroups(ctx):
    import torch

    x, d = _series(np.random.default_rng(2))
    n = (1 << 22) + 3
    prm, xd = P.ks_params_init(0.05), P.to_device(x)
    prm.max_K = 300

    def run(desc, num):
        cps = torch.zeros(num * 2 * 48, dtype=torch.uint8, device="cuda")
        counts = torch.full((num,), 77, dtype=torch.int32, device="cuda")
        P.ks_segment_batch(ctx.handle, xd, desc, num, prm, 0, 2, cps, counts)
        torch.cuda.synchronize()
        return cps, counts.view(torch.uint8)

    small, big = run(P.to_device(d), len(d)), run(_tiled(d, n), n)
    _repeats(big[0], small[0], n, 96)
    _repeats(big[1], small[1], n, 4)
