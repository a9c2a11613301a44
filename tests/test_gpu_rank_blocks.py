"""Windows of more than 256 rows in the segmentation (ranks counted in blocks and
searched for in the others, the walk over groups of equal keys eight positions at
a time): bit-equal to the oracle's at the edges of the blocks, and a first level
that keeps up with the plain scan.
"""

import numpy as np
import pytest

import oracle as O
import paper_2511_05958_amd as P

from test_gpu_learned import _pack
from test_gpu_segment import check_series
from test_gpu_segment import run as run_segment
from test_gpu_split import _sweep
from test_gpu_split_placement import _us

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx(dev):
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("K", [255, 256, 257, 320, 511, 512, 513, 767, 1023, 1024, 1025, 1281, 2047, 2048])
@pytest.mark.parametrize("kind", ["level", "ties", "wide", "equal"])
def test_windows_around_the_blocks(ctx, K, kind):
    rng = np.random.default_rng(K)
    ss = [_sweep(rng, k, n, kind) for k, n in ((K, 3), (K, 40))]
    ss[1][K // 2:] += 700 if kind != "wide" else 0  # opens a window of each size
    ss[1][:K // 3] += 90 if kind != "wide" else 0
    if kind == "level":  # keys in order, in reverse and in runs
        ss.append(np.repeat((np.arange(K) + 100)[:, None], 2, axis=1).astype(np.uint32))
        ss.append(ss[-1][::-1].copy())
        ss.append((np.arange(K) // 9 % 30 + 100)[:, None].astype(np.uint32))
    x, d = _pack(ss, gap=1)
    cps, counts = run_segment(ctx, x, d, K)
    for t, r in enumerate(ss):
        check_series(cps[t], int(counts[t]), O.segment(r), t)


@pytest.mark.parametrize("num,K,N", [(512, 2048, 8), (2048, 1024, 8)])
def test_first_level_keeps_up_with_the_scan(ctx, num, K, N):
    """One level of windows, within half as much again as the scan of the batch."""
    import torch

    x = torch.randint(200, 400, (num * K * N,), dtype=torch.int32, device="cuda")
    d = P.to_device(P.make_desc(np.arange(num, dtype=np.int64) * K * N, [K] * num, [N] * num))
    prm, out = P.ks_params_init(0.05), P.empty_results(num)
    prm.max_K = K
    counts = torch.empty(num, dtype=torch.int32, device="cuda")
    scan = _us(lambda: P.ks_scan_batch(ctx.handle, x, d, num, prm, out))
    assert _us(lambda: P.ks_segment_batch(ctx.handle, x, d, num, prm, 1, 1, out, counts)) <= 1.5 * scan
