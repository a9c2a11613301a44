"""The scan of few series when max_K is far above the rows: results bit-equal to
the oracle's for every placement of its workgroups, and no slower than one
workgroup per series.
"""

import numpy as np
import pytest

import paper_2511_05958_amd as P

from test_gpu_split import _check_scan, _sweep

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx(dev):
    c = P.Context(0)
    yield c
    c.close()


# either side of 256 series (slots turned by the series, or slot after slot over
# whole turns of the XCDs), 1, 5, 16 and 32 slots of which few have rows
@pytest.mark.parametrize("num", [3, 8, 255, 256, 257, 264, 300, 384])
@pytest.mark.parametrize("max_K", [64, 300, 1024, 2048])
def test_slots_of_every_series(ctx, num, max_K):
    rng = np.random.default_rng(num * 4099 + max_K)
    ss = [_sweep(rng, int(rng.integers(2, 65)), int(rng.integers(1, 40)), "level") for _ in range(num)]
    for t in (0, num // 2, num - 1):  # and some with a row in the last slot
        ss[t] = _sweep(rng, max_K, 3, "level")
    ss[1] = _sweep(rng, 64, 70000, "level")  # past the one-launch scan's mean size for few series
    _check_scan(ctx, ss, max_K)


def _us(call):
    import torch

    a, b = torch.cuda.Event(True), torch.cuda.Event(True)
    best = float("inf")
    for _ in range(8):
        a.record()
        for _ in range(10):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    return best


@pytest.mark.parametrize("num,K,N", [(384, 64, 4), (384, 256, 64), (256, 64, 64), (256, 256, 4)])
def test_default_keeps_up_with_the_ordered_grid(ctx, num, K, N):
    """Under max_K 0, within a fifth of the recorded ordered plan (variant 0)."""
    import torch

    x = torch.randint(100, 400, (num * K * N,), dtype=torch.int32, device="cuda")
    d = P.to_device(P.make_desc(np.arange(num, dtype=np.int64) * K * N, [K] * num, [N] * num))
    prm, out = P.ks_params_init(0.05), P.empty_results(num)
    scan = lambda: P.ks_scan_batch(ctx.handle, x, d, num, prm, out)
    default = _us(scan)
    P.ks_launch_set(ctx.handle, 0, num, P.KS_LAUNCH_ORDERED, 1 << 20, 0, variant=0)
    assert default <= 1.2 * _us(scan)
