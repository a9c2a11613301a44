"""What calls allocate: the scan of few series has a workspace of its own, taken
by the first call that runs it and by ks_reserve; without it the ordered grid runs.
"""

import numpy as np
import pytest

import paper_2511_05958_amd as P

from test_gpu_launch_plans import Batch, captured, ordered

pytestmark = pytest.mark.gpu


@pytest.fixture
def ctx(dev):
    c = P.Context(0)
    yield c
    c.close()


def _free():
    import torch

    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("call", ["stats", "ordered grid", "one-launch scan"])
def test_calls_without_the_scan_of_few_series_take_none_of_its_workspace(ctx, call):
    import torch

    b = Batch(400 if call == "stats" else 2000 if call == "ordered grid" else 384, 2, 4, max_K=64)
    stats = torch.empty(b.n * 2 * 32, dtype=torch.uint8, device="cuda")
    before = _free()
    if call == "stats":
        P.ks_stats_batch(ctx.handle, b.samples, b.desc, b.n, 64, stats)
    else:
        b.scan(ctx)
    assert before - _free() < 8 << 20  # 31 MB of it serve 384 series of any K


def test_reserved_scans_allocate_nothing(ctx):
    batches = [Batch(1, 64, 64, max_K=0), Batch(384, 16, 4, max_K=0), Batch(300, 1024, 2), Batch(384, 300, 3)]
    P.ks_reserve(ctx.handle, 384, 0)
    before = _free()
    for b in batches:
        b.scan(ctx)
    assert _free() == before


def test_captured_scan_without_its_workspace_runs_the_ordered_grid(ctx):
    Batch(400, 16, 4, max_K=1024).scan(ctx)  # grows the ordered plan's workspace
    b = Batch(53, 600, 5)
    assert captured(lambda st: b.scan(ctx, st)) == ordered(53, 2)
    spread = b.kernels(ctx)
    assert len(spread) == 3
    assert captured(lambda st: b.scan(ctx, st)) == spread


@pytest.mark.parametrize("n", [1, 57, 384])
def test_workspace_of_the_scan_does_not_move(ctx, n):
    import torch

    small, large = Batch(n, 300, 5), Batch(384, 2048, 2)
    small.scan(ctx)
    want = small.out.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        small.scan(ctx, torch.cuda.current_stream().cuda_stream)
    g.replay()
    before = _free()
    large.scan(ctx)
    assert _free() == before
    for _ in range(3):
        small.out.zero_()
        g.replay()
        large.scan(ctx)
        torch.cuda.synchronize()
        assert torch.equal(small.out, want)
