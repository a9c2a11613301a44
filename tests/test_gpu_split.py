"""GPU parity of the launches that split a series over workgroups, at the
batch sizes where the split changes: integers and statistics bit-equal to the
oracle's, as in the tests of the unsplit launches.
"""

import numpy as np
import pytest

import oracle as O
import paper_2511_05958_amd as P

from test_gpu_learned import _pack, gpu_features, series
from test_gpu_segment import check_series
from test_gpu_segment import run as run_segment
from test_gpu_stats import gpu_stats, same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(dev):
    c = P.Context(0)
    yield c
    c.close()


def _rows(rng, K, N, wide):
    """Latency rows with a level change; `wide` spreads a row over more than the window and the fast moments' range."""
    r = rng.integers(200, 700, (K, N)).astype(np.uint32)
    r[K // 2:] += 150
    if K > 2:
        r[1] = 77  # equal samples
    if wide:
        r[0, -1] = 9500
        r[-1, 0] = 1 << 31
        r[K // 2, N // 3] = 1
    return r


# one launch for all classes up to 16 series; 16 and 17 on either side of it; 700
# with several chunks a series; rows of 4099 / 4100 on either side of the streamed
# class, K of 1 to a few steps of the workgroups' waves
@pytest.mark.parametrize("num", [2, 16, 17, 700])
def test_row_passes_split_over_chunks(ctx, num):
    rng = np.random.default_rng(num)
    Ns = [4, 255, 256, 257, 1027, 1028, 2051, 2052, 4099, 4100, 9001]
    ss = []
    for t in range(num):
        N = Ns[t % len(Ns)] if t < 64 else int(rng.choice([64, 255, 256, 300]))
        K = int(rng.choice([2, 3, 7, 8, 9, 16, 17, 33])) if t < 64 else int(rng.integers(2, 20))
        ss.append(_rows(rng, K, N, t % 3 == 2))
    if num == 2:  # few long rows: every wave of a workgroup on one row
        ss = [_rows(rng, 33, 4100, True), _rows(rng, 2, 40001, False)]
    x, d = _pack(ss, gap=3)
    g = gpu_stats(ctx, x, d, 64)
    f = gpu_features(ctx, x, d, 64)
    for t, r in enumerate(ss):
        a = int(d[t]["aux_offset"])
        assert same(g[a:a + len(r)], O.row_stats(r)), (t, r.shape)
        assert np.array_equal(f[a:a + len(r)], O.features(series(x, d, t))), (t, r.shape)


def test_streamed_rows_a_wave_each(ctx):
    """Chunks of two rows per wave and more: streamed rows a wave each."""
    rng = np.random.default_rng(5)
    ss = [_rows(rng, 2, 64, False) for _ in range(1100)] + [_rows(rng, 64, 4100, True), _rows(rng, 33, 4101, False)]
    x, d = _pack(ss, gap=1)
    g = gpu_stats(ctx, x, d, 64)
    f = gpu_features(ctx, x, d, 64)
    for t in [0, 1099, 1100, 1101]:
        a = int(d[t]["aux_offset"])
        assert same(g[a:a + len(ss[t])], O.row_stats(ss[t])), t
        assert np.array_equal(f[a:a + len(ss[t])], O.features(ss[t])), t


def _sweep(rng, K, N, kind):
    r = rng.integers(200, 260, (K, N)).astype(np.uint32)
    r[K // 3:] += 30
    if kind == "ties":  # groups of equal keys
        r = np.repeat((np.arange(K) // 5 % 7 * 3 + 100)[:, None], N, axis=1).astype(np.uint32)
    elif kind == "wide":  # keys of 53 bits and more
        r[rng.integers(0, K, max(1, K // 4)), 0] = 0xFFFFFFFF - rng.integers(0, 3)
    elif kind == "equal":
        r[:] = 7
    return r


def _check_scan(ctx, ss, max_K, gap=1):
    import torch

    x, d = _pack(ss, gap=gap)
    prm = P.ks_params_init(0.05)
    prm.max_K = max_K
    out = P.empty_results(len(d))
    allU = torch.full((int(d["K"].sum()),), 77, dtype=torch.int32, device="cuda")
    P.ks_scan_batch(ctx.handle, P.to_device(x), P.to_device(d), len(d), prm, out, allU)
    torch.cuda.synchronize()
    g = P.results_to_numpy(out)
    o, oU, _ = O.scan_batch(x, d["offset"], d["K"], d["N"], want_allU=True)
    assert np.array_equal(g["flags"] & P.KS_SIGNIFICANT, o["significant"])
    for k in ("cp", "n", "m", "U", "D", "lambda"):
        assert np.array_equal(g[k], o[k]), k
    assert np.allclose(g["p"], o["p"], rtol=1e-12, atol=0)
    assert np.array_equal(allU.cpu().numpy().view(np.uint32), oU)


# K around the edges of the 64-row and 64-candidate slots and of the K classes;
# the mean series size on both sides of the one-launch scan's limit
@pytest.mark.parametrize("K", [2, 3, 63, 64, 65, 66, 128, 129, 256, 257, 1025, 2048])
@pytest.mark.parametrize("kind", ["level", "ties", "wide", "equal"])
def test_split_scan_edges(ctx, K, kind):
    rng = np.random.default_rng(K)
    _check_scan(ctx, [_sweep(rng, k, n, kind) for k, n in ((K, 5), (max(2, K - 1), 257), (K, 33))], K)
    _check_scan(ctx, [_sweep(rng, K, n, kind) for n in (513, 66000 // K + 1)], K, gap=2)


@pytest.mark.parametrize("num", [1, 2, 384, 385, 1024, 1025])
def test_split_scan_series_counts(ctx, num):
    """Long rows shared by a workgroup's waves (few rows in all), and both sides of the largest batches that are split or
    scanned in one launch."""
    rng = np.random.default_rng(num)
    kmax = 300 if num < 1000 else 64
    if num <= 2:
        ss = [_sweep(rng, 9 + t, 40001 + t, "level") for t in range(num)]
    else:
        ss = [_sweep(rng, int(rng.integers(2, kmax)), int(rng.integers(1, 700)), "level") for _ in range(num)]
    _check_scan(ctx, ss, kmax if num > 2 else 2048)
    d = P.make_desc([0], [3], [4])
    d["K"] = 1  # a bad shape beside good ones is flagged by both paths alike
    for n in (1, 300):
        import torch

        dd = np.concatenate([d, P.make_desc(np.zeros(n - 1), [3] * (n - 1), [4] * (n - 1))]) if n > 1 else d
        prm = P.ks_params_init(0.05)
        prm.max_K = 64
        out = P.empty_results(n)
        P.ks_scan_batch(ctx.handle, P.to_device(np.arange(12, dtype=np.uint32)), P.to_device(dd), n, prm, out)
        torch.cuda.synchronize()
        g = P.results_to_numpy(out)
        assert g["flags"][0] == P.KS_BAD_SHAPE and g["cp"][0] == 0 and (g["flags"][1:] & P.KS_BAD_SHAPE == 0).all()


@pytest.mark.parametrize("num,K", [(1, 2), (3, 65), (2, 1025), (1, 2048), (511, 24), (512, 24)])
@pytest.mark.parametrize("kind", ["level", "ties", "wide"])
def test_segment_edges(ctx, num, K, kind):
    """Windows around the 64-row and 64-candidate slots and past the workgroup's
    threads; both sides of the batch size from which a workgroup streams its rows."""
    rng = np.random.default_rng(K)
    ss = [_sweep(rng, K if num < 8 else int(rng.integers(2, K)), 7 if K > 100 else 12, kind) for _ in range(num)]
    if K > 100:  # more levels, so that windows of every size open
        for r in ss:
            r[K // 2:K // 2 + 40] += 500
            r[K - 70:] += 900
    x, d = _pack(ss, gap=1)
    cps, counts = run_segment(ctx, x, d, K)
    for t, r in enumerate(ss):
        if num < 8 or t % 37 == 0:
            check_series(cps[t], int(counts[t]), O.segment(r), t)
