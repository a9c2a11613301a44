"""Row passes cut into chunks of a series' rows: batches around a whole round of
resident workgroups, rows that leave a chunk short or empty, against numpy's sort
and exact integer sums.

Bar: order statistics equal; the mean is one correctly rounded division.
"""

import numpy as np
import pytest

import paper_2511_05958_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("series,K,N", [(17, 2, 64), (300, 33, 255), (600, 5, 2060), (700, 9, 1030),
                                        (1025, 13, 70), (1100, 30, 256), (2100, 5, 2052), (8193, 2, 129)])
def test_every_row_of_every_chunk(dev, series, K, N):
    import torch

    rng = np.random.default_rng(series * 4099 + K * 67 + N)
    x = rng.integers(200, 900, size=(series * K, N), dtype=np.uint32)
    d = P.make_desc(np.arange(series, dtype=np.int64) * K * N, [K] * series, [N] * series)
    ctx = P.Context(0)
    try:
        xd, dd = P.to_device(x.ravel()), P.to_device(d)
        out = torch.full((series * K * 32,), 0xFF, dtype=torch.uint8, device="cuda")
        P.ks_stats_batch(ctx.handle, xd, dd, series, K, out)
        fe = torch.full((series * K * 9,), -1.0, dtype=torch.float32, device="cuda")
        P.ks_features(ctx.handle, xd, dd, series, K, fe)
        torch.cuda.synchronize()
        g = out.cpu().numpy().view(P.ROW_STATS_DTYPE)
        f = fe.cpu().numpy().reshape(series, K, 9)
    finally:
        ctx.close()
    s = np.sort(x, axis=1)
    assert (g["min"] == s[:, 0]).all() and (g["max"] == s[:, -1]).all()
    assert (g["p50"] == s[:, (N - 1) // 2]).all() and (g["p95"] == s[:, 95 * (N - 1) // 100]).all()
    assert np.array_equal(g["mean"], s.sum(axis=1, dtype=np.uint64).astype(np.float64) / N)
    dec = s[:, [k * (N - 1) // 10 for k in range(1, 10)]].reshape(series, K, 9).astype(np.float64)
    m = s[:, 0].reshape(series, K).min(axis=1).astype(np.float64)[:, None, None]
    assert np.array_equal(f, ((dec - m) / np.maximum(m, 1.0)).astype(np.float32))
