"""GPU parity of the launches that split a series over workgroups, at the
batch sizes where the split changes: integers and statistics bit-equal to the
oracle's, as in the tests of the unsplit launches.
"""

import numpy as np
import pytest

import oracle as O
import paper_2511_05958_amd as P

from test_gpu_learned import _pack, gpu_features, series
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
    if wide:
        r[0, -1] = 9500
        r[-1, 0] = 1 << 31
        r[K // 2, N // 3] = 1
    return r


# one launch for all classes up to 64 series; 64 and 65 on either side of it; 700
# with three chunks a series; rows of 4099 / 4100 on either side of the streamed
# class, K of 1 to a few steps of the workgroups' waves
@pytest.mark.parametrize("num", [2, 64, 65, 700])
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
