"""Network kernels at the edges of their tiles, on the grid cases of
test_gpu_network (bit-exact with the oracle): 116-row forward tiles, 120-row
backward tiles, 64-row weight-gradient tiles over the slot rows, and more tiles
than resident workgroups.
"""

import numpy as np
import pytest

import paper_2511_05958_amd as P
from oracle import cnn as C

from test_gpu_network import NA, device_grads, device_logits, device_trace, grid_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(dev):
    c = P.Context(0)
    yield c
    c.close()


EDGES = [4, 15, 16, 99, 100, 115, 116, 117, 119, 120, 121, 231, 232, 233, 239, 240, 241, 256]


def test_forward_tile_edges(ctx):
    theta, feats, _ = grid_case(11, EDGES)
    caches = [C.forward(f, theta, round_bf16=True) for f in feats]
    assert C.exact_in_fp32([c for _, c in caches], theta)
    z = device_logits(ctx, theta, feats, 256)
    tr, _ = device_trace(ctx, theta, feats, 256)
    for K, zg, (zo, _), (a, _) in zip(EDGES, z, caches, tr):
        assert np.array_equal(zg, zo) and np.array_equal(a[:, NA - 1], zo), K


@pytest.mark.parametrize("K", [60, 64, 116, 119, 120, 121, 128, 241])
def test_backward_tile_edges(ctx, K):
    theta, feats, dzs = grid_case(200 + K, [K, 5, K - 1], 0.0)
    dzs[0][[1, K // 2]] = 0.0625  # first and middle rows of one series, the last of another
    dzs[2][K - 2] = -0.125
    caches = [C.forward(f, theta, round_bf16=True) for f in feats]
    assert C.exact_in_fp32([c for _, c in caches], theta, dzs)
    go = np.zeros(C.NUM_PARAMS)
    for (_, cache), dz in zip(caches, dzs):
        go += C.backward(dz, theta, cache, round_bf16=True)
    assert np.count_nonzero(go)
    assert np.array_equal(device_grads(ctx, theta, feats, dzs, 256), go)


def test_more_tiles_than_workgroups(ctx):
    """1100 short series: every resident workgroup takes several tiles."""
    rng = np.random.default_rng(3)
    Ks = [int(k) for k in rng.integers(2, 12, 1100)]
    theta, feats, dzs = grid_case(12, Ks, 0.0)
    for t in (0, 511, 512, 1023, 1099):
        dzs[t][1] = 0.25
    caches = [C.forward(f, theta, round_bf16=True) for f in feats]
    use = [t for t in range(1100) if np.any(dzs[t])]
    assert C.exact_in_fp32([caches[t][1] for t in use], theta, [dzs[t] for t in use])
    z = device_logits(ctx, theta, feats, 16)
    assert all(np.array_equal(zg, zo) for zg, (zo, _) in zip(z, caches))
    go = np.zeros(C.NUM_PARAMS)
    for t in use:
        go += C.backward(dzs[t], theta, caches[t][1], round_bf16=True)
    assert np.array_equal(device_grads(ctx, theta, feats, dzs, 16), go)
