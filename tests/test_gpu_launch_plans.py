"""Which kernels a recorded launch plan, the default plan and the launch options run.

A call is captured into a graph (never launched) and the captured kernels'
workgroup sizes are compared with the plan's: the ordered plan is its planning
kernel (1024 threads, one workgroup) and one workgroup of the variant's size per
series. Results under a replayed graph are bit-equal to the oracle's.
"""

import ctypes

import numpy as np
import pytest

import paper_2511_05958_amd as P
from paper_2511_05958_amd import synth as S

from test_gpu_scan import assert_parity, batch_arrays, oracle_batch, run_gpu

pytestmark = pytest.mark.gpu

THREADS = (256, 128, 512, 256, 256, 256)  # per scan-kernel variant (ks_launch.variant)


@pytest.fixture
def ctx(dev):
    c = P.Context(0)
    yield c
    c.close()


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNode(ctypes.Structure):
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def _hip():
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    return ctypes.CDLL(path)


def captured(call):
    """(grid, block) of every kernel that call(stream) launches, in capture order."""
    import torch

    hip, st, graph, n = _hip(), torch.cuda.Stream(), ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(st.cuda_stream), 1) == 0
    try:
        call(st.cuda_stream)
    finally:
        rc = hip.hipStreamEndCapture(ctypes.c_void_p(st.cuda_stream), ctypes.byref(graph))
    assert rc == 0 and graph.value
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    got = []
    for node in nodes:
        k = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(k)) == 0
        got.append(((k.grid.x, k.grid.y), k.block.x))
    assert hip.hipGraphDestroy(graph) == 0
    return got


class Batch:
    def __init__(self, num, K, N, max_K=None, opts=0):
        import torch

        self.n, self.prm = num, P.ks_params_init(0.05)
        self.prm.max_K, self.prm.opts = K if max_K is None else max_K, opts
        self.samples = torch.randint(100, 400, (num * K * N,), dtype=torch.int32, device="cuda")
        self.desc = P.to_device(P.make_desc(np.arange(num, dtype=np.int64) * K * N, [K] * num, [N] * num))
        self.out = P.empty_results(num)

    def scan(self, ctx, stream=None, fn=P.ks_scan_batch):
        fn(ctx.handle, self.samples, self.desc, self.n, self.prm, self.out, stream=stream)

    def kernels(self, ctx, fn=P.ks_scan_batch):
        self.scan(ctx, fn=fn)  # grows the workspace
        return captured(lambda st: self.scan(ctx, st, fn))


def ordered(num, variant):
    return [((1, 1), 1024), ((num, 1), THREADS[variant])]


@pytest.mark.parametrize("num,K,N", [(1, 64, 64), (53, 2048, 5), (384, 256, 8), (1024, 64, 8)])
@pytest.mark.parametrize("variant", range(P.KS_SCAN_VARIANTS))
def test_recorded_ordered_plan_is_run(ctx, num, K, N, variant):
    b = Batch(num, K, N)
    P.ks_launch_set(ctx.handle, K, num, P.KS_LAUNCH_ORDERED, 1 << 20, 0, variant=variant)
    assert b.kernels(ctx) == ordered(num, variant)


@pytest.mark.parametrize("num,K,N", [(1, 64, 64), (53, 2048, 5), (1100, 1024, 4)])
def test_recording_the_default_changes_nothing(ctx, num, K, N):
    b = Batch(num, K, N)
    default = b.kernels(ctx)
    c = P.ks_launch_get(ctx.handle, K, num)
    assert (c.mode, c.chunk_bytes, c.graph, c.variant) == (P.KS_LAUNCH_ORDERED, 1 << 20, 1, 0)
    P.ks_launch_set(ctx.handle, K, num, c.mode, c.chunk_bytes, c.graph, variant=c.variant)
    assert b.kernels(ctx) == default
    assert b.kernels(ctx, P.ks_scan_batch_noalloc) == ordered(num, 2 if K >= 1024 else 0)


@pytest.mark.parametrize("chunk,variant", [(2 << 20, 0), (1 << 20, 1), (1 << 20, 2)])
def test_ordered_graph_of_few_series_with_new_buffers(ctx, chunk, variant):
    """A recorded ordered graph is updated to each call's buffers and replayed."""
    for first in (0, 40, 80):
        x, d = batch_arrays(S.make_batch(3, num_series=40, first_series=first))
        g, gU = run_gpu(ctx, x, d, max_K=512, launch=(P.KS_LAUNCH_ORDERED, chunk, 1), variant=variant)
        o, oU, _ = oracle_batch(x, d)
        assert_parity(g, gU, o, oU, d)


@pytest.mark.parametrize("num,K,N", [(1, 64, 64), (53, 2048, 5), (1100, 1024, 4), (600, 300, 700)])
def test_no_graph_option_changes_no_kernel(ctx, num, K, N):
    """KS_OPT_NO_GRAPH replaces the graph of the plan, the default's kernels stay."""
    assert Batch(num, K, N, opts=P.KS_OPT_NO_GRAPH).kernels(ctx) == Batch(num, K, N).kernels(ctx)
    P.ks_launch_set(ctx.handle, K, num, P.KS_LAUNCH_ORDERED, 1 << 20, 1, variant=1)
    assert Batch(num, K, N, opts=P.KS_OPT_NO_GRAPH).kernels(ctx) == ordered(num, 1)


@pytest.mark.parametrize("num,N,threads", [(600, 300, 256), (600, 321, 512), (10240, 321, 512), (10241, 321, 256)])
def test_default_variant_of_512_row_series(ctx, num, N, threads):
    """Eight waves per series above 160 Ki samples on average, in batches of up to 40 series per CU (of 256); the
    descriptors share one series' samples, num_samples counts as in a batch that does not."""
    import torch

    b = Batch(1, 512, N)
    d = P.to_device(P.make_desc(np.zeros(num, np.int64), [512] * num, [N] * num, np.zeros(num, np.int64)))
    b.n, b.desc, b.out = num, d, P.empty_results(num)
    b.samples = torch.randint(100, 400, (num * 512 * N,), dtype=torch.int32, device="cuda")
    assert b.kernels(ctx) == [((1, 1), 1024), ((num, 1), threads)]
