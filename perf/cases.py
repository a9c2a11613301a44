"""Performance cases of the K-S change-point library: what a user of it runs, from one small
sweep to a batch that fills the card, through the public entry points.

A case is a dict of plain values:
  op        the call or chain of calls (see run)
  S, K, N   series (sweeps), rows per series (array sizes), samples per row
  uneven    K and N drawn per series, log-uniform on [K / 16, K] and [N / 64, N]
            (the shapes come from the case alone, the samples from the seed)
  packed    series follow each other without padding, so rows start at any
            4-byte offset; otherwise each series starts on 256 bytes
  noise     "plain" (one change, lognormal jitter), "levels" (one to four
            changes, 1% outliers) or "hard" (adjacent levels 1.05 - 1.2 apart, 5%
            outliers, Pareto tails)
  all_U     also write every split's statistic
  tuned     run under a recorded launch plan (ks_launch_set, as a tuning cache
            file gives it) instead of the default plan
The samples are made on the device from the seed; `exact` restates the method in
64-bit torch and numpy.
"""

from __future__ import annotations

import json
import math
from pathlib import Path

import numpy as np
import torch

import paper_2511_05958_amd as P

_MODELS = Path(P.__file__).resolve().parent / "models"
_ALPHA = 0.05
_LR = 1e-3
_CHUNK = 1 << 27  # samples generated at a time
_MAX_CP = 64
_LINE_J, _LINE_A = 16, 32
_ctx_handle = None


def listed():
    return [
        # one sweep of one memory element, the smallest call: launch latency
        dict(name="scan one sweep", op="scan", S=1, K=64, N=256, noise="plain"),
        # the sweeps of one GPU's memory elements, one per cache level, with the curve of every split
        dict(name="scan six sweeps", op="scan", S=6, K=1024, N=2048, noise="levels", all_U=True),
        # a batch of equal sweeps (the shape that the proposal network is trained on)
        dict(name="scan batch", op="scan", S=4096, K=256, N=1024, noise="levels"),
        # thousands of uneven sweeps in one call, rows at any 4-byte offset
        dict(name="scan uneven", op="scan", S=8192, K=512, N=4096, noise="levels", uneven=True),
        # the largest batch: long rows, adjacent levels, heavy tails, a tuned launch plan
        dict(name="scan large", op="scan", S=2048, K=1024, N=2048, noise="hard", tuned=True),
        # per-row statistics of a few sweeps with very long rows (streamed, odd length)
        dict(name="stats long rows", op="stats", S=8, K=64, N=65537, noise="levels"),
        # workflow step 3 of a few sweeps: detection, per-row statistics, outlier check
        dict(name="check eight sweeps", op="check", S=8, K=256, N=1024, noise="levels"),
        # cache-line-size scoring: statistics of many short rows, then the scores
        dict(name="line size", op="line", S=256, K=_LINE_J * _LINE_A, N=256, noise="plain"),
        # every level boundary of each sweep
        dict(name="segment", op="segment", S=512, K=256, N=1024, noise="levels"),
        # proposal by the trained network and the exact refine, on a batch
        dict(name="learned step", op="learned", S=1024, K=256, N=1024, noise="levels"),
        # the network alone, on features kept from earlier passes
        dict(name="network forward", op="forward", S=512, K=1024, N=0),
        # four optimizer steps of the training loop's batch, then the weights
        dict(name="training steps", op="train", S=256, K=256, N=0, steps=4),
    ]


def _logu(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: every op, sizes log-uniform over what the listed ones span, at most 2 GiB of samples."""
    op = rng.choice(["scan", "scan", "scan", "stats", "check", "line", "segment", "learned", "forward", "train"])
    if op == "forward":
        K = _logu(rng, 32, 2048)
        return dict(op=op, S=min(_logu(rng, 1, 4096), (1 << 20) // K + 1), K=K, N=0)
    if op == "train":
        return dict(op=op, S=_logu(rng, 16, 512), K=_logu(rng, 48, 512), N=0, steps=rng.choice([1, 2, 4]))
    noise = rng.choice(["plain", "levels", "hard"])
    if op == "line":
        return dict(op=op, S=_logu(rng, 8, 512), K=_LINE_J * _LINE_A, N=_logu(rng, 64, 1024), noise="plain")
    K = _logu(rng, 32, 2048)
    N = _logu(rng, 64, 65536 if op in ("scan", "stats") else 4096)
    cap = (1 << 29) // (K * N)
    S = max(1, min(_logu(rng, 1, 8192), cap, 512 if op == "segment" else 8192))
    c = dict(op=op, S=S, K=K, N=N, noise=noise, packed=rng.random() < 0.5)
    if op in ("scan", "stats", "learned") and K >= 512 and N >= 4096:
        c["uneven"] = True
    if op == "scan":
        c["all_U"] = rng.random() < 0.25
    return c


# ---------------------------------------------------------------- inputs


def _shapes(case):
    """K and N of every series, and the first sample of each, and the total; from the case alone."""
    S, K, N = case["S"], case["K"], case["N"]
    Ks, Ns = np.full(S, K, np.int64), np.full(S, N, np.int64)
    if case.get("uneven"):
        r = np.random.default_rng(S * 1000003 + K * 1009 + N)
        Ks = np.rint(np.exp(r.uniform(math.log(max(2, K / 16)), math.log(K), S))).astype(np.int64)
        Ns = np.rint(np.exp(r.uniform(math.log(max(1, N / 64)), math.log(N), S))).astype(np.int64)
    size = Ks * Ns
    room = size if case.get("packed") else (size + 63) // 64 * 64
    off = np.concatenate([[0], np.cumsum(room)])
    return Ks, Ns, off[:-1], int(off[-1])


def _samples(case, seed):
    """uint32 latencies (an int32 tensor) of every series, in the layout of _shapes."""
    Ks, Ns, off, total = _shapes(case)
    S, noise = case["S"], case["noise"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    most = 1 if noise == "plain" else 4
    Kd = torch.from_numpy(Ks).cuda()
    n_change = torch.randint(1, most + 1, (S, 1), device="cuda", generator=g)
    at = 1 + (torch.rand((S, most), device="cuda", generator=g, dtype=torch.float64) * (Kd[:, None] - 1)).long()
    at = torch.where(torch.arange(most, device="cuda")[None, :] < n_change, at, 1 << 30).sort(1).values
    # "hard": adjacent levels close together; otherwise rising steps of the load latencies of a GPU's memory elements
    if noise == "hard":
        first = 120.0 * (0.9 + 0.2 * torch.rand((S, 1), device="cuda", generator=g))
        ratio = 1.05 + 0.15 * torch.rand((S, most), device="cuda", generator=g)
        level = torch.cat([first, first * torch.cumprod(ratio, 1)], 1)
    else:
        ladder = torch.tensor([120.0, 300.0, 550.0, 850.0, 1300.0, 1300.0, 1300.0, 1300.0, 1300.0], device="cuda")
        step0 = (torch.rand((S, 1), device="cuda", generator=g) * (5 - n_change)).long()
        level = ladder[step0 + torch.arange(most + 1, device="cuda")[None, :]]
        level = level * (0.9 + 0.2 * torch.rand((S, most + 1), device="cuda", generator=g))
    sid = torch.repeat_interleave(torch.arange(S, device="cuda"), Kd)
    start = torch.cumsum(Kd, 0) - Kd
    row = torch.arange(len(sid), device="cuda") - start[sid]
    row_level = level[sid, (at[sid] <= row[:, None]).sum(1)]
    # samples per row, a series' padding counted with its last row
    count = np.repeat(Ns, Ks)
    last = np.cumsum(Ks) - 1
    count[last] += np.diff(np.concatenate([off, [total]])) - Ks * Ns
    ends = np.cumsum(count)
    count_d = torch.from_numpy(count).cuda()
    out = torch.empty(max(total, 1), dtype=torch.int32, device="cuda")
    sigma = 0.05 if noise == "plain" else 0.08
    p_out = {"plain": 0.0, "levels": 0.01, "hard": 0.05}[noise]
    a = 0
    while a < len(count):
        e0 = int(ends[a - 1]) if a else 0
        b = max(a + 1, int(np.searchsorted(ends, e0 + _CHUNK, side="right")))
        n = int(ends[b - 1]) - e0
        x = torch.repeat_interleave(row_level[a:b], count_d[a:b], output_size=n)
        z = torch.randn(n, device="cuda", generator=g).mul_(sigma).exp_()
        if p_out:
            u = torch.rand(n, device="cuda", generator=g)
            v = torch.rand(n, device="cuda", generator=g)
            if noise == "hard":
                z = torch.where(u < p_out + 0.095, (1.0 - v).clamp_(min=1e-9).pow_(-1 / 2.5), z)
            z = torch.where(u < p_out, 1.0 + 4.0 * v, z)
        out[e0:e0 + n] = x.mul_(z).round_().clamp_(1.0, 2.0e9).to(torch.int32)
        a = b
    return out


def _weights(seed):
    """Parameters of the network: He-uniform weights, small biases."""
    r = np.random.default_rng(seed)
    parts = []
    for cin, cout in ((11, 64), (64, 64), (64, 64), (64, 1)):
        a = math.sqrt(6.0 / (5 * cin))
        parts += [r.uniform(-a, a, cout * cin * 5), r.uniform(-0.1, 0.1, cout)]
    return np.concatenate(parts).astype(np.float32)


def _features(S, K, seed):
    """Decile features of S sweeps of K rows: nine rising values per row, relative to the sweep's minimum, and the labels."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    at = torch.randint(1, K, (S, 1), device="cuda", generator=g)
    t = torch.arange(K, device="cuda")[None, :]
    level = 1.3 + torch.rand((S, 1), device="cuda", generator=g) * (t >= at)
    q = torch.tensor([-1.28, -0.84, -0.52, -0.25, 0.0, 0.25, 0.52, 0.84, 1.28], device="cuda")
    jitter = 0.004 * torch.randn((S, K, 9), device="cuda", generator=g)
    f = level[:, :, None] * (torch.exp(0.08 * q)[None, None, :] + jitter) - 1.0
    return f.sort(2).values.contiguous(), at[:, 0].to(torch.int32)


# ---------------------------------------------------------------- the calls


def _ctx():
    """The program's one context."""
    global _ctx_handle
    if _ctx_handle is None:
        _ctx_handle = P.Context(0)
    return _ctx_handle


def _results(buf, n):
    """A ks_result buffer as its whole numbers and its floats (views, nothing is copied)."""
    i = buf.view(torch.int32).view(n, 12)
    return {"cp_n_m_U": i[:, :4], "flags": i[:, 10:], "D_lambda_p": buf.view(torch.float64).view(n, 6)[:, 2:5]}


def _row_stats(buf, rows):
    return {"mean_std": buf.view(torch.float64).view(rows, 4)[:, :2], "min_p50_p95_max": buf.view(torch.int32).view(rows, 8)[:, 4:]}


def prepare(case, seed):
    op, S, K = case["op"], case["S"], case["K"]
    st = {"op": op, "S": S, "K": K, "ctx": _ctx(), "steps": case.get("steps", 1)}
    prm = P.ks_params_init(_ALPHA)
    prm.max_K = K
    st["prm"] = prm
    if op in ("forward", "train"):
        st["model"] = P.Model(st["ctx"])
        P.ks_model_set_params(st["model"].handle, _weights(seed))
        st["batches"] = []
        for j in range(st["steps"]):
            f, lab = _features(S, K, seed + 7919 * j)
            d = P.to_device(P.make_desc(np.zeros(S), np.full(S, K), np.full(S, 1)))
            st["batches"].append((f.view(-1), d, lab))
        st["logits"] = torch.zeros(S * K, dtype=torch.float32, device="cuda")
        st["loss"] = torch.zeros(st["steps"], dtype=torch.float32, device="cuda")
        return st
    Ks, Ns, off, _ = _shapes(case)
    st["samples"] = _samples(case, seed)
    st["desc"] = P.to_device(P.make_desc(off, Ks, Ns))
    rows = int(Ks.sum())
    if op in ("scan", "check", "learned"):
        st["out"] = P.empty_results(S)
        st["results"] = _results(st["out"], S)
    if case.get("all_U"):
        st["all_U"] = torch.zeros(rows, dtype=torch.int32, device="cuda")
    if case.get("tuned"):
        P.ks_launch_set(st["ctx"].handle, K, S, P.KS_LAUNCH_PERSISTENT, 16 << 20, 1, 2)
    if op in ("stats", "check", "line"):
        st["stats"] = torch.empty(rows * 32, dtype=torch.uint8, device="cuda")
        st["row_stats"] = _row_stats(st["stats"], rows)
    if op == "check":
        st["check"] = torch.empty(S * 32, dtype=torch.uint8, device="cuda")
    if op == "line":
        st["strides"] = torch.arange(16, 16 * (_LINE_J + 1), 16, dtype=torch.int32, device="cuda")
        st["lines"] = torch.empty(S * 24, dtype=torch.uint8, device="cuda")
        i = st["lines"].view(torch.int32).view(S, 6)
        st["line_out"] = {"line_jstar_flags": i[:, :3], "jump": st["lines"].view(torch.float64).view(S, 3)[:, 2:]}
    if op == "segment":
        st["cps"] = torch.zeros(S * _MAX_CP * 48, dtype=torch.uint8, device="cuda")
        st["counts"] = torch.empty(S, dtype=torch.int32, device="cuda")
        st["results"] = _results(st["cps"], S * _MAX_CP)
    if op == "learned":
        st["model"] = P.Model(st["ctx"])
        P.ks_model_load(st["model"].handle, _MODELS / "proposal_r4.ckpt")
        prm.tau = json.loads((_MODELS / "proposal_r4.json").read_text())["tau"]
        st["features"] = torch.zeros(rows * 9, dtype=torch.float32, device="cuda")
        st["proposal"] = torch.empty(S, dtype=torch.int32, device="cuda")
        st["confidence"] = torch.empty(S, dtype=torch.float32, device="cuda")
    return st


def run(st):
    op, ctx, S, prm = st["op"], st["ctx"].handle, st["S"], st["prm"]
    if op == "scan":
        P.ks_scan_batch(ctx, st["samples"], st["desc"], S, prm, st["out"], st.get("all_U"))
        return {"results": st["results"], "all_U": st["all_U"]} if "all_U" in st else {"results": st["results"]}
    if op == "stats":
        P.ks_stats_batch(ctx, st["samples"], st["desc"], S, st["K"], st["stats"])
        return {"stats": st["row_stats"]}
    if op == "check":
        P.ks_scan_batch(ctx, st["samples"], st["desc"], S, prm, st["out"])
        P.ks_stats_batch(ctx, st["samples"], st["desc"], S, st["K"], st["stats"])
        P.ks_check_batch(ctx, st["desc"], S, st["K"], st["out"], st["stats"], st["check"])
        return {"results": st["results"], "stats": st["row_stats"], "check": st["check"]}
    if op == "line":
        P.ks_stats_batch(ctx, st["samples"], st["desc"], S, st["K"], st["stats"])
        P.ks_line_batch(ctx, st["desc"], S, st["stats"], _LINE_J, st["strides"], st["lines"])
        return {"stats": st["row_stats"], "lines": st["line_out"]}
    if op == "segment":
        P.ks_segment_batch(ctx, st["samples"], st["desc"], S, prm, 0, _MAX_CP, st["cps"], st["counts"])
        return {"counts": st["counts"], "results": st["results"]}
    if op == "learned":
        P.ks_propose(ctx, st["model"].handle, st["samples"], st["desc"], S, prm, st["proposal"], st["confidence"],
                     st["features"])
        P.ks_refine(ctx, st["desc"], S, st["samples"].numel(), st["proposal"], st["confidence"], prm, st["out"])
        return {"features": st["features"], "proposal": st["proposal"], "confidence": st["confidence"],
                "results": st["results"]}
    if op == "forward":
        f, d, _ = st["batches"][0]
        P.ks_cnn_forward(ctx, st["model"].handle, f, d, S, st["K"], st["logits"])
        return {"logits": st["logits"]}
    for j, (f, d, lab) in enumerate(st["batches"]):
        P.ks_train_step(ctx, st["model"].handle, f, d, lab, S, st["K"], _LR, st["loss"][j:])
    return {"loss": st["loss"], "weights": P.ks_model_get_params(st["model"].handle)}


def work(case):
    """Each sample, feature and weight read once, each output written once; the network's multiplications and additions."""
    op, S, K = case["op"], case["S"], case["K"]
    params = 4 * P.KS_CNN_PARAMS
    macs = 5 * (11 * 64 + 64 * 64 + 64 * 64 + 64)
    if op == "forward":
        return {"bytes": S * K * 40 + params, "flops": 2 * macs * S * K}
    if op == "train":
        # forward, input gradients of three layers, weight gradients of four
        back = 5 * (64 + 64 * 64 + 64 * 64) + macs
        n = case["steps"]
        return {"bytes": n * (S * K * 36 + 6 * params), "flops": n * 2 * (macs + back) * S * K}
    Ks, Ns, _, _ = _shapes(case)
    rows = int(Ks.sum())
    reads = 4 * int((Ks * Ns).sum())
    writes = {"scan": 48 * S + (4 * rows if case.get("all_U") else 0), "stats": 32 * rows, "check": 80 * S + 32 * rows,
              "line": 24 * S + 32 * rows, "segment": 52 * S, "learned": 56 * S + 36 * rows}[op]
    return {"bytes": reads + writes, "flops": 2 * macs * rows if op == "learned" else 0}


# ---------------------------------------------------------------- 64-bit restatement


def _series_rows(case, x):
    """Per group of series of one shape: their indices and their samples as [series, K, N] int64."""
    Ks, Ns, off, _ = _shapes(case)
    s = 0
    while s < len(Ks):
        K, N = int(Ks[s]), int(Ns[s])
        e = s + 1
        while e < len(Ks) and Ks[e] == K and Ns[e] == N and (e - s + 1) * K * N <= 1 << 26:
            e += 1
        step = int(off[s + 1] - off[s]) if e > s + 1 else K * N
        block = torch.as_strided(x, (e - s, K, N), (step, N, 1), int(off[s]))
        yield range(s, e), block.to(torch.int64)
        s = e


def _splits(Q):
    """U_c, c = 1 .. K - 1, of one series' reduced values Q (exact integers)."""
    K = len(Q)
    q, order = torch.sort(Q)
    c = torch.arange(1, K, device=Q.device)
    i = torch.cumsum((order[None, :] < c[:, None]).to(torch.int32), 1)
    p = torch.arange(1, K + 1, device=Q.device)
    end = torch.ones(K, dtype=torch.bool, device=Q.device)
    end[:-1] = q[1:] != q[:-1]
    return torch.where(end[None, :], (K * i - c[:, None] * p[None, :]).abs(), 0).amax(1)


def _kolmogorov(l2):
    """The asymptotic Kolmogorov tail of lambda^2."""
    l2 = np.asarray(l2, np.float64)
    k = np.arange(1, 101, dtype=np.float64)[:, None]
    with np.errstate(divide="ignore", over="ignore", invalid="ignore"):
        tail = 2 * ((-1.0) ** (k + 1) * np.exp(-2 * k * k * l2)).sum(0)
        body = 1 - np.sqrt(2 * np.pi) / np.sqrt(l2) * np.exp(-((2 * k - 1) ** 2) * np.pi**2 / (8 * l2)).sum(0)
    return np.where(l2 <= 0, 1.0, np.where(2 * l2 > 700, 0.0, np.where(l2 >= 1, tail, body)))


def _choice(U, K):
    """cp, n, m, U and D, lambda, p of the most significant split."""
    c = torch.arange(1, K, device=U.device, dtype=torch.float64)
    Ud = U.to(torch.float64)
    j = int(torch.argmax(Ud * Ud / (c * (K - c))))  # the first on ties
    u, n = int(U[j]), j + 1
    l2 = u * u / (n * (K - n) * K)
    return (n, n, K - n, u), (u / (n * (K - n)), math.sqrt(l2), float(_kolmogorov([l2])[0]))


def _result_arrays(ints, floats, significant):
    i = np.array(ints, np.int32).reshape(-1, 4)
    return {"cp_n_m_U": i, "flags": np.stack([significant, np.zeros_like(significant)], 1), "D_lambda_p": np.array(floats, np.float64).reshape(-1, 3)}


def _significant(ints):
    i = np.array(ints, np.float64).reshape(-1, 4)
    return (i[:, 3] ** 2 > -0.5 * math.log(_ALPHA / 2) * i[:, 1] * i[:, 2] * (i[:, 1] + i[:, 2])).astype(np.int32)


def _moments(block):
    """Reduced values of each row, as exact integers."""
    m = block.amin((1, 2))
    return (block - m[:, None, None]).square().sum(2)


def _exact_scan(case, x):
    ints, floats, curves = [], [], []
    for series, block in _series_rows(case, x):
        Q = _moments(block)
        for t in range(len(series)):
            U = _splits(Q[t])
            a, b = _choice(U, len(Q[t]))
            ints.append(a)
            floats.append(b)
            if case.get("all_U"):
                curves.append(np.concatenate([[0], U.cpu().numpy()]).astype(np.int32))
    got = {"results": _result_arrays(ints, floats, _significant(ints))}
    if case.get("all_U"):
        got["all_U"] = np.concatenate(curves)
    return got


def _exact_stats(case, x):
    ms, order = [], []
    for _, block in _series_rows(case, x):
        N = block.shape[2]
        s1, s2 = block.sum(2), block.square().sum(2)
        var = (N * s2 - s1 * s1).to(torch.float64) / float(N) ** 2
        ms.append(torch.stack([s1.to(torch.float64) / N, var.sqrt()], 2).reshape(-1, 2).cpu().numpy())
        v = block.sort(2).values
        pick = [0, (N - 1) // 2, 95 * (N - 1) // 100, N - 1]
        order.append(v[:, :, pick].to(torch.int32).reshape(-1, 4).cpu().numpy())
    return {"mean_std": np.concatenate(ms), "min_p50_p95_max": np.concatenate(order)}


def _exact_segment(case, x):
    S = case["S"]
    counts = np.zeros(S, np.int32)
    ints, floats, flags = np.zeros((S, _MAX_CP, 4), np.int32), np.zeros((S, _MAX_CP, 3)), np.zeros((S, _MAX_CP, 2), np.int32)
    for series, block in _series_rows(case, x):
        low = block.amin(2)
        for t, s in enumerate(series):
            found, todo = [], [(0, case["K"], 0)]
            while todo:
                a, b, depth = todo.pop()
                if b - a < 2:
                    continue
                w = block[t, a:b]
                i, f = _choice(_splits((w - low[t, a:b].min()).square().sum(1)), b - a)
                if not _significant([i])[0]:
                    continue
                found.append((a + i[0], i, f, depth))
                todo += [(a, a + i[0], depth + 1), (a + i[0], b, depth + 1)]
            counts[s] = len(found)
            for j, (cp, i, f, depth) in enumerate(sorted(found, key=lambda v: v[0])[:_MAX_CP]):
                ints[s, j], floats[s, j], flags[s, j] = (cp, *i[1:]), f, (1, depth)
    return {"counts": counts, "results": {"cp_n_m_U": ints.reshape(-1, 4), "flags": flags.reshape(-1, 2), "D_lambda_p": floats.reshape(-1, 3)}}


def _exact_features(case, x):
    got = []
    for _, block in _series_rows(case, x):
        N = block.shape[2]
        v = block.sort(2).values[:, :, [k * (N - 1) // 10 for k in range(1, 10)]].to(torch.float64)
        m = block.amin((1, 2)).to(torch.float64)[:, None, None]
        got.append(((v - m) / m.clamp(min=1.0)).reshape(-1).cpu().numpy())
    return np.concatenate(got)


def _layers(p):
    """The weights as [5 cin, cout] matrices (tap-major) and biases."""
    got, at = [], 0
    for cin, cout in ((11, 64), (64, 64), (64, 64), (64, 1)):
        w = p[at:at + cout * cin * 5].view(cout, cin, 5).permute(2, 1, 0).reshape(5 * cin, cout)
        at += cout * cin * 5
        got.append((w, p[at:at + cout]))
        at += cout
    return got


def _network(f, p):
    S, K, _ = f.shape
    t = torch.arange(K, device=f.device, dtype=torch.float64)
    pos = torch.stack([t / max(K - 1, 1), 4 * t * (K - t) / (K * K)], 1)
    h = torch.cat([f.to(torch.float64), pos[None].expand(S, K, 2)], 2)
    for l, (w, b) in enumerate(_layers(p)):
        pad = torch.nn.functional.pad(h, (0, 0, 2, 2))
        cols = torch.cat([pad[:, k:k + K] for k in range(5)], 2)
        h = (cols.reshape(S * K, -1) @ w + b).view(S, K, -1)
        if l < 3:
            h = h.relu()
    return h[:, :, 0]


def exact(case, seed):
    op, S, K = case["op"], case["S"], case["K"]
    if op == "forward":
        f, _ = _features(S, K, seed)
        p = torch.from_numpy(_weights(seed)).cuda().double()
        return {"logits": torch.cat([_network(f[a:a + 64], p).reshape(-1) for a in range(0, S, 64)])}
    if op == "train":
        p = torch.from_numpy(_weights(seed)).cuda().double()
        m1, m2, losses = torch.zeros_like(p), torch.zeros_like(p), []
        for j in range(case["steps"]):
            f, lab = _features(S, K, seed + 7919 * j)
            p.requires_grad_(True)
            z = _network(f, p)[:, 1:]
            loss = torch.nn.functional.cross_entropy(z, lab.long() - 1)
            (g,) = torch.autograd.grad(loss, p)
            losses.append(loss.item())
            m1, m2 = 0.9 * m1 + 0.1 * g, 0.999 * m2 + 0.001 * g * g
            p = p.detach() - _LR * (m1 / (1 - 0.9 ** (j + 1))) / ((m2 / (1 - 0.999 ** (j + 1))).sqrt() + 1e-8)
        return {"loss": np.array(losses), "weights": p}
    if op == "segment" and S * K > 1 << 17:
        return None  # a window at a time: minutes
    x = _samples(case, seed)
    if op == "scan":
        return _exact_scan(case, x)
    if op == "stats":
        return {"stats": _exact_stats(case, x)}
    if op == "check":
        return {**_exact_scan(case, x), "stats": _exact_stats(case, x), "check": None}
    if op == "line":
        return {"stats": _exact_stats(case, x), "lines": None}
    if op == "segment":
        return _exact_segment(case, x)
    # the proposal is the argmax of 16-bit logits, and confidence and refine follow it
    return {"features": _exact_features(case, x), "proposal": None, "confidence": None, "results": None}
