"""What a user of the library has it do, as cases that can be timed.

Each case is one whole call through the Python binding: the exact top-k of a
series in device memory, the same without an allocation, the one-shot call on a
host series, a stream session, and a batch of requests to the server.  Sizes,
intervals and generators are those of the benchmark, the tests and the serving
mix (random walk, Wafer-like, ECG-like).

listed()            the cases
draw(rng)           one more of the same ranges
prepare(case, seed) what a program holds before the call
run(state)          one call, and its outputs
work(case)          bytes and operations that one call cannot do without
exact(case, seed)   the distances that run() reports, by brute force in FP64
"""
import math

import numpy as np
import torch

from paper_2607_17481_amd import pmp, synth

DEVICE = "cuda:0"
PRECISION = {"fp64": pmp.PREC_FP64, "fp32": pmp.PREC_FP32, "bf16": pmp.PREC_BF16}
SERVER_BYTES = 24 << 30
SERVER_SLOTS = 4
APPEND = 65536                   # samples per append of a stream
EXACT_FLOPS = 2.5e14             # the largest brute force that exact() takes on


def _case(name, call, series, n, m_min, m_max, m_step, excl, budget, precision="fp64", **more):
    return dict(name=name, call=call, series=series, n=n, m_min=m_min, m_max=m_max, m_step=m_step,
                excl=excl, k=20, budget=budget, precision=precision, **more)


def listed():
    return [
        # the smallest request of the tests: a random walk with planted pairs
        _case("walk4k", "device", "walk", 4000, 32, 82, 1, 64, 16),
        # a small series from code that may not allocate (the library's own scratch)
        _case("ecg5k_noalloc", "noalloc", "ecg", 5000, 100, 400, 6, 100, 16),
        # the one-shot call on a host series, a ragged size of the serving mix
        _case("wafer30k_host", "host", "wafer", 30011, 23, 61, 1, 23, 16),
        # short windows over a noisy series, in the FP32 form, as served
        _case("ecg50k_short_fp32", "device", "ecg", 50021, 24, 67, 1, 24, 16, "fp32"),
        # the longest windows of the serving mix, BF16 keys
        _case("wafer40k_long_bf16", "device", "wafer", 40009, 480, 520, 1, 480, 16, "bf16"),
        # the ordinary request: Wafer-like, 51 lengths
        _case("wafer100k", "device", "wafer", 100000, 50, 100, 1, 50, 8),
        # a noisy series where the threshold join does most of the work
        _case("ecg250k_fp32", "device", "ecg", 250000, 100, 400, 6, 100, 8, "fp32"),
        # the benchmark's two workloads at full size, in the plain form
        _case("ecg1m", "device", "ecg", 1000000, 100, 400, 6, 100, 8),
        _case("wafer5m", "device", "wafer", 5000000, 50, 100, 1, 50, 8),
        # stream sessions: samples ingested in batches of `excl`, then the one-pass answer
        _case("stream_ecg100k", "stream", "ecg", 100000, 100, 400, 6, 100, 16),
        _case("stream_wafer100k", "stream", "wafer", 100000, 50, 100, 1, 50, 16),
        # eight requests of the serving mix at once, on four slots
        _case("server_mix8", "server", "mix", 40000, 16, 512, 1, 16, 16, requests=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["device"] * 8 + ["noalloc", "host", "stream", "server"])
    series = rng.choice(["wafer", "ecg", "ecg", "walk"])
    precision = rng.choice(["fp64", "fp64", "fp32", "bf16"])
    budget = rng.choice([8, 16])
    if call == "server":
        c = _case("", call, "mix", _log_int(rng, 12000, 60000), 16, 512, 1, 16, budget, precision,
                  requests=rng.randint(4, 10))
    elif call == "stream":
        series = rng.choice(["wafer", "ecg"])
        m_min = rng.randint(32, 120)
        span = rng.randint(16, 64)
        c = _case("", call, series, _log_int(rng, 8000, 120000), m_min, m_min + span,
                  rng.choice([1, 2]), rng.randint(m_min // 2, m_min), budget)
    else:
        m_min = rng.randint(16, 512)
        m_step = rng.choice([1, 1, 1, 6])
        span = rng.randint(8, 64) * m_step
        lengths = len(range(m_min, m_min + span, m_step))
        if call == "noalloc":
            n = rng.randint(3000, max(3001, min(12000, 380000 // lengths)))
        elif series == "wafer":
            n = _log_int(rng, 10000, 2000000)
        else:
            n = _log_int(rng, 4000, 150000)
        n = max(n, 4 * (m_min + span))
        if call == "noalloc":
            n = min(n, 380000 // lengths)
        c = _case("", call, series, n, m_min, m_min + span - 1, m_step, m_min, budget, precision)
    del c["name"]
    return c


def _series(kind, n, seed):
    if kind == "walk":
        return synth.random_walk_planted(n, seed=seed)[0]
    return synth.wafer_like(n, seed) if kind == "wafer" else synth.ecg_like(n, seed)


def _requests(case, seed):
    """The server's batch: (series, m_min, m_max) with lengths as in the serving mix."""
    rng = np.random.Generator(np.random.PCG64(seed))
    shape = np.random.Generator(np.random.PCG64(case["n"]))      # the sizes are the case's own
    out = []
    for x in range(case["requests"]):
        n = int(round(math.exp(shape.uniform(math.log(8000), math.log(case["n"])))))
        m_min = int(shape.integers(case["m_min"], case["m_max"] + 1))
        span = int(shape.integers(8, 65))
        out.append((_series("ecg" if x % 2 else "wafer", n, int(rng.integers(1 << 30))), m_min,
                    m_min + span - 1))
    return out


def _options(case):
    return pmp.options(m_step=case["m_step"], precision=PRECISION[case["precision"]])


# one workspace and one server per process, as a program keeps them
_workspace = pmp.Workspace(DEVICE)
_server = None


def prepare(case, seed):
    global _server
    s = dict(case, opts=_options(case))
    if case["call"] == "server":
        if _server is None:
            _server = pmp.Server(0, SERVER_BYTES, SERVER_SLOTS)
        s["batch"] = _requests(case, seed)
        return s
    t = _series(case["series"], case["n"], seed)
    if case["call"] in ("device", "noalloc"):
        s["t"] = torch.from_numpy(t).to(DEVICE)
    else:
        s["t"] = t
    if case["call"] == "device":
        _workspace.get(pmp.workspace_bytes(case["n"], case["m_min"], case["m_max"], case["k"],
                                           s["opts"]))
    return s


def _outputs(motifs):
    return {"i": np.array([x.i for x in motifs], dtype=np.int64),
            "j": np.array([x.j for x in motifs], dtype=np.int64),
            "m": np.array([x.m for x in motifs], dtype=np.int64),
            "dist": np.array([x.dist for x in motifs], dtype=np.float64)}


def run(s):
    call, args = s["call"], (s["m_min"], s["m_max"], s["k"], s["excl"], s["budget"])
    if call == "device":
        return _outputs(pmp.run_device(s["t"], *args, opts=s["opts"], workspace=_workspace)[0])
    if call == "noalloc":
        return _outputs(pmp.run_device_noalloc(s["t"], *args, opts=s["opts"])[0])
    if call == "host":
        return _outputs(pmp.open_host(s["t"], *args, opts=s["opts"]))
    if call == "server":
        ids = [_server.submit(t, lo, hi, s["k"], lo, s["budget"], s["opts"])
               for t, lo, hi in s["batch"]]
        return [_outputs(_server.wait(x)[0]) for x in ids]
    with pmp.Stream(s["n"], *args, opts=s["opts"]) as st:
        for x in range(0, s["n"], APPEND):
            st.append(s["t"][x:x + APPEND])
        st.flush()
        rows = [st.profile(a) for a in range(st.info()["anchors"])]
        return {"top": _outputs(st.topk()), "P": np.concatenate([p for p, _ in rows]),
                "I": np.concatenate([i for _, i in rows])}


def _lengths(case):
    return list(range(case["m_min"], case["m_max"] + 1, case["m_step"]))


def _shapes(case):
    """(samples, lengths) of each series of a call."""
    if case["call"] == "server":
        return [(len(t), list(range(lo, hi + 1))) for t, lo, hi in _requests(case, 0)]
    ms = _lengths(case)
    if case["call"] == "stream":
        ms = [m for x, m in enumerate(ms) if x % 16 == 0 or x == len(ms) - 1]
    return [(case["n"], ms)]


def work(case):
    """The samples in, the answer out; every window's moments (8 operations by
    running sums) and its 15 spectral bins (10 operations each by the slide)."""
    cells = sum(n - m + 1 for n, ms in _shapes(case) for m in ms)
    nbytes = sum(8 * n + 32 * case["k"] for n, _ in _shapes(case))
    if case["call"] == "stream":
        nbytes += 16 * cells
    return {"bytes": nbytes, "flops": 158 * cells}


def _row_minima(t, m, excl, keep):
    """The `keep` smallest row minima of one length, as (distance, start)."""
    x = t.unfold(0, m, 1)
    live = (x != x[:, :1]).any(1)
    z = x - x.mean(1, keepdim=True)
    z = z / torch.where(live, (z * z).mean(1).sqrt(), torch.ones_like(z[:, 0]))[:, None]
    w = z.shape[0]
    best = torch.full((w,), math.inf, dtype=torch.float64, device=t.device)
    arg = torch.zeros(w, dtype=torch.int64, device=t.device)
    step = max(1, (1 << 27) // w)
    dead = ~live
    for a in range(0, w, step):
        b = min(w, a + step)
        d2 = torch.mm(z[a:b], z.t()).mul_(-2.0).add_(2.0 * m)
        d2[:, dead] = math.inf
        lo, hi = max(0, a - excl), min(w, b + excl)
        near = (torch.arange(a, b, device=t.device)[:, None]
                - torch.arange(lo, hi, device=t.device)[None, :]).abs() < excl
        d2[:, lo:hi][near] = math.inf
        best[a:b], arg[a:b] = d2.min(1)
    best[dead] = math.inf
    start = torch.topk(best, min(keep, w), largest=False).indices
    start = start[torch.isfinite(best[start])]
    # the distances themselves without the cancellation of the product form
    d = (z[start] - z[arg[start]]).square().sum(1).sqrt()
    d = torch.where(d < 1e-6, torch.zeros_like(d), d)
    return d.cpu().numpy(), start.cpu().numpy()


def _exact_topk(t, ms, excl, k):
    t = torch.from_numpy(t).to(DEVICE)
    cells = []
    for m in ms:
        d, i = _row_minima(t, m, excl, k * (m + 1))
        cells += [(float(x), m, int(y)) for x, y in zip(d, i)]
    taken = []
    for d, m, i in sorted(cells):
        if not any(q == m and 2 * abs(p - i) <= m for _, q, p in taken):
            taken.append((d, m, i))
            if len(taken) == k:
                break
    return {"i": None, "j": None, "m": None,
            "dist": np.array([d for d, _, _ in taken], dtype=np.float64)}


def exact(case, seed):
    # a stream's profile depends on the candidates that its keys choose
    if case["call"] == "stream" or sum(2.0 * n * n * m for n, ms in _shapes(case)
                                       for m in ms) > EXACT_FLOPS:
        return None
    if case["call"] == "server":
        return [_exact_topk(t, range(lo, hi + 1), lo, case["k"])
                for t, lo, hi in _requests(case, seed)]
    t = _series(case["series"], case["n"], seed)
    return _exact_topk(t, _lengths(case), case["excl"], case["k"])
