"""Work that a program using this library has it do, for timing.

``listed()`` names the cases and ``draw(rng)`` makes more of the same ranges. ``prepare(case, seed)`` builds what a
program holds before a call (frames in device memory, a plan, batch or server, output buffers), ``run(state)`` is one
pass through the public entry points, ``work(case)`` the bytes and integer operations a pass cannot do without, and
``exact(case, seed)`` the floating results of the first pass in 64 bits, from plain torch.

Kinds of case:
  plan     one call of a ``Plan`` on a frame [T][F][N] (``compute_into``, continuing the running normaliser), the
           stream of one array; ``entry`` "fresh" lets the call allocate its outputs (``compute``)
  noalloc  ``compute_noalloc`` (fresh normaliser, no plan) and ``channel_stats`` over its values
  batch    one call of a ``Batch`` of many uneven problems
  server   frames of two arrays submitted to a ``Server`` in turn, until all are done
  mc       ``calibrate_mc``, the threshold simulation
"""
import math
import random

import numpy as np
import torch

import paper_1808_10365_amd as sk

WANT = {"sums": sk.DEFAULT_OUTPUTS, "all": sk.ALL_OUTPUTS, "flags": ("v", "flags")}
FLOATS = ("v", "sk_i", "significance")
BATCH_WANT = ("s1", "s2", "v", "flags", "n_eff")
ITEM = {"s1": 4, "s2": 4, "r1": 8, "r2": 8, "v": 4, "flags": 1, "n_eff": 4, "sk_i": 4, "significance": 4}
OPS_PER_SAMPLE = 7      # the paper's count for the multi-receiver estimate, (7n + 2)N + 6 per n N samples
OPS_PER_DRAW = 40       # simulated sample: one 64-bit mixing function, two quantised components, power, two sums
EST = {"hat": sk.EST_HAT, "tilde": sk.EST_TILDE}


def _plan(name, N, F, T, M, L, est="hat", mask=False, want="sums", entry="into"):
    c = dict(kind="plan", inputs=N, channels=F, samples=T, block=M, window=L, est=est, mask=mask, want=want, entry=entry)
    return dict(c, name=name) if name else c


def _noalloc(name, N, F, T, M, L, est, mask, want):
    c = dict(kind="noalloc", inputs=N, channels=F, samples=T, block=M, window=L, est=est, mask=mask, want=want)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: 16 inputs, one channel, 64 KiB a call. Latency and launches.
        _plan("tiny", 16, 1, 4096, 256, 4),
        # One frame of the smaller serving array (48 MiB), shorter than its window of 256 blocks.
        _plan("frame256", 256, 4, 49152, 256, 256),
        # One frame of the larger serving array (384 MiB).
        _plan("frame2048", 2048, 4, 49152, 256, 256),
        # The Pathfinder: 256 inputs, 8 channels a GPU (256 MiB a call).
        _plan("pathfinder", 256, 8, 1 << 17, 256, 256),
        # CHIME: 2048 inputs, 4 channels, 2 GiB a call, blocks of 256 samples as deployed.
        _plan("chime256", 2048, 4, 1 << 18, 256, 256),
        # The same array with four times longer blocks.
        _plan("chime1024", 2048, 4, 1 << 18, 1024, 64),
        # An array whose input count is a multiple of 4 and not of 16 (some correlator inputs not connected).
        _plan("inputs1000", 1000, 3, 1 << 15, 256, 16),
        # An odd input count and a block length that is no power of two; a caller that lets the call allocate.
        _plan("inputs509", 509, 5, 25600, 100, 7, entry="fresh"),
        # The paper's deployed form (rescaled, own-block mean) in a loop that may not allocate, dead inputs masked,
        # every output exported, then the common-mode diagnostic over the call's values.
        _noalloc("masked_export", 1024, 4, 1 << 16, 256, 1, "tilde", True, "all"),
        # Many uneven streams in one call.
        dict(kind="batch", name="batch12", problems=12, shapes=4, most=1 << 17),
        # Two arrays served together, four frames each, from submit until all are done.
        dict(kind="server", name="server", small=256, large=2048, channels=4, samples=49152, block=256, window=256,
             frames=4),
        # Threshold calibration for a 16-input array: 2^18 simulated estimates.
        dict(kind="mc", name="calibrate", inputs=16, block=256, sims=1 << 18, est="tilde", sigma=2.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _inputs(rng):
    """Input counts: multiples of 16 mostly, then multiples of 4, then any."""
    n = _log(rng, 16, 4096)
    k = rng.random()
    return max(16, n // 16 * 16) if k < 0.55 else max(4, n // 4 * 4) if k < 0.75 else n


def _shape(rng, most_bytes):
    N, F = _inputs(rng), rng.choice([1, 1, 2, 3, 4, 5, 8])
    M = rng.choice([64, 128, 256, 256, 512, 1024]) if rng.random() < 0.7 else _log(rng, 30, 1200)
    B = max(1, _log(rng, 1 << 17, most_bytes) // (N * F * M))
    return N, F, M, B


def draw(rng):
    k = rng.random()
    if k < 0.7:
        N, F, M, B = _shape(rng, 1 << 30)
        L = rng.choice([0, 1, 2, 4, 7, 16, 64, (1 << 16) // M, (1 << 16) // M, max(1, (1 << 16) // M)])
        est = "tilde" if L == 1 and rng.random() < 0.6 else "hat"
        return _plan("", N, F, M * B, M, L, est, rng.random() < 0.25, rng.choice(["sums", "sums", "all", "flags"]),
                     rng.choice(["into", "into", "fresh"]))
    if k < 0.8:
        N, F, M, B = _shape(rng, 1 << 28)
        return _noalloc("", N, F, M * B, M, rng.choice([0, 1, 1]), "hat", rng.random() < 0.5,
                        rng.choice(["sums", "all"]))
    if k < 0.88:
        return dict(kind="batch", problems=rng.randint(3, 12), shapes=rng.randint(10, 10 ** 6), most=_log(rng, 4096, 1 << 16))
    if k < 0.94:
        M = rng.choice([128, 256, 512])
        return dict(kind="server", small=16 * _log(rng, 2, 20), large=16 * _log(rng, 32, 128), channels=rng.choice([1, 2, 4]),
                    samples=M * _log(rng, 16, 49152 // M), block=M, window=(1 << 16) // M, frames=rng.randint(2, 4))
    M = rng.choice([64, 128, 256, 500])
    return dict(kind="mc", inputs=_log(rng, 1, 64), block=M, sims=_log(rng, 1 << 10, 1 << 15),
                est=rng.choice(["tilde", "hat"]), sigma=round(rng.uniform(1.3, 3.0), 3))


# ---------------------------------------------------------------------------------------------------- inputs

def _problems(case):
    """(N, F, T, M, L) of each problem of a batch."""
    r = random.Random(case["shapes"])
    out = []
    for _ in range(case["problems"]):
        N, M, F = r.choice([64, 256, 1024, 2048]), r.choice([64, 256, 1024]), r.choice([1, 4, 8])
        out.append((N, F, M * r.randint(1, max(1, case["most"] // M)), M, (1 << 16) // M))
    return out


def _frame(T, F, N, gen, sigma):
    """[T][F][N] bytes on the GPU: each input's components Gaussian of its own RMS, rounded and bounded to [-7, 7];
    in a twentieth of the cells of 256 samples of a channel, interference doubles the RMS."""
    x = torch.empty((T, F, N), dtype=torch.uint8, device="cuda")
    gain = 1.0 + (torch.rand(((T + 255) // 256, F, 1), generator=gen, device="cuda") < 0.05).float()
    rows = max(256, (1 << 25) // (F * N) // 256 * 256)
    for t in range(0, T, rows):
        n = min(rows, T - t)
        z = torch.randn((2, n, F, N), generator=gen, device="cuda")
        z *= sigma
        z *= gain[t // 256:(t + n + 255) // 256].repeat_interleave(256, 0)[:n]
        z.round_().clamp_(-7, 7).add_(8)
        x[t:t + n] = (z[0] * 16 + z[1]).to(torch.uint8)
    return x


def _gen(seed, k=0):
    return torch.Generator(device="cuda").manual_seed(seed * 1000003 + k)


def _sigma(N, gen):
    return 1.5 + 2.0 * torch.rand(N, generator=gen, device="cuda")


def _stream(case, seed):
    """Frame, mask and flag parameters of a plan or noalloc case."""
    T, F, N = case["samples"], case["channels"], case["inputs"]
    gen = _gen(seed)
    sigma = _sigma(N, gen)
    x = _frame(T, F, N, gen, sigma)
    mask = (torch.rand((F, N), generator=gen, device="cuda") > 0.05).to(torch.uint8) if case["mask"] else None
    delta, spread = sk.digitised_expectation(sigma.cpu().numpy().astype(np.float64), case["block"])
    return x, mask, delta, spread


def _outputs(F, B, N, want):
    kinds = {"s1": torch.int32, "s2": torch.int32, "r1": torch.int64, "r2": torch.int64, "v": torch.float32,
             "flags": torch.uint8, "n_eff": torch.int32, "sk_i": torch.float32, "significance": torch.float32}
    return sk.Result(**{k: torch.empty((F, B, N) if k in ("s1", "s2", "sk_i") else (F, B), dtype=t, device="cuda")
                        if k in want else None for k, t in kinds.items()})


def _server_arrays(case):
    base = dict(n_channels=case["channels"], n_samples=case["samples"], block_len=case["block"],
                norm_window=case["window"])
    return [dict(base, n_inputs=case["small"]), dict(base, n_inputs=case["large"])]


def _server_frames(case, seed):
    frames = []
    for a, kw in enumerate(_server_arrays(case)):
        gen = _gen(seed, a)
        sigma = _sigma(kw["n_inputs"], gen)
        frames.append([_frame(kw["n_samples"], kw["n_channels"], kw["n_inputs"], gen, sigma)
                       for _ in range(case["frames"])])
    return frames


def _batch_inputs(case, seed):
    xs = []
    for j, (N, F, T, M, L) in enumerate(_problems(case)):
        gen = _gen(seed, j)
        sigma = _sigma(N, gen)
        xs.append(_frame(T, F, N, gen, sigma))
    return xs


# ------------------------------------------------------------------------------------------------- the passes

def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind in ("plan", "noalloc"):
        x, mask, delta, spread = _stream(case, seed)
        st.update(x=x, mask=mask)
        N, F, T, M = case["inputs"], case["channels"], case["samples"], case["block"]
        if kind == "plan":
            st["plan"] = sk.Plan(N, F, T, M, norm_window=case["window"], estimator=EST[case["est"]], k_sigma=5.0,
                                 expect_offset=delta, sigma_override=spread)
            st["out"] = st["plan"].alloc_outputs(x.device, WANT[case["want"]]) if case["entry"] == "into" else None
        else:
            st["out"] = _outputs(F, T // M, N, WANT[case["want"]])
            st["kw"] = dict(block_len=M, norm_window=case["window"], estimator=EST[case["est"]], k_sigma=5.0,
                            expect_offset=delta, sigma_override=spread)
    elif kind == "batch":
        plans = [dict(n_inputs=N, n_channels=F, n_samples=T, block_len=M, norm_window=L)
                 for N, F, T, M, L in _problems(case)]
        st["batch"] = sk.Batch(plans, _batch_inputs(case, seed), want=BATCH_WANT)
    elif kind == "server":
        st["frames"] = _server_frames(case, seed)
        st["server"] = sk.Server(8 << 30, max_inflight=12, n_streams=4)
        ids = [st["server"].add_array(**kw) for kw in _server_arrays(case)]
        st["outs"] = [[st["server"].alloc_outputs(a, "cuda", BATCH_WANT) for _ in f] for a, f in zip(ids, st["frames"])]
        st["ids"] = ids
        torch.cuda.synchronize()
    else:
        st["seed"] = seed
    return st


def _named(out, want):
    return {k: getattr(out, k) for k in want}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "plan":
        want = WANT[case["want"]]
        if case["entry"] == "into":
            return _named(state["plan"].compute_into(state["x"], state["out"], mask=state["mask"]), want)
        return _named(state["plan"].compute(state["x"], mask=state["mask"], want=want), want)
    if kind == "noalloc":
        out = sk.compute_noalloc(state["x"], state["out"], mask=state["mask"], **state["kw"])
        mean, var, n_eff, count = sk.channel_stats(out.v, case["block"])
        return dict(_named(out, WANT[case["want"]]), channels=[mean, var, n_eff, count])
    if kind == "batch":
        return [_named(r, BATCH_WANT) for r in state["batch"].compute()]
    if kind == "server":
        server, tickets = state["server"], []
        for k in range(case["frames"]):
            for a, frames, outs in zip(state["ids"], state["frames"], state["outs"]):
                tickets.append(server.submit(a, frames[k], outs[k]))
        server.drain()
        for t in tickets:
            server.poll(t)
        return [[_named(r, BATCH_WANT) for r in outs] for outs in state["outs"]]
    moments, values = sk.calibrate_mc(case["inputs"], case["block"], case["sigma"], case["sims"], state["seed"],
                                      estimator=EST[case["est"]], return_values=True)
    return dict(moments=moments, values=values)


# ------------------------------------------------------------------------------------------------- work

def _call_work(N, F, T, M, L, want, mask=False):
    B = T // M
    out = sum(ITEM[k] * F * B * (N if k in ("s1", "s2", "sk_i") else 1) for k in want)
    state = 2 * 4 * F * N * min(B, max(L - 1, 0))        # window blocks handed from call to call
    return N * F * T + out + state + (F * N if mask else 0), OPS_PER_SAMPLE * N * F * T


def work(case):
    kind = case["kind"]
    if kind in ("plan", "noalloc"):
        L = case["window"] if kind == "plan" else 0
        w = [_call_work(case["inputs"], case["channels"], case["samples"], case["block"], L, WANT[case["want"]],
                        case["mask"])]
    elif kind == "batch":
        w = [_call_work(N, F, T, M, L, BATCH_WANT) for N, F, T, M, L in _problems(case)]
    elif kind == "server":
        w = [_call_work(kw["n_inputs"], kw["n_channels"], kw["n_samples"], kw["block_len"], kw["norm_window"],
                        BATCH_WANT) for kw in _server_arrays(case)] * case["frames"]
    else:
        w = [(8 * case["sims"], OPS_PER_DRAW * case["sims"] * case["inputs"] * case["block"])]
    return {"bytes": sum(b for b, _ in w), "flops": sum(f for _, f in w)}


# ------------------------------------------------------------------------------------------------- 64-bit results

def _sums(x, M):
    """S1, S2 [F][B][N] (int64) of a frame."""
    T, F, N = x.shape
    B = T // M
    s1 = torch.empty((B, F, N), dtype=torch.int64, device=x.device)
    s2 = torch.empty_like(s1)
    step = max(1, (1 << 26) // (M * F * N))
    for b in range(0, B, step):
        n = min(step, B - b)
        y = x[b * M:(b + n) * M].view(n, M, F, N)
        re, im = (y >> 4).to(torch.int32) - 8, (y & 15).to(torch.int32) - 8
        p = re * re + im * im
        s1[b:b + n] = p.sum(1, dtype=torch.int64)
        s2[b:b + n] = (p * p).sum(1, dtype=torch.int64)
    return s1.permute(1, 0, 2), s2.permute(1, 0, 2)


def _values(s1, s2, M, L, est, mask=None, delta=0.0, spread=0.0, want=()):
    """The floating outputs of a call, in 64 bits, for sums [F][B'][N] of the blocks since the normaliser began."""
    F, B, N = s1.shape
    if L == 0:
        P = s1
    else:
        c = torch.nn.functional.pad(s1.cumsum(1), (0, 0, 1, 0))
        at = torch.arange(1, B + 1, device=s1.device)
        P = c[:, 1:] - c[:, (at - L).clamp(min=0)]
    inc = P > 0
    if mask is not None:
        inc = inc & (mask != 0)[:, None, :]
    n = inc.sum(2).double()
    K = n * M
    zero = torch.zeros((), dtype=torch.float64, device=s1.device)
    if L == 0:
        r1, r2 = (torch.where(inc, s, 0).sum(2).double() for s in (s1, s2))
        V = (K + 1) / (K - 1) * (K * r2 / (r1 * r1) - 1)
        bad = (K < 2) | (r1 == 0)
    else:
        w = torch.where(inc, 1.0 / P.clamp(min=1).double(), zero)
        A = (s1.double() * w).sum(2)
        Q = (s2.double() * w * w).sum(2)
        V = (M + 1) / (M - 1) * (M * Q / n - 1) if est == "tilde" else (K + 1) / (K - 1) * (K * Q / (A * A) - 1)
        bad = (K < 2) | (A == 0)
    V = torch.where(bad, math.nan, V)
    got = {"v": V}
    if "sk_i" in want:
        a, b = s1.double(), s2.double()
        got["sk_i"] = torch.where(s1 == 0, math.nan, (M + 1) / (M - 1) * (M * b / (a * a) - 1))
    if "significance" in want:
        e0 = ((K + 1) * (M - 1)) / ((K - 1) * (M + 1)) if est == "hat" and L == 1 else 1.0
        got["significance"] = (V - (e0 + delta)) / (spread if spread > 0 else torch.sqrt(4.0 / K))
    return {k: got.get(k) for k in want}


def _mix(z):
    """The output function of SplitMix64 on int64 (wrapping)."""
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * (0xBF58476D1CE4E5B9 - (1 << 64))
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * (0x94D049BB133111EB - (1 << 64))
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _exact_mc(case, seed):
    N, M, S, clip = case["inputs"], case["block"], case["sims"], 7
    thr = [min(max(math.floor(0.5 * math.erfc(-((k - clip + 0.5) / case["sigma"]) / math.sqrt(2.0)) * 4294967296.0), 0), 4294967295)
           for k in range(2 * clip)]
    thr = torch.tensor(thr, dtype=torch.int64, device="cuda")
    key = int(_mix(torch.tensor([seed], dtype=torch.int64))[0])
    gold = 0x9E3779B97F4A7C15 - (1 << 64)
    values = torch.empty(S, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 25) // (N * M))
    for s in range(0, S, step):
        n = min(step, S - s)
        at = torch.arange(s * N * M + 1, (s + n) * N * M + 1, dtype=torch.int64, device="cuda")
        r = _mix(at * gold + key)
        re = torch.bucketize((r >> 32) & 0xFFFFFFFF, thr, right=True) - clip
        im = torch.bucketize(r & 0xFFFFFFFF, thr, right=True) - clip
        p = (re * re + im * im).view(n, N, M)
        s1, s2 = p.sum(2).double(), (p * p).sum(2).double()
        live = s1 > 0
        q = torch.where(live, s2 / (s1 * s1), torch.zeros_like(s1)).sum(1)
        m = live.sum(1).double()
        K = m * M
        V = (M + 1) / (M - 1) * (M * q / m - 1) if case["est"] == "tilde" else (K + 1) / (K - 1) * (K * q / (m * m) - 1)
        values[s:s + n] = torch.where(K >= 2, V, math.nan)
    v = values[~values.isnan()]
    e = v - v.mean()
    m2, m3, m4 = (float((e ** k).mean()) for k in (2, 3, 4))
    moments = [float(v.mean()), m2 * len(v) / (len(v) - 1), m3 / m2 ** 1.5, m4 / m2 ** 2 - 3.0]
    return dict(moments=np.array(moments), values=values)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("plan", "noalloc"):
        x, mask, delta, spread = _stream(case, seed)
        s1, s2 = _sums(x, case["block"])
        want = WANT[case["want"]]
        got = _values(s1, s2, case["block"], case["window"], case["est"], mask, delta, spread, want)
        if kind == "plan":
            return got
        v = got["v"].float().double()          # the diagnostic is over the call's own values
        cnt = (~v.isnan()).sum(1)
        mean = torch.nanmean(v, 1)
        var = torch.nansum((v - mean[:, None]) ** 2, 1) / (cnt - 1)
        return dict(got, channels=[mean, var, 4.0 / (case["block"] * var), None])
    if kind == "batch":
        got = []
        for (N, F, T, M, L), x in zip(_problems(case), _batch_inputs(case, seed)):
            s1, s2 = _sums(x, M)
            got.append(_values(s1, s2, M, L, "hat", want=BATCH_WANT))
        return got
    if kind == "server":
        got, B = [], case["samples"] // case["block"]
        for frames in _server_frames(case, seed):
            sums = [_sums(x, case["block"]) for x in frames]
            s1, s2 = (torch.cat([s[k] for s in sums], 1) for k in (0, 1))
            v = _values(s1, s2, case["block"], case["window"], "hat", want=("v",))["v"]
            got.append([dict({k: None for k in BATCH_WANT}, v=v[:, k * B:(k + 1) * B]) for k in range(case["frames"])])
        return got
    return _exact_mc(case, seed)
