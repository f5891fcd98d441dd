"""Measured workloads of the sampler: what a program that uses it does, from
one small trace to the largest that it is built for.

Every trace is synthetic and made on the GPU from the seed alone, with the
statistics of the recipes in ``tracegen/`` (the C generators there would take
seconds per preparation):

* ``mix``: 55 % allocations with log-uniform sizes in [16 B, 1 MiB], 45 % frees
  of a uniformly chosen live object (an object allocated at event s is still
  live at event t with probability (s/t)^4.5), a few never freed, Zipf lines,
  70 % Python; optionally copy events (log-uniform bytes) and timer events
  (exponential delay, mean 50 us) among them.
* ``life``: 95 % small Python objects of 16 k bytes, 5 % native arrays of
  1-256 MiB, exponential lifetimes with a mean of 1e4 events, Zipf lines.

A case names its path: ``profile`` (one trace through Sampler.profile, the
whole profile on the host), ``fetch`` (the same through the C calls, into
page-locked arrays that the program keeps), ``resident`` (one trace already
in GPU memory, its samples and per-line arrays kept there), ``batch`` (many
traces in one launch, some profiles fetched, the others released with their
counts),
``served`` (a burst of requests in pinned host memory through serve.serve) and
``rate`` (the rate-based sampler).  Launch parameters, timing events and
options are the library's defaults unless the case says otherwise.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

import paper_2212_07597_amd as smp
from paper_2212_07597_amd import serve

KiB, MiB = 1 << 10, 1 << 20
DEV = "cuda"


def _case(name, path, mix, n, lines, T, **kw):
    c = {"name": name, "path": path, "mix": mix, "n": n, "lines": lines, "T": T, "Tc": T, "zipf": 1.1, "leak": 0.01,
         "copy": 0.0, "timer": 0.0, "options": 0, "source": "device", "traces": 1, "shape_seed": 0}
    c.update(kw)
    return c


def listed():
    return [
        # The shortest trace of a batch workload, alone: nothing but launches, latencies and the copy out.
        _case("profile_1k", "profile", "mix", 1_000, 1_000, 256 * KiB),
        # A short program's trace, recorded on the host and profiled with one call.
        _case("profile_100k_host", "profile", "mix", 100_000, 64, MiB, source="host"),
        # A ragged trace with every option in use: copy and timer events, a prime threshold, a copy threshold that
        # is no power of two and differs from T, and the last tracked object resolved at the end of the trace.
        _case("profile_777k_options", "profile", "mix", 777_777, 1_003, 3 * MiB + 1, Tc=5_000_011, copy=0.1, timer=0.01,
              options=smp.OPT_PRIME_T | smp.OPT_RESOLVE_AT_END),
        # A burst of requests at a profiling service: log-normal lengths (median 5e4 events), in pinned host memory,
        # each answered with its whole profile.
        _case("served_burst_32", "served", "mix", 50_000, 64, MiB, source="pinned", traces=32, shape_seed=4),
        # A fleet's traces in one launch: 1,024 of them, 1e3 to 1e6 events each (about 1.5e8), three thresholds.
        _case("batch_1024", "batch", "mix", 31_623, 1_000, MiB, traces=1024, shape_seed=3),
        # A long-running program with objects and arrays, its whole profile fetched into page-locked memory.
        _case("fetch_10m_life", "fetch", "life", 10_000_000, 10_000, 10 * MiB, zipf=1.2, leak=0.001),
        # The headline workload: 1e8 events in GPU memory, results kept there.
        _case("resident_100m_life", "resident", "life", 100_000_000, 10_000, 10 * MiB, zipf=1.2, leak=0.001),
        # A program that copies and computes, with a threshold far above what a few hundred events move.
        _case("fetch_20m_copy_timer", "fetch", "mix", 20_000_000, 100_000, 64 * MiB, zipf=1.05, leak=0.0001, copy=0.1,
              timer=0.01),
        # The longest trace: 5e8 events with copies and timers over 1e6 lines.
        _case("resident_500m_copy_timer", "resident", "mix", 500_000_000, 1_000_000, 64 * MiB, zipf=1.05, leak=0.0001,
              copy=0.1, timer=0.01),
        # The rate-based sampler beside it, on a short trace (caller that may not allocate) ...
        _case("rate_100k_noalloc", "rate", "mix", 100_000, 64, MiB, noalloc=True),
        # ... and on the headline trace.
        _case("rate_100m_life", "rate", "life", 100_000_000, 10_000, 10 * MiB, zipf=1.2, leak=0.001),
    ]


def _log_uniform(rng, lo, hi):
    return int(lo * (hi / lo) ** rng.random())


def draw(rng):
    path = rng.choice(["profile", "profile", "fetch", "resident", "resident", "batch", "served", "rate"])
    mix = rng.choice(["mix", "mix", "life"])
    lines = _log_uniform(rng, 64, 200_000)
    T = rng.choice([256 * KiB, MiB, 10 * MiB, 64 * MiB, _log_uniform(rng, 128 * KiB, 128 * MiB) | 1])
    kw = {"zipf": rng.choice([1.05, 1.1, 1.2]), "leak": rng.choice([0.01, 0.001, 0.0001]), "shape_seed": rng.randrange(1 << 20)}
    if mix == "mix" and path != "rate" and rng.random() < 0.4:
        kw.update(copy=0.1, timer=0.01, Tc=rng.choice([T, _log_uniform(rng, MiB, 64 * MiB)]))
    if path == "profile":
        n = _log_uniform(rng, 500, 2_000_000)
        kw["source"] = rng.choice(["host", "pinned", "device"])
        kw["options"] = rng.randrange(4)
    elif path == "fetch":
        n = _log_uniform(rng, 500_000, 20_000_000)
        T = max(T, 10 * MiB)
        kw["options"] = rng.randrange(4)
    elif path == "resident":
        n = _log_uniform(rng, 100_000, 150_000_000)
    elif path == "batch":
        n, kw["traces"] = _log_uniform(rng, 5_000, 60_000), rng.randrange(40, 700)
        lines = _log_uniform(rng, 64, 2_000)
    elif path == "served":
        n, kw["traces"], kw["source"] = _log_uniform(rng, 5_000, 100_000), rng.randrange(2, 40), "pinned"
        lines = _log_uniform(rng, 64, 2_000)
    else:
        n = _log_uniform(rng, 10_000, 150_000_000)
        kw["noalloc"] = rng.random() < 0.5
    c = _case("", path, mix, n | 1, lines, T, **kw)
    del c["name"]
    return c


# ------------------------------------------------------------------ traces --

def _shapes(case):
    """(events, threshold) of each trace: the seed of the inputs does not
    change how much work a case is."""
    n, k, T = case["n"], case["traces"], case["T"]
    if k == 1:
        return [(n, T)]
    r = np.random.default_rng(case["shape_seed"])
    if case["path"] == "batch":  # log-uniform over three decades around n, three thresholds
        lens = n * 10 ** (3 * (np.arange(k) + r.random(k)) / k - 1.5)
        r.shuffle(lens)
        Ts = r.choice([max(T // 4, 1), T, 10 * T], k)
    else:  # log-normal around n
        lens = np.minimum(np.exp(math.log(n) + 1.5 * r.standard_normal(k)), 20_000_000)
        Ts = np.full(k, T)
    return [(max(int(x), 1), int(t)) for x, t in zip(lens, Ts)]


def _zipf_lines(g, n, lines, s, out):
    """Zipf ranks mapped to ids spread over [0, lines), into out (int64)."""
    w = np.arange(1, lines + 1, dtype=np.float64) ** -s
    cdf = torch.from_numpy(np.cumsum(w) / w.sum()).to(DEV)
    for a in range(0, n, 1 << 26):
        b = min(a + (1 << 26), n)
        rank = torch.searchsorted(cdf, torch.rand(b - a, generator=g, device=DEV, dtype=torch.float64)).clamp_(max=lines - 1)
        out[a:b] = (rank * 7919 + 17) % lines


def _trace(case, n, seed):
    """One trace of n records as a CUDA uint8 tensor.  Objects get an
    allocation time and a free time on an integer clock (4096 ticks per
    event); sorting all times gives the order of the memory events."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)

    def uni(k):
        return torch.rand(k, generator=g, device=DEV, dtype=torch.float64)

    aux = case["copy"] + case["timer"]
    kind = None
    m = n
    if aux:
        u = torch.rand(n, generator=g, device=DEV)
        kind = (u < case["copy"]).to(torch.int8) + 2 * ((u >= case["copy"]) & (u < aux)).to(torch.int8)
        del u
        m = int((kind == 0).sum())
    life = case["mix"] == "life"
    objects = int((0.51 if life else 0.56) * m) + 600
    every = 2.0 if life else 1 / 0.55
    t_alloc = (-torch.log1p(-uni(objects)) * every * 4096).to(torch.int64).add_(1).cumsum_(0)
    if life:
        t_free = t_alloc + (-torch.log1p(-uni(objects)) * 1e4 * 4096).to(torch.int64) + 1
    else:
        t_free = ((t_alloc + 4096) * (1 - uni(objects)) ** (-1 / 4.5)).to(torch.int64) + 1
    t_free[uni(objects) < case["leak"]] = 1 << 62
    order = torch.sort(torch.cat([t_alloc, t_free]), stable=True)[1][:m]
    del t_alloc, t_free
    if life:
        small = uni(objects) < 0.95
        k = (torch.log1p(-uni(objects)) / math.log(0.75)).to(torch.int64).add_(1).clamp_(max=32)
        big = torch.exp2(20 + 8 * uni(objects)).to(torch.int64)
        size, native = torch.where(small, 16 * k, big), ~small
        del small, k, big
    else:
        size = torch.exp2(4 + 16 * uni(objects)).to(torch.int64)
        native = uni(objects) >= 0.7
    obj = order % objects
    size = size[obj]
    size = torch.where(order >= objects, -size, size)
    del order
    rec = torch.empty((n, 3), dtype=torch.int64, device=DEV)
    line = torch.empty(n, dtype=torch.int64, device=DEV)
    _zipf_lines(g, n, case["lines"], case["zipf"], line)
    if kind is None:
        rec[:, 0], rec[:, 1], rec[:, 2] = size, (obj + 1) | (line << 32), native[obj].to(torch.int64)
        return rec.view(-1).view(torch.uint8)
    rec[:, 0] = torch.where(kind == 1, torch.exp2(4 + 16 * uni(n)).to(torch.int64),
                            (-torch.log1p(-uni(n)) * 50 + 0.5).to(torch.int64))
    rec[:, 1] = line << 32
    rec[:, 2] = kind.to(torch.int64) * 2
    at = torch.nonzero(kind == 0).view(-1)
    del kind
    rec[:, 0][at] = size
    rec[:, 1][at] += obj + 1
    rec[:, 2][at] = native[obj].to(torch.int64)
    return rec.view(-1).view(torch.uint8)


def _placed(ev, source):
    if source == "device":
        return ev
    host = ev.cpu()
    return host.pin_memory() if source == "pinned" else host.numpy()


# ------------------------------------------------------------------- cases --

def _room(case, n, T):
    """Rows for the samples of a trace: one per T bytes that its events move
    (mean size of an event of the mix), with a margin."""
    mean = 2.42e6 if case["mix"] == "life" else 94.6e3
    return min(n, int(1.1 * mean * n / T)) + 1024


def prepare(case, seed):
    shapes = _shapes(case)
    traces = [_placed(_trace(case, n, seed * 1_000_003 + i), case["source"]) for i, (n, _) in enumerate(shapes)]
    st = {"case": case, "traces": traces}
    L, path = case["lines"], case["path"]
    if path == "rate":
        if case.get("noalloc"):
            st["counts"] = torch.empty(L, dtype=torch.int64, device=DEV)
            st["result"] = torch.empty(2, dtype=torch.int64, device=DEV)
        else:
            st["ws"] = torch.empty(smp.rate_workspace_bytes(case["n"]), dtype=torch.uint8, device=DEV)
        return st
    st["params"] = [smp.make_params(T, L, case["Tc"] if case["traces"] == 1 else T, 10_000, case["options"])
                    for _, T in shapes]
    on_dev = case["source"] == "device"
    need = sum(smp.workspace_bytes(n, p, ev_on_device=on_dev) + 256 for (n, _), p in zip(shapes, st["params"]))
    st["sampler"] = smp.Sampler(workspace=smp.sampler_fixed_bytes() + need + MiB)
    if path == "batch":
        st["params"] = (smp.Params * len(shapes))(*st["params"])
        shapes = shapes[::FETCHED]
    # where the program keeps its samples and tracked objects
    rows = sum(_room(case, n, T) for n, T in shapes)
    if path == "resident":
        st["samples"] = torch.zeros((rows, 4), dtype=torch.int64, device=DEV)
        st["hist"] = torch.zeros((len(smp.HIST_NAMES), L), dtype=torch.int64, device=DEV)
    elif path == "fetch":
        for name, shape, dtype in (("samples", (rows, 4), torch.int64), ("tracked", (rows, 4), torch.int32),
                                   ("hist", (len(smp.HIST_NAMES), L), torch.int64),
                                   ("leak", (len(smp.LEAK_NAMES), L), torch.int64),
                                   ("gates", (len(smp.GATE_NAMES), L), torch.uint8)):
            st[name] = torch.zeros(shape, dtype=dtype, pin_memory=True).numpy()
    else:
        st["samples"] = np.zeros((rows, 4), dtype=np.int64)
        st["tracked"] = np.zeros((rows, 4), dtype=np.int32)
    return st


FETCHED = 64  # a batch program looks at the whole profile of every 64th trace


def _kept(st, profiles):
    """Profiles field by field, one after another; samples and tracked
    objects in the program's own arrays."""
    out = {k: np.concatenate([np.atleast_1d(p[k]) for p in profiles]) if len(profiles) > 1 else profiles[0][k]
           for k in profiles[0] if k not in ("samples", "tracked")}
    for name, dtype in (("samples", np.int64), ("tracked", np.int32)):
        at = 0
        for p in profiles:
            rows = p[name].view(dtype).reshape(-1, 4)
            st[name][at:at + len(rows)] = rows
            at += len(rows)
        out[name] = st[name]
    return out


def _run_profile(st):
    c = st["case"]
    return _kept(st, [st["sampler"].profile(st["traces"][0], c["T"], c["lines"], c["Tc"], 10_000, c["options"])])


def _run_fetch(st):
    s = st["sampler"]
    tid = s.submit_trace(st["traces"][0], st["params"][0])
    s.run()
    sizes = smp.ProfileSizes()
    out = smp.Profile(*(st[k].ctypes.data for k in ("samples", "tracked", "hist", "leak", "gates")))
    if smp.lib().fetch_profile(s.h, tid, ctypes.byref(sizes), None):
        raise RuntimeError("fetch_profile")
    if sizes.n_samples > len(st["samples"]):
        raise RuntimeError("more samples than the program has room for")
    if smp.lib().fetch_profile(s.h, tid, ctypes.byref(sizes), ctypes.byref(out)):
        raise RuntimeError("fetch_profile")
    return {**{k: st[k] for k in ("samples", "tracked", "hist", "leak", "gates")},
            **{k: getattr(out, k) for k in ("final_F", "peak_F", "peak_sampled_F", "threshold_used", "n_samples",
                                            "n_tracked", "status")}}


def _run_resident(st):
    """Sample the trace, copy its results to the program's own GPU arrays and
    release it."""
    s = st["sampler"]
    tid = s.submit_trace(st["traces"][0], st["params"][0])
    s.run()
    samples, hist, k = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_uint64()
    if smp.lib().trace_device_results(s.h, tid, ctypes.byref(samples), ctypes.byref(hist), ctypes.byref(k)):
        raise RuntimeError("trace_device_results")
    a, b = samples.value - s.ws.data_ptr(), hist.value - s.ws.data_ptr()
    st["samples"][:k.value].copy_(s.ws[a:a + 32 * k.value].view(torch.int64).view(-1, 4))
    st["hist"].copy_(s.ws[b:b + 8 * st["hist"].numel()].view(torch.int64).view(st["hist"].shape))
    count, status = s.release(tid)
    return {"K": count, "status": status, "samples": st["samples"], "hist": st["hist"]}


def _run_batch(st):
    """All traces in one launch; the profiles of a few are fetched, the rest
    answer with their sample counts."""
    s = st["sampler"]
    ids = s.submit_traces(st["traces"], st["params"])
    s.run(blocking=True)
    fetched = ids[::FETCHED]
    profiles = [s.fetch_profile(t) for t in fetched]
    chosen = set(fetched)
    counts = s.release_traces([t for t in ids if t not in chosen])
    return {"counts": np.array(counts, dtype=np.int64), **_kept(st, profiles)}


def _run_served(st):
    reqs = [serve.Request(i, 0, ev, p, ev.numel() // 24) for i, (ev, p) in enumerate(zip(st["traces"], st["params"]))]
    outcomes, _ = serve.serve(st["sampler"], reqs, keep_profiles=True)
    return _kept(st, [outcomes[i].profile for i in range(len(reqs))])


def _run_rate(st):
    c = st["case"]
    if c.get("noalloc"):
        smp.rate_run_noalloc(st["traces"][0], c["T"], c["lines"], st["counts"], st["result"])
        return {"counts": st["counts"], "result": st["result"]}
    counts, result = smp.rate_run(st["traces"][0], c["T"], c["lines"], workspace=st["ws"], sync=False)
    return {"counts": counts, "result": result}


def run(state):
    return {"profile": _run_profile, "fetch": _run_fetch, "resident": _run_resident, "batch": _run_batch, "served": _run_served,
            "rate": _run_rate}[state["case"]["path"]](state)


def work(case):
    """Every record once in; the per-line arrays and an estimate of the
    sample records once out (a few adds and compares per event are no bound)."""
    events = sum(n for n, _ in _shapes(case))
    if case["path"] == "rate":
        return {"bytes": 24 * events + 8 * case["lines"], "flops": 0}
    # measured on both mixes: about one sample per 8 T (life) or 3 T (mix) moved
    per_event = min(1.0, 0.13 * 2.42e6 / case["T"] if case["mix"] == "life" else 0.31 * 94.6e3 / case["T"])
    arrays = 96 if case["path"] == "resident" else 130
    return {"bytes": 24 * events + 32 * per_event * events + arrays * case["lines"] * case["traces"], "flops": 0}


# --------------------------------------------------------- reference values --

def _prime_from(v):
    while v < 2 or any(v % d == 0 for d in range(2, math.isqrt(v) + 1)):
        v += 1
    return v


def _exact_rate(case, seed):
    w = _trace(case, case["n"], seed * 1_000_003).view(torch.int64).view(-1, 3)
    vol = torch.cumsum(w[:, 0].abs(), 0) // case["T"]
    took = torch.diff(vol, prepend=torch.zeros(1, dtype=torch.int64, device=DEV))
    counts = torch.zeros(case["lines"], dtype=torch.int64, device=DEV)
    counts.scatter_add_(0, w[:, 1] >> 32, took)
    return {"counts": counts, "result": torch.stack([vol[-1], torch.zeros_like(vol[-1])])}


def exact(case, seed):
    """The paper's counters, one event after another in Python's integers
    (short single traces; the rate-based sampler at every size)."""
    if case["path"] == "rate":
        return _exact_rate(case, seed)
    if case["path"] != "profile" or case["n"] > 1_000_000:
        return None
    w = _trace(case, case["n"], seed * 1_000_003).view(torch.int64).view(-1, 3).cpu().numpy()
    L, Tc = case["lines"], case["Tc"]
    T = _prime_from(case["T"]) if case["options"] & smp.OPT_PRIME_T else case["T"]
    hist = {k: [0] * L for k in smp.HIST_NAMES}
    samples, tracked = [], []
    F = P = F_at = P_at = peak = peak_s = hwm = copied = 0
    rows = zip(w[:, 0].tolist(), (w[:, 1] & 0xFFFFFFFF).tolist(), (w[:, 1] >> 32).tolist(), w[:, 2].tolist())
    for i, (d, ptr, line, flags) in enumerate(rows):
        if flags >> 1 == 1:
            hist["copy_exact"][line] += d
            hist["copy_sampled"][line] += Tc * ((copied + d) // Tc - copied // Tc)
            copied += d
        elif flags >> 1 == 2:
            hist["py_time_us"][line] += 10_000
            hist["nat_time_us"][line] += d
        else:
            F += d
            P += 0 if flags & 1 else d
            peak = max(peak, F)
            if d < 0 and tracked and tracked[-1][2] == ptr:
                tracked[-1][3] = 1
            if abs(F - F_at) >= T:
                moved, py = F - F_at, P - P_at
                samples.append((i, line, F, py, moved - py))
                hist["py_bytes"][line] += py
                hist["nat_bytes"][line] += moved - py
                which = "growth" if moved > 0 else "shrink"
                hist[which + "_n"][line] += 1
                hist[which + "_bytes"][line] += abs(moved)
                peak_s = max(peak_s, F)
                if moved > 0 and F > hwm:
                    hwm = F
                    tracked.append([i, line, ptr, 0])
                F_at, P_at = F, P
    last = len(tracked) if case["options"] & smp.OPT_RESOLVE_AT_END else len(tracked) - 1
    for k, (_, line, _, freed) in enumerate(tracked):
        hist["leak_mallocs"][line] += 1
        hist["leak_frees"][line] += freed if k < last else 0
    out = {k: np.array(v, dtype=np.int64) for k, v in hist.items()}
    m, f = out["leak_mallocs"], out["leak_frees"]
    seen = m > 0
    for name, num, den in (("lap", m - f + 1, m + 2), ("lit", m - 2 * f + 1, m - f + 2)):
        div = np.gcd(num, den)
        out[name + "_num"] = np.where(seen, num // div, 0)
        out[name + "_den"] = np.where(seen, den // div, 0)
        out[name + "_gate"] = (seen & (20 * num > 19 * den)).astype(np.uint8)
    for name, rows, dtype in (("samples", [(i | line << 32, F, py, nat) for i, line, F, py, nat in samples], np.int64),
                              ("tracked", tracked, np.int32)):
        out[name] = np.zeros((_room(case, case["n"], case["T"]), 4), dtype=dtype)
        out[name][:len(rows)] = np.array(rows, dtype=np.int64).reshape(-1, 4)
    out.update(status=0, K=len(samples), H=len(tracked), final_F=F, peak_F=peak, peak_sampled_F=peak_s, threshold_used=T)
    return out
