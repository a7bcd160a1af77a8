"""What the replay library is timed on: batches of cluster replays as policy studies run them.

A case says how many traces there are, how many subscription-ratio caps each is replayed under, the shape
of the cluster, the policy and the traffic. Traces follow the recipes of ``tracegen`` (same distributions,
same session streams, same order of events), drawn on the GPU so that large batches are quick to make.

``mode`` is the way the library is called:
  keep    the handle exists already (traces in device memory, validated): run, then read the results
  fresh   a new set of traces: create, run, read the results and the bills, destroy
  static  the entry point that allocates nothing, into a result buffer of the caller's
  study   ``sweep.run_policies`` on a host-side batch: upload, the replay under its own policy with bills,
          then the same traces under the Batch baseline
"""
import math

import numpy as np
import torch

from paper_2503_20591_amd import replay, sweep
from paper_2503_20591_amd import tracegen as tg

DEVICE = "cuda:0"
PRICE = 10_000_000        # micro-dollars per host-hour
STATS_BYTES = replay.STATS_DTYPE.itemsize

# policy -> flags and the configuration that goes with them
MIG, OUT, IN = tg.F_MIGRATE, tg.F_SCALE_OUT, tg.F_SCALE_IN
POLICIES = {
    "plain": dict(flags=0),
    "migrate": dict(flags=MIG),
    "grow": dict(flags=MIG | OUT),
    "scale": dict(flags=MIG | OUT | IN),
    "auto": dict(flags=MIG | IN | tg.F_AUTOSCALE | tg.F_DYNAMIC_SR, autoscale_f_milli=1050, scaling_buffer_hosts=32),
    # the remaining variants together: sticky executor, pre-warmed containers, dynamic limit
    "variants": dict(flags=MIG | OUT | tg.F_STICKY_EXECUTOR | tg.F_WARM_POOL | tg.F_DYNAMIC_SR,
                     warm_pool_per_host=2, warm_migration_delay_ms=2_000, prewarm_delay_ms=60_000),
    "batch": dict(flags=tg.F_BATCH_MODE, batch_start_delay_ms=15_000),
    "batch_grow": dict(flags=tg.F_BATCH_MODE | OUT, batch_start_delay_ms=15_000),
    "closed": dict(flags=MIG | tg.F_CLOSED_LOOP),
    "closed_grow": dict(flags=MIG | OUT | tg.F_CLOSED_LOOP),
}

# traffic -> ramp, gap, duration, GPU requests, END events (the recipes of tracegen's workloads c1 to c5)
TRAFFIC = {
    "steady": dict(ramp=600_000, gap=("exp", 60.0), dur=("logn", 30.0, 1.0), gpus="uniform"),
    "pareto": dict(ramp=3_600_000, gap=("pareto", 1.5, 10.0), dur=("logn", 60.0, 1.2), gpus="uniform"),
    "heavy": dict(ramp=3_600_000, gap=("pareto", 1.5, 10.0), dur=("pareto", 1.3, 5.0), gpus="weighted"),
    "diurnal": dict(ramp=tg.DAY_MS, gap=("logn", 60.0, 2.06), base_gap=240_000, dur=("logn", 120.0, 1.36),
                    gpus="weighted", end=True),
    "bursty": dict(ramp=600_000, gap=("mmpp", 10.0, 300.0, 0.1), dur=("logn", 30.0, 1.0), gpus="uniform"),
}


def _case(name, mode, policy, traffic, traces, caps, cap_lo, cap_hi, hosts, hosts_max, sessions, cells, gpus=8, ragged=False):
    return dict(name=name, mode=mode, policy=policy, traffic=traffic, traces=traces, caps=caps, cap_lo=cap_lo,
                cap_hi=cap_hi, hosts=hosts, hosts_max=hosts_max, sessions=sessions, cells=cells, gpus=gpus, ragged=ragged)


def listed():
    return [
        # one small cluster looked at once: a lone replay, where latency and the calls around it count
        _case("one_small_cluster", "fresh", "plain", "steady", 1, 1, 2000, 2000, 8, 8, 50, 2_000),
        # a serving loop's what-if query: short traces on small clusters, no allocation allowed
        _case("what_if_static", "static", "grow", "bursty", 300, 1, 1000, 4000, 16, 24, 60, 1_500),
        # the cap swept finely on a fixed mid-size cluster (workload c2)
        _case("cap_sweep", "keep", "migrate", "pareto", 1024, 1, 1000, 3000, 30, 30, 400, 50_000),
        # heavy-tailed cells, every trace under four caps (workload c3): the chip full of replays
        _case("heavy_tails", "keep", "migrate", "heavy", 1024, 4, 1500, 4000, 64, 64, 1_000, 100_000),
        # very many small bursty clusters that may grow (workload c5)
        _case("bursty_many", "keep", "grow", "bursty", 4096, 4, 1000, 4000, 16, 24, 120, 20_000),
        # large clusters over days, growing and shrinking (workload c4, the benchmark's default)
        _case("large_scaling", "keep", "scale", "diurnal", 256, 1, 2000, 2000, 512, 768, 8_000, 500_000),
        # the periodic auto-scaler sizes the cluster (workload c4a), fewer replays than compute units
        _case("auto_scaler", "keep", "auto", "diurnal", 192, 1, 4000, 4000, 256, 768, 8_000, 250_000),
        # the Batch baseline on large clusters (workload c4b)
        _case("batch_large", "keep", "batch", "diurnal", 256, 1, 2000, 2000, 512, 512, 8_000, 250_000),
        # users who wait for their cells: closed loops on mid-size clusters (workload c2l) ...
        _case("closed_mid", "keep", "closed", "pareto", 1024, 1, 1000, 3000, 30, 30, 400, 50_000),
        # ... and on large ones (workload c4l)
        _case("closed_large", "keep", "closed_grow", "diurnal", 256, 1, 2000, 2000, 512, 768, 8_000, 250_000),
        # the policy study end to end, from traces in host memory to the table's rows
        _case("policy_study", "study", "grow", "diurnal", 4, 5, 1000, 4000, 16, 256, 1_000, 60_000),
        # new traces of uneven length with every other option switched on, odd cluster size
        _case("uneven_variants", "fresh", "variants", "diurnal", 150, 3, 1500, 3500, 93, 117, 1_301, 70_003, ragged=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    mode = rng.choice(["keep", "keep", "keep", "keep", "fresh", "fresh", "static", "study"])
    policy = {"study": "grow", "static": rng.choice(["plain", "migrate", "grow", "scale"])}.get(mode) or rng.choice(list(POLICIES))
    traffic = "diurnal" if mode == "study" else rng.choice(list(TRAFFIC))
    hosts = _log_uniform(rng, 8, 48 if mode == "static" else 16 if mode == "study" else 700)
    grows = policy in ("grow", "scale", "auto", "variants", "batch_grow", "closed_grow")
    hosts_max = hosts if not grows else min(int(hosts * rng.uniform(1.1, 2.0)) + 1, 64 if mode == "static" else 1024)
    if mode == "study":
        hosts_max = _log_uniform(rng, 64, 256)
    sessions = max(3, min(int(max(hosts, hosts_max // 2) * rng.uniform(5.0, 16.0)), 60 if mode == "static" else 6_000))
    cells = min(int(sessions * rng.uniform(15.0, 130.0)), 60_000 if mode == "study" else 180_000)
    caps = rng.choice([1, 1, 2, 3, 5]) if mode != "study" else 5
    # batches from one replay to what a launch of that cluster size is used for
    most = 4 if mode == "study" else max(1, min(4096, 40_000_000 // cells, 300 if mode == "static" else 1 << 30) // caps)
    traces = _log_uniform(rng, 1, most) if most > 1 else 1
    cap_lo = rng.choice([1000, 1300, 2000])
    return {k: v for k, v in _case("", mode, policy, traffic, traces, caps, cap_lo, cap_lo + rng.choice([0, 700, 2000]), hosts,
                                   hosts_max, sessions, cells, gpus=rng.choice([8, 8, 8, 4]),
                                   ragged=rng.random() < 0.5 and mode != "study").items() if k != "name"}


def _kept(case):
    """Events that every trace keeps (uneven batches: each trace ends somewhere in its last 60 %)."""
    total = case["sessions"] * (2 if TRAFFIC[case["traffic"]].get("end") else 1) + case["cells"]
    if not case["ragged"]:
        return [total] * case["traces"]
    return [max(1, int(total * (1.0 - 0.6 * ((k * 0.6180339887) % 1.0)))) for k in range(case["traces"])]


def _caps(case):
    n, k = case["traces"], case["caps"]
    steps = k if k > 1 else n
    at = [case["cap_lo"] + (case["cap_hi"] - case["cap_lo"]) * j // max(steps - 1, 1) for j in range(steps)]
    return [at[j if k > 1 else t] for t in range(n) for j in range(k)]


def _config(case):
    return tg.base_config(hosts_initial=case["hosts"], hosts_max=case["hosts_max"], gpus_per_host=case["gpus"],
                          min_hosts=case["hosts"] // 2 if case["policy"] == "auto" else case["hosts"],
                          **POLICIES[case["policy"]])


def _sample(gen, shape, spec):
    """Integer milliseconds, 1 ms to 24 h."""
    kind, u = spec[0], torch.rand(shape, generator=gen, device=DEVICE, dtype=torch.float64)
    if kind == "exp":
        sec = -spec[1] * torch.log1p(-u)
    elif kind == "pareto":
        sec = spec[2] * torch.pow(1.0 - u, -1.0 / spec[1])
    elif kind == "logn":
        sec = torch.exp(math.log(spec[1]) + spec[2] * torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float64))
    else:                     # two-state process per session: a fast and a slow mean, switched with a probability per cell
        slow = torch.cumsum((torch.rand(shape, generator=gen, device=DEVICE) < spec[3]).to(torch.int32), dim=-1) & 1
        sec = -torch.where(slow == 0, spec[1], spec[2]) * torch.log1p(-u)
    return torch.clamp(torch.floor(sec * 1000.0), 1, tg.MAX_DUR_MS).to(torch.int64)


def _traces(case, gen, n):
    """Event times, durations, session | kind words [n][events] and GPU requests [n][sessions] of n traces."""
    tr = TRAFFIC[case["traffic"]]
    N, E, G = case["sessions"], case["cells"], case["gpus"]
    M = -(-E // N)
    per = torch.full((N,), E // N, device=DEVICE, dtype=torch.int64)
    per[: E % N] += 1
    live = torch.arange(M, device=DEVICE) < per[:, None]
    start = torch.floor(torch.rand((n, N), generator=gen, device=DEVICE, dtype=torch.float64) * tr["ramp"]).to(torch.int64)
    u = torch.rand((n, N), generator=gen, device=DEVICE)
    at = torch.tensor([0.25, 0.5, 0.75] if tr["gpus"] == "uniform" else [0.5, 0.75, 0.9], device=DEVICE)
    g = torch.clamp(torch.pow(2, torch.bucketize(u, at, right=True)), max=G).to(torch.uint8)
    d = _sample(gen, (n, N, M), tr["dur"])
    gap = _sample(gen, (n, N, M), tr["gap"])
    if "base_gap" in tr:      # diurnal: every gap is divided by 1 + 0.5 sin(2 pi t / 24 h) at the time it begins
        gap += tr["base_gap"]
        t = start.clone()
        tc = torch.empty_like(gap)
        for k in range(M):
            m = 1.0 + 0.5 * torch.sin(2.0 * math.pi * (t % tg.DAY_MS).to(torch.float64) / tg.DAY_MS)
            tc[:, :, k] = t + torch.clamp(torch.floor(gap[:, :, k] / m), 1, tg.MAX_DUR_MS).to(torch.int64)
            t = tc[:, :, k] + d[:, :, k]
    else:
        tc = start[:, :, None] + torch.cumsum(gap + d, dim=-1) - d
    del gap
    sid = torch.arange(N, device=DEVICE, dtype=torch.int64)[:, None] << 16
    seq = torch.arange(1, M + 1, device=DEVICE, dtype=torch.int64)
    never = torch.iinfo(torch.int64).max
    key = torch.where(live, (torch.clamp(tc, max=tg.MAX_TIME_MS) << 32) | sid | seq, never)
    parts, durs = [(start << 32) | sid[:, 0], key.view(n, -1)], [torch.zeros_like(start), d.view(n, -1)]
    if tr.get("end"):
        last = (per - 1).clamp(min=0).expand(n, N)[:, :, None]
        over = torch.gather(tc + d, 2, last)[:, :, 0]
        over = torch.clamp(torch.where(per > 0, over, start), max=tg.MAX_TIME_MS)
        parts.append((over << 32) | sid[:, 0] | (M + 1))
        durs.append(torch.zeros_like(start))
    del tc
    key, order = torch.sort(torch.cat(parts, dim=1), dim=1)
    count = N * (2 if tr.get("end") else 1) + E
    key, order = key[:, :count], order[:, :count]
    dur = torch.gather(torch.cat(durs, dim=1), 1, order).to(torch.int32)
    place = key & 0xFFFF
    kind = torch.where(place == 0, tg.EV_START, torch.where(place == M + 1, tg.EV_END, tg.EV_CELL))
    return (key >> 32).to(torch.int32), dur, (((key >> 16) & 0xFFFF) | (kind << 24)).to(torch.int32), g


def _device_inputs(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    kept = _kept(case)
    step = max(1, 30_000_000 // max(kept))          # bounds the temporaries of the generator
    total = sum(kept)
    out = {k: torch.empty(total, dtype=torch.int32, device=DEVICE) for k in ("ev_time_ms", "ev_dur_ms", "ev_sess_kind")}
    gpus, at = [], 0
    for k0 in range(0, case["traces"], step):
        n = min(step, case["traces"] - k0)
        t, d, s, g = _traces(case, gen, n)
        gpus.append(g.reshape(-1))
        size = sum(kept[k0:k0 + n])
        rows = None
        if case["ragged"]:
            rows = torch.arange(t.shape[1], device=DEVICE) < torch.tensor(kept[k0:k0 + n], device=DEVICE)[:, None]
        for key, v in (("ev_time_ms", t), ("ev_dur_ms", d), ("ev_sess_kind", s)):
            out[key][at:at + size] = v.reshape(-1) if rows is None else v[rows]
        at += size
    on = lambda v, dt: torch.tensor(np.asarray(v), dtype=dt, device=DEVICE)
    out["ev_offset"] = on(np.concatenate([[0], np.cumsum(np.asarray(kept, np.int64))]), torch.int64)
    out["sess_offset"] = on(np.arange(case["traces"] + 1) * case["sessions"], torch.int32)
    out["sess_gpus"] = torch.cat(gpus)
    out["trace_of_replay"] = on(np.repeat(np.arange(case["traces"]), case["caps"]), torch.int32)
    out["cap_milli"] = on(_caps(case), torch.int32)
    torch.cuda.synchronize()
    return out


def _host_study(case, seed):
    kw = tg.recipe("c4")["kw"]
    traces = [tg.make_trace(1_000 * seed + k, case["sessions"], case["cells"], **kw) for k in range(case["traces"])]
    for _, _, _, g in traces:
        np.minimum(g, case["gpus"], out=g)
    tor = [t for t in range(case["traces"]) for _ in range(case["caps"])]
    return tg.pack(_config(case), traces, tor, _caps(case), "study")


def prepare(case, seed):
    if case["mode"] == "study":
        return {"mode": "study", "batch": _host_study(case, seed)}
    state = {"mode": case["mode"], "config": _config(case), "inputs": _device_inputs(case, seed), "sessions": case["sessions"]}
    n = case["traces"] * case["caps"]
    if case["mode"] == "keep":
        state["handle"] = replay.Replay(state["config"], state["inputs"])
    elif case["mode"] == "static":
        state["replays"] = n
        state["out"] = torch.zeros(n * STATS_BYTES, dtype=torch.uint8, device=DEVICE)
    return state


def _fields(records):
    return {k: records[k] for k in records.dtype.names}


def run(state):
    mode = state["mode"]
    if mode == "study":
        rows = sweep.run_policies(state["batch"], price_micro_per_host_hour=PRICE)
        return {k: np.array([r[k] for r in rows]) for k in rows[0]}        # the table's columns
    if mode == "keep":
        h = state["handle"]
        h.run()
        return _fields(h.stats())
    if mode == "fresh":
        h = replay.Replay(state["config"], state["inputs"])
        h.run()
        out = _fields(h.stats())
        out["bills"] = _fields(h.billing(PRICE))
        h.close()
        return out
    replay.run_static(state["config"], state["inputs"], state["sessions"], state["out"])
    return _fields(replay.stats_from_tensor(state["out"], state["replays"]))


def work(case):
    """Bytes: 12 per event and 1 per session of every trace and 8 per replay read, one result record per
    replay written (a trace that several replays share is counted once). The study does it once per policy."""
    events, replays = sum(_kept(case)), case["traces"] * case["caps"]
    once = 12 * events + case["traces"] * case["sessions"] + replays * (8 + STATS_BYTES)
    return {"bytes": once * (2 if case["mode"] == "study" else 1), "flops": 0}


def tolerance(case):
    return "exact"            # integer milliseconds and counts throughout
