"""The work that users of this library have it do, as cases that can be timed and compared.

Every case is one call (or the short run of calls that belongs together) of the public entry points of
`paper_2408_00741_amd` on a synthetic request trace: arrivals with a constant, hourly, daily or weekly rate,
log-normal token counts, profile tables that follow simple laws in load, frequency and tensor parallelism.  The
kinds are the entry points that a program calls in its loop:

  ingest      dyn_trace_ingest: a raw request log becomes the cell-sorted trace
  select      dyn_eval_select: every candidate of every (window, class), least-cost choice, window totals
  plan        dyn_eval_space, dyn_select_config, dyn_account: the same in separate calls, with the bill
  ticks       dyn_eval_select_ticks: the load followed tick by tick inside a window
  mixed       dyn_eval_select_mixed: pools that mix instance types
  path        dyn_select_path: selection with re-sharding overheads between windows, on an evaluated space
  hierarchy   dyn_hierarchy: node counts, layouts and frequencies top down

`exact` computes the same quantities in float64 with plain torch and NumPy, without this library.
"""
import math

import numpy as np
import torch

import paper_2408_00741_amd as dyn

F_LO, F_HI = 880, 1980                      # MHz, the frequency range of the profiles


# ---- the cases ----------------------------------------------------------------------------------------------

def _case(kind, name=None, **kw):
    c = {"kind": kind, "n_req": 10_000_000, "n_window": 1440, "window_s": 60.0, "rate": "day", "n_model": 1,
         "in_bins": 5, "out_bins": 5, "tp": "2,4,8", "f_lo": F_LO, "f_step": 100, "n_inst": 16, "n_rho": 64,
         "f_between": False, "prefill": "flat", "idle": 0.0, "budget": 0, "pct": 99, "runs": 1}
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a day of a production log (ten million requests in time order), filed into one-minute windows
        _case("ingest", "ingest-day"),
        # the logs of six front ends of a four-model service, one after the other: not in time order
        _case("ingest", "ingest-merged", n_req=6_000_000, n_model=4, in_bins=3, out_bins=3, runs=6),
        # a controller that looks at the last minute only: the smallest call, latency
        _case("select", "select-minute", n_req=10_000, n_window=1, rate="const", in_bins=3, out_bins=3, f_step=220, n_inst=4, n_rho=16),
        # the last hour, minute by minute
        _case("select", "select-hour", n_req=1_000_000, n_window=60, rate="hour", in_bins=3, out_bins=3, n_rho=32),
        # a day in one-minute windows: the ordinary planning run
        _case("select", "select-day"),
        # a week of four models with the full frequency range: the largest run, eleven gigabytes written
        _case("select", "select-week-models", n_req=100_000_000, n_window=2016, window_s=300.0, rate="week", n_model=4, tp="1,2,4,8",
              f_lo=480, n_inst=32, idle=0.1),
        # odd sizes: 487 windows, 15 classes, candidates between the profiled frequencies, a budget, an idle
        # term; separate calls, because the program looks at the space before it selects, and then the bill
        _case("plan", "plan-odd", n_req=3_333_333, n_window=487, window_s=300.0, in_bins=3, n_inst=13, n_rho=48, f_between=True, idle=0.05, budget=72),
        # a day with five-second ticks
        _case("ticks", "ticks-day", n_tick=12),
        # an hour with five-second ticks and a prefill time that grows with the load
        _case("ticks", "ticks-hour-load", n_req=1_000_000, n_window=60, rate="hour", in_bins=3, out_bins=3, n_rho=32, prefill="load", n_tick=12),
        # a day of mixed pools: eight shares of the load, 32 GPUs a class
        _case("mixed", "mixed-day", shares=8, budget=32),
        # a day of choices with re-sharding overheads between 48 layouts
        _case("path", "path-day"),
        # a day under the three controllers, five-second ticks
        _case("hierarchy", "hierarchy-day", n_tick=12, epoch=6, overheads=False, spill=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ingest", "ingest", "select", "select", "select", "plan", "ticks", "ticks", "mixed", "path", "hierarchy"])
    c = _case(kind, n_req=_log(rng, 3_000, 20_000_000), n_window=_log(rng, 1, 2016), window_s=rng.choice([30.0, 60.0, 60.0, 300.0]),
              rate=rng.choice(["const", "hour", "day", "week"]), n_model=rng.choice([1, 1, 1, 2, 4]), in_bins=rng.randint(1, 5),
              out_bins=rng.randint(1, 5), tp=rng.choice(["2,4,8", "1,2,4,8", "4,8", "8"]), f_step=rng.choice([100, 110, 220]),
              n_inst=rng.randint(1, 32), n_rho=rng.randint(8, 72), f_between=rng.random() < 0.25,
              prefill=rng.choice(["flat", "flat", "load"]), idle=rng.choice([0.0, 0.0, 0.1]), budget=rng.choice([0, 0, 48]),
              pct=rng.choice([99, 99, 99, 95, 90]))
    # no more than the listed ones cost: at most 4e7 (cell, candidate) pairs, 4e8 look-ups in the ticks
    def shrink(limit, per_window):
        c["n_window"] = max(1, min(c["n_window"], int(limit // max(1, per_window))))
    G, K = _n_class(c), _n_cand(c)
    if kind == "ingest":
        c["runs"] = rng.choice([1, 1, 1, rng.randint(2, 9)])
        if c["runs"] > 1:
            c["n_req"] = min(c["n_req"], 9_000_001)
    elif kind in ("select", "plan"):
        shrink(4e7, G * K)
    elif kind == "ticks":
        c["n_tick"] = rng.choice([1, 5, 6, 10, 12, 30])
        c["n_req"] = min(c["n_req"], 4_000_001)
        shrink(1.5e8, G * K * c["n_tick"])
    elif kind == "mixed":
        c["shares"] = rng.randint(1, 8)
        c["budget"] = rng.choice([16, 24, 32])
        shrink(36_000, G)
    elif kind == "path":
        c["n_inst"] = min(c["n_inst"], 64 // len(c["tp"].split(",")))
        shrink(4e7, G * _n_cand(c))
    else:
        c.update(n_tick=rng.choice([5, 6, 12]), epoch=rng.choice([1, 6, 30]), spill=rng.random() < 0.3)
        c["overheads"] = rng.random() < 0.3
        c["n_inst"] = min(c["n_inst"], 64 // len(c["tp"].split(",")))
        shrink(450_000, G * c["n_tick"])
    return c


def _tp(c):
    return np.asarray([int(x) for x in c["tp"].split(",")], np.int32)


def _freqs(c):
    return np.arange(c["f_lo"], F_HI + 1, c["f_step"]).astype(np.float64)


def _n_class(c):
    return c["n_model"] * c["in_bins"] * c["out_bins"]


def _n_cand(c):
    return len(_tp(c)) * (len(_freqs(c)) - (1 if c["f_between"] else 0)) * c["n_inst"]


def _n_max(c):
    return [max(1, c["budget"] // int(t)) for t in _tp(c)]


# ---- what a program has in hand: the log, the profile, the candidates, the objective ------------------------------

def _edges(c):
    def axis(bins, three):
        if bins == 3:
            return three
        return [int(round(64 * 128 ** (i / bins))) for i in range(1, bins)]
    ie, oe = axis(c["in_bins"], [256, 2048]), axis(c["out_bins"], [128, 512])
    return {"in_edge": np.tile(np.asarray(ie, np.int32), (c["n_model"], 1)).reshape(c["n_model"], len(ie)),
            "out_edge": np.tile(np.asarray(oe, np.int32), (c["n_model"], 1)).reshape(c["n_model"], len(oe))}


_MIX = {1: [1.0], 2: [0.6, 0.4], 4: [0.4, 0.3, 0.2, 0.1]}
_PEAK = {"const": 1.0, "hour": 1.3, "day": 1.6, "week": 1.8}


def _rate(shape, t):
    if shape == "const":
        return np.ones_like(t)
    if shape == "hour":
        return 1.0 + 0.3 * np.sin(2.0 * math.pi / 3600.0 * t)
    day = 1.0 + 0.6 * np.sin(2.0 * math.pi / 86400.0 * (t - 6.0 * 3600.0))
    return day if shape == "day" else day * np.where(np.floor(t / 86400.0) % 7 >= 5, 0.6, 1.0)


def _log_of(c, seed):
    """The request log on the GPU: timestamps, input tokens, output tokens, model (None for a single one)."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 1_000_003 + 17)
    n, horizon = c["n_req"], c["n_window"] * c["window_s"]
    grid = np.linspace(0.0, horizon, 8193)
    cum = np.concatenate([[0.0], np.cumsum(_rate(c["rate"], 0.5 * (grid[1:] + grid[:-1])))])
    cum = torch.from_numpy(cum / cum[-1]).to(dev)
    u = torch.rand(n, generator=gen, device=dev, dtype=torch.float64)
    i = torch.clamp(torch.searchsorted(cum, u, right=True) - 1, 0, 8191)
    t = (i + (u - cum[i]) / (cum[i + 1] - cum[i])) * (horizon / 8192.0)
    del u, i
    t = torch.clamp(t, 0.0, math.nextafter(horizon, 0.0))
    if c["runs"] == 1:
        t = torch.sort(t).values
    else:                                    # one sorted run per front end, concatenated
        cut = [n * r // c["runs"] for r in range(c["runs"] + 1)]
        t = torch.cat([torch.sort(t[a:b]).values for a, b in zip(cut[:-1], cut[1:])])

    def tokens(median, sigma):
        z = torch.randn(n, generator=gen, device=dev, dtype=torch.float32)
        return torch.clamp(torch.round(torch.exp(math.log(median) + sigma * z)), 1.0, 8192.0).to(torch.int32)
    x, y = tokens(1000.0, 1.0), tokens(250.0, 0.8)
    model = None
    if c["n_model"] > 1:
        upto = torch.tensor(np.cumsum(_MIX[c["n_model"]])[:-1], dtype=torch.float32, device=dev)
        model = torch.bucketize(torch.rand(n, generator=gen, device=dev), upto).to(torch.int32)
    return t, x, y, model


def _profile(c, seed):
    """Prefill time, TBT, power and capacity over (class, TP, frequency, load): time falls with frequency and TP, TBT
    grows as 1 / (1 - load), power as f^3 times the load; capacities put a busy class at 0.6 of the largest pool."""
    r = np.random.RandomState(int(seed) % (1 << 31))
    tp, f, rho = _tp(c), _freqs(c), np.linspace(0.0, 0.95, c["n_rho"])
    cpm, G = c["in_bins"] * c["out_bins"], _n_class(c)
    shape = (G, tp.size, f.size, rho.size)
    pf, tb, pw, ml = np.empty(shape), np.empty(shape), np.empty(shape), np.empty(shape[:3])
    peak = c["n_req"] / (c["n_window"] * c["window_s"]) * _PEAK[c["rate"]]
    p = tp.astype(np.float64)[:, None]
    for j in range(c["n_model"]):
        a, b = r.uniform(0.6, 1.0), r.uniform(0.6, 0.9)
        kp, kd = r.uniform(0.05, 0.2, cpm) * 2 ** j, r.uniform(15.0, 40.0, cpm) * 2 ** j
        unit = np.mean(p[-1, 0] ** (1 + b) * 1000.0 / kd)
        scale = peak * _MIX[c["n_model"]][j] * 2000.0 / math.sqrt(cpm) / (c["n_inst"] * 0.6 * unit)
        slow = (f[-1] / f)[None, :] ** a / p ** b
        more = 1.0 + (0.8 * rho ** 2 if c["prefill"] == "load" else 0.0 * rho)
        for i in range(cpm):
            g = j * cpm + i
            pf[g] = (kp[i] * slow)[:, :, None] * more
            tb[g] = np.minimum((kd[i] * slow)[:, :, None] / (1.0 - rho), 1000.0)
            pw[g] = p[:, :, None] * (100.0 + 600.0 * ((f / f[-1]) ** 3)[None, :, None] * rho)
            ml[g] = scale * p * 1000.0 / (kd[i] * slow)
    return {"tp": tp, "f_mhz": f, "rho": rho, "prefill_ms_per_tok": pf, "tbt_ms": tb, "power_w": pw, "max_load_tps": ml}


def _candidates(c):
    f = _freqs(c)
    f = 0.4 * f[:-1] + 0.6 * f[1:] if c["f_between"] else f
    t, f, n = np.meshgrid(np.arange(len(_tp(c))), f, np.arange(1, c["n_inst"] + 1), indexing="ij")
    return {"n_inst": n.ravel().astype(np.int32), "tp_index": t.ravel().astype(np.int32), "f_mhz": f.ravel()}


def _slos(c, prof):
    ib = (np.arange(_n_class(c)) % (c["in_bins"] * c["out_bins"])) // c["out_bins"]
    upper = np.concatenate([_edges(c)["in_edge"][0], [8192]])
    return {"slo_ttft_ms": 5.0 * upper[ib] * prof["prefill_ms_per_tok"][:, -1, -1, 0], "slo_tbt_ms": np.full(_n_class(c), 100.0)}


def _layouts(c):
    """Distinct (TP, instances) pairs, the pair of every candidate, and the overhead in joules of going from one to
    another: GPUs that join are loaded, a change of TP re-shards all of them."""
    cand = _candidates(c)
    key, lay = np.unique(cand["tp_index"].astype(np.int64) * 1000 + cand["n_inst"], return_inverse=True)
    ti, n = key // 1000, key % 1000
    gpus = _tp(c)[ti].astype(np.int64) * n
    unit = 0.02 * 300.0 * c["window_s"]
    cost = unit * np.maximum(0, gpus[None, :] - gpus[:, None]) + 0.5 * unit * (ti[None, :] != ti[:, None]) * gpus[None, :]
    return lay.astype(np.int32), cost.astype(np.float64), n.astype(np.int32), ti.astype(np.int32)


def _budget(c):
    return np.full(_n_class(c), c["budget"], np.int32) if c["budget"] else None


def _carbon(c):
    return torch.from_numpy(300.0 + 120.0 * np.sin(np.arange(c["n_window"]) * (c["window_s"] * 2.0 * math.pi / 86400.0))).cuda()


_PRICE = (2.1, 0.12)                         # per GPU-hour, per kWh


def prepare(case, seed):
    c, s = case, {"case": case}
    t, x, y, model = _log_of(c, seed)
    NW, G, edges = c["n_window"], _n_class(c), _edges(c)
    if c["kind"] == "ingest":
        ws = torch.empty(max(256, dyn.dyn_trace_ingest_workspace(c["n_req"], NW, G)), dtype=torch.uint8, device="cuda")
        s.update(log=(t, x, y, model), edges=edges, ws=ws)
        return s
    prof = _profile(c, seed)
    s["slos"] = _slos(c, prof)
    s["prof"] = dyn.dyn_profile_load(prof)
    n_tick = c.get("n_tick", 1)
    s["fine"] = dyn.dyn_trace_ingest(t, x, y, model, edges, NW * n_tick, c["window_s"] / n_tick)[:3]
    cells, K = NW * G, _n_cand(c)
    dev = t.device

    def empty(*shape, dtype=torch.float64):
        return torch.empty(shape, dtype=dtype, device=dev)

    def workspace(n):
        return torch.empty(max(256, n), dtype=torch.uint8, device=dev)
    totals = {"window_energy_j": empty(NW), "window_infeasible": empty(NW, dtype=torch.int32)}
    if c["kind"] in ("select", "plan", "ticks", "path"):
        s["plan"] = dyn.Plan(_candidates(c), s["slos"], (c["pct"], 100), _budget(c), c["idle"])
        s["space"] = {"energy_j": empty(cells, K), "p99_ttft_ms": empty(cells, K), "p99_tbt_ms": empty(cells, K), "flags": empty(cells, K, dtype=torch.uint8)}
        s["sel"] = {"sel": empty(cells, dtype=torch.int32), "sel_energy_j": empty(cells), "sel_cost": empty(cells), **totals}
        s["ws"] = workspace(dyn.dyn_eval_ticks_workspace(c["n_req"], NW, n_tick, G, K) if c["kind"] == "ticks" else dyn.dyn_eval_space_workspace(NW, G, K))
    if c["kind"] == "plan":
        s["carbon"] = _carbon(c)
    elif c["kind"] == "mixed":
        s["plan"] = dyn.MixedPlan(c["shares"], _n_max(c), s["slos"], (c["pct"], 100), _budget(c))
        T = len(_tp(c))
        s["sel"] = {"energy_j": empty(cells), **{k: empty(cells, T, dtype=torch.int32) for k in ("n_inst", "f_index", "share")}, **totals}
        s["ws"] = workspace(dyn.dyn_mixed_workspace(s["prof"], NW, s["plan"]))
    elif c["kind"] == "path":
        s["layout"], s["transition"] = _layouts(c)[:2]
        dyn.dyn_eval_space(s["prof"], *s["fine"], NW, c["window_s"], s["plan"], out=s["space"], workspace=s["ws"])
        s["sel"] = {"sel": empty(cells, dtype=torch.int32), "sel_energy_j": empty(cells), "path_cost": empty(G), **totals}
        s["ws"] = workspace(dyn.dyn_select_path_workspace(NW, G, K, s["transition"].shape[0]))
    elif c["kind"] == "hierarchy":
        s["coarse"] = dyn.dyn_trace_ingest(t, x, y, model, edges, NW, c["window_s"])[:3]
        _, tr, n, ti = _layouts(c)
        s["lay"], s["transition"] = (n, ti), tr if c["overheads"] else None
        n_epoch = -(-NW // c["epoch"])
        s["out"] = {"nodes": empty(n_epoch, G, dtype=torch.int32), "layout_sel": empty(cells, dtype=torch.int32), "f_sel": empty(NW * n_tick, G, dtype=torch.int32),
                    "energy_j": empty(cells), "violations": empty(cells, dtype=torch.int32), **totals}
        if c["overheads"]:
            s["out"]["path_cost"] = empty(G)
        if c["spill"]:
            s["out"]["keep"] = empty(n_epoch, G)
        s["ws"] = workspace(dyn.dyn_hierarchy_workspace(NW, n_tick, G, n.size))
    return s


def run(state):
    s, c = state, state["case"]
    NW, win = c["n_window"], c["window_s"]
    if c["kind"] == "ingest":
        ins, outs, off, _ = dyn.dyn_trace_ingest(*s["log"], s["edges"], NW, win, workspace=s["ws"])
        return {"in": ins, "out": outs, "off": off}
    if c["kind"] == "select":
        dyn.dyn_eval_select(s["prof"], *s["fine"], NW, win, s["plan"], out=s["space"], sel=s["sel"], workspace=s["ws"])
        return {"space": s["space"], "sel": s["sel"]}
    if c["kind"] == "plan":
        dyn.dyn_eval_space(s["prof"], *s["fine"], NW, win, s["plan"], out=s["space"], workspace=s["ws"])
        dyn.dyn_select_config(s["prof"], s["space"], NW, win, s["plan"], out=s["sel"])
        bill, _ = dyn.dyn_account(s["prof"], s["sel"]["sel"], s["sel"]["window_energy_j"], s["plan"], NW, win, *_PRICE, s["carbon"])
        return {"space": s["space"], "sel": s["sel"], "bill": bill}
    if c["kind"] == "ticks":
        dyn.dyn_eval_select_ticks(s["prof"], *s["fine"], NW, c["n_tick"], win / c["n_tick"], s["plan"], out=s["space"], sel=s["sel"], workspace=s["ws"])
        return {"space": s["space"], "sel": s["sel"]}
    if c["kind"] == "mixed":
        dyn.dyn_eval_select_mixed(s["prof"], *s["fine"], NW, win, s["plan"], out=s["sel"], workspace=s["ws"])
        return {"sel": s["sel"]}
    if c["kind"] == "path":
        dyn.dyn_select_path(s["prof"], s["space"], NW, win, s["plan"], s["layout"], s["transition"], out=s["sel"], workspace=s["ws"])
        return {"sel": s["sel"]}
    out, _ = dyn.dyn_hierarchy(s["prof"], s["coarse"], s["fine"], NW, c["n_tick"], win / c["n_tick"], c["epoch"], len(_tp(c)) - 1, len(_freqs(c)) - 1, 8,
                               *s["lay"], s["slos"], (c["pct"], 100), out=s["out"], workspace=s["ws"], transition_j=s["transition"], spill=c["spill"])
    return {"out": out}


def work(case):
    """Each request, offset, table and selection once; per look-up the divisions (one operation each), the
    interpolation of three quantities, the energy and the percentile: 18 operations."""
    c = case
    R, G, K = c["n_req"], _n_class(c), _n_cand(c)
    cells, n_tick = c["n_window"] * G, c.get("n_tick", 1)
    table = 8 * (3 * c["n_rho"] + 1) * G * len(_tp(c)) * len(_freqs(c))
    trace = 8 * R + 8 * cells * n_tick + table
    totals = 12 * c["n_window"]
    if c["kind"] == "ingest":
        return {"bytes": (28 + (4 if c["n_model"] > 1 else 0)) * R + 8 * cells, "flops": R}
    if c["kind"] in ("select", "plan", "ticks"):
        again = 9 * cells * K + 60 * c["n_window"] if c["kind"] == "plan" else 0
        return {"bytes": trace + 25 * cells * K + 20 * cells + totals + again, "flops": 18 * cells * K * n_tick}
    if c["kind"] == "mixed":
        entries = sum(_n_max(c)) * c["shares"]
        return {"bytes": trace + cells * (8 + 12 * len(_tp(c))) + totals, "flops": cells * entries * (18 * len(_freqs(c)) + 1)}
    if c["kind"] == "path":
        L = len(_tp(c)) * c["n_inst"]
        return {"bytes": 9 * cells * K + 12 * cells + totals, "flops": cells * (K + 2 * L * L)}
    L = len(_tp(c)) * c["n_inst"]
    return {"bytes": 16 * R + 8 * cells * (n_tick + 1) + table + cells * (16 + 4 * n_tick) + totals,
            "flops": 18 * cells * (L + n_tick * len(_freqs(c))) + (2 * cells * L * L if c["overheads"] else 0)}


def tolerance(case):
    if case["kind"] == "ingest":
        return "exact"                       # whole numbers, moved and counted
    # float64 throughout: sums in another order differ in the last bits, and a choice or a flag flips where two
    # totals, or a latency and its limit, agree to the last bits (measured against `exact`: at most 5e-16)
    return {"rel": 4e-15, "max": 1e-12, "differ": 1e-5}


# ---- the same in plain float64 -------------------------------------------------------------------------------

def _stats(c, log, n_window, window_s):
    """Per cell: requests, tokens a second, the percentile of the input lengths; and the sorted trace."""
    t, x, y, model = log
    G = _n_class(c)
    e = _edges(c)
    key = torch.floor(t / window_s).long() * G
    g = torch.bucketize(x, torch.from_numpy(e["in_edge"][0]).cuda(), right=True).long() * c["out_bins"]
    g += torch.bucketize(y, torch.from_numpy(e["out_edge"][0]).cuda(), right=True)
    if model is not None:
        g += model.long() * (c["in_bins"] * c["out_bins"])
    key += g
    cells = n_window * G
    m = torch.bincount(key, minlength=cells)
    tok = torch.zeros(cells, dtype=torch.int64, device=key.device).index_add_(0, key, x.long() + y.long())
    xs = torch.sort(key * 16384 + x.long()).values % 16384
    beg = torch.cumsum(m, 0) - m
    rank = torch.where(m > 0, (c["pct"] * m + 99) // 100, torch.ones_like(m))
    xp = torch.where(m > 0, xs[torch.clamp(beg + rank - 1, max=xs.numel() - 1)], torch.zeros_like(m)).double()
    return {"m": m, "load": tok.double() / window_s, "xp": xp, "xs": xs, "beg": beg, "rank": rank}


class _Tables:
    def __init__(self, prof):
        dev = torch.device("cuda")
        self.pf, self.tb, self.pw = (torch.from_numpy(prof[k]).to(dev).reshape(-1) for k in ("prefill_ms_per_tok", "tbt_ms", "power_w"))
        self.ml = torch.from_numpy(prof["max_load_tps"]).to(dev)
        self.rho = torch.from_numpy(prof["rho"]).to(dev)
        self.G, self.T, self.F = prof["max_load_tps"].shape
        self.R = prof["rho"].size

    def look(self, load, n, g, ti, lo, u):
        """(prefill, TBT, power, overloaded) at load / (n * capacity) for index tensors that broadcast with `load`."""
        two = bool((u != 0).any())
        hi = torch.clamp(lo + 1, max=self.F - 1)
        ml = self.ml[g, ti, lo]
        if two:
            ml = (1.0 - u) * ml + u * self.ml[g, ti, hi]
        rho = load / (n * ml)
        top = self.rho[-1]
        rc = torch.minimum(rho, top)
        j = torch.clamp(torch.searchsorted(self.rho, rc.contiguous(), right=True) - 1, 0, self.R - 2)
        w = (rc - self.rho[j]) / (self.rho[j + 1] - self.rho[j])
        row = ((g * self.T + ti) * self.F + lo) * self.R
        row_hi = ((g * self.T + ti) * self.F + hi) * self.R

        def at(tab):
            a = (1.0 - w) * tab[row + j] + w * tab[row + j + 1]
            if two:
                a = (1.0 - u) * a + u * ((1.0 - w) * tab[row_hi + j] + w * tab[row_hi + j + 1])
            return a
        return at(self.pf), at(self.tb), at(self.pw), rho > top


def _cand_tensors(c):
    cand, f = _candidates(c), _freqs(c)
    lo = np.clip(np.searchsorted(f, cand["f_mhz"], side="right") - 1, 0, max(0, len(f) - 2))
    u = (cand["f_mhz"] - f[lo]) / (f[lo + 1] - f[lo]) if len(f) > 1 else np.zeros(len(lo))
    up = u == 1.0
    lo, u = lo + up, np.where(up, 0.0, u)
    put = lambda a, d: torch.from_numpy(np.ascontiguousarray(a)).to("cuda", d)
    return put(cand["n_inst"], torch.float64), put(cand["tp_index"], torch.int64), put(lo, torch.int64), put(u, torch.float64)


def _pick(c, tab, energy, flags, cells_g, window_s):
    """Least cost among the feasible candidates of each row: (energy, cost, candidate)."""
    n, ti, lo, u = _cand_tensors(c)
    cost = energy
    if c["idle"]:
        pw0 = tab.look(torch.zeros_like(energy), n, cells_g[:, None], ti, lo, u)[2]
        cost = energy + c["idle"] * ((n * pw0) * window_s)
    cost = torch.where(flags, cost, torch.full_like(cost, math.inf))
    best, k = cost.min(1)
    e = torch.where(torch.isfinite(best), energy.gather(1, k[:, None])[:, 0], best)
    return e, best, torch.where(torch.isfinite(best), k, -torch.ones_like(k)), cost


def _exact_space(c, st, tab, slos, keep_cost=False):
    """The evaluated space and its choices, a run of cells at a time."""
    G, K, n_tick = _n_class(c), _n_cand(c), c.get("n_tick", 1)
    cells = c["n_window"] * G
    dev = torch.device("cuda")
    n, ti, lo, u = _cand_tensors(c)
    st_t, st_b = (torch.from_numpy(slos[k]).to(dev) for k in ("slo_ttft_ms", "slo_tbt_ms"))
    over = torch.zeros(K, dtype=torch.bool, device=dev)
    if c["budget"]:
        over = n * torch.from_numpy(_tp(c)).to(dev)[ti] > c["budget"]
    E, P, B = (torch.empty((cells, K), dtype=torch.float64, device=dev) for _ in range(3))
    se, sc = (torch.empty(cells, dtype=torch.float64, device=dev) for _ in range(2))
    sel = torch.empty(cells, dtype=torch.int64, device=dev)
    costs = torch.empty((cells, K), dtype=torch.float64, device=dev) if keep_cost else None
    tick_s = c["window_s"] / n_tick
    depth = 1
    if n_tick > 1:
        per = lambda v: v.view(c["n_window"], n_tick, G).transpose(1, 2).reshape(cells, n_tick)
        m_t, load_t, beg_t = per(st["m"]), per(st["load"]), per(st["beg"])
        m = m_t.sum(1)
        j = m - torch.where(m > 0, (c["pct"] * m + 99) // 100, m) + 1
        depth = int(j.max())
        if float(cells) * K * n_tick * min(depth, int(m_t.max())) > 6e9:
            return None
    step = max(1, int(3e7 // (K * n_tick * (depth if n_tick > 1 else 1))))
    for a in range(0, cells, step):
        b = min(cells, a + step)
        g = torch.arange(a, b, device=dev) % G
        if n_tick == 1:
            pf, tb, pw, ov = tab.look(st["load"][a:b, None], n, g[:, None], ti, lo, u)
            e = (n * pw) * c["window_s"]
            p, q = st["xp"][a:b, None] * pf, tb * (st["m"][a:b, None] > 0)
        else:
            pf, tb, pw, ov = tab.look(load_t[a:b, :, None], n, g[:, None, None], ti, lo, u)
            e = ((n * pw) * tick_s).sum(1)
            ov = ov.any(1)
            # the j-th largest of the requests' TTFTs: only each tick's j longest inputs can be among them
            mt, jj = m_t[a:b], j[a:b]
            d = int(min(depth, int(mt.max()))) or 1
            at = torch.arange(d, device=dev)
            idx = beg_t[a:b, :, None] + mt[:, :, None] - 1 - at
            x = torch.where(at < mt[:, :, None], st["xs"][torch.clamp(idx, 0, st["xs"].numel() - 1)].double(), -math.inf)
            v = torch.where(torch.isfinite(x)[..., None], torch.clamp(x, min=0.0)[..., None] * pf[:, :, None, :], -math.inf).reshape(b - a, n_tick * d, K)
            v = torch.sort(v, dim=1, descending=True).values
            p = v.gather(1, torch.clamp(jj - 1, 0, n_tick * d - 1)[:, None, None].expand(-1, 1, K))[:, 0]
            o = torch.sort(tb, dim=1, descending=True)
            cum = torch.cumsum(mt[:, :, None].expand(-1, -1, K).gather(1, o.indices), 1)
            first = torch.clamp((cum < jj[:, None, None]).sum(1, keepdim=True), max=n_tick - 1)
            q = o.values.gather(1, first)[:, 0]
            some = (m[a:b] > 0)[:, None]
            p, q = torch.where(some, p, torch.zeros_like(p)), torch.where(some, q, torch.zeros_like(q))
        ok = ~ov & ~(p > st_t[g][:, None]) & ~(q > st_b[g][:, None]) & ~over
        E[a:b], P[a:b], B[a:b] = e, p, q
        se[a:b], sc[a:b], sel[a:b], cost = _pick(c, tab, e, ok, g, c["window_s"])
        if keep_cost:
            costs[a:b] = cost
    return {"energy_j": E, "p99_ttft_ms": P, "p99_tbt_ms": B, "flags": None}, se, sc, sel, costs


def _window_sum(c, e):
    e = e.view(c["n_window"], -1)
    return torch.where(torch.isfinite(e), e, torch.zeros_like(e)).sum(1)


def _chain(cost, tr):
    """cost [windows, classes, layouts], +inf where not allowed -> layouts of the least total per class (-1: none), totals."""
    NW, G, L = cost.shape
    pred = np.zeros((NW, G, L), np.int64)
    V = np.empty((NW, G, L))
    gap = ~np.isfinite(cost).any(2)
    total, out = np.zeros(G), np.full((NW, G), -1, np.int64)
    for w in range(NW):
        if w:
            arr = V[w - 1][:, :, None] + tr[None]
            pred[w] = arr.argmin(1)
            arr = np.take_along_axis(arr, pred[w][:, None, :], 1)[:, 0]
            arr = np.where(gap[w - 1][:, None], 0.0, arr)
        else:
            arr = 0.0
        V[w] = np.where(np.isfinite(cost[w]), arr + np.where(np.isfinite(cost[w]), cost[w], 0.0), np.inf)
        ends = ~gap[w] & (gap[w + 1] if w + 1 < NW else True)
        total[ends] += V[w].min(1)[ends]
    state = np.full(G, -1)
    for w in range(NW - 1, -1, -1):
        here = np.where(state < 0, V[w].argmin(1), 0)
        if w + 1 < NW:
            here = np.where(state < 0, here, np.take_along_axis(pred[w + 1], np.maximum(state, 0)[:, None], 1)[:, 0])
        state = np.where(gap[w], -1, here)
        out[w] = state
    return out, total


def _exact_mixed(c, st, tab, slos):
    dev, G, S = torch.device("cuda"), _n_class(c), c["shares"]
    cells = c["n_window"] * G
    U = c["budget"]
    tp, n_max = _tp(c), _n_max(c)
    st_t, st_b = (torch.from_numpy(slos[k]).to(dev) for k in ("slo_ttft_ms", "slo_tbt_ms"))
    best = torch.empty(cells, dtype=torch.float64, device=dev)
    a_sh = torch.arange(1, S + 1, device=dev, dtype=torch.float64)
    f = torch.arange(tab.F, device=dev)
    zero = torch.zeros((), dtype=torch.float64, device=dev)
    step = max(1, int(2e7 // (max(n_max) * S * tab.F)))
    for a in range(0, cells, step):
        b = min(cells, a + step)
        g = (torch.arange(a, b, device=dev) % G)[:, None, None, None]
        D = torch.full((b - a, U + 1, S + 1), math.inf, dtype=torch.float64, device=dev)
        D[:, 0, 0] = 0.0
        for i in range(len(tp)):
            n = torch.arange(1, n_max[i] + 1, device=dev, dtype=torch.float64)[:, None, None]
            load = (st["load"][a:b, None, None, None] * a_sh[:, None]) / S
            pf, tb, pw, ov = tab.look(load, n, g, torch.full_like(f, i), f, zero)
            m = (st["m"][a:b] > 0)[:, None, None, None]
            bad = ov | (st["xp"][a:b, None, None, None] * pf > st_t[g]) | (tb * m > st_b[g])
            E = torch.where(bad, torch.full_like(pw, math.inf), (n * pw) * c["window_s"]).min(3).values
            new = D.clone()
            for q in range(1, n_max[i] + 1):
                k = q * int(tp[i])
                if k > U:
                    break
                for x in range(1, S + 1):
                    new[:, k:, x:] = torch.minimum(new[:, k:, x:], D[:, :U + 1 - k, :S + 1 - x] + E[:, q - 1, x - 1, None, None])
            D = new
        best[a:b] = D[:, :, S].min(1).values
    return {"sel": {"energy_j": best, "n_inst": None, "f_index": None, "share": None, "window_energy_j": _window_sum(c, best), "window_infeasible": None}}


def _exact_hierarchy(c, log, tab, prof, slos):
    dev, G, NW, n_tick = torch.device("cuda"), _n_class(c), c["n_window"], c["n_tick"]
    tick_s = c["window_s"] / n_tick
    co, fi = _stats(c, log, NW, c["window_s"]), _stats(c, log, NW * n_tick, tick_s)
    tr, n_l, t_l = _layouts(c)[1:]
    tp, ew = _tp(c), c["epoch"]
    st_t, st_b = (torch.from_numpy(slos[k]).to(dev) for k in ("slo_ttft_ms", "slo_tbt_ms"))
    n_epoch = -(-NW // ew)
    A = torch.zeros((n_epoch * ew, G), dtype=torch.float64, device=dev)
    A[:NW] = co["load"].view(NW, G)
    A = A.view(n_epoch, ew, G)
    lf = fi["load"].view(NW, n_tick, G)
    epoch = torch.arange(NW, device=dev) // ew
    keep, nodes = torch.ones((n_epoch, G), dtype=torch.float64, device=dev), torch.ones((n_epoch, G), dtype=torch.float64, device=dev)
    node = max(1, 8 // int(tp[-1])) * torch.from_numpy(prof["max_load_tps"][:, -1, -1]).to(dev) * prof["rho"][-1]
    S, Sf = torch.empty_like(A), torch.empty_like(lf)
    fwd, ffwd = torch.zeros_like(A[:, :, 0]), torch.zeros_like(lf[:, :, 0])
    for g in range(G):
        arr = A[:, :, g] + fwd
        peak = arr.max(1).values
        q = peak / node[g]
        spill = (torch.floor(q) >= 1) & (torch.floor(q) < q) if c["spill"] and g < G - 1 else torch.zeros_like(q, dtype=torch.bool)
        nodes[:, g] = torch.where(spill, torch.floor(q), torch.clamp(torch.ceil(q), min=1.0))
        keep[:, g] = torch.where(spill, torch.floor(q) * node[g] / peak * (1.0 - 2.0 ** -40), torch.ones_like(q))
        S[:, :, g] = keep[:, g, None] * arr
        fwd = arr - S[:, :, g]
        af = lf[:, :, g] + ffwd
        Sf[:, :, g] = keep[epoch, g][:, None] * af
        ffwd = af - Sf[:, :, g]
    load = S.reshape(-1, G)[:NW].reshape(-1)
    gi = torch.arange(NW * G, device=dev) % G
    nl, tl = torch.from_numpy(n_l).to(dev), torch.from_numpy(t_l).to(dev).long()
    zero = torch.zeros((), dtype=torch.float64, device=dev)
    fr = torch.full_like(tl, tab.F - 1)
    pf, tb, pw, ov = tab.look(load[:, None], nl.double(), gi[:, None], tl, fr, zero)
    fits = nl * torch.from_numpy(tp).to(dev)[tl] <= (nodes[epoch].reshape(-1) * 8)[:, None]
    bad = ov | (co["xp"][:, None] * pf > st_t[gi][:, None]) | (tb * (co["m"] > 0)[:, None] > st_b[gi][:, None]) | ~fits
    E = torch.where(bad, torch.full_like(pw, math.inf), (nl.double() * pw) * c["window_s"])
    path_cost = None
    if c["overheads"]:
        lay, path_cost = _chain(E.view(NW, G, -1).cpu().numpy(), tr)
        lay = torch.from_numpy(lay.reshape(-1)).to(dev)
    else:
        lay = torch.where(torch.isfinite(E.min(1).values), E.argmin(1), -torch.ones_like(gi))
    some, l = lay >= 0, torch.clamp(lay, min=0)
    n_c, t_c = nl[l].double().view(NW, 1, G, 1), tl[l].view(NW, 1, G, 1)
    energy = torch.zeros((NW, G), dtype=torch.float64, device=dev)
    f = torch.arange(tab.F, device=dev)
    g4 = torch.arange(G, device=dev).view(1, 1, G, 1)
    pf, tb, pw, ov = tab.look(Sf[..., None], n_c, g4, t_c, f, zero)
    bad = ov | (fi["xp"].view(NW, n_tick, G, 1) * pf > st_t.view(1, 1, G, 1)) | (tb * (fi["m"] > 0).view(NW, n_tick, G, 1) > st_b.view(1, 1, G, 1))
    least = torch.where(bad, torch.full_like(pw, math.inf), pw).min(3).values
    power = torch.where(torch.isfinite(least), least, pw[..., -1])
    energy = ((n_c[..., 0] * power) * tick_s).sum(1).reshape(-1)
    energy = torch.where(some, energy, torch.full_like(energy, math.inf))
    out = {"nodes": None, "layout_sel": None, "f_sel": None, "energy_j": energy, "violations": None, "window_energy_j": _window_sum(c, energy), "window_infeasible": None}
    if c["overheads"]:
        out["path_cost"] = torch.from_numpy(path_cost)
    if c["spill"]:
        out["keep"] = keep
    return {"out": out}


def exact(case, seed):
    c = case
    if c["kind"] == "ingest":
        return None
    log = _log_of(c, seed)
    prof = _profile(c, seed)
    slos, tab = _slos(c, prof), _Tables(prof)
    if c["kind"] == "hierarchy":
        return _exact_hierarchy(c, log, tab, prof, slos)
    n_tick = c.get("n_tick", 1)
    st = _stats(c, log, c["n_window"] * n_tick, c["window_s"] / n_tick)
    if c["kind"] == "mixed":
        return _exact_mixed(c, st, tab, slos)
    got = _exact_space(c, st, tab, slos, keep_cost=c["kind"] == "path")
    if got is None:
        return None
    space, se, sc, sel, costs = got
    none = {"sel": None, "window_infeasible": None}
    if c["kind"] == "path":
        lay, tr = _layouts(c)[:2]
        L, NW, G = tr.shape[0], c["n_window"], _n_class(c)
        least = torch.stack([costs[:, torch.from_numpy(np.flatnonzero(lay == l)).cuda()].min(1).values for l in range(L)], 1)
        pick, total = _chain(least.view(NW, G, L).cpu().numpy(), tr)
        pick = torch.from_numpy(pick.reshape(-1)).cuda()
        member = torch.from_numpy(lay).cuda()[None, :] == pick[:, None]
        k = torch.where(member, costs, torch.full_like(costs, math.inf)).argmin(1)
        e = torch.where(pick >= 0, space["energy_j"].gather(1, k[:, None])[:, 0], torch.full_like(se, math.inf))
        return {"sel": {"sel_energy_j": e, "path_cost": torch.from_numpy(total), "window_energy_j": _window_sum(c, e), **none}}
    we = _window_sum(c, se)
    out = {"space": space, "sel": {"sel_energy_j": se, "sel_cost": sc, "window_energy_j": we, **none}}
    if c["kind"] == "plan":
        n, ti = _cand_tensors(c)[:2]
        per = n * torch.from_numpy(_tp(c)).cuda()[ti]
        used = torch.where(sel >= 0, per[torch.clamp(sel, min=0)], torch.zeros_like(se)).view(c["n_window"], -1).sum(1)
        hours, kwh, co2 = used * c["window_s"] / 3600.0, we / 3.6e6, _carbon(c)
        rows = [hours, hours * _PRICE[0], kwh * _PRICE[1], kwh * co2, torch.ceil(used / 8)]
        out["bill"] = {"gpus": None, "gpu_cost": rows[1], "energy_cost": rows[2], "carbon_g": rows[3], "totals": torch.stack([r.sum() for r in rows])}
    return out
