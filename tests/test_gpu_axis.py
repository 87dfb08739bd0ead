"""Forms of the load axis (evenly spaced points, buckets, search) on a real MI355X against the CPU oracle, with loads that fall on the
points and a rounding beside them, and TBT rows for which only some ticks are asked."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_hierarchy import _layouts, assert_same as same_hierarchy, gpu_hier
from tests.test_gpu_mixed import check as same_mixed, gpu_mixed
from tests.test_gpu_ticks import assert_same, gpu_ticks, ora_ticks
from workloads import SPECS, make

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dyn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00741_amd as d
    return d


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


GRIDS = {
    "two": np.asarray([0.0, 0.95]),
    "even": np.linspace(0.0, 0.95, 33),
    "summed": np.cumsum(np.r_[0.0, np.full(40, 0.95 / 40)]),                       # spacings a few roundings apart
    "many": np.linspace(0.0, 0.95, 900),                                           # a row of 21 KB
    "jitter": np.linspace(0.0, 0.95, 33) * (1.0 + 1e-9 * np.sin(np.arange(33.0))),    # more than the even form allows
    "late": np.linspace(0.0, 0.95, 33) + np.r_[0.0, np.linspace(0.3, 0.9, 31), 0.0] * (0.95 / 32),    # points late in their buckets
    "crowded": np.linspace(0.0, 0.95, 33) + np.r_[0.0, np.full(31, 0.95), 0.0] * (0.95 / 32),      # so late that the even form takes them
    "uneven": np.r_[0.0, np.geomspace(0.01, 0.95, 20)],
}


def _case(grid, tbt, n_req=4000, NW=3):
    """A profile over `grid` whose capacities put the cells' loads (and half of them) on grid points, up to the rounding of a quotient."""
    w = make(SPECS[1].scaled(n_req, NW))
    rng = np.random.default_rng(len(grid))
    P, G = w["profile"], w["n_class"]
    n_tp, n_f, R = P["tp"].size, 4, grid.size
    w["configs"] = {"n_inst": np.tile(np.arange(1, 9), n_tp * n_f).astype(np.int32), "tp_index": np.repeat(np.arange(n_tp), 8 * n_f).astype(np.int32),
                    "f_mhz": np.tile(np.repeat(P["f_mhz"][:n_f], 8), n_tp).astype(float)}
    st = oracle.ingest(w["trace"], w["edges"], NW, w["window_s"])
    tok = np.asarray([st["in_tok"][a:b].sum() + st["out_tok"][a:b].sum() for a, b in zip(st["cell_off"][:-1], st["cell_off"][1:])]).reshape(NW, G)
    load = np.maximum(tok, 1) / w["window_s"]
    shape = (G, n_tp, n_f)
    at = rng.integers(1, R, shape)
    ml = load[rng.integers(0, NW, shape), np.arange(G)[:, None, None]] / (grid[at] * rng.integers(1, 9, shape))
    base = rng.uniform(5.0, 40.0, shape)[..., None]
    tb = {"rising": base / (1.0 - grid), "capped": np.minimum(base / (1.0 - grid), 1.5 * base), "flat": base + 0.0 * grid, "level": base * (1.0 + 1e-14 * np.arange(R)),
          "falling": base * (2.0 - grid)}[tbt]
    w["profile"] = {"tp": P["tp"], "f_mhz": P["f_mhz"][:n_f], "rho": grid, "max_load_tps": ml, "tbt_ms": tb, "prefill_ms_per_tok": rng.uniform(0.05, 0.2, shape)[..., None] + 0.0 * grid,
                    "power_w": rng.uniform(100.0, 200.0, shape)[..., None] * (1.0 + grid)}
    w["slos"] = {"slo_ttft_ms": np.full(G, 400.0), "slo_tbt_ms": np.full(G, 60.0)}
    return w, st


@pytest.mark.parametrize("tbt", ["rising", "capped", "flat", "level", "falling"])
@pytest.mark.parametrize("grid", list(GRIDS))
def test_every_form_of_the_axis(dyn, grid, tbt):
    w, st = _case(GRIDS[grid], tbt)
    prof = dyn.dyn_profile_load(w["profile"])
    space, sel, ws = dyn.dyn_eval_select(prof, _dev(st["in_tok"]), _dev(st["out_tok"]), _dev(st["cell_off"]), w["n_window"], w["window_s"],
                                         dyn.Plan(w["configs"], w["slos"], w["pct"], None, 0.1))
    o = oracle.evaluate(w["profile"], st, w["n_window"], w["window_s"], w["configs"], w["slos"], w["pct"], None, 0.1)
    for k in ("energy_j", "p99_ttft_ms", "p99_tbt_ms", "flags"):
        np.testing.assert_array_equal(space[k].cpu().numpy(), o[k], err_msg=k)
    np.testing.assert_array_equal(sel["sel"].cpu().numpy(), o["sel"])
    prof.free()
    for n_tick in (1, 2, 5, 40):
        g, fine = gpu_ticks(dyn, w, n_tick)
        assert g["status"] == 0
        assert_same(w, g, ora_ticks(w, fine, n_tick))
    n_max = [3] * w["profile"]["tp"].size
    if grid != "many":                       # whose rows mixed pools refuse: four of them do not fit in LDS
        g, s = gpu_mixed(dyn, w, 4, n_max)
        same_mixed(w, g, oracle.mixed(w["profile"], s, w["n_window"], w["window_s"], 4, n_max, w["slos"], w["pct"], None, want_types=True), 4, n_max, None)
    lay_n, lay_tp = _layouts(w, 4)
    tick = w["window_s"] / 5
    g, _, _ = gpu_hier(dyn, w["profile"], w["trace"], w["edges"], w["n_window"], 5, tick, 2, w["profile"]["tp"].size - 1, 3, 8, lay_n, lay_tp, w["slos"], w["pct"])
    st_f = oracle.ingest(w["trace"], w["edges"], w["n_window"] * 5, tick)
    o = oracle.hierarchy(w["profile"], st, st_f, w["n_window"], 5, tick, 2, w["profile"]["tp"].size - 1, 3, 8, lay_n, lay_tp, w["slos"], w["pct"])
    same_hierarchy(g, o, w["n_window"], w["n_class"])


@pytest.mark.parametrize("apart", [0, 1, 3, 1 << 10, 1 << 20])
def test_ticks_whose_loads_are_close(dyn, apart):
    """One class, ticks of the same number of tokens or `apart` more in one: which tick has the largest TBT is then a matter of roundings.  Lengths of
    2^16 and more: the cell is walked with lists, which asks every tick."""
    w, _ = _case(GRIDS["even"], "rising", 2000, 1)
    n_tick, per = 8, 12
    n = n_tick * per
    rng = np.random.default_rng(apart)
    x = np.tile(rng.permutation(np.arange(1 << 18, (1 << 18) + per)), n_tick).astype(np.int64)
    x[per * int(rng.integers(n_tick))] += apart
    w["trace"] = {"t_s": (np.repeat(np.arange(n_tick), per) + 0.5) * (w["window_s"] / n_tick), "in_tok": x.astype(np.int32), "out_tok": np.ones(n, np.int32), "model": np.zeros(n, np.int32)}
    P = w["profile"]
    total = x.sum() / w["window_s"]
    P["max_load_tps"][...] = total / (4.0 * P["rho"][np.random.default_rng(1).integers(1, 33, P["max_load_tps"].shape)])
    g, fine = gpu_ticks(dyn, w, n_tick, pct=(90, 100))
    assert g["status"] == 0
    assert_same(w, g, ora_ticks(w, fine, n_tick, pct=(90, 100)))


DENSE, GENERAL, TIGHT = 1, 16, 32               # of a cell's plan


def _close_case(tokens, seed):
    """One populated cell of 6 ticks of 680 requests whose loads are `tokens`, the same again, and 1 to 400 fewer (2^-20 is 32 to 38 of them), and TBT
    rows that rise by so little that a token is about a rounding, or less, with utilizations on both sides of the rows' bounds; capacities put the
    largest load on, below and above grid points and the last one."""
    w, _ = _case(GRIDS["even"], "rising", 2000, 1)
    rng = np.random.default_rng(seed)
    n_tick, per, P = 6, 680, w["profile"]
    w["window_s"] = float(n_tick)               # a tick of one second: loads are token counts
    x = rng.integers(tokens // per - 2500, tokens // per + 2500, (n_tick, per))
    lack = tokens - np.asarray([0, 0, 1, 40, 200, 400])[rng.permutation(n_tick)] - per - x.sum(1)      # an output token each
    x += (lack // per)[:, None]
    x[:, 0] += lack % per
    x = x[:, rng.permutation(per)]
    assert x.min() > 1000 and x.max() < 65535
    w["trace"] = {"t_s": np.repeat(np.arange(n_tick), per) + 0.5, "in_tok": x.ravel().astype(np.int32), "out_tok": np.ones(n_tick * per, np.int32), "model": np.zeros(n_tick * per, np.int32)}
    n_tp, n_f, rho = P["tp"].size, 16, P["rho"]
    w["configs"] = {"n_inst": np.tile(np.arange(1, 9), n_tp * n_f).astype(np.int32), "tp_index": np.repeat(np.arange(n_tp), 8 * n_f).astype(np.int32),
                    "f_mhz": np.tile(np.repeat(1000.0 + np.arange(n_f), 8), n_tp)}
    shape = (w["n_class"], n_tp, n_f)
    at = np.r_[rho[-1] * np.asarray([1.0, 1.0 - 2.0 ** -21, 1.0 + 2.0 ** -21, 1.0 + 1e-9, 1.2]), 0.7, 0.3, rho[rng.integers(1, 32, 5)]]
    rise = rng.choice([1e-3, 0.1, 1.0, 1.1, 2.0, 5.0, 100.0, 1e4], shape)[..., None]      # the bound is near 1 / rise
    w["profile"] = {"tp": P["tp"], "f_mhz": 1000.0 + np.arange(n_f), "rho": rho, "max_load_tps": tokens / (rng.choice(at, shape) * rng.integers(1, 4, shape)),
                    "prefill_ms_per_tok": rng.uniform(0.005, 0.02, shape)[..., None] + 0.0 * rho, "power_w": rng.uniform(100.0, 200.0, shape)[..., None] * (1.0 + rho),
                    "tbt_ms": rng.uniform(5.0, 40.0, shape)[..., None] * (1.0 + rise * 2.0 ** -28 * rho)}
    return w, n_tick


@pytest.mark.parametrize("tokens", [1 << 25, (1 << 25) + 1, (1 << 25) + 33, 40_000_003])
def test_walk_without_lists_and_close_loads(dyn, tokens):
    """Which tick has the largest TBT is then a matter of roundings, and the walk without lists asks only ticks near the largest load."""
    for seed in range(6):
        w, n_tick = _close_case(tokens, seed)
        prof = dyn.dyn_profile_load(w["profile"])
        ins, outs, off, _ = dyn.dyn_trace_ingest(*(_dev(w["trace"][k]) for k in ("t_s", "in_tok", "out_tok", "model")), w["edges"], n_tick, 1.0)
        space, sel, ws = dyn.dyn_eval_select_ticks(prof, ins, outs, off, 1, n_tick, 1.0, dyn.Plan(w["configs"], w["slos"], (90, 100), None, 0.0))
        torch.cuda.synchronize()
        fine = {"in_tok": ins.cpu().numpy(), "out_tok": outs.cpu().numpy(), "cell_off": off.cpu().numpy()}
        o = oracle.evaluate_ticks(w["profile"], fine, 1, n_tick, 1.0, w["configs"], w["slos"], (90, 100), None, 0.0)
        for k in ("energy_j", "p99_ttft_ms", "p99_tbt_ms", "flags"):
            np.testing.assert_array_equal(space[k].cpu().numpy(), o[k], err_msg=k)
        np.testing.assert_array_equal(sel["sel"].cpu().numpy(), o["sel"])
        # the cell's plan in the workspace: j, x_j, flags
        j = fine["in_tok"].size - -(-90 * fine["in_tok"].size // 100) + 1
        words = ws[: ws.numel() // 4 * 4].view(torch.int32).cpu().numpy()
        i = np.flatnonzero((words[:-3] == j) & (words[1:-2] == np.sort(fine["in_tok"])[-j]))
        assert i.size == 1 and words[i[0] + 2] & (DENSE | GENERAL | TIGHT) == DENSE | TIGHT
        prof.free()


def test_blocks_of_many_windows_and_of_few(dyn):
    """Cells enough for the walk to begin with blocks of many windows: 25 classes in 1440 windows, the last block not full."""
    w = make(SPECS[2].scaled(150_000, 1439))
    g, fine = gpu_ticks(dyn, w, 12)
    assert g["status"] == 0
    assert_same(w, g, ora_ticks(w, fine, 12))


def test_powers_of_zero_with_a_sign(dyn):
    """-0.0 passes as a power: its energy is the least, equal to that of +0.0, for every entry point that selects."""
    w, st = _case(GRIDS["even"], "rising")
    P, NW, G = w["profile"], w["n_window"], w["n_class"]
    P["power_w"][:, 1] = -0.0
    P["power_w"][:, 2, ::2] = 0.0
    P["max_load_tps"] *= 4.0
    prof = dyn.dyn_profile_load(P)
    for idle in (0.0, 0.1):
        _, sel, _ = dyn.dyn_eval_select(prof, _dev(st["in_tok"]), _dev(st["out_tok"]), _dev(st["cell_off"]), NW, w["window_s"], dyn.Plan(w["configs"], w["slos"], w["pct"], None, idle))
        o = oracle.evaluate(P, st, NW, w["window_s"], w["configs"], w["slos"], w["pct"], None, idle)
        np.testing.assert_array_equal(sel["sel"].cpu().numpy(), o["sel"])
    prof.free()
    g, fine = gpu_ticks(dyn, w, 5)
    assert_same(w, g, ora_ticks(w, fine, 5))
    n_max = [3] * P["tp"].size
    g, s = gpu_mixed(dyn, w, 4, n_max)
    same_mixed(w, g, oracle.mixed(P, s, NW, w["window_s"], 4, n_max, w["slos"], w["pct"], None, want_types=True), 4, n_max, None)
    tick = w["window_s"] / 5
    st_f = oracle.ingest(w["trace"], w["edges"], NW * 5, tick)
    lay_n, lay_tp = _layouts(w, 4)
    for keep in (lay_tp != 2, lay_tp >= 0):
        g, _, _ = gpu_hier(dyn, P, w["trace"], w["edges"], NW, 5, tick, 2, 0, 3, 64, lay_n[keep], lay_tp[keep], w["slos"], w["pct"])
        o = oracle.hierarchy(P, st, st_f, NW, 5, tick, 2, 0, 3, 64, lay_n[keep], lay_tp[keep], w["slos"], w["pct"])
        same_hierarchy(g, o, NW, G)
        assert (o["energy_j"] == 0.0).any()
