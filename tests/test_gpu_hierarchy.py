"""The controller hierarchy (Section IV-B "Hierarchical Control") on a real MI355X against the CPU oracle."""
import numpy as np
import pytest

import oracle
from workloads import SPECS, make

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

INT_KEYS = ("nodes", "layout_sel", "f_sel", "violations")


@pytest.fixture(scope="module")
def dyn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00741_amd as d
    return d


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _layouts(w, n_max):
    """Every (instances, TP) pair up to n_max instances, TP-major."""
    T = w["profile"]["tp"].size
    lay = [(n, ti) for ti in range(T) for n in range(1, n_max + 1)]
    return np.asarray([l[0] for l in lay], np.int32), np.asarray([l[1] for l in lay], np.int32)


def gpu_hier(dyn, profile, tr, edges, n_window, n_tick, tick_s, epoch_windows, tp_ref, f_ref, gpn, lay_n, lay_tp, slos,
             pct=(99, 100), transition=None, spill=False):
    d = [_dev(tr[k]) for k in ("t_s", "in_tok", "out_tok", "model")]
    ci, co, coff, ws1 = dyn.dyn_trace_ingest(*d, edges, n_window, tick_s * n_tick)
    fi, fo, foff, ws2 = dyn.dyn_trace_ingest(*d, edges, n_window * n_tick, tick_s)
    assert dyn.dyn_workspace_status(ws1) == 0 and dyn.dyn_workspace_status(ws2) == 0
    prof = dyn.dyn_profile_load(profile)
    out, ws = dyn.dyn_hierarchy(prof, (ci, co, coff), (fi, fo, foff), n_window, n_tick, tick_s, epoch_windows, tp_ref, f_ref,
                                gpn, lay_n, lay_tp, slos, pct, transition_j=transition, spill=spill)
    status = dyn.dyn_workspace_status(ws)
    torch.cuda.synchronize()
    r = {k: v.cpu().numpy() for k, v in out.items()}
    r["status"] = status
    coarse = {"in_tok": ci.cpu().numpy(), "out_tok": co.cpu().numpy(), "cell_off": coff.cpu().numpy()}
    fine = {"in_tok": fi.cpu().numpy(), "out_tok": fo.cpu().numpy(), "cell_off": foff.cpu().numpy()}
    prof.free()
    return r, coarse, fine


def assert_same(g, o, n_window, G):
    assert g["status"] == 0
    for k in INT_KEYS:
        np.testing.assert_array_equal(g[k], o[k], err_msg=k)
    np.testing.assert_array_equal(g["energy_j"], o["energy_j"], err_msg="energy_j")
    we, wi = oracle.window_totals(o["layout_sel"], o["energy_j"], n_window, G)
    np.testing.assert_array_equal(g["window_energy_j"], we)
    np.testing.assert_array_equal(g["window_infeasible"], wi)


CASES = {
    # name: (spec, ticks per window, windows per epoch, instances per TP in the layout list, GPUs per node)
    "cfg0-T12": (SPECS[0], 12, 3, 6, 8),
    "cfg0-T7-epoch1": (SPECS[0], 7, 1, 4, 8),
    "cfg1-60k-T12": (SPECS[1].scaled(60_000, 48), 12, 6, 8, 8),
    "cfg2-300k-T12": (SPECS[2].scaled(300_000, 40), 12, 6, 16, 8),
    "cfg3-100k-T4": (SPECS[3].scaled(100_001, 9), 4, 2, 12, 8),
    "cfg4-250k-T6": (SPECS[4].scaled(250_000, 24), 6, 5, 40, 8),
    "cfg2-day-T12": (SPECS[2], 12, 6, 16, 8),                       # full size: a day of 5-minute windows, 25-second ticks
}


@pytest.mark.parametrize("name", list(CASES))
def test_hierarchy_matches_oracle(dyn, name):
    spec, T, epoch, n_max, gpn = CASES[name]
    w = make(spec)
    lay_n, lay_tp = _layouts(w, n_max)
    P = w["profile"]
    tp_ref, f_ref = P["tp"].size - 1, P["f_mhz"].size - 1
    tick = w["window_s"] / T
    g, coarse, fine = gpu_hier(dyn, P, w["trace"], w["edges"], w["n_window"], T, tick, epoch, tp_ref, f_ref, gpn, lay_n, lay_tp,
                               w["slos"], w["pct"])
    st_c = oracle.ingest(w["trace"], w["edges"], w["n_window"], tick * T)
    st_f = oracle.ingest(w["trace"], w["edges"], w["n_window"] * T, tick)
    for a, b in ((coarse, st_c), (fine, st_f)):
        for k in ("in_tok", "out_tok", "cell_off"):
            np.testing.assert_array_equal(a[k], b[k])
    o = oracle.hierarchy(P, st_c, st_f, w["n_window"], T, tick, epoch, tp_ref, f_ref, gpn, lay_n, lay_tp, w["slos"], w["pct"])
    assert_same(g, o, w["n_window"], w["n_class"])
    assert (o["layout_sel"] >= 0).any()
    # the case exercises the lower controller: some tick runs below the reference frequency
    assert (o["f_sel"][o["f_sel"] >= 0] < f_ref).any()


def _gpu_overheads(w, lay_n, lay_tp, unit_j):
    """Overhead table in the shape of the paper's Table VI: proportional to the GPUs whose weights move."""
    gpus = lay_n.astype(np.int64) * w["profile"]["tp"][lay_tp]
    return unit_j * np.abs(gpus[:, None] - gpus[None, :]).astype(np.float64)


@pytest.mark.parametrize("name", ["cfg0-T12", "cfg1-60k-T12", "cfg2-300k-T12", "cfg4-250k-T6", "cfg2-day-T12"])
def test_hierarchy_with_overheads_matches_oracle(dyn, name):
    spec, T, epoch, n_max, gpn = CASES[name]
    w = make(spec)
    lay_n, lay_tp = _layouts(w, min(n_max, 16))           # the sequence selection keeps n_layout^2 overheads in LDS
    P = w["profile"]
    tp_ref, f_ref = P["tp"].size - 1, P["f_mhz"].size - 1
    tick = w["window_s"] / T
    args = (P, w["trace"], w["edges"], w["n_window"], T, tick, epoch, tp_ref, f_ref, gpn, lay_n, lay_tp, w["slos"], w["pct"])
    plain, coarse, fine = gpu_hier(dyn, *args)
    e = plain["energy_j"][np.isfinite(plain["energy_j"])]
    trans = _gpu_overheads(w, lay_n, lay_tp, 0.02 * float(np.median(e)))
    g, _, _ = gpu_hier(dyn, *args, transition=trans)
    o = oracle.hierarchy(P, coarse, fine, w["n_window"], T, tick, epoch, tp_ref, f_ref, gpn, lay_n, lay_tp, w["slos"], w["pct"],
                         transition=trans)
    np.testing.assert_array_equal(g["path_cost"], o["path_cost"])
    assert_same(g, o, w["n_window"], w["n_class"])
    if w["n_window"] > 1:
        changes = lambda a: int((np.diff(a["layout_sel"].reshape(w["n_window"], -1), axis=0) != 0).sum())
        assert changes(g) < changes(plain)                # the overheads do remove layout changes
    # a zero table is the plain hierarchy
    z, _, _ = gpu_hier(dyn, *args, transition=np.zeros_like(trans))
    for k in INT_KEYS + ("energy_j", "window_energy_j", "window_infeasible"):
        np.testing.assert_array_equal(z[k], plain[k], err_msg=k)


@pytest.mark.parametrize("seed", [1, 2, 3, 4, 6, 8])
def test_random_overheads(dyn, seed):
    """Load that rises and falls over 16 windows (layouts change, some windows have no admissible layout, so the
    sequences have gaps) and a random, asymmetric overhead table."""
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(seed, 3, 3, 6000, 16)
    rng = np.random.default_rng(900 + seed)
    tr = dict(tr, t_s=NW * T * tick * rng.beta(2.0, 3.0, tr["t_s"].size))
    slo = {k: v * 1.6 for k, v in slo.items()}
    plain, coarse, fine = gpu_hier(dyn, prof, tr, edges, NW, T, tick, 4, 2, 2, 8, lay_n, lay_tp, slo)
    fin = plain["energy_j"][np.isfinite(plain["energy_j"])]
    trans = rng.uniform(0, 0.3, (lay_n.size, lay_n.size)) * np.median(fin); np.fill_diagonal(trans, 0.0)
    g, _, _ = gpu_hier(dyn, prof, tr, edges, NW, T, tick, 4, 2, 2, 8, lay_n, lay_tp, slo, transition=trans)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, 4, 2, 2, 8, lay_n, lay_tp, slo, transition=trans)
    np.testing.assert_array_equal(g["path_cost"], o["path_cost"])
    assert_same(g, o, NW, 2)
    assert (g["layout_sel"] != plain["layout_sel"]).any() and (g["layout_sel"] < 0).any()


def _node_capacity_for(w, T, nodes_at_peak):
    """Profile of `w` with max_load_tps scaled so that the busiest (window, class) needs `nodes_at_peak` nodes: the
    synthetic profiles leave most pools below one node, where the fragmentation rule has nothing to do."""
    P = dict(w["profile"])
    st = oracle.ingest(w["trace"], w["edges"], w["n_window"], w["window_s"])
    o = st["cell_off"]
    tok = np.concatenate([[0], np.cumsum(st["in_tok"].astype(np.int64) + st["out_tok"])])
    load = ((tok[o[1:]] - tok[o[:-1]]) / w["window_s"]).reshape(w["n_window"], -1)
    cap = P["max_load_tps"][:, -1, -1] * P["rho"][-1]
    P["max_load_tps"] = P["max_load_tps"] * float((load / cap).max() / nodes_at_peak)
    return P


@pytest.mark.parametrize("name", ["cfg0-T12", "cfg0-T7-epoch1", "cfg1-60k-T12", "cfg2-300k-T12", "cfg4-250k-T6", "cfg2-day-T12"])
def test_hierarchy_with_spill_matches_oracle(dyn, name):
    """Section IV-B "Handling fragmentation": node counts, kept fractions and everything the lower controllers decide
    under the loads left after forwarding, bit for bit."""
    spec, T, epoch, n_max, gpn = CASES[name]
    w = make(spec)
    lay_n, lay_tp = _layouts(w, n_max)
    P = _node_capacity_for(w, T, 6.5)
    tp_ref, f_ref = P["tp"].size - 1, P["f_mhz"].size - 1
    tick = w["window_s"] / T
    args = (P, w["trace"], w["edges"], w["n_window"], T, tick, epoch, tp_ref, f_ref, gpn, lay_n, lay_tp, w["slos"], w["pct"])
    g, coarse, fine = gpu_hier(dyn, *args, spill=True)
    o = oracle.hierarchy(P, coarse, fine, w["n_window"], T, tick, epoch, tp_ref, f_ref, gpn, lay_n, lay_tp, w["slos"], w["pct"],
                         spill=True)
    np.testing.assert_array_equal(g["keep"], o["keep"])
    assert_same(g, o, w["n_window"], w["n_class"])
    plain, _, _ = gpu_hier(dyn, *args)
    assert (o["keep"] < 1.0).any() and (o["keep"][:, -1] == 1.0).all()
    assert g["nodes"].sum() < plain["nodes"].sum()        # fewer nodes in all: that is what the rule is for
    assert (o["layout_sel"] >= 0).any()


@pytest.mark.parametrize("seed,n_tick,NW,epoch", [(0, 3, 9, 2), (1, 2, 150, 70), (2, 4, 30, 1000), (3, 1, 7, 3)])
def test_spill_on_random_cases(dyn, seed, n_tick, NW, epoch):
    """Small capacities (pools of several nodes), epochs longer than a wave has lanes and longer than the trace, with
    and without the overhead table."""
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(seed, n_tick, 3, 400 * NW, NW)
    prof = dict(prof, max_load_tps=prof["max_load_tps"] * 0.3)
    slo = {k: v * 1.5 for k, v in slo.items()}
    g, coarse, fine = gpu_hier(dyn, prof, tr, edges, NW, T, tick, epoch, 2, 2, 8, lay_n, lay_tp, slo, spill=True)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, epoch, 2, 2, 8, lay_n, lay_tp, slo, spill=True)
    np.testing.assert_array_equal(g["keep"], o["keep"])
    assert_same(g, o, NW, 2)
    assert (o["keep"][:, 0] < 1.0).any()
    fin = o["energy_j"][np.isfinite(o["energy_j"])]
    trans = np.random.default_rng(seed).uniform(0, 0.2, (lay_n.size, lay_n.size)) * (np.median(fin) if fin.size else 1.0)
    g, _, _ = gpu_hier(dyn, prof, tr, edges, NW, T, tick, epoch, 2, 2, 8, lay_n, lay_tp, slo, transition=trans, spill=True)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, epoch, 2, 2, 8, lay_n, lay_tp, slo, transition=trans, spill=True)
    np.testing.assert_array_equal(g["keep"], o["keep"])
    np.testing.assert_array_equal(g["path_cost"], o["path_cost"])
    assert_same(g, o, NW, 2)


def _random_case(seed, n_tick, n_f, R, NW):
    """Small random profile (not monotone across TP or frequency), two classes, nine random layouts."""
    rng = np.random.default_rng(4100 + seed)
    n_tp, n_rho, G = 3, 4, 2
    fg = np.sort(rng.uniform(600, 2000, n_f))
    rg = np.concatenate([[0.0], np.sort(rng.uniform(0.1, 0.95, n_rho - 1))])
    shape = (G, n_tp, n_f, n_rho)
    prof = {"tp": np.asarray([2, 4, 8], np.int32), "f_mhz": fg, "rho": rg,
            "prefill_ms_per_tok": rng.uniform(0.02, 0.1, shape),
            "tbt_ms": np.sort(rng.uniform(10, 150, shape), axis=-1),
            "power_w": np.sort(rng.uniform(100, 3000, shape), axis=-1),
            "max_load_tps": rng.uniform(300, 1500, shape[:3])}
    tick = 5.0
    tr = {"t_s": rng.uniform(0, NW * n_tick * tick, R), "in_tok": rng.integers(1, 500, R).astype(np.int32),
          "out_tok": rng.integers(1, 300, R).astype(np.int32), "model": np.zeros(R, np.int32)}
    edges = {"in_edge": np.asarray([[200]], np.int32), "out_edge": np.zeros((1, 0), np.int32)}
    slo = {"slo_ttft_ms": rng.uniform(25, 70, G), "slo_tbt_ms": rng.uniform(80, 150, G)}
    lay_n = rng.integers(1, 6, 9).astype(np.int32)
    lay_tp = rng.integers(0, n_tp, 9).astype(np.int32)
    return prof, tr, edges, slo, lay_n, lay_tp, NW, n_tick, tick


@pytest.mark.parametrize("seed,n_tick,n_f,R,NW,epoch", [(0, 3, 3, 500, 5, 2), (1, 1, 1, 300, 4, 4), (2, 5, 7, 3000, 9, 3),
                                                        (3, 2, 2, 40, 6, 1), (4, 16, 4, 20_000, 11, 100)])
def test_random_profiles_and_layouts(dyn, seed, n_tick, n_f, R, NW, epoch):
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(seed, n_tick, n_f, R, NW)
    g, coarse, fine = gpu_hier(dyn, prof, tr, edges, NW, T, tick, epoch, 2, n_f - 1, 8, lay_n, lay_tp, slo)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, epoch, 2, n_f - 1, 8, lay_n, lay_tp, slo)
    assert_same(g, o, NW, 2)
    # violations and infeasible windows both occur across these seeds; here only: the arrays agree
    assert o["nodes"].min() >= 1


def _on_grid(prof, rg, seed):
    """The profile's capacities with random tables over the load points `rg`."""
    rng = np.random.default_rng(seed)
    shape = prof["max_load_tps"].shape + (rg.size,)
    return dict(prof, rho=rg, prefill_ms_per_tok=rng.uniform(0.02, 0.1, shape), tbt_ms=np.sort(rng.uniform(10, 150, shape), axis=-1),
                power_w=np.sort(rng.uniform(100, 3000, shape), axis=-1))


@pytest.mark.parametrize("kind,n_rho,NW", [("even", 1500, 5), ("even", 1800, 5), ("even", 1800, 800), ("jitter", 1000, 5), ("jitter", 1000, 800), ("uneven", 300, 9),
                                           ("uneven", 3000, 5), ("uneven", 3000, 700), ("even", 4500, 3), ("uneven", 9700, 3)])
def test_long_load_axes(dyn, kind, n_rho, NW):
    """Axes that a block keeps in LDS, and that it reads from global memory because they are long or the blocks many, in every form."""
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(n_rho, 2, 3, 400 + 8 * NW, NW)
    rg = np.linspace(0.0, 0.95, n_rho)
    if kind == "jitter":
        rg = rg * (1.0 + 1e-9 * np.sin(np.arange(n_rho)))
    if kind == "uneven":
        rg = np.r_[0.0, np.geomspace(0.01, 0.95, n_rho - 1)]
    prof = _on_grid(prof, rg, n_rho)
    slo = {k: v * 2.0 for k, v in slo.items()}          # so that every axis has windows with a layout
    g, coarse, fine = gpu_hier(dyn, prof, tr, edges, NW, T, tick, 3, 2, 2, 8, lay_n, lay_tp, slo)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, 3, 2, 2, 8, lay_n, lay_tp, slo)
    assert_same(g, o, NW, 2)
    assert (o["layout_sel"] >= 0).any()


def test_load_axes_beyond_what_is_taken(dyn):
    """9730 points, with their bucket index, are the longest axis that fits a compute unit's LDS; more are refused."""
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(0, 2, 3, 300, 3)
    prof = _on_grid(prof, np.linspace(0.0, 0.95, 9800), 1)
    with pytest.raises(dyn.DynError):
        gpu_hier(dyn, prof, tr, edges, NW, T, tick, 3, 2, 2, 8, lay_n, lay_tp, slo)


@pytest.mark.parametrize("n_tick,n_f", [(64, 3), (65, 3), (130, 2), (3, 128), (3, 129), (70, 150)])
def test_many_ticks_and_many_frequencies(dyn, n_tick, n_f):
    """More ticks than a block keeps at a time, whose sums and violations run on, and more frequencies than it tables."""
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(11, n_tick, n_f, 40 * n_tick, 4)
    prof = dict(prof, max_load_tps=prof["max_load_tps"] * 0.3)
    g, coarse, fine = gpu_hier(dyn, prof, tr, edges, NW, T, tick, 2, 2, n_f - 1, 8, lay_n, lay_tp, slo)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, 2, 2, n_f - 1, 8, lay_n, lay_tp, slo)
    assert_same(g, o, NW, 2)
    assert (o["layout_sel"] >= 0).any() and o["violations"].sum() > 0


@pytest.mark.parametrize("G,n_tick,NW", [(1, 1, 5003), (1, 5, 1030), (1, 12, 2017), (1, 65, 600), (3, 5, 2000), (9, 12, 1025), (25, 12, 7), (48, 12, 3), (100, 12, 5)])
def test_windows_and_classes_packed_into_blocks(dyn, G, n_tick, NW):
    """Blocks of several windows (the last not full), of more look-ups than threads, and runs of classes; some cells without a layout, some without requests."""
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(G, n_tick, 3, 40 * n_tick * G + 6 * NW * n_tick, NW)
    rng = np.random.default_rng(G)
    a = 1 if G in (1, 3) else {9: 3, 25: 5, 48: 6, 100: 10}[G]
    edges = {"in_edge": np.linspace(1, 500, a + 1)[1:-1].astype(np.int32).reshape(1, -1), "out_edge": np.linspace(1, 300, G // a + 1)[1:-1].astype(np.int32).reshape(1, -1)}
    shape = (G,) + prof["tbt_ms"].shape[1:]
    prof = dict(prof, prefill_ms_per_tok=rng.uniform(0.02, 0.1, shape), tbt_ms=np.sort(rng.uniform(10, 150, shape), axis=-1), power_w=np.sort(rng.uniform(100, 3000, shape), axis=-1),
                max_load_tps=rng.uniform(300, 1500, shape[:3]) * (0.3 / min(G, 2)))
    slo = {"slo_ttft_ms": rng.uniform(25, 70, G), "slo_tbt_ms": rng.uniform(80, 150, G)}
    g, coarse, fine = gpu_hier(dyn, prof, tr, edges, NW, T, tick, 5, 2, 2, 8, lay_n, lay_tp, slo)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, 5, 2, 2, 8, lay_n, lay_tp, slo)
    assert_same(g, o, NW, G)
    assert (o["layout_sel"] >= 0).any() and (o["layout_sel"] < 0).any()


def test_more_than_64_layouts_and_ties(dyn):
    """Layout list longer than a wave with repeated entries: the lowest index of equal energies is chosen."""
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(5, 4, 3, 4000, 6)
    lay_n = np.tile(lay_n, 23)[:200]; lay_tp = np.tile(lay_tp, 23)[:200]
    g, coarse, fine = gpu_hier(dyn, prof, tr, edges, NW, T, tick, 2, 2, 2, 8, lay_n, lay_tp, slo)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, 2, 2, 2, 8, lay_n, lay_tp, slo)
    assert_same(g, o, NW, 2)
    assert (o["layout_sel"] < 9).all()


def test_load_grid_with_points_closer_than_a_bucket(dyn):
    """Grid points 1e-5 apart: several fall into one bucket of the load-axis index, which then only
    narrows the bracket search instead of deciding it."""
    prof, tr, edges, slo, lay_n, lay_tp, NW, T, tick = _random_case(6, 4, 5, 6000, 8)
    rng = np.random.default_rng(77)
    rg = np.asarray([0.0, 0.2, 0.41, 0.41001, 0.41002, 0.41003, 0.7, 0.95])
    shape = prof["tbt_ms"].shape[:3] + (rg.size,)
    prof = dict(prof, rho=rg, prefill_ms_per_tok=rng.uniform(0.02, 0.1, shape),
                tbt_ms=np.sort(rng.uniform(10, 150, shape), axis=-1), power_w=np.sort(rng.uniform(100, 3000, shape), axis=-1))
    g, coarse, fine = gpu_hier(dyn, prof, tr, edges, NW, T, tick, 3, 2, 4, 8, lay_n, lay_tp, slo)
    o = oracle.hierarchy(prof, coarse, fine, NW, T, tick, 3, 2, 4, 8, lay_n, lay_tp, slo)
    assert_same(g, o, NW, 2)
    assert (o["layout_sel"] >= 0).any()


def test_tight_slo_counts_violations_and_marks_infeasible_windows(dyn):
    w = make(SPECS[0])
    P = w["profile"]
    T = 6
    tick = w["window_s"] / T
    lay_n, lay_tp = _layouts(w, 3)
    slos = {k: v * 0.3 for k, v in w["slos"].items()}
    tp_ref, f_ref = P["tp"].size - 1, P["f_mhz"].size - 1
    g, coarse, fine = gpu_hier(dyn, P, w["trace"], w["edges"], w["n_window"], T, tick, 4, tp_ref, f_ref, 8, lay_n, lay_tp, slos,
                               w["pct"])
    o = oracle.hierarchy(P, coarse, fine, w["n_window"], T, tick, 4, tp_ref, f_ref, 8, lay_n, lay_tp, slos, w["pct"])
    assert_same(g, o, w["n_window"], w["n_class"])
    assert o["violations"].sum() > 0 and (o["layout_sel"] < 0).any()


def test_empty_trace(dyn):
    w = make(SPECS[0])
    P = w["profile"]
    tr = {k: v[:0] for k, v in w["trace"].items()}
    lay_n, lay_tp = _layouts(w, 2)
    g, coarse, fine = gpu_hier(dyn, P, tr, w["edges"], 4, 3, 10.0, 2, 0, 0, 8, lay_n, lay_tp, w["slos"])
    o = oracle.hierarchy(P, coarse, fine, 4, 3, 10.0, 2, 0, 0, 8, lay_n, lay_tp, w["slos"])
    assert_same(g, o, 4, w["n_class"])
    assert (g["nodes"] == 1).all() and (g["violations"] == 0).all()


def test_argument_errors(dyn):
    w = make(SPECS[0])
    P = w["profile"]
    lay_n, lay_tp = _layouts(w, 2)
    d = [_dev(w["trace"][k]) for k in ("t_s", "in_tok", "out_tok", "model")]
    T = 3
    tick = w["window_s"] / T
    c = dyn.dyn_trace_ingest(*d, w["edges"], w["n_window"], w["window_s"])[:3]
    f = dyn.dyn_trace_ingest(*d, w["edges"], w["n_window"] * T, tick)[:3]
    prof = dyn.dyn_profile_load(P)
    args = dict(n_window=w["n_window"], n_tick=T, tick_s=tick, epoch_windows=2, tp_ref_index=0, f_ref_index=0, gpus_per_node=8,
                lay_n=lay_n, lay_tp_index=lay_tp, slos=w["slos"])
    for bad in (dict(epoch_windows=0), dict(tp_ref_index=P["tp"].size), dict(f_ref_index=-1), dict(gpus_per_node=0),
                dict(lay_n=np.zeros_like(lay_n)), dict(lay_tp_index=lay_tp + 100)):
        with pytest.raises(dyn.DynError):
            dyn.dyn_hierarchy(prof, c, f, **{**args, **bad})
    with pytest.raises((dyn.DynError, ValueError)):         # the coarse trace in place of the tick-level one
        dyn.dyn_hierarchy(prof, c, c, **args)
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(dyn.DynError):
        dyn.dyn_hierarchy(prof, c, f, **args, workspace=ws)
    many_n = np.tile(lay_n, 40); many_tp = np.tile(lay_tp, 40)         # 240 layouts: fine without overheads, too many with
    dyn.dyn_hierarchy(prof, c, f, **{**args, "lay_n": many_n, "lay_tp_index": many_tp})
    with pytest.raises(dyn.DynError):
        dyn.dyn_hierarchy(prof, c, f, **{**args, "lay_n": many_n, "lay_tp_index": many_tp},
                          transition_j=np.zeros((many_n.size, many_n.size)))
    bad_t = np.zeros((lay_n.size, lay_n.size)); bad_t[0, 1] = -1.0
    with pytest.raises(dyn.DynError):
        dyn.dyn_hierarchy(prof, c, f, **args, transition_j=bad_t)
    bad_t[0, 1] = np.nan
    with pytest.raises(dyn.DynError):
        dyn.dyn_hierarchy(prof, c, f, **args, transition_j=bad_t)
    out, _ = dyn.dyn_hierarchy(prof, c, f, **args)
    torch.cuda.synchronize()
    assert out["nodes"].min().item() >= 1
    prof.free()


def test_workspaces_of_every_size_that_is_taken(dyn):
    """The path's pieces and the long cells' scratch follow the least workspace, in this order of need: without either, with the
    scratch alone, a word short of the pieces, with all.  Outputs are the same; a word short of the least is refused."""
    NW, T, n_lay, G = 300, 1, 9, 1
    prof, _, _, slo, lay_n, lay_tp, _, _, tick = _random_case(2, 3, 3, 600, 6)
    prof = {k: (v[:G] if v.ndim >= 3 else v) for k, v in prof.items()}
    slo = {k: np.full(G, 1e9) for k in slo}
    rng = np.random.default_rng(17)
    n = 9001 * NW * T + 1                                  # long cells at both levels
    off = np.concatenate([[0], np.sort(rng.integers(0, n + 1, NW - 1)), [n]]).astype(np.int64)
    x, y = (_dev(rng.integers(1, 4000, n).astype(np.int32)) for _ in range(2))
    trace = (x, y, _dev(off))
    tok = np.diff(np.concatenate([[0], np.cumsum(x.cpu().numpy().astype(np.int64) + y.cpu().numpy())])[off]) / tick
    prof["max_load_tps"] = prof["max_load_tps"] * (tok.max() / prof["max_load_tps"].mean() / 3.0)      # some windows need several instances
    h = dyn.dyn_profile_load(prof)
    trans = rng.uniform(0.0, 1.0, (n_lay, n_lay)) * 0.05 * 300.0 * tick
    np.fill_diagonal(trans, 0.0)
    up = lambda b: (b + 255) // 256 * 256   # noqa: E731
    full = dyn.dyn_hierarchy_workspace(NW, T, G, n_lay)
    pieces = 2 * up(NW * G * n_lay * 8) + up(G * 4)
    scratch = up(4 * (64 + 1024 + 1088 + 2048 * min(1024, 4 * NW * G * T)))
    sizes = {"least": full - pieces - scratch, "no pieces": full - pieces, "almost": full - 256, "all": full}
    call = lambda b: dyn.dyn_hierarchy(h, trace, trace, NW, T, tick, 4, 2, 2, 8, lay_n[:n_lay], lay_tp[:n_lay], slo, transition_j=trans,   # noqa: E731
                                       workspace=torch.empty(b, dtype=torch.uint8, device="cuda"))
    out = {}
    for k, b in sizes.items():
        out[k], ws = call(b)
        assert dyn.dyn_workspace_status(ws) == 0
        for q in out[k]:
            assert torch.equal(out[k][q], out["least"][q]), (k, q)
    st = {"in_tok": x.cpu().numpy(), "out_tok": y.cpu().numpy(), "cell_off": off}
    o = oracle.hierarchy(prof, st, st, NW, T, tick, 4, 2, 2, 8, lay_n[:n_lay], lay_tp[:n_lay], slo, transition=trans)
    assert_same({**{k: v.cpu().numpy() for k, v in out["all"].items()}, "status": 0}, o, NW, G)
    np.testing.assert_array_equal(out["all"]["path_cost"].cpu().numpy(), o["path_cost"])
    assert (o["layout_sel"] >= 0).any()
    with pytest.raises(dyn.DynError):
        call(sizes["least"] - 256)
    h.free()
