"""Calls on small problems beside a kernel of another stream that fills the device: their blocks fit beside it."""
import numpy as np
import pytest

from tests.beside import calls_through_early
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


@pytest.mark.parametrize("n_win", [60, 487])
def test_account(dyn, n_win):
    w = make(SPECS[1].scaled(1000, 2))
    G = w["n_class"]
    prof = dyn.dyn_profile_load(w["profile"])
    plan = dyn.Plan(w["configs"], w["slos"], w["pct"], None, 0.0)
    rng = np.random.default_rng(n_win)
    sel = _dev(rng.integers(-1, w["configs"]["n_inst"].size, n_win * G).astype(np.int32))
    e, ci = _dev(rng.uniform(0.0, 1e9, n_win)), _dev(rng.uniform(80.0, 700.0, n_win))
    early, _ = calls_through_early(lambda: dyn.dyn_account(prof, sel, e, plan, n_win, 300.0, 11.06, 0.0832, ci, 8))
    prof.free()
    assert early >= 2, early


@pytest.mark.parametrize("n_win", [1, 60])
@pytest.mark.parametrize("idle", [0.0, 0.1])
def test_evaluate_and_select(dyn, n_win, idle):
    w = make(SPECS[1].scaled(2500 * n_win, n_win))
    tr = w["trace"]
    ins, outs, off, _ = dyn.dyn_trace_ingest(_dev(tr["t_s"]), _dev(tr["in_tok"]), _dev(tr["out_tok"]), _dev(tr["model"]), w["edges"], n_win, w["window_s"])
    prof = dyn.dyn_profile_load(w["profile"])
    plan = dyn.Plan(w["configs"], w["slos"], w["pct"], None, idle)
    early, (space, ws) = calls_through_early(lambda: dyn.dyn_eval_space(prof, ins, outs, off, n_win, w["window_s"], plan))
    assert early >= 2, early
    early, _ = calls_through_early(lambda: dyn.dyn_eval_select(prof, ins, outs, off, n_win, w["window_s"], plan))
    assert early >= 2, early
    early, sel = calls_through_early(lambda: dyn.dyn_select_config(prof, space, n_win, w["window_s"], plan))
    assert early >= 2, early
    prof.free()


def test_ticks(dyn):
    """An hour of 540 cells whose lists the block kernel builds."""
    w = make(SPECS[1].scaled(60_000, 60))
    tr, T = w["trace"], 12
    ins, outs, off, _ = dyn.dyn_trace_ingest(_dev(tr["t_s"]), _dev(tr["in_tok"]), _dev(tr["out_tok"]), _dev(tr["model"]), w["edges"], 60 * T, w["window_s"] / T)
    prof = dyn.dyn_profile_load(w["profile"])
    plan = dyn.Plan({k: v[:8] for k, v in w["configs"].items()}, w["slos"], w["pct"], None, 0.0)
    early, _ = calls_through_early(lambda: dyn.dyn_eval_select_ticks(prof, ins, outs, off, 60, T, w["window_s"] / T, plan))
    prof.free()
    assert early >= 2, early


@pytest.mark.parametrize("n_layout", [12, 48, 64])
def test_path(dyn, n_layout):
    """Sequences over enough windows for the walk in pieces."""
    n_win = 320
    w = make(SPECS[1].scaled(1000, 2))
    G, rng = w["n_class"], np.random.default_rng(n_layout)
    cfg = {"n_inst": rng.integers(1, 5, n_layout).astype(np.int32), "tp_index": np.zeros(n_layout, np.int32), "f_mhz": np.full(n_layout, w["profile"]["f_mhz"][0])}
    prof = dyn.dyn_profile_load(w["profile"])
    plan = dyn.Plan(cfg, w["slos"], w["pct"], None, 0.0)
    space = {"energy_j": _dev(rng.uniform(1e4, 5e4, (n_win * G, n_layout))), "flags": _dev(np.ones((n_win * G, n_layout), np.uint8))}
    tr = rng.uniform(0.0, 1e4, (n_layout, n_layout))
    early, _ = calls_through_early(lambda: dyn.dyn_select_path(prof, space, n_win, 60.0, plan, np.arange(n_layout, dtype=np.int32), tr))
    prof.free()
    assert early >= 2, early


@pytest.mark.parametrize("n_win,n_tick", [(60, 12), (240, 12), (20, 30)])
def test_hierarchy(dyn, n_win, n_tick):
    """Windows of 25 classes with more ticks than a block of four waves has threads."""
    w = make(SPECS[2].scaled(400 * n_win, n_win))
    raw = [_dev(w["trace"][k]) for k in ("t_s", "in_tok", "out_tok", "model")]
    coarse = dyn.dyn_trace_ingest(*raw, w["edges"], n_win, w["window_s"])[:3]
    fine = dyn.dyn_trace_ingest(*raw, w["edges"], n_win * n_tick, w["window_s"] / n_tick)[:3]
    prof = dyn.dyn_profile_load(w["profile"])
    n, t = np.meshgrid(np.arange(1, 17, dtype=np.int32), np.arange(3, dtype=np.int32))
    early, _ = calls_through_early(lambda: dyn.dyn_hierarchy(prof, coarse, fine, n_win, n_tick, w["window_s"] / n_tick, 6, 2, w["profile"]["f_mhz"].size - 1, 8,
                                                             n.ravel(), t.ravel(), w["slos"], w["pct"]))
    prof.free()
    assert early >= 2, early
