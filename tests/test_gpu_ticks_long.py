"""Ticks of long cells, which many blocks share, and lists of short cells taken from a wave's registers, against the CPU oracle."""
import numpy as np
import pytest

from tests.test_gpu_ticks import _one_class, assert_same, dyn, gpu_ticks, ora_ticks  # noqa: F401
from workloads import SPECS, make

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(n_req, NW, prefill, one_class=True, stride=7):
    w = make(SPECS[1].scaled(n_req, NW))
    if one_class:
        w = _one_class(w)
    r = w["profile"]["rho"]
    pf = w["profile"]["prefill_ms_per_tok"]
    if prefill == "load":
        pf = pf * (1.0 + 0.8 * r * r)
    elif prefill == "wild":                # a factor of 6 between neighbouring load points: no table is wide enough
        pf = pf * np.where(np.arange(r.size) % 2 == 0, 1.0, 6.0)
    w["profile"]["prefill_ms_per_tok"] = pf
    w["configs"] = {k: v[::stride].copy() for k, v in w["configs"].items()}
    return w


def _check(d, w, T, pct=(99, 100)):
    g, fine = gpu_ticks(d, w, T, pct=pct)
    assert g["status"] == 0
    assert_same(w, g, ora_ticks(w, fine, T, pct=pct))


@pytest.mark.parametrize("n_req,NW,T,crowd", [(4096, 1, 3, 0), (4097, 1, 3, 0), (20_000, 1, 1, 0), (40_000, 1, 2, 9000), (60_000, 2, 12, 0), (70_000, 1, 7, 30_000), (50_000, 1, 64, 3000)])
@pytest.mark.parametrize("prefill", ["flat", "load", "wild"])
def test_long_cells(dyn, n_req, NW, T, crowd, prefill):   # noqa: F811
    """One class; the smallest long cell and one request less, one tick and the most, a tick that holds much of the cell."""
    w = _case(n_req, NW, prefill)
    if crowd:
        w["trace"]["t_s"][:crowd] = 0.6 * w["window_s"] / T
        w["trace"]["t_s"].sort()
    _check(dyn, w, T)


@pytest.mark.parametrize("pct", [(1, 1), (1, 2), (1, 100), (9, 10), (9999, 10000)])
@pytest.mark.parametrize("prefill", ["flat", "load"])
def test_ranks_of_long_cells(dyn, pct, prefill):   # noqa: F811
    _check(dyn, _case(30_000, 1, prefill), 6, pct)


@pytest.mark.parametrize("prefill", ["flat", "load"])
@pytest.mark.parametrize("lengths", ["few", "short", "wide", "edge"])
def test_lengths_of_long_cells(dyn, lengths, prefill):   # noqa: F811
    """Ties everywhere, lengths below 64 (exact bins), lengths of 2^16 and more (lists instead), lengths around 2^16."""
    w = _case(30_000, 1, prefill)
    rng = np.random.default_rng(5)
    n = w["trace"]["in_tok"].size
    w["trace"]["in_tok"] = {"few": rng.integers(0, 3, n) * 900, "short": rng.integers(0, 64, n), "wide": rng.integers(0, 1 << 24, n),
                            "edge": rng.integers((1 << 16) - 40, (1 << 16) + (0 if prefill == "flat" else 40), n)}[lengths].astype(np.int32)
    _check(dyn, w, 5)


def test_several_long_cells_beside_short_ones(dyn):   # noqa: F811
    _check(dyn, _case(150_000, 2, "load", one_class=False), 10, (95, 100))


def test_a_negative_count_in_a_long_cell_is_reported(dyn):   # noqa: F811
    w = _case(20_000, 1, "load")
    w["trace"]["out_tok"][777] = -5
    tr = w["trace"]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()   # noqa: E731
    prof = dyn.dyn_profile_load(w["profile"])
    off = torch.tensor([0, 9000, 20_000], dtype=torch.int64, device="cuda")
    ws = dyn.dyn_eval_select_ticks(prof, dev(tr["in_tok"]), dev(tr["out_tok"]), off, 1, 2, 5.0, dyn.Plan(w["configs"], w["slos"], w["pct"], None, 0.0))[2]
    assert dyn.dyn_workspace_status(ws) == dyn.DYN_WS_BAD_REQUEST
    prof.free()


def test_a_workspace_without_room_for_sharing(dyn):   # noqa: F811
    """The size that the query returned before cells were shared is still taken, with the same outputs."""
    w = _case(30_000, 1, "load")
    tr = w["trace"]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()   # noqa: E731
    ins, outs, off, _ = dyn.dyn_trace_ingest(dev(tr["t_s"]), dev(tr["in_tok"]), dev(tr["out_tok"]), dev(tr["model"]), w["edges"], 6, w["window_s"] / 6)
    prof = dyn.dyn_profile_load(w["profile"])
    plan = dyn.Plan(w["configs"], w["slos"], w["pct"], None, 0.0)
    K = len(w["configs"]["n_inst"])
    n = dyn.dyn_eval_ticks_workspace(30_000, 1, 6, 1, K)
    former = n - 7 * 8192 - (46384 * 4 + 255) // 256 * 256   # seven slots and the tables
    got = []
    for size in (n, former):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        space, sel, _ = dyn.dyn_eval_select_ticks(prof, ins, outs, off, 1, 6, w["window_s"] / 6, plan, workspace=ws)
        got.append({k: v.clone() for k, v in {**space, **sel}.items()})
    for k in got[0]:
        assert torch.equal(got[0][k], got[1][k]), k
    with pytest.raises(dyn.DynError):
        dyn.dyn_eval_select_ticks(prof, ins, outs, off, 1, 6, w["window_s"] / 6, plan, workspace=ws[:former - 256])
    prof.free()


@pytest.mark.parametrize("n_req,T,pct", [(5_000, 3, (99, 100)), (60_000, 1, (99, 100)), (60_000, 5, (99, 100)), (60_000, 12, (95, 100)), (40_000, 9, (9, 10))])
def test_lists_from_registers(dyn, n_req, T, pct):   # noqa: F811
    """1200 cells of a few to 50 requests with lists of 1 to 6 places: up to 4 are taken from the registers of the wave that read the cell."""
    w = _case(n_req, 1200, "load", stride=41)
    _check(dyn, w, T, pct)


@pytest.mark.parametrize("T,m,windows,rest", [(13, 4420, 1, 0), (13, 4421, 2, 0), (64, 21_760, 2, 0), (64, 21_761, 1, 0), (64, 21_761, 265, 264 * 14_100), (64, 21_761, 266, 265 * 14_100)])
def test_lists_and_tables_of_long_cells(dyn, T, m, windows, rest):   # noqa: F811
    """The longest cell whose ticks' lists are made and the shortest that gets tables, of few ticks and of most; 265 and 266 cells of 64 ticks and 220
    requests a tick, where tables are made and where all lists are: one long cell, and `rest` requests in the others."""
    w = _case(m + rest, windows, "load", stride=61)
    w["trace"]["t_s"] = np.concatenate([(np.arange(m) + 0.5) * (w["window_s"] / m), w["window_s"] * (1.0 + (windows - 1) * (np.arange(rest) + 0.5) / max(rest, 1))])
    _check(dyn, w, T)


@pytest.mark.parametrize("prefill", ["load", "wild"])
@pytest.mark.parametrize("longest", [63, 64, 127, 128, 8191, 8192, 8319, 65_535, 65_536, 70_000])
def test_tables_end_at_the_longest_request(dyn, longest, prefill):   # noqa: F811
    """The percentile among the longest requests, which many share, at the ends of the counted ranges of lengths and beyond those that are counted;
    the first tick has twice the load of the others."""
    w = _case(30_000, 1, prefill)
    tr, rng = w["trace"], np.random.default_rng(7)
    tr["in_tok"] = np.minimum(rng.integers(1, max(2, 2 * longest), 30_000), longest).astype(np.int32)
    tr["in_tok"][rng.random(30_000) < 0.7] = 1 + longest // 3
    tr["t_s"][:4000] = 0.05 * w["window_s"]
    tr["t_s"].sort()
    _check(dyn, w, 7)
    tr["in_tok"][rng.integers(0, 30_000, 40)] = longest + 300     # fewer than the percentile's rank: longer than all that counts
    _check(dyn, w, 7)
