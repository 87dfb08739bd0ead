"""The orders a request log can come in, each through the route it takes, at the sizes where tiles and runs end."""
import numpy as np
import pytest

import oracle
from tests.beside import calls_through_early

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TILE = 8192          # requests a large block of the general sort moves at a time, a small one (logs of up to a million) SMALL
SMALL = 2048
MILLION = 1 << 20
WINDOW = 12288       # requests a block of the window route moves at a time (512, 2048 or 4096 where windows are short)


@pytest.fixture(scope="module")
def dyn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00741_amd as d
    return d


def _edges(n_in, n_out, n_model=1):
    tile = lambda e: np.tile(e.astype(np.int32), (n_model, 1)).reshape(n_model, e.size) + 7 * np.arange(n_model, dtype=np.int32)[:, None]
    return {"in_edge": tile(np.linspace(100, 8000, n_in - 1)), "out_edge": tile(np.linspace(90, 7900, n_out - 1))}


def _log(seed, n, horizon, n_model=1):
    rng = np.random.default_rng(seed)
    return {"t_s": rng.uniform(0, horizon, n), "in_tok": rng.integers(1, 8193, n).astype(np.int32),
            "out_tok": rng.integers(1, 8193, n).astype(np.int32), "model": rng.integers(0, n_model, n).astype(np.int32)}


def _call(dyn, tr, edges, n_window, window_s, **kw):
    d = [torch.from_numpy(np.ascontiguousarray(tr[k])).cuda() for k in ("t_s", "in_tok", "out_tok", "model")]
    return dyn.dyn_trace_ingest(*d[:3], d[3] if len(edges["in_edge"]) > 1 else None, edges, n_window, window_s, **kw)


def _check(got, tr, edges, n_window, window_s):
    want = oracle.ingest(tr, edges, n_window, window_s)
    np.testing.assert_array_equal(got[2].cpu().numpy(), want["cell_off"])
    np.testing.assert_array_equal(got[0].cpu().numpy(), want["in_tok"])
    np.testing.assert_array_equal(got[1].cpu().numpy(), want["out_tok"])


# one, two and three passes; digits of 5 to 10 bits; less than a wave (1200 classes: the sort is forced), a tile and one more, many
# tiles a block; the longest log that small blocks sort and one more
@pytest.mark.parametrize("n,n_window,n_in,n_out", [(1, 1, 40, 30), (2, 2, 40, 30), (63, 5, 40, 30), (SMALL - 1, 9, 5, 5), (SMALL, 40, 5, 5), (SMALL + 1, 300, 2, 1), (TILE - 1, 9, 5, 5), (TILE, 40, 5, 5), (TILE + 1, 41, 5, 5),
                                                   (2 * TILE + 65, 1000, 5, 5), (100_000, 3, 40, 30), (300_001, 2000, 16, 20), (MILLION, 1440, 5, 5), (MILLION + 1, 1440, 5, 5), (2_500_000, 1440, 5, 5)])
def test_general_sort_is_stable(dyn, n, n_window, n_in, n_out):
    edges = _edges(n_in, n_out)
    tr = _log(n, n, n_window * 10.0)
    got = _call(dyn, tr, edges, n_window, 10.0)
    assert dyn.dyn_workspace_status(got[3]) == 0
    _check(got, tr, edges, n_window, 10.0)


# a window of one request, of a wave, of a tile, of one more and of several tiles; empty windows; one class, and the most
# that the route takes; several models; edges that stay in global memory
@pytest.mark.parametrize("n,n_window,n_in,n_out,n_model", [(1, 1, 1, 1, 1), (64, 1, 2, 2, 1), (WINDOW, 1, 5, 5, 1), (WINDOW + 1, 1, 5, 5, 1), (50_000, 7, 32, 32, 1),
                                                           (3 * WINDOW, 2, 8, 8, 4), (513, 1000, 5, 5, 1), (200_000, 31, 3, 3, 4), (100_000, 7, 2, 2, 256),
                                                           (20_000, 70, 5, 5, 1), (60_000, 70, 5, 5, 2), (120_000, 70, 32, 32, 1), (400_000, 3, 5, 5, 1)])
@pytest.mark.parametrize("skewed", [False, True])
def test_log_in_time_order(dyn, n, n_window, n_in, n_out, n_model, skewed):
    edges = _edges(n_in, n_out, n_model)
    tr = _log(n, n, n_window * 10.0, n_model)
    if skewed:           # half of the requests in the last tenth: windows of several tiles beside short ones
        tr["t_s"][::2] = n_window * 9.0 + 0.1 * tr["t_s"][::2]
    tr["t_s"].sort()
    got = _call(dyn, tr, edges, n_window, 10.0)
    assert dyn.dyn_workspace_status(got[3]) == 0
    _check(got, tr, edges, n_window, 10.0)


# the logs of several front ends, one after the other: fewer and more runs than the route takes, a run of one request, runs
# of different parts of the day, windows of several tiles, and (2000 windows of 30 000 requests) the sort all the same
@pytest.mark.parametrize("n,n_window,n_run,n_model", [(2, 2, 2, 1), (5_000, 5, 5, 1), (100_000, 100, 48, 1), (100_000, 100, 49, 4), (100_000, 100, 50, 1), (100_000, 60, 300, 1),
                                                      (30_000, 2000, 9, 1), (900_000, 45, 7, 4), (1_500_000, 60, 3, 1)])
@pytest.mark.parametrize("apart", [False, True])
def test_log_of_several_runs(dyn, n, n_window, n_run, n_model, apart):
    edges = _edges(5, 5, n_model)
    tr = _log(n, n, n_window * 10.0, n_model)
    cut = [n * r // n_run for r in range(n_run + 1)]
    if n_run > 2:
        cut[1] = 1
    for r, (a, b) in enumerate(zip(cut[:-1], cut[1:])):
        if apart:        # a run covers a part of the windows: others have no piece of it
            tr["t_s"][a:b] = n_window * 10.0 * (r % 3 + tr["t_s"][a:b] / (n_window * 10.0)) / 3.0
        tr["t_s"][a:b] = np.sort(tr["t_s"][a:b])
    got = _call(dyn, tr, edges, n_window, 10.0)
    assert dyn.dyn_workspace_status(got[3]) == 0
    _check(got, tr, edges, n_window, 10.0)


def test_edges_that_stay_in_global_memory(dyn):
    """One class axis of 900 bins and three models: 2697 edges, more than a block stages (and more classes than the window route)."""
    edges = _edges(900, 1, 3)
    for order in (True, False):
        tr = _log(5, 50_000, 30.0, 3)
        if order:
            tr["t_s"].sort()
        _check(_call(dyn, tr, edges, 3, 10.0), tr, edges, 3, 10.0)


def test_no_requests_and_more_classes_than_the_window_route_counts(dyn):
    edges = _edges(40, 30)
    got = _call(dyn, _log(0, 0, 1.0), edges, 3, 10.0)
    assert got[2].cpu().numpy().tolist() == [0] * (3 * 1200 + 1)


def test_sorts_on_eight_streams_at_once(dyn):
    """More sorts than the device holds whole: every one forms its team from the blocks that run."""
    edges = _edges(5, 5)
    logs = [_log(q, 400_000 + q, 3600.0) for q in range(8)]
    streams = [torch.cuda.Stream() for _ in logs]
    got = []
    for tr, st in zip(logs, streams):
        with torch.cuda.stream(st):
            got.append(_call(dyn, tr, edges, 60, 60.0))
    torch.cuda.synchronize()
    for tr, g in zip(logs, got):
        assert dyn.dyn_workspace_status(g[3]) == 0
        _check(g, tr, edges, 60, 60.0)


def _squeezed(seed, n, n_window, first, used, n_model=1):
    """A log whose requests lie in `used` windows of 10 s from window `first` on."""
    tr = _log(seed, n, used * 10.0, n_model)
    tr["t_s"] += first * 10.0
    return tr


def _us(call):
    """Least time of a few calls on the GPU, in microseconds."""
    call()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


# the sort where most cells are empty: before the first request, between two tiles, behind the last (1200 classes force the
# sort, so a log of one request takes it too)
@pytest.mark.parametrize("n", [1, 63, 64, 65, TILE, TILE + 1, 3 * TILE + 5])
@pytest.mark.parametrize("first", [0, 17, 39])
@pytest.mark.parametrize("n_in,n_out", [(5, 5), (40, 30)])
def test_sort_of_a_log_in_a_small_part_of_the_grid(dyn, n, first, n_in, n_out):
    edges = _edges(n_in, n_out)
    tr = _squeezed(n, n, 40, first, 1)
    if n > 1:
        tr["t_s"][-1], tr["t_s"][0] = 10.0 * first, 399.0       # out of order also where all lie in one window
    got = _call(dyn, tr, edges, 40, 10.0)
    _check(got, tr, edges, 40, 10.0)


def test_sort_is_as_quick_where_most_cells_are_empty(dyn):
    """A day's log of the last minute, unordered: its empty cells before it are filled by all threads (one thread: 13 times as long)."""
    edges = _edges(5, 5)
    us = []
    for used in (2000, 1):
        tr = _squeezed(7, 300_000, 2000, 2000 - used, used)
        tr["t_s"][1000::1000] = 0.0                             # more breaks than the runs route takes
        d = [torch.from_numpy(tr[k]).cuda() for k in ("t_s", "in_tok", "out_tok")]
        us.append(_us(lambda: dyn.dyn_trace_ingest(*d, None, edges, 2000, 10.0)))
    assert us[1] < 4.0 * us[0], us


def _counted(seed, counts, n_run=1, n_model=1):
    """A log with counts[w] requests in window w of 10 s: in time order, or as n_run ordered runs that each take part in every window."""
    n = int(np.sum(counts))
    tr = _log(seed, n, 1.0, n_model)
    tr["t_s"] = np.repeat(10.0 * np.arange(len(counts)), counts) + 9.0 * tr["t_s"]
    tr["t_s"].sort()
    if n_run > 1:
        for k in tr:
            tr[k] = np.concatenate([tr[k][r::n_run] for r in range(n_run)])
    return tr


# uneven logs: a window longer than the tile that the mean window asks for is left to larger blocks (512, 2048, 4096 and
# 4 x 12 288 requests, and one more; several of them; all but one), one that alone takes longer than the sort has the log sorted
@pytest.mark.parametrize("counts,n_run,left,sorts", [
    ([512, 513] + [100] * 20, 1, 1, False), ([500] * 20 + [2048, 2049], 1, 1, False), ([1500] * 20 + [4097, 4096], 1, 1, False),
    ([6000] * 400 + [4 * WINDOW + 1, 4 * WINDOW], 1, 1, False), ([4000] * 20 + [4 * WINDOW], 1, None, True), ([0] * 600 + [520] * 300, 1, 300, False), ([0] * 99 + [12_000], 1, 1, False), ([0] * 99 + [25_000], 1, None, True),
    ([200] * 2000 + [20_000, 100], 1, 1, False), ([200] * 2000 + [60_000, 100], 1, None, True), ([0] * 2000 + [90_000] * 2, 1, None, True),
    ([200] * 2000 + [60_000, 100], 2, None, True), ([0] * 2000 + [90_000] * 2, 6, None, True), ([200] * 200 + [15_000, 100], 6, 0, False)])
@pytest.mark.parametrize("n_model", [1, 4])
def test_uneven_log(dyn, counts, n_run, left, sorts, n_model):
    edges = _edges(5, 5, n_model)
    tr = _counted(len(counts), counts, n_run, n_model)
    got = _call(dyn, tr, edges, len(counts), 10.0)
    assert dyn.dyn_workspace_status(got[3]) == 0
    _check(got, tr, edges, len(counts), 10.0)
    words = got[3][:256].view(torch.int32).cpu().numpy()        # 8: breaks, or past 48 where the log is sorted; 12: windows left
    assert (words[8] > 48) == sorts and (sorts or words[8] == n_run - 1)
    assert sorts or words[12] == left


@pytest.mark.parametrize("n_run", [1, 6])
def test_log_of_a_few_long_windows_is_as_quick_as_an_even_one(dyn, n_run):
    """Three million requests in three of 2016 windows (by window one block each: 19 and 14 times as long)."""
    edges = _edges(5, 5)
    us = []
    for counts in ([1488] * 2016, [0] * 2013 + [1_000_000] * 3):
        tr = _counted(3, counts, n_run)
        d = [torch.from_numpy(np.ascontiguousarray(tr[k])).cuda() for k in ("t_s", "in_tok", "out_tok")]
        us.append(_us(lambda: dyn.dyn_trace_ingest(*d, None, edges, 2016, 10.0)))
    assert us[1] < 8.0 * us[0], us


def test_sort_beside_another_kernel_is_not_left_to_a_few_blocks(dyn):
    """The device is full when the sort starts: its first block waits for the others as long as that pays."""
    edges = _edges(5, 5)
    tr = _log(20, 4_000_000, 14400.0)
    d = [torch.from_numpy(tr[k]).cuda() for k in ("t_s", "in_tok", "out_tok")]
    full = torch.rand(1 << 28, device="cuda")
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        for _ in range(12):
            torch.erfinv(full, out=full)
    got = dyn.dyn_trace_ingest(*d, None, edges, 1440, 10.0)
    torch.cuda.synchronize()
    assert dyn.dyn_workspace_status(got[3]) == 0
    _check(got, tr, edges, 1440, 10.0)
    assert int(got[3][:256].view(torch.int32)[11]) >= 64         # blocks that sorted


# in time order, of six runs, of long windows that are left, unordered
@pytest.mark.parametrize("counts,n_run,shuffled", [([300] * 60, 1, False), ([700] * 1000, 1, False), ([60] * 100, 6, False), ([0] * 99 + [9000], 1, False), ([200] * 1000, 1, True)])
def test_small_log_does_not_wait_for_another_stream(dyn, counts, n_run, shuffled):
    """A kernel on another stream fills the device: the ingest's blocks fit beside it, and it is through long before that kernel."""
    edges = _edges(5, 5)
    tr = _counted(9, counts, n_run)
    if shuffled:
        p = np.random.default_rng(9).permutation(len(tr["t_s"]))
        tr = {k: v[p] for k, v in tr.items()}
    d = [torch.from_numpy(np.ascontiguousarray(tr[k])).cuda() for k in ("t_s", "in_tok", "out_tok")]
    call = lambda: dyn.dyn_trace_ingest(*d, None, edges, len(counts), 10.0)
    early, got = calls_through_early(call)
    _check(got, tr, edges, len(counts), 10.0)
    assert early >= 2, early
