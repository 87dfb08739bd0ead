"""Token sums and percentile length of single cells at the sizes where the reduction changes its form: few cells of many requests (a
wave each, a block for a long one), more cells or fewer requests (a wave each), many small ones."""
import numpy as np
import pytest

from workloads import SPECS, make

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dyn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2408_00741_amd as d
    return d


SIZES = [0, 1, 2, 63, 64, 65, 100, 101, 256, 511, 512, 513, 1024, 1025, 2047, 2048, 2049, 3072, 3073, 4096, 4097, 8191, 8192, 8193, 20_001, 0, 3]


# (cells, requests in those that SIZES does not name): the block form asks for at most 1024 cells and more than 1000 requests a cell
@pytest.mark.parametrize("cells,each", [(len(SIZES), 0), (1024, 1010), (1024, 930), (1025, 1010), (1025, 5), (3000, 400)])
@pytest.mark.parametrize("pct", [(99, 100), (1, 2), (1, 1000), (1, 1)])
@pytest.mark.parametrize("kind", ["tokens", "equal", "wide", "negative"])
def test_cell_statistics(dyn, cells, each, pct, kind):
    rng = np.random.default_rng(cells + pct[0])
    m = np.concatenate([SIZES, rng.integers(each - each // 20 if each > 900 else 0, each + 1 if each < 900 else each + each // 20, cells - len(SIZES))]).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(m)])
    n = int(off[-1])
    assert (cells <= 1024 and n > 1000 * cells) == ((cells, each) in ((len(SIZES), 0), (1024, 1010)))
    x, y = (rng.integers(0, {"tokens": 8193, "equal": 3, "wide": 1 << 31, "negative": 8193}[kind], n).astype(np.int32) for _ in range(2))
    if kind == "negative":
        x[off[20]] = -5                            # cell 20 holds one: its sums count it, its status says so
    w = make(SPECS[1].scaled(1000, 2))
    G = 1
    prof = dyn.dyn_profile_load({k: (v[:G] if v.ndim >= 3 else v) for k, v in w["profile"].items()})
    plan = dyn.Plan({k: v[:3] for k, v in w["configs"].items()}, {k: v[:G] for k, v in w["slos"].items()}, pct, None, 0.0)
    dev = lambda a: torch.from_numpy(a).cuda()
    _, ws = dyn.dyn_eval_space(prof, dev(x), dev(y), dev(off), cells, 60.0, plan)
    tin, tout, p99 = (t.cpu().numpy() for t in dyn.dyn_cell_stats(ws, cells, G))
    assert dyn.dyn_workspace_status(ws) == (dyn.DYN_WS_BAD_REQUEST if kind == "negative" else 0)
    sums = lambda a: np.concatenate([[0], np.cumsum(a.astype(np.int64))])
    np.testing.assert_array_equal(tin, sums(x)[off[1:]] - sums(x)[off[:-1]])
    np.testing.assert_array_equal(tout, sums(y)[off[1:]] - sums(y)[off[:-1]])
    for c in range(cells):
        if kind == "negative" and c == 20:
            continue
        v = np.sort(x[off[c]:off[c + 1]])
        rank = -(-pct[0] * v.size // pct[1])
        assert p99[c] == (v[rank - 1] if v.size else 0), (c, v.size)
    prof.free()


# Cells that many blocks share: edges of what a block keeps, of a block's piece and of the bins; lengths around the widths of a bin's
# parts (2^15), a rank in every kind of bin, offsets out of order that claim
# more long cells than a sound trace can hold; more cells than there are copies of counters for.
@pytest.mark.parametrize("sizes", [[300_000], [8192, 8193, 0, 12_288, 12_289, 1, 70_001, 0], [4096 * 30, 4096 * 30 + 1, 5, 4096 * 3 - 1], [1_500_000, 3, 9000], [9100] * 70 + [8192] * 5 + [60_000] * 3])
@pytest.mark.parametrize("pct", [(99, 100), (1, 2), (1, 1_000_000), (1, 1)])
@pytest.mark.parametrize("kind", ["tokens", "equal", "near 2^15", "wide", "negative"])
def test_long_cells(dyn, sizes, pct, kind):
    rng = np.random.default_rng(len(sizes) + pct[0])
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n, cells = int(off[-1]), len(sizes)
    assert n > 9000 * cells and n > 20_000
    lo, hi = {"tokens": (0, 8193), "equal": (7000, 7002), "near 2^15": (32_000, 34_000), "wide": (0, (1 << 31) - 1), "negative": (0, 8193)}[kind]
    x, y = (rng.integers(lo, hi + 1, n).astype(np.int32) for _ in range(2))
    if kind == "negative":
        y[n // 2] = -1                             # sums count it, the status says so, the lengths do not see it
    _check(dyn, x, y, off, cells, pct, [(int(off[c]), int(off[c + 1])) for c in range(cells)], dyn.DYN_WS_BAD_REQUEST if kind == "negative" else 0)


def test_long_cells_that_overlap(dyn):
    n = 100_000
    off = np.array([0, n, 0, n, 0, n, 0, n, 0, n], np.int64)
    x, y = (np.random.default_rng(k).integers(1, 9000, n).astype(np.int32) for k in range(2))
    _check(dyn, x, y, off, 9, (99, 100), [(0, n) if c % 2 == 0 else (0, 0) for c in range(9)], dyn.DYN_WS_BAD_OFFSETS)


def _check(dyn, x, y, off, cells, pct, spans, status):
    w = make(SPECS[1].scaled(1000, 2))
    prof = dyn.dyn_profile_load({k: (v[:1] if v.ndim >= 3 else v) for k, v in w["profile"].items()})
    plan = dyn.Plan({k: v[:3] for k, v in w["configs"].items()}, {k: v[:1] for k, v in w["slos"].items()}, pct, None, 0.0)
    dev = lambda a: torch.from_numpy(a).cuda()
    _, ws = dyn.dyn_eval_space(prof, dev(x), dev(y), dev(off), cells, 60.0, plan)
    tin, tout, p99 = (t.cpu().numpy() for t in dyn.dyn_cell_stats(ws, cells, 1))
    assert dyn.dyn_workspace_status(ws) == status
    for c, (b, e) in enumerate(spans):
        v = np.sort(x[b:e])
        rank = -(-pct[0] * v.size // pct[1])
        got = (tin[c], tout[c], p99[c])
        assert got == (v.sum(dtype=np.int64), y[b:e].sum(dtype=np.int64), v[rank - 1] if v.size else 0), (c, e - b)
    prof.free()
