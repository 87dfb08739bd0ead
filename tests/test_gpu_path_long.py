"""Path selection over many windows, whose walk is cut into pieces, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_path import check, dyn, run_path  # noqa: F401
from workloads import SPECS, make

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(rng, NW, NL, K, digits=3):
    w = make(SPECS[0])
    G = w["n_class"]
    cfg = {"n_inst": rng.integers(1, 5, K).astype(np.int32), "tp_index": rng.integers(0, w["profile"]["tp"].size, K).astype(np.int32),
           "f_mhz": rng.choice(w["profile"]["f_mhz"], K)}
    energy = np.round(rng.uniform(1, 50, (NW * G, K)), digits)
    flags = np.where(rng.uniform(0, 1, (NW * G, K)) < 0.8, 1, 4).astype(np.uint8)
    lay = rng.permutation(np.arange(K) % NL).astype(np.int32)
    tr = np.round(rng.uniform(0, 6, (NL, NL)), digits)
    tr[np.diag_indices(NL)] = 0.0
    return w, G, cfg, energy, flags, lay, tr


def _run(d, w, cfg, energy, flags, NW, lay, tr, G, workspace=None):
    feas = (flags & 1).astype(np.uint8)
    o_sel, o_pc = oracle.select_path(energy, feas, NW, G, lay, tr)
    prof = d.dyn_profile_load(w["profile"])
    plan = d.Plan(cfg, w["slos"], w["pct"], None, 0.0)
    if workspace is None:
        g = run_path(d, prof, plan, energy, flags, NW, 60.0, lay, tr)
    else:
        space = {"energy_j": torch.from_numpy(energy).cuda(), "flags": torch.from_numpy(flags).cuda()}
        g = {k: v.cpu().numpy() for k, v in d.dyn_select_path(prof, space, NW, 60.0, plan, lay, tr, workspace=workspace)[0].items()}
    same = check(g, o_sel, o_pc, energy, feas, energy, lay, tr, NW, G)
    prof.free()
    return same


@pytest.mark.parametrize("NW,NL", [(299, 48), (300, 1), (303, 16), (335, 17), (336, 33), (337, 48), (400, 49), (521, 64), (1440, 5)])
def test_pieces(dyn, NW, NL):   # noqa: F811
    """Window counts around the line and the pieces' ends, layout counts around the tiers, gaps of one window and of many."""
    rng = np.random.default_rng(NW * 100 + NL)
    w, G, cfg, energy, flags, lay, tr = _case(rng, NW, NL, NL + 5)
    f = flags.reshape(NW, G, -1)
    for at in (0, 15, 16, 47, 48, 49, 200, NW - 1):
        f[at, at % G] = 8
    f[210:290, 1] = 8
    assert _run(dyn, w, cfg, energy, flags, NW, lay, tr, G) == G


@pytest.mark.parametrize("kind", ["equal windows", "equal layouts", "coarse", "free"])
def test_ties(dyn, kind):   # noqa: F811
    """Many sources reach the least: which of them is taken depends on the last bit of the totals, or on the candidates' order."""
    rng = np.random.default_rng(5)
    NW, NL = 600, 40
    w, G, cfg, energy, flags, lay, tr = _case(rng, NW, NL, NL, 1 if kind == "coarse" else 3)
    e = energy.reshape(NW, G, -1)
    flags[:] = 1
    if kind == "equal windows":
        e[100:500] = e[100]
    elif kind == "equal layouts":
        e[:, :, :] = e[:, :, :1]
        tr = np.full((NL, NL), 0.1)
        tr[np.diag_indices(NL)] = 0.0
    elif kind == "free":
        tr[:] = 0.0
    _run(dyn, w, cfg, energy, flags, NW, lay, tr, G)


@pytest.mark.parametrize("scale", [30.0, 1e4, 1.7e308])
def test_overheads_that_outlast_a_piece(dyn, scale):   # noqa: F811
    """Changes so dear that what was chosen hundreds of windows ago still decides: those classes are walked as a whole."""
    rng = np.random.default_rng(6)
    NW, NL = 500, 20
    w, G, cfg, energy, flags, lay, tr = _case(rng, NW, NL, NL)
    flags[:] = 1
    tr = tr / 6.0 * scale
    _run(dyn, w, cfg, energy, flags, NW, lay, tr, G)


def test_a_workspace_without_room_for_pieces(dyn):   # noqa: F811
    """The size that the query returned before is still taken, with the same outputs; one less is refused."""
    rng = np.random.default_rng(7)
    NW, NL = 420, 9
    w, G, cfg, energy, flags, lay, tr = _case(rng, NW, NL, NL)
    up = lambda n: (n + 255) // 256 * 256   # noqa: E731
    n = dyn.dyn_select_path_workspace(NW, G, NL, NL)
    former = n - 2 * up(NW * G * NL * 8) - up((G + 1) * 4)
    assert _run(dyn, w, cfg, energy, flags, NW, lay, tr, G, torch.empty(former, dtype=torch.uint8, device="cuda")) == G
    with pytest.raises(dyn.DynError):
        _run(dyn, w, cfg, energy, flags, NW, lay, tr, G, torch.empty(former - 256, dtype=torch.uint8, device="cuda"))


def _whole(ws, G):
    """Windows of each class that were walked with all sums: the last part of the workspace."""
    n = (G * 4 + 255) // 256 * 256
    return ws[-n:].view(torch.int32)[:G].cpu().numpy()


# How a piece of 48 windows is walked: of the one named source (plain), where some have none (gaps), where few windows have several (few
# ties); with all sums where many have (ties), where what was chosen 16 windows before still decides (dear), with costs below zero.
@pytest.mark.parametrize("NW,NL", [(300, 16), (481, 17), (624, 48), (577, 64)])
@pytest.mark.parametrize("kind", ["plain", "gaps", "few ties", "ties", "dear", "some dear", "below zero", "mixed"])
def test_how_pieces_are_walked(dyn, NW, NL, kind):   # noqa: F811
    rng = np.random.default_rng(NW + NL + len(kind))
    w, G, cfg, energy, flags, lay, tr = _case(rng, NW, NL, NL, 9)
    e, f, tr = energy.reshape(NW, G, NL), flags.reshape(NW, G, NL), tr / 100.0
    f[:] = 1
    lo, hi = 96, 96 + 48                       # a piece
    if kind in ("gaps", "mixed"):
        for at in (1, 47, 48, 100, 143, 200, NW - 2):
            f[at] = 8
        f[150:155, : G // 2] = 8
    if kind in ("few ties", "mixed"):          # two layouts of one kind: whoever leaves one could as well leave the other
        tr[1], tr[:, 1] = tr[0], tr[:, 0]
        for at in (50, 95, 110, 190):
            e[at, :, :2] = 0.0
    if kind == "ties":
        e[lo:hi, :, 1:] = e[lo:hi, :, :1]
        tr[:] = 0.0
    if kind in ("dear", "some dear", "mixed"):
        scale = 1e5 if kind == "dear" else 2e3
        tr = tr * scale + 5.0 * (tr > 0)
    if kind == "below zero":
        e[lo:lo + 3] -= 100.0
    prof = dyn.dyn_profile_load(w["profile"])
    ws = torch.empty(dyn.dyn_select_path_workspace(NW, G, NL, NL), dtype=torch.uint8, device="cuda")
    feas = (flags & 1).astype(np.uint8)
    o_sel, o_pc = oracle.select_path(energy, feas, NW, G, lay, tr)
    plan = dyn.Plan(cfg, w["slos"], w["pct"], None, 0.0)
    space = {"energy_j": torch.from_numpy(energy).cuda(), "flags": torch.from_numpy(flags).cuda()}
    for _ in range(2):                         # a workspace that holds another call's parts
        g = {k: v.cpu().numpy() for k, v in dyn.dyn_select_path(prof, space, NW, 60.0, plan, lay, tr, workspace=ws)[0].items()}
        check(g, o_sel, o_pc, energy, feas, energy, lay, tr, NW, G)
    whole = _whole(ws, G)
    prof.free()
    if kind in ("plain", "gaps"):
        assert (whole == 0).all(), whole
    elif kind == "few ties":
        assert (whole < 48).any(), whole
    elif kind == "ties":
        assert (whole >= 48).all(), whole
    elif kind == "dear":
        assert (whole > NW // 2).any(), whole
    elif kind == "below zero":
        assert (whole >= 48).all() and (whole < 200).all(), whole


@pytest.mark.parametrize("scale", [5.0, 20.0, 100.0])
def test_dear_changes_cost_no_more_than_the_whole_walk(dyn, scale):   # noqa: F811
    """Overheads at which pieces are of less use, against the same call in a workspace without room for them."""
    w = make(SPECS[2].scaled(200_000, 960))
    NW, G = 960, w["n_class"]
    rng = np.random.default_rng(11)
    n, ti = np.meshgrid(np.arange(1, 17), np.arange(3), indexing="ij")
    n, ti = n.ravel(), ti.ravel()
    gpus = n * w["profile"]["tp"][ti]
    base = np.maximum(8.0, 60.0 + 40.0 * np.sin(np.arange(NW) / 150.0))[:, None] * rng.uniform(0.5, 1.0, G)[None, :]
    base = base[..., None] * rng.uniform(0.9, 1.1, (NW, G, 1))
    energy = 6000.0 * gpus + 12_000.0 * base * (1.0 + 0.1 * ti)                                  # idle GPUs, and the load's own part
    flags = np.where(gpus >= base, 1, 4).astype(np.uint8)
    tr = 360.0 * np.maximum(0, gpus[None, :] - gpus[:, None]) + 180.0 * (ti[None, :] != ti[:, None]) * gpus[None, :]
    cfg = {"n_inst": n.astype(np.int32), "tp_index": ti.astype(np.int32), "f_mhz": np.full(n.size, w["profile"]["f_mhz"][0])}
    prof = dyn.dyn_profile_load(w["profile"])
    plan = dyn.Plan(cfg, w["slos"], w["pct"], None, 0.0)
    space = {"energy_j": torch.from_numpy(energy.reshape(NW * G, -1)).cuda(), "flags": torch.from_numpy(flags.reshape(NW * G, -1)).cuda()}
    full = dyn.dyn_select_path_workspace(NW, G, n.size, n.size)
    up = lambda x: (x + 255) // 256 * 256   # noqa: E731
    lay, us = np.arange(n.size, dtype=np.int32), {}
    sizes = {"pieces": full, "whole": full - 2 * up(NW * G * n.size * 8) - up((G + 1) * 4)}
    ws = {k: torch.empty(b, dtype=torch.uint8, device="cuda") for k, b in sizes.items()}
    out = {}
    for _ in range(5):
        for k in ws:
            out[k] = dyn.dyn_select_path(prof, space, NW, 60.0, plan, lay, tr * scale, workspace=ws[k])[0]
            torch.cuda.synchronize()
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                dyn.dyn_select_path(prof, space, NW, 60.0, plan, lay, tr * scale, workspace=ws[k])
            b.record()
            torch.cuda.synchronize()
            us.setdefault(k, []).append(a.elapsed_time(b) * 100.0)
    prof.free()
    for k in out["pieces"]:
        assert torch.equal(out["pieces"][k], out["whole"][k]), k
    # the pieces themselves and predecessors over all sources take a tenth or so where every piece is walked as a whole after all
    assert min(us["pieces"]) < 1.15 * min(us["whole"]), us
