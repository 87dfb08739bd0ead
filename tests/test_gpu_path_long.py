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
