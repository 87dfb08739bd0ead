"""Entries of the mixed pools' per-type search that are twice another entry, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_mixed import check, dyn, gpu_mixed  # noqa: F401
from workloads import SPECS, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 2, 3, 4, 7, 8, 16])
@pytest.mark.parametrize("n_max", [[1, 2, 3], [4, 5, 0], [8, 7, 6]])
def test_odd_and_even_counts(dyn, S, n_max):   # noqa: F811
    """Odd and even instance limits and shares, powers of two (an entry four and eight times another) and a type that is not there."""
    w = make(SPECS[2].scaled(6_000, 3))
    n_max = (n_max * 2)[:w["profile"]["tp"].size]
    g, st = gpu_mixed(dyn, w, S, n_max, None)
    o = oracle.mixed(w["profile"], st, w["n_window"], w["window_s"], S, n_max, w["slos"], w["pct"], None, want_types=True)
    assert sum(check(w, g, o, S, n_max, None)) == w["n_window"] * w["n_class"]
    assert np.isfinite(o["energy_j"]).any()
