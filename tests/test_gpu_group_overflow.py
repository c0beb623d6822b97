"""Two column groups of records of which one outgrows its buffer while the
other is being scanned: the level falls back to atomics as a whole, whichever
group it is, and the next level is binned again.  Bit-exact with the oracle."""
import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("busy", ["first", "second", "both", "neither"])
@pytest.mark.parametrize("C", [2, 7])
def test_one_group_overflows(C, busy, monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    monkeypatch.setenv("AGP_AGGREGATION", "binned")
    monkeypatch.setenv("AGP_RECORD_GROUPS", "2")
    monkeypatch.setenv("AGP_RECORD_CAP", "4000")
    g = inputs.chung_lu(20011, 10, 2.3, seed=5)
    G, sg = agp.Graph.from_inputs(g, validate=True), oracle.degree_sort(g)
    # columns of a wide signal make records by the thousand, a single source
    # behind a coarse threshold a few, empty columns none
    wide = {"first": range((C + 1) // 2), "second": range((C + 1) // 2, C), "both": range(C), "neither": []}[busy]
    src = np.random.default_rng(C).choice(np.flatnonzero(np.diff(g.row_ptr) > 0), size=C)
    x = inputs.one_hot(g.n, src) if busy == "neither" else np.zeros((g.n, C), dtype=np.float32)
    x[:, list(wide)] = inputs.features_normal(g.n, C, seed=C)[:, list(wide)]
    X = torch.from_numpy(x).to("cuda:0")
    w, eps = inputs.weights_tp(4), 2e-2 if busy == "neither" else 1e-4
    ref, cnt = oracle.propagate(sg, 0.0, 1.0, w, x, eps, 4, wp=32, threads=8)
    for _ in range(3):
        out, st = agp.propagate(G, 0.0, 1.0, w, X, eps, 4, stats=True)
        assert np.array_equal(out.cpu().numpy().astype(np.float64), ref)
        assert np.array_equal(st["acc"][:5], cnt["acc"].sum(axis=0).astype(np.uint64)[:5])
