"""Records are read four at a time: bit-exact with the oracle when a level's
records end anywhere in a group of four (bins, segments and buffers alike),
with and without the overflow of small buffers."""
import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", ["1", "2"])
@pytest.mark.parametrize("cap", [None, "1", "61", "402"])
@pytest.mark.parametrize("C", [1, 3, 5])
def test_record_tails(C, cap, groups, monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    monkeypatch.setenv("AGP_AGGREGATION", "binned")
    monkeypatch.setenv("AGP_RECORD_GROUPS", groups)
    if cap:
        monkeypatch.setenv("AGP_RECORD_CAP", cap)
    g = inputs.chung_lu(9001, 8, 2.3, seed=C)
    G, sg = agp.Graph.from_inputs(g, validate=True), oracle.degree_sort(g)
    x = inputs.one_hot(g.n, np.random.default_rng(C).choice(g.n, size=C)).astype(np.float32)
    X = torch.from_numpy(x).to("cuda:0")
    seen = set()
    for seed in range(4):  # other counts of records per bin and segment
        eps = 2e-3 / (seed + 1)
        ref, cnt = oracle.propagate(sg, 0.0, 1.0, inputs.weights_tp(4), x, eps, seed, wp=32)
        out, st = agp.propagate(G, 0.0, 1.0, inputs.weights_tp(4), X, eps, seed, stats=True)
        assert np.array_equal(out.cpu().numpy().astype(np.float64), ref), seed
        assert np.array_equal(st["acc"][:5], cnt["acc"].sum(axis=0).astype(np.uint64)[:5])
        seen |= {int(a) % 4 for a in st["acc"][:4] if a}
    assert len(seen) > 1
