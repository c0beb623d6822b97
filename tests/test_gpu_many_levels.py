"""Level counts around the 64 whose parameters travel with the launch, and the
most a call may have: estimates and counters of every level equal the
oracle's, launched kernel by kernel and replayed."""
import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", ["direct", "captured", "noalloc", "f64"])
@pytest.mark.parametrize("L", [63, 64, 255])
def test_many_levels(L, entry, monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    if entry == "captured":
        monkeypatch.setenv("AGP_CAPTURE", "1")
    g = inputs.chung_lu(1500, 8, 2.3, seed=L)
    G, sg = agp.Graph.from_inputs(g, validate=True), oracle.degree_sort(g)
    wp = 64 if entry == "f64" else 32
    w = inputs.weights_ppr(1.0 / (L + 1), L)  # mass at every level
    x = inputs.one_hot(g.n, inputs.sources_uniform(g, 3, seed=1)).astype(np.float64 if wp == 64 else np.float32)
    X = torch.from_numpy(x).to("cuda:0")
    for seed in (4, 5, 6):  # (a captured loop is replayed with other parameters)
        ref, cnt = oracle.propagate(sg, 0.0, 1.0, w, x, 1e-4, seed, wp=wp)
        assert cnt["acc"].sum(axis=0)[L - 1] > 0
        out, st = agp.propagate(G, 0.0, 1.0, w, X, 1e-4, seed, stats=True)
        if entry == "noalloc":
            out = agp.propagate_noalloc(G, 0.0, 1.0, w, X, 1e-4, seed)
        assert np.array_equal(out.cpu().numpy().astype(np.float64), ref), seed
        for k in ("frontier", "hash", "det", "cand", "acc", "runs"):
            assert np.array_equal(st[k][:L + 1], cnt[k].sum(axis=0).astype(np.uint64)[:L + 1]), k
