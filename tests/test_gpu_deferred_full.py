"""Lists of deferred work that fill while many waves add to them.

A wave reads the list's counter once for all of its lanes, takes slots for
those that defer in one addition, and keeps what does not get one.  Whatever
the lists hold (nothing but one entry, part of a wave's, all), the estimate
and the counters are the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 2, 17, 63, 64, 65, 1000])
@pytest.mark.parametrize("a,b,eps", [(0.0, 0.0, 1e-3), (0.5, 0.5, 1e-5)])
def test_lists_that_fill(rows, a, b, eps, monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    g = inputs.chung_lu(6000, 60, 2.1, seed=12)
    G, sg = agp.Graph.from_inputs(g, validate=True), oracle.degree_sort(g)
    C = 48
    x = inputs.features_normal(g.n, C, seed=2)
    x[:, ::2] = inputs.one_hot(g.n, np.argsort(np.diff(g.row_ptr))[-C:])[:, ::2]  # half of them the hubs
    w = inputs.weights_katz(0.01, 4) if a == 0.0 else inputs.weights_ppr(0.2, 4)
    ref, cnt = oracle.propagate(sg, a, b, w, x, eps, 6, wp=32, threads=8)
    X = torch.from_numpy(x).to("cuda:0")
    monkeypatch.setenv("AGP_BIG_ROWS", str(rows))
    try:
        for aggregation in (0, 1):
            agp.set_tuning(G, C, a, b, {"aggregation": aggregation, "big_row": 64, "big_items": 1})
            out, st = agp.propagate(G, a, b, w, X, eps, 6, stats=True)
            assert np.array_equal(out.cpu().numpy().astype(np.float64), ref)
            for k in ("frontier", "hash", "det", "cand", "acc", "runs"):
                assert np.array_equal(st[k][:5], cnt[k].sum(axis=0).astype(np.uint64)[:5]), k
    finally:
        agp.set_tuning(G, C, a, b, None)
