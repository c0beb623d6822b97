"""More queries at once than a block sums in LDS (128 slots), and more slots
than keep several sets of counter rows (8192): results and counters of every
query equal the oracle's, for first and for recycled slots."""
import time

import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [127, 128, 129, 300, 8191, 8192])
def test_served_slots(slots):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    g = inputs.chung_lu(2000, 8, 2.3, seed=7)
    G, sg = agp.Graph.from_inputs(g, validate=True), oracle.degree_sort(g)
    nq = 320
    srv = agp.Server(G, max_slots=slots, queue_capacity=1024, memory_bytes=256 << 20)
    models = [(0.0, 1.0, inputs.weights_ppr(0.2, 5), 1e-3), (0.0, 0.0, inputs.weights_katz(0.02, 4), 1e-2),
              (0.5, 0.5, inputs.weights_hkpr(2.0, 3), 1e-3)]
    src = inputs.sources_uniform(g, nq, seed=3)
    qs = []
    for i in range(nq):
        a, b, w, eps = models[i % 3]
        out = torch.full((g.n,), float("nan"), dtype=torch.float32, device="cuda:0")
        if i % 5 == 4:  # a signal of several entries, one of them negative
            ids = np.random.default_rng(i).choice(g.n, 9, replace=False)
            vals = np.where(np.arange(9) == 4, -1.0, 1.0).astype(np.float32)
        else:
            ids, vals = np.array([src[i]]), np.ones(1, dtype=np.float32)
        x = (ids, vals) if ids.size > 1 else None
        qs.append((ids, vals, out, srv.submit(int(ids[0]), a, b, w, eps, 11, i, out, x=x)))
    res = [None] * nq
    t0 = time.time()
    while any(r is None for r in res):
        res = [r if r is not None else srv.poll(q[3]) for r, q in zip(res, qs)]
        assert time.time() - t0 < 60, "server did not finish"
        time.sleep(0.001)
    srv.close()
    for i, (ids, vals, out, _) in enumerate(qs):
        a, b, w, eps = models[i % 3]
        x = np.zeros(g.n, dtype=np.float32)
        x[ids] = vals
        ref, cnt = oracle.propagate(sg, a, b, w, x, eps, 11, wp=32, qids=[i])
        assert res[i]["status"] == agp.AGP_OK
        assert np.array_equal(out.cpu().numpy().astype(np.float64), ref.reshape(g.n)), i
        assert res[i]["frontier"] == int(cnt["frontier"].sum())
        assert res[i]["pushes"] == int(cnt["det"].sum() + cnt["acc"].sum())
        assert res[i]["candidates"] == int(cnt["cand"].sum())
