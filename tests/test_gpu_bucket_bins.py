"""Up to 8192 cells for each of 1024 buckets (512 per column group) the
partitioned records are summed bucket by bucket, above by bins of buckets:
bit-exact with the oracle on both sides of that size, at one bin and two."""
import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", ["1", "2"])
@pytest.mark.parametrize("n,C", [(4096, 2), (8193, 2), (131071, 64), (131072, 64), (131073, 64)])
def test_bucket_bins(n, C, groups, monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    monkeypatch.setenv("AGP_AGGREGATION", "binned")
    monkeypatch.setenv("AGP_RECORD_GROUPS", groups)
    g = inputs.chung_lu(n, 6, 2.3, seed=n)
    # the last node, in the last bin, and others
    src = np.random.default_rng(C).choice(np.flatnonzero(np.diff(g.row_ptr) > 0), size=C)
    src[-1] = np.flatnonzero(np.diff(g.row_ptr) > 0)[-1]
    x = inputs.one_hot(g.n, src).astype(np.float32)
    w, eps = inputs.weights_tp(3), 1e-4
    ref, cnt = oracle.propagate(oracle.degree_sort(g), 0.0, 1.0, w, x, eps, 6, wp=32)
    assert cnt["acc"].sum() > 0
    G = agp.Graph.from_inputs(g, validate=True)
    for _ in range(2):
        out, st = agp.propagate(G, 0.0, 1.0, w, torch.from_numpy(x).to("cuda:0"), eps, 6, stats=True)
        assert np.array_equal(out.cpu().numpy().astype(np.float64), ref)
        assert np.array_equal(st["acc"][:4], cnt["acc"].sum(axis=0).astype(np.uint64)[:4])
