"""Calls whose levels make more pushes than 1 / eps per column.

At (a, b) = (0, 1) the residue mass never grows along the arcs that the factor
degrees count, and the call need not be ready for levels of many pushes.
Along in-edges it can grow by in-degree over out-degree: such a call keeps its
record buffers (seen in the device memory that a graph's first call takes) and
equals the oracle."""
import gc

import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu

FOLLOWERS, ACCOUNTS, STARS = 1 << 18, 800, 12


def _graph():
    rng = np.random.default_rng(1)
    n = FOLLOWERS + ACCOUNTS + STARS
    acc = STARS + np.arange(ACCOUNTS)
    fol = STARS + ACCOUNTS + np.arange(FOLLOWERS)
    src = np.concatenate([np.repeat(acc, 4), np.repeat(fol, 4)])
    dst = np.concatenate([rng.integers(0, STARS, ACCOUNTS * 4), STARS + rng.integers(0, ACCOUNTS, FOLLOWERS * 4)])
    return inputs.directed_from_pairs(n, src, dst)


@pytest.mark.parametrize("reverse", [True, False])
def test_record_buffers_follow_the_push_bound(reverse, monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    g = _graph()
    x = inputs.one_hot(g.n, np.arange(STARS) if reverse else g.n - 1 - np.arange(STARS))
    X = torch.from_numpy(x).to("cuda:0")
    out = torch.empty_like(X)
    w, eps = inputs.weights_tp(2), 0.5
    # the library's code and the runtime's own memory come with its first calls
    monkeypatch.setenv("AGP_AGGREGATION", "binned")
    G = agp.Graph.from_inputs(g, directed=True, reverse=reverse)
    agp.propagate(G, 0.0, 1.0, w, X, eps, 3, out=out, stats=True)
    G.close()
    taken = {}
    for aggregation in ("atomic", "auto"):
        monkeypatch.setenv("AGP_AGGREGATION", aggregation)
        G = agp.Graph.from_inputs(g, directed=True, reverse=reverse)
        gc.collect()  # (what the collector frees meanwhile would count)
        torch.cuda.synchronize()
        gc.disable()
        try:
            free = torch.cuda.mem_get_info()[0]
            _, st = agp.propagate(G, 0.0, 1.0, w, X, eps, 3, out=out, stats=True)
            taken[aggregation] = free - torch.cuda.mem_get_info()[0]
        finally:
            gc.enable()
        ref, cnt = oracle.propagate(oracle.directed(g, reverse), 0.0, 1.0, w, x, eps, 3, wp=32, threads=8)
        assert np.array_equal(out.cpu().numpy().astype(np.float64), ref)
        for k in ("frontier", "hash", "det", "cand", "acc", "runs"):
            assert np.array_equal(st[k][:3], cnt[k].sum(axis=0).astype(np.uint64)[:3]), k
        G.close()
    pushes = int(st["det"].max() + st["acc"].max())
    assert (pushes > 100 * STARS / eps) == reverse
    buffers = 2 * 4 * g.n * STARS * 4  # two of four 4-byte records a cell
    assert (taken["auto"] - taken["atomic"] > buffers // 2) == reverse, taken
