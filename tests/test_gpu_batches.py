"""The split of a level's work among the waves: batches of entries sized by
the frontier, work items sized by their expected draws, and batches whose
entries together make many pushes or items, which leave for the grid-wide
kernels; bit-exact with the oracle around every edge of those rules."""
import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    return torch, agp


def _hub_graph(degrees, n, seed):
    rng = np.random.default_rng(seed)
    src, dst = [rng.integers(0, n, size=3 * n)], [rng.integers(0, n, size=3 * n)]
    for h, d in enumerate(degrees):
        src.append(np.full(d, h))
        dst.append(rng.choice(np.arange(len(degrees), n), size=d, replace=False))
    return inputs.csr_from_pairs(n, np.concatenate(src), np.concatenate(dst))


def _check(torch, agp, g, x, a, b, w, eps, wp=32):
    G = agp.Graph.from_inputs(g, validate=True)
    ref, cnt = oracle.propagate(oracle.degree_sort(g), a, b, w, x, eps, 31, wp=wp)
    out, st = agp.propagate(G, a, b, w, torch.from_numpy(x).to("cuda:0"), eps, 31, stats=True)
    assert np.array_equal(out.cpu().numpy().astype(np.float64), ref)
    for k in ("frontier", "hash", "det", "cand", "acc", "runs"):
        assert np.array_equal(st[k], cnt[k].sum(axis=0).astype(np.uint64)), k
    return cnt


# hubs of 130 and 600 neighbours in 64 columns: rows that are short by themselves
# but 64 of which make one batch of more than 2048 pushes or 512 items
@pytest.mark.parametrize("aggregation", ["atomic", "binned", "auto"])
@pytest.mark.parametrize("model", ["det", "sampled", "general"])
def test_batches_of_one_hub(env, model, aggregation, monkeypatch):
    torch, agp = env
    monkeypatch.setenv("AGP_AGGREGATION", aggregation)
    g = _hub_graph((130, 600, 900), 3000, 5)
    src = [1] * 31 + [0] * 20 + [2] * 13
    x = inputs.one_hot(g.n, src)
    a, b, w, eps = {
        "det": (0.0, 0.0, inputs.weights_katz(0.01, 3), 1e-4),
        "sampled": (0.0, 0.0, inputs.weights_katz(0.4, 4), 0.9),   # c just below theta: up to 64 draws a window
        "general": (0.5, 0.5, inputs.weights_ppr(0.2, 5), 1e-2),
    }[model]
    cnt = _check(torch, agp, g, x.astype(np.float32), a, b, w, eps)
    assert cnt["det" if model == "det" else "cand"][:, :2].sum() > 2048


# frontiers around one entry per resident wave (4096), one batch per resident
# wave (262144) and ragged last batches
@pytest.mark.parametrize("n,C,wp", [(4095, 1, 32), (4096, 1, 32), (4097, 1, 64), (8193, 1, 32), (4096, 64, 32),
                                    (4099, 64, 32), (2731, 3, 64)])
def test_full_frontiers(env, n, C, wp):
    torch, agp = env
    g = inputs.chung_lu(n, 6, 2.5, seed=n, self_loops=True)
    x = inputs.features_normal(n, C, seed=C).astype(np.float32 if wp == 32 else np.float64)
    _check(torch, agp, g, x, 0.5, 0.5, inputs.weights_hkpr(2.0, 3), 2.0 / n, wp=wp)
