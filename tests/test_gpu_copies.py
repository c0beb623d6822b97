"""Calls of few cells keep their next residues in four copies, added up as the
next frontier is listed (1024 cells a block); above 2^20 cells, and where a
level's pushes stay below cells / 32, there is one.  Bit-exact with the oracle
around the block's edges, at the smallest calls and on both sides of that
size and of 2^18 cells (level 0 over every cell), call after call on one
graph's scratch."""
import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu

# (n, C): cells 1, 257, around 1024 and 2048, ragged widths, around 2^18 and 2^20
SHAPES = [(1, 1), (257, 1), (1023, 1), (1024, 1), (1025, 1), (683, 3), (16383, 16), (16384, 16), (16385, 16),
          (65536, 16), (65537, 16)]


@pytest.mark.parametrize("entry", ["f32", "f64", "noalloc", "captured"])
@pytest.mark.parametrize("n,C", SHAPES)
def test_copies(n, C, entry, monkeypatch):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    if entry == "captured":
        monkeypatch.setenv("AGP_CAPTURE", "1")
    if n == 1:
        g = inputs.add_self_loops(1, np.zeros(2, np.int64), np.zeros(0, np.uint32))
    else:
        g = inputs.chung_lu(n, 6, 2.3, seed=n, self_loops=True)
    G, sg = agp.Graph.from_inputs(g, validate=True), oracle.degree_sort(g)
    wp = 64 if entry == "f64" else 32
    rng = np.random.default_rng(C)
    signed = inputs.features_normal(n, C, seed=C)
    onehot = inputs.one_hot(n, rng.integers(0, n, size=C))
    w = inputs.weights_ppr(0.2, 6)
    # other columns in between: the copies have to be left clear
    for x, eps in ((onehot, 1e-5), (signed, 1e-5), (onehot[:, :1], 1e-4), (onehot, 1e-2)):
        x = np.ascontiguousarray(x).astype(np.float32 if wp == 32 else np.float64)
        ref, _ = oracle.propagate(sg, 0.0, 1.0, w, x, eps, 9, wp=wp)
        X = torch.from_numpy(x).to("cuda:0")
        run = agp.propagate_noalloc if entry == "noalloc" else agp.propagate
        out = torch.empty_like(X)
        if entry == "noalloc":  # an allocating call makes the degree tables it needs
            agp.propagate(G, 0.0, 1.0, w, X, eps, 9)
        for _ in range(2):  # (a captured loop is replayed)
            run(G, 0.0, 1.0, w, X, eps, 9, out=out)
            assert np.array_equal(out.cpu().numpy().astype(np.float64), ref), (x.shape, eps)
