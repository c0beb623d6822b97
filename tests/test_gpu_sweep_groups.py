"""The batched sweep orders all columns of a group in one sort and parts them
by a stable pass over the bits a column number needs: sizes and conductances
bit-exact with the oracle's sweep at the widths where the bits, the groups of
64 and the last group change, with ties across columns and signed values."""
import math

import numpy as np
import pytest

import oracle
from paper_2106_03058_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 700, 17000])
@pytest.mark.parametrize("C", [1, 2, 3, 32, 33, 64, 65, 130])
def test_group_widths(n, C):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_03058_amd import agp

    g = inputs.chung_lu(n, 5, 2.3, seed=n)
    G = agp.Graph.from_inputs(g)
    rng = np.random.default_rng(C)
    # few distinct values: the same keys in many columns and nodes; zeros, both signs
    P = (rng.integers(-2, 6, size=(n, C)) * 0.125).astype(np.float32)
    P[:, C // 2] = 0.0
    size, phi = agp.sweep_batch(G, torch.from_numpy(P).to("cuda:0"))
    for c in range(0, C, max(1, C // 9)):
        rs, rphi, _ = oracle.sweep(g, P[:, c].astype(np.float64))
        assert (size[c], phi[c]) == (rs, rphi) or (size[c] == rs == 0 and math.isinf(phi[c])), c
