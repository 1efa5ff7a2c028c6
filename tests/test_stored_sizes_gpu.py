"""Forwards whose packed tensors lie on both sides of the size from which they are
stored non-temporally, on the per-lane and the node-per-wave layers and as separate
calls, sampled rows against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_07400_amd import bitlogic as bl
from paper_2602_07400_amd.workloads import draw_connectivity, draw_tables

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n,d,b,widths,k,specialize", [
    (150000, 128, 8, (9000, 400), 6, False),      # node per wave, 169 MB
    (140000, 128, 8, (9000, 400), 4, False),      # per lane, 158 MB
    (150000, 128, 8, (9000, 400), 3, False),      # per lane, 169 MB
    (150000, 128, 8, (9000, 400), 4, 0.0),        # specialized tables
    (700000, 300, 8, (300, 200), 5, False),       # 210 MB of wires
])
def test_forward(n, d, b, widths, k, specialize):
    rng = np.random.default_rng(n + k)
    layers, w_in = [], d * b
    for w in widths:
        layers.append((draw_connectivity(rng, w, k, w_in), draw_tables(rng, w, k)))
        w_in = w
    x = rng.integers(0, 256, size=(n, d), dtype=np.uint8)
    th = rng.integers(0, 256, size=(d, b), dtype=np.uint8)
    model = bl.BitlogicModel.from_numpy(th, layers, 10, device=DEV, specialize=specialize)
    out, am = model.forward(torch.from_numpy(x).to(DEV))
    rows = np.r_[0:64, n - 64:n, rng.integers(0, n, 2000)]
    want, best = oracle.forward(x[rows], th, layers, 10)
    assert np.array_equal(out.cpu().numpy()[rows], want)
    assert np.array_equal(am.cpu().numpy()[rows], best)


def test_separate_calls():
    rng = np.random.default_rng(2)
    n, d, b, w, k = 160000, 1100, 8, 9000, 4                # 176 and 180 MB
    x = rng.integers(0, 256, size=(n, d), dtype=np.uint8)
    th = rng.integers(0, 256, size=(d, b), dtype=np.uint8)
    conn, tab = draw_connectivity(rng, w, k, d * b), draw_tables(rng, w, k)
    bits = bl.bitlogic_encode(torch.from_numpy(x).to(DEV), torch.from_numpy(th).to(DEV))
    out = bl.bitlogic_lut_layer(bits, torch.from_numpy(conn).to(DEV),
                                torch.from_numpy(tab.view(np.int64)).to(DEV))
    scores, _ = bl.bitlogic_groupsum_head(out, n, 10)
    rows = np.r_[0:64, n - 64:n, rng.integers(0, n, 1000)]
    want, _ = oracle.forward(x[rows], th, [(conn, tab)], 10)
    assert np.array_equal(scores.cpu().numpy()[rows], want)
