"""Small batches, which run by 64-sample columns, against the oracle and against
the slab kernels (an environment switch keeps those), in one block a column and
stage by stage: one to many columns and nodes a lane, ragged batches, every
encoder width and fan-in, heads whose classes sit in one block or several, groups
smaller than a wave and larger than a block's rounds, inputs staged in LDS and
not, and both class heads.  Each case names the path that its sizes are to take
(they need wires for the counts' scratch: 32 a class in large batches)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_07400_amd import bitlogic as bl
from paper_2602_07400_amd.workloads import draw_connectivity
from paths import each_path

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def check(monkeypatch, path, n, d, b, widths, k, c, dsp=False, binary=False, seed=0):
    rng = np.random.default_rng([n, d, b, c, seed])
    ks = [k] * len(widths) if isinstance(k, int) else list(k)
    layers, w_in = [], d * b
    for w, kk in zip(widths, ks):
        # whole 64-bit tables: bits past 2^k are ignored
        layers.append((draw_connectivity(rng, w, min(kk, w_in), w_in),
                       rng.integers(0, 1 << 63, size=w, dtype=np.uint64) * np.uint64(2)
                       + rng.integers(0, 2, size=w, dtype=np.uint64)))
        w_in = w
    x = rng.integers(0, 256, size=(n, d), dtype=np.uint8)
    th = rng.integers(0, 256, size=(d, b), dtype=np.uint8)
    q = rng.integers(-128, 128, size=(c, c)).astype(np.int8) if dsp else None
    kw = dict(encoder="binary", n_features=d, n_bits=b) if binary else {}
    model = bl.BitlogicModel.from_numpy(None if binary else th, layers, c, device=DEV,
                                        head_weights=q, **kw)
    want, best = oracle.forward(x, th, layers, c, binary_bits=b if binary else 0)
    if dsp:
        want, best = oracle.grouped_dsp(want, q)
    xd = torch.from_numpy(x).to(DEV)
    assert model.path(n) == path
    for switch in each_path(monkeypatch, model, n):
        ws = torch.full((model.workspace_bytes(n),), 0xA5, dtype=torch.uint8, device=DEV)
        out, am = model.forward(xd, workspace=ws)
        none, only = model.forward(xd, workspace=ws, want_scores=False)
        assert none is None
        assert np.array_equal(out.cpu().numpy(), want), switch
        assert np.array_equal(am.cpu().numpy(), best), switch
        assert np.array_equal(only.cpu().numpy(), best), switch
        # with stage events the stages are kernels of their own
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(len(layers) + 3)]
        for e in ev:
            e.record()
        out, am = model.forward(xd, workspace=ws, events=ev)
        torch.cuda.synchronize()
        assert all(ev[i].elapsed_time(ev[i + 1]) >= 0 for i in range(len(layers) + 2))
        assert np.array_equal(out.cpu().numpy(), want), switch
        assert np.array_equal(am.cpu().numpy(), best), switch


# features of a group at b wires per feature
GROUP = {1: 64, 2: 32, 3: 16, 4: 16, 5: 12, 6: 8, 7: 8, 8: 8}


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000])
@pytest.mark.parametrize("b", range(1, 9))
def test_encoder_widths_and_batches(monkeypatch, n, b):
    check(monkeypatch, "block", n, 97 + b + (256 if b < 4 else 0), b, (300, 130), 1 + b % 6, 10,
          dsp=b % 2 == 0, binary=b % 3 == 0)
    # rows shorter than a group of features
    short = 3 if n <= 65 else GROUP[b] - 1
    check(monkeypatch, "block", n, short, b, (70, 66), min(3, 1 + b % 6), 1, binary=b % 3 == 1)


@pytest.mark.parametrize("k", range(1, 7))
def test_fan_ins(monkeypatch, k):
    check(monkeypatch, "block", 200, 60, 4, (257, 511, 640), k, 10)
    check(monkeypatch, "block", 129, 60, 4, (300, 260), (k, 7 - k), 13, dsp=True)


@pytest.mark.parametrize("path,n,d,widths,k,c", [
    ("block", 130, 40, (500, 7), 4, 7),      # one node a class: 64 classes in a wave's word
    ("block", 130, 410, (500, 300), 4, 300),     # more classes than waves
    ("block", 65, 40, (200, 3990), 3, 10),       # one head block, 399 nodes a class
    ("columns", 65, 40, (200, 12000), 3, 10),    # classes over several blocks
    ("columns", 65, 40, (200, 10000), 3, 2),     # a class longer than a block's rounds
    ("columns", 65, 40, (21001, 900), 3, 10),    # input rows past the LDS: gathered
    ("columns", 70, 40, (19999, 900), 2, 10),    # input rows that just fit
    ("columns", 64 * 40, 400, (12001, 100), 2, 10),      # two columns a lane
    ("columns", 64 * 60 - 1, 400, (12001, 100), 2, 10),  # four, a ragged group
    ("columns", 64 * 61, 400, (12001, 100), 4, 10),
    ("columns", 64 * 1000 + 1, 40, (20, 10), 4, 1),      # near the most columns
    ("slab", 64 * 1024 + 1, 40, (20, 10), 4, 1),         # one past them
])
def test_shapes(monkeypatch, path, n, d, widths, k, c):
    check(monkeypatch, path, n, d, 3, widths, k, c)
    if c <= 128:
        check(monkeypatch, path, n, d, 3, widths, k, c, dsp=True, seed=1)



@pytest.mark.parametrize("path,d,widths,c", [("block", 50, (1000, 900, 800, 700), 10),
                                             ("columns", 50, (60, 70, 80, 90, 100), 5),
                                             ("block", 970, (1025, 1024, 1030), 206)])
def test_depths_in_one_block_and_deeper(monkeypatch, path, d, widths, c):
    check(monkeypatch, path, 300, d, 2, widths, [2, 6, 1, 3, 5][:len(widths)], c)
