"""bitlogic_lut_layer on row-major bits against the oracle: windows of 16 words
whole and ragged, rows of odd word counts and 8-byte aligned buffers, one-pass and
multi-pass node blocks with whole and partial blocks, every fan-in."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_07400_amd import bitlogic as bl
from paper_2602_07400_amd.workloads import draw_connectivity

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def buffer(rows, words, shift):
    """int64 [rows][words] whose first word is `shift` words into an allocation."""
    return torch.full((rows * words + shift,), -1, dtype=torch.int64,
                      device=DEV)[shift:].view(rows, words)


def run(w_in, w, k, W, shift, seed):
    rng = np.random.default_rng(seed)
    bits = rng.integers(0, 1 << 63, size=(w_in, W), dtype=np.uint64) << np.uint64(1)
    bits |= rng.integers(0, 2, size=bits.shape, dtype=np.uint64)
    conn = draw_connectivity(rng, w, k, w_in)
    tab = rng.integers(0, 1 << 63, size=w, dtype=np.uint64) << np.uint64(1)
    src, dst = buffer(w_in, W, shift), buffer(w, W, shift)
    src.copy_(torch.from_numpy(bits.view(np.int64)))
    out = bl.bitlogic_lut_layer(src, torch.from_numpy(conn).to(DEV),
                                torch.from_numpy(tab.view(np.int64)).to(DEV), bits_out=dst)
    # every word, or of long rows the first and last windows and 32 others
    cols = (np.arange(W) if W <= 64 else
            np.r_[0:16, np.sort(rng.choice(np.arange(16, W - 16), 32, replace=False)), W - 16:W])
    v = np.unpackbits(np.ascontiguousarray(bits[:, cols]).view(np.uint8), axis=1,
                      bitorder="little").T
    want = oracle.lut_layer(np.ascontiguousarray(v), conn, tab)
    got = out[:, torch.from_numpy(cols).to(DEV)].cpu().numpy()
    got = np.unpackbits(got.view(np.uint8), axis=1, bitorder="little").T
    assert np.array_equal(got, want)


@pytest.mark.parametrize("k", range(1, 7))
@pytest.mark.parametrize("W", [1, 15, 16, 17, 33, 64])
def test_windows(k, W):
    run(50 + k, 131, k, W, W % 2, 10 * W + k)
    run(40, 32, k, W, 1, 10 * W + k + 1)


@pytest.mark.parametrize("w_in,w,W,shift", [
    (60, 70, 16, 0),                  # one window, nodes in a short pass
    (60, 70, 48, 16),                 # buffers that start a line later
    (60, 70, 48, 2),                  # and inside one
    (300, 64 * 3 + 1, 1024, 0),       # a row of 8 KB
    (5859, 70, 1024, 0),              # the most rows of it, and one more
    (5860, 70, 1024, 0),
    (300, 256 * 136 + 5, 480, 0),     # multi-pass blocks, the last of 5 nodes
    (24000, 70, 480, 0),              # 88 and 92 MiB of input
    (25200, 70, 480, 0),
    (2000, 70, 1030, 0),              # rows of parts of lines, 15.7 and 16.1 MiB
    (2050, 70, 1030, 1),
])
def test_lanes_a_node_at_fan_in_6(w_in, w, W, shift):
    run(w_in, w, 6, W, shift, w_in + W)


@pytest.mark.parametrize("W,shift", [(1563, 0), (1564, 0), (1560, 0), (1560, 8), (1560, 1),
                                     (1568, 0)])
@pytest.mark.parametrize("k", [2, 6])
def test_tensors_past_the_cache(k, W, shift):
    # 173 MB of output, in parts of lines, half lines and whole lines
    run(40, 13800, k, W, shift, W + k + shift)


@pytest.mark.parametrize("k", [1, 3, 4, 5, 6])
def test_multi_pass_blocks(k):
    # 2097 node blocks of 128 nodes, the last of 5, over two windows
    run(3000, 128 * 2096 + 5, k, 17 + k % 2, k % 2, k)
