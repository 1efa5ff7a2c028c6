"""The encoders' feature tiles on the GPU against the oracle, bit-exact: rows
around whole numbers of tiles (the last tile then starts earlier and repeats
features it does not write), rows shorter than a tile or a dword, rows at any
byte address, and batches that end inside a column or leave whole padding
columns."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_07400_amd import bitlogic as bl

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
# features of one tile at b wires per feature
TILE = {1: 64, 2: 32, 3: 64, 4: 32, 5: 36, 6: 40, 7: 32, 8: 32}


def unpack(bits, n):
    v = np.unpackbits(bits.cpu().numpy().view(np.uint8), axis=1, bitorder="little")
    return np.ascontiguousarray(v[:, :n].T)


@pytest.mark.parametrize("b", sorted(TILE))
@pytest.mark.parametrize("n", [1, 63, 1100])
def test_feature_tiles(b, n):
    t = TILE[b]
    rng = np.random.default_rng(100 * b + n)
    for d in (1, 3, 4, 5, t - 1, t, t + 1, t + 5, 2 * t + 16, 3 * t - 2):
        for shift in (0, 1, 4):                   # byte address of the first row
            buf = rng.integers(0, 256, size=shift + n * d, dtype=np.uint8)
            x = torch.from_numpy(buf).to(DEV)[shift:].view(n, d)
            th = rng.integers(0, 256, size=(d, b), dtype=np.uint8)
            host = buf[shift:].reshape(n, d)
            got = bl.bitlogic_encode(x, torch.from_numpy(th).to(DEV))
            assert np.array_equal(unpack(got, n), oracle.encode(host, th)), (d, shift)
            got = bl.bitlogic_encode_binary(x, b)
            assert np.array_equal(unpack(got, n), oracle.encode_binary(host, b)), (d, shift)
