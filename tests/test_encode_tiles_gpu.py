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
# features of one tile at b wires per feature, in large launches (half of it in
# small ones at b = 3 and b >= 5)
TILE = {1: 64, 2: 32, 3: 64, 4: 32, 5: 48, 6: 32, 7: 32, 8: 32}


def unpack(bits, n):
    v = np.unpackbits(bits.cpu().numpy().view(np.uint8), axis=1, bitorder="little")
    return np.ascontiguousarray(v[:, :n].T)


@pytest.mark.parametrize("b", sorted(TILE))
@pytest.mark.parametrize("n", [1, 63, 1100])
def test_feature_tiles(b, n):
    t = TILE[b]
    rng = np.random.default_rng(100 * b + n)
    for d in (1, 3, 4, 5, t // 2 - 1, t // 2 + 1, t - 1, t, t + 1, t + 5, 2 * t + 16, 3 * t - 2):
        for shift in (0, 1, 4):                   # byte address of the first row
            buf = rng.integers(0, 256, size=shift + n * d, dtype=np.uint8)
            x = torch.from_numpy(buf).to(DEV)[shift:].view(n, d)
            th = rng.integers(0, 256, size=(d, b), dtype=np.uint8)
            host = buf[shift:].reshape(n, d)
            got = bl.bitlogic_encode(x, torch.from_numpy(th).to(DEV))
            assert np.array_equal(unpack(got, n), oracle.encode(host, th)), (d, shift)
            got = bl.bitlogic_encode_binary(x, b)
            assert np.array_equal(unpack(got, n), oracle.encode_binary(host, b)), (d, shift)


@pytest.mark.parametrize("b", sorted(TILE))
def test_large_tiles(b):
    # 65 column tiles by 17 and more feature tiles: past the bound of the large size
    rng = np.random.default_rng(b)
    n, d = 64 * 1024 + 65, 32 * TILE[b] + 7 * b
    x = rng.integers(0, 256, size=(n, d), dtype=np.uint8)
    th = rng.integers(0, 256, size=(d, b), dtype=np.uint8)
    xd = torch.from_numpy(x).to(DEV)
    rows = np.r_[0:200, n - 200:n, rng.integers(0, n, 400)]
    for got, want in ((bl.bitlogic_encode(xd, torch.from_numpy(th).to(DEV)),
                       oracle.encode(x[rows], th)),
                      (bl.bitlogic_encode_binary(xd, b), oracle.encode_binary(x[rows], b))):
        word = got[:, torch.from_numpy(rows // 64).to(DEV)].cpu().numpy().view(np.uint64)
        bits = ((word >> (rows % 64).astype(np.uint64)) & np.uint64(1)).astype(np.uint8).T
        assert np.array_equal(bits, want)


def test_every_pixel_value_against_every_threshold():
    # 256 samples, sample v holding value v in every feature; feature f's
    # thresholds walk all 256 values
    x = torch.arange(256, dtype=torch.uint8, device=DEV)[:, None].expand(256, 64).contiguous()
    th = np.arange(256, dtype=np.uint8).reshape(64, 4)
    assert np.array_equal(unpack(bl.bitlogic_encode(x, torch.from_numpy(th).to(DEV)), 256),
                          oracle.encode(x.cpu().numpy(), th))
    for b in range(1, 9):
        assert np.array_equal(unpack(bl.bitlogic_encode_binary(x, b), 256),
                              oracle.encode_binary(x.cpu().numpy(), b))
