"""Quantile fitting on the GPU against the oracle around its 16-byte columns: rows
shorter than one, of whole columns and a few bytes more or less, of more columns
than a block has threads, groups that split a column, row counts that are no
multiple of a block's rows, and pixels that all fall into one bin."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_07400_amd import bitlogic as bl

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def check(x, b, groups, shift=0):
    buf = torch.empty(x.size + shift, dtype=torch.uint8, device=DEV)
    xd = buf[shift:].view(x.shape)
    xd.copy_(torch.from_numpy(x))
    th = bl.bitlogic_fit_quantile_thresholds(xd, b, groups)
    assert np.array_equal(th.cpu().numpy(), oracle.fit_quantiles(x, b, groups))


@pytest.mark.parametrize("d,groups", [(1, 1), (15, 5), (16, 1), (17, 1), (18, 3), (31, 1),
                                      (33, 11), (48, 3), (63, 7), (999, 3), (1021, 1),
                                      (16400, 2), (16397, 1)])
@pytest.mark.parametrize("n", [1, 7, 1300])
def test_columns(n, d, groups):
    rng = np.random.default_rng(n * 7 + d)
    n = max(1, n // 20) if d > 10000 else n
    x = (rng.random((n, d)) ** 1.7 * 256).astype(np.uint8)
    check(x, 1 + d % 8, groups, d % 3)


@pytest.mark.parametrize("n", [19, 20, 21, 500, 511, 512, 513])
@pytest.mark.parametrize("d,groups", [(784, 1), (3072, 3), (12, 4)])
def test_few_rows(n, d, groups):
    # 20, 5 or 1024 rows a block where the batch has fewer than 512 times as many
    rng = np.random.default_rng(n * 3 + d)
    check((rng.random((n, d)) ** 2 * 256).astype(np.uint8), 4, groups, 1)


@pytest.mark.parametrize("value", [0, 255])
def test_one_bin(value):
    check(np.full((600, 37), value, dtype=np.uint8), 3, 1, 1)
