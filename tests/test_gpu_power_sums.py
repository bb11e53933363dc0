"""Power sums of constant and extreme rows (the largest intermediate sums) and
of rows around the steps of 16384 samples, enough of them for several steps a
workgroup, against exact integers."""

import numpy as np
import pytest

import paper_2401_13834_amd as tx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nchan,nt", [(3, 1), (3, 15), (5, 16384), (5, 16385), (2048, 16384 * 9 - 7), (3000, 16384 * 6 + 33)])
def test_extreme_rows(nchan, nt):
    import torch
    pitch = (nt + 15) // 16 * 16
    d = torch.randint(0, 256, (nchan, pitch), dtype=torch.uint8, device="cuda")
    for row, v in ((0, 0), (1, 255), (2, 128)):
        d[row] = v
    sums = torch.empty((nchan, 4), dtype=torch.int64, device="cuda")
    tx.tx_channel_power_sums(d, nchan, nt, sums)
    x = d[:, :nt].to(torch.int64)
    for k in range(4):
        assert torch.equal(sums[:, k], (x ** (k + 1)).sum(dim=1))
    assert [int(s) for s in sums[1]] == [nt * 255 ** (k + 1) for k in range(4)]
