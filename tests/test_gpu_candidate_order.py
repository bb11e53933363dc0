"""The order in which tx_candidates lists what it finds in blocks of up to 1280
rows of up to 65536 samples, one workgroup a row: every 64 starts of a row are
listed together in their order, and the row's wavefronts take turns."""

import numpy as np
import pytest

import paper_2401_13834_amd as tx
from gpu_helpers import as_tuples, gpu_candidates
from oracle import c_oracle
from test_gpu_boxcar import device

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 4, 8]


@pytest.mark.parametrize("rows,nt", [(1, 4096), (1, 4100), (5, 12289), (2, 65536), (128, 8192), (1280, 4097)])
def test_wavefronts_take_turns(rows, nt):
    import torch
    print(rows, nt, flush=True)
    g = np.random.Generator(np.random.PCG64(rows + nt))
    y = g.integers(1000, 1040, (rows, nt), dtype=np.int32)
    # every start is a candidate in the last row, a few in the others
    want = c_oracle.boxcar_candidates(y, WIDTHS, 2.5)
    n, rec = gpu_candidates(device(y, 0), nt, WIDTHS, 2.5)
    assert n == len(want) and sorted(as_tuples(rec)) == want
    raw = torch.zeros((nt, 3), dtype=torch.int64, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    tx.tx_candidates(device(y[-1:], 0), nt, WIDTHS, -1e6, raw, count)
    assert int(count.item()) == nt
    t = raw[:, 1].cpu().numpy()                             # as listed
    assert np.array_equal(np.sort(t), np.arange(nt))
    lead = np.flatnonzero(t % 64 == 0)                      # groups of 64 starts, in their order
    for i in lead:
        assert np.array_equal(t[i:i + min(64, nt - t[i])], t[i] + np.arange(min(64, nt - t[i])))
    # listed one wavefront after the other the first tile would be 4 runs of 16 groups
    wave = t[lead][t[lead] < 4096] // 64 % 4
    assert len(wave) == 64 and np.count_nonzero(np.diff(wave)) > 16
