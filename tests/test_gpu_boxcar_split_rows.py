"""Rows that no part of a split row can judge alone: a value out of range in
one part, a constant row, a row constant but for its last part.  Peaks are split
over workgroups from 3 tiles of 4096 starts a row, candidate lists from 17."""

import numpy as np
import pytest

import oracle
from gpu_helpers import as_tuples, gpu_candidates, gpu_peaks
from test_gpu_boxcar import device

pytestmark = pytest.mark.gpu

WIDTHS = [1, 4, 64]


@pytest.mark.parametrize("nt", [4096 * 3 + 1, 4096 * 17 - 3, 4096 * 66 + 11])
@pytest.mark.parametrize("shift", [0, 1])
def test_flagged_and_constant_rows(nt, shift):
    print(nt, shift, flush=True)
    y = np.random.Generator(np.random.PCG64(nt)).integers(0, 100, (8, nt), dtype=np.int32)
    y[0, nt - 1] = 2 ** 21                    # out of range in the last part
    y[1, 5] = -1                              # and in the first
    y[2] = 77                                 # constant
    y[3] = 77
    y[3, nt - 2:] = 78                        # constant but for the last part
    y[4] = 0
    y[5, nt // 2] = -2 ** 31
    y[6, nt // 2:nt // 2 + 9] = 900
    good = [2, 3, 4, 6, 7]
    want = oracle.boxcar_peaks(y[good], WIDTHS)
    cands = [(good[c[0]],) + tuple(c[1:]) for c in oracle.boxcar_candidates(y[good], WIDTHS, 6.0)]
    assert any(c[0] == 3 for c in cands) and any(c[0] == 6 for c in cands)
    d = device(y, shift)
    n, rec, listed = gpu_candidates(d, nt, WIDTHS, 6.0, with_peaks=True)
    assert n == len(cands) and as_tuples(rec) == cands
    for snr, wid, tim in (gpu_peaks(d, nt, WIDTHS), listed):
        for a, b in zip((snr, wid, tim), want):
            assert np.array_equal(a[good], b)
        for r in (0, 1, 5):
            assert np.isnan(snr[r]) and wid[r] == -1 and tim[r] == -1
        for r in (2, 4):
            assert (snr[r], wid[r], tim[r]) == (0.0, WIDTHS[0], 0)
