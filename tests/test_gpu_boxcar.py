"""The matched filter against the oracle where equal sums compete and rows are
split over workgroups: few and many tiles (4096 starts each), the earliest of
equal peaks in different lanes, wavefronts, tiles and parts, candidates in many tiles and up to the row's end, unaligned rows,
and a capture (which is not split)."""

import numpy as np
import pytest

import paper_2401_13834_amd as tx
from gpu_helpers import as_tuples, gpu_candidates, gpu_peaks
from oracle import c_oracle

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 5, 16, 100, 1024]
# rows, samples: below one tile to many, whole tiles and remainders
SHAPES = [(1, 4096), (3, 8193), (5, 12288), (2, 4096 * 65 + 7), (127, 4096 * 3 + 1), (128, 4096 * 6 - 1),
          (129, 4096 * 5 + 5), (300, 4096 * 9 + 33), (4, 900)]


def rows(ndm, nt):
    g = np.random.Generator(np.random.PCG64(ndm * 7 + nt))
    y = g.integers(1000, 1040, (ndm, nt), dtype=np.int32)
    for d in range(ndm):
        # equal pulses (a flat patch each, so that starts within it tie too)
        for t in range(d % 50 + 17, nt - 40, 4096 + 255):
            y[d, t:t + 40] = 1100
        y[d, nt - 3:] = 1090                               # windows that end with the row
    return y


def device(y, shift):
    """int32 rows starting `shift` elements past a 16-byte boundary."""
    import torch
    ndm, nt = y.shape
    pitch = nt + (nt & 1) + 2
    flat = torch.zeros(ndm * pitch + 4, dtype=torch.int32, device="cuda")
    d = torch.as_strided(flat, (ndm, pitch), (pitch, 1), shift)
    d[:, :nt] = torch.from_numpy(y).to("cuda")
    return d


@pytest.mark.parametrize("shape", SHAPES)
def test_matches_oracle(shape):
    print(shape, flush=True)
    y = rows(*shape)
    nt = shape[1]
    want = c_oracle.boxcar_peaks(y, WIDTHS)
    cands = c_oracle.boxcar_candidates(y, WIDTHS, 6.0)
    for shift in (0, 1):
        d = device(y, shift)
        for a, b in zip(gpu_peaks(d, nt, WIDTHS), want):
            assert np.array_equal(a, b)
        got = gpu_candidates(d, nt, WIDTHS, 6.0, with_peaks=True)
        assert got[0] == len(cands) and sorted(as_tuples(got[1])) == cands
        for a, b in zip(got[2], want):
            assert np.array_equal(a, b)


def test_capture():
    import torch
    y = rows(4, 4096 * 12 + 9)
    d = device(y, 0)
    out = (torch.empty(4, dtype=torch.float64, device="cuda"), torch.empty(4, dtype=torch.int32, device="cuda"),
           torch.empty(4, dtype=torch.int64, device="cuda"))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        tx.tx_boxcar_snr(d, y.shape[1], WIDTHS, *out, stream=torch.cuda.current_stream())
    for k in range(3):
        d += 1
        for o in out:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, c_oracle.boxcar_peaks(y + k + 1, WIDTHS)):
            assert np.array_equal(a.cpu().numpy(), b)
