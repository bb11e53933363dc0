"""The normalised dedispersion bit for bit: float32 sums of the once-rounded
samples in the stated order (the channels of a sub-band, then the sub-bands),
in the first stage that shares a channel's samples among trials and in the
general one, which give the same bits.  The form that a plan takes shows in its
scratch: series of whole 1280-sample tiles in the general form, of multiples of
16 samples in the shared one."""

import ctypes

import numpy as np
import pytest

import oracle
import synth
import test_gpu_norm
import test_gpu_norm_shared
import paper_2401_13834_amd as tx
from gpu_helpers import device_block

SHAPES = [(s, True) for s in test_gpu_norm_shared.SHAPES] + [(s, False) for s in test_gpu_norm.SHAPES[1:4]]


def series(plan, nt):
    """Floats per first-stage series."""
    b = ctypes.c_int64()
    assert tx.lib().tx_dedisperse_norm_ws_size(plan._h, nt, ctypes.byref(b)) == 0
    return b.value // (4 * plan.info["ngroups"] * plan.info["nsub"])


@pytest.mark.parametrize("shape,shared", SHAPES, ids=[f"s{i}" for i in range(len(SHAPES))])
def test_form(shape, shared):
    nchan, nsub, ndm, nt, ft, fb, ts, dmmax = shape
    plan = tx.tx_plan(synth.band_centres(ft, fb, nchan), ts, np.linspace(0.0, dmmax, ndm), nsub, host_only=True)
    # over a tile of lengths, so that none is whole by chance
    whole = [series(plan, n) % 1280 == 0 for n in range(nt, nt + 2000, 40)]
    assert all(whole) != shared


def in_float32(x, ref, nt, scale, offset):
    """Samples times scale minus offset, exact in float64 (8 by 24 bits, and an
    offset of at most 2^9 scales), rounded to float32 once; sums in float32."""
    z = (x.astype(np.float64) * scale[:, None] - offset[:, None]).astype(np.float32)
    z = np.pad(z, ((0, 0), (0, nt)))
    y = np.zeros((len(ref.dms), nt), dtype=np.float32)
    for j in range(ref.ngroups):
        rows = [i for i in range(len(ref.dms)) if i // ref.g == j]
        rel = np.array([ref.d_fine_sub[i] - ref.d_coarse_sub[j] for i in rows])
        n = nt + int(rel.max())                           # (a sub-band of a smaller reach uses fewer)
        b = np.zeros((ref.nsub, n), dtype=np.float32)
        for ch in range(x.shape[0]):
            d = int(ref.d_coarse_chan[j, ch])
            b[ch // ref.m] += z[ch, d:d + n]
        for i, r in zip(rows, rel):
            for s in range(ref.nsub):
                y[i] += b[s, r[s]:r[s] + nt]
    return y


@pytest.mark.gpu
@pytest.mark.parametrize("shape,shared", SHAPES, ids=[f"s{i}" for i in range(len(SHAPES))])
def test_bits(shape, shared):
    import torch
    print(shape, flush=True)
    nchan, nsub, ndm, nt, ft, fb, ts, dmmax = shape
    freqs, dms = synth.band_centres(ft, fb, nchan), np.linspace(0.0, dmmax, ndm)
    ref = oracle.make_plan(freqs, ts, dms, nsub)
    plan = tx.tx_plan(freqs, ts, dms, nsub)
    x = test_gpu_norm._varied_block(nchan, nt + ref.overlap, nchan)
    g = np.random.Generator(np.random.PCG64(nt))
    scale = g.uniform(0.02, 0.4, nchan).astype(np.float32)
    offset = (scale * g.uniform(60.0, 190.0, nchan)).astype(np.float32)
    out = torch.zeros((ndm, nt), dtype=torch.float32, device="cuda")
    tx.tx_dedisperse_norm(plan, device_block(x), nt, torch.from_numpy(scale).to("cuda"),
                          torch.from_numpy(offset).to("cuda"), out)
    torch.cuda.synchronize()
    want = in_float32(x, ref, nt, scale.astype(np.float64), offset.astype(np.float64))
    assert np.array_equal(out.cpu().numpy().view(np.int32), want.view(np.int32))
