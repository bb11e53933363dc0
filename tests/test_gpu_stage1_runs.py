"""The matrix-core first stage where a workgroup takes a run of several tiles:
rows of the next tile loaded during the current one, stores of the last tile
still on their way, one staging buffer and two carried from tile to tile, several
rounds of channels a tile, dropped channels, wavefronts with nothing to do in
some tiles of a run.  A run is as many tiles (at most 8) as 2048 goes into a
call's tiles of 1152 samples x sub-bands x 16 trials."""

import numpy as np
import pytest

import oracle
import synth
import paper_2401_13834_amd as tx
from test_gpu_stage1_mx import exact_block, mx_variant

pytestmark = pytest.mark.gpu

# name: (channels, sub-bands, trials, DM step, block, LDS bytes, runs of at least)
CASES = {
    "m3": (96, 32, 17, 2.0, 75001, 0, 2),
    "m3 one buffer": (96, 32, 17, 2.0, 75001, 6000, 2),
    "m7 one buffer, two rounds": (224, 32, 17, 1.0, 75011, 6000, 2),
    "m21 two rounds": (336, 16, 33, 1.0, 100003, 0, 2),
    "m21 three rounds": (336, 16, 33, 1.0, 100003, 23000, 2),
    "spread trials": (96, 32, 16, 300.0, 148003, 0, 2),
    "spread trials, one buffer": (96, 32, 16, 300.0, 148003, 6000, 2),
    "longest runs": (192, 64, 17, 2.0, 150001, 0, 8),
    "ends with a run": (64, 64, 15, 0.1, 1152 * 72 - 15, 0, 2),
}


@pytest.mark.parametrize("case", list(CASES))
def test_matches_oracle(case):
    import torch
    print(case, flush=True)
    nchan, nsub, ndm, step, nt, lds, run = CASES[case]
    assert (nt // 1152 + 2) * nsub * ((ndm + 15) // 16) // 2048 >= run
    f = synth.band_centres(1500.0, 1200.0, nchan)
    dms = np.arange(ndm) * step
    ref = oracle.make_plan(f, 256e-6, dms, nsub, g=1)
    plan = tx.tx_plan(f, 256e-6, dms, nsub, dms_per_group=1)
    plan.set_tiles(mx_variant(), lds, -1, 0)
    assert plan.resolved_tiles(nt)[0] == mx_variant()
    x = synth.uniform_u8(nchan, nt + ref.overlap, 9)
    d = exact_block(x)
    y = torch.full((ndm, nt + (nt & 1)), -3, dtype=torch.int32, device="cuda")
    tx.tx_dedisperse(plan, d, nt, y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy()[:, :nt], oracle.dedisperse_subband(x, ref, nt))
    mask = np.ones(nchan, dtype=np.uint8)
    mask[1::3] = 0
    mask[-1] = 0
    plan.set_mask(mask)
    tx.tx_dedisperse(plan, d, nt, y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy()[:, :nt], oracle.dedisperse_subband(x * mask[:, None], ref, nt))
