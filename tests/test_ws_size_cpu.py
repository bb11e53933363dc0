"""Scratch sized for a block serves every shorter one, also where the library
takes another first stage for it: the matrix-core form holds blocks of up to a
length that falls with the number of sub-bands.  Host plans, no device."""

import numpy as np
import pytest

import synth
import paper_2401_13834_amd as tx


def limit(plan):
    """The longest block of the matrix-core form (the last variant)."""
    mx = len(tx.tx_tile_variants(1)) - 1
    lo, hi = 1, 1 << 28
    assert plan.resolved_tiles(lo)[0] == mx and plan.resolved_tiles(hi)[0] != mx
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if plan.resolved_tiles(mid)[0] == mx:
            lo = mid
        else:
            hi = mid
    return lo


# (channels, sub-bands, tsamp, DM step, trials per group); the first two need
# more for the longest block of the matrix-core form than the general form
# rounds up to for one sample more
PLANS = [
    (512, 32, 0.00012808027139335297, 0.8052640145545372, 16),
    (512, 32, 0.00013996178143800558, 0.8911451740669624, 16),
    (1024, 64, 153.12e-6, 0.2, 4),
    (512, 8, 153.12e-6, 0.05, 1),
]


@pytest.mark.parametrize("shape", PLANS, ids=[f"p{i}" for i in range(len(PLANS))])
def test_shorter_blocks_need_no_more(shape):
    nchan, nsub, tsamp, step, g = shape
    f = synth.band_centres(1712.0, 856.0, nchan)
    plan = tx.tx_plan(f, tsamp, np.arange(16 * g) * step, nsub, dms_per_group=g, host_only=True)
    n = limit(plan)
    most = 0
    for nt in list(range(1, 6000, 7)) + list(range(n - 5000, n + 5000)):
        b = plan.ws_size(nt)
        assert b >= most, (nt, n, b, most)
        most = b
