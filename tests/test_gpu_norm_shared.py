"""The first stage of normalised data in the form that shares a channel's
normalised samples among trials, within the rounding bound of the general
form's test: blocks around a tile of 1280, coarse trials around multiples of 4
and 16, odd numbers of channels per sub-band, trials further apart than the 8
samples that one reading serves, delays far beyond a tile."""

import pytest

import test_gpu_norm

pytestmark = pytest.mark.gpu

SHAPES = [  # (nchan, nsub, ndm, nt, f_top, f_bot, tsamp, dm_max): plans of few windows and little padding
    (12, 4, 96, 1281, 1712.0, 856.0, 306.24e-6, 3.0),
    (64, 4, 200, 1280, 1712.0, 856.0, 306.24e-6, 20.0),
    (40, 8, 330, 2600, 1500.0, 1100.0, 1e-3, 60.0),
    (256, 2, 130, 1300, 1712.0, 856.0, 153.12e-6, 12.0),
    (28, 4, 700, 5003, 1712.0, 856.0, 153.12e-6, 90.0),
    (96, 12, 57, 1025, 1500.0, 1100.0, 1e-3, 30.0),
    (128, 8, 160, 1290, 1400.0, 1000.0, 64e-6, 40.0),
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"s{i}" for i in range(len(SHAPES))])
@pytest.mark.parametrize("weighting", [0, 1])
def test_within_rounding_bound(shape, weighting):
    test_gpu_norm.test_dedisperse_norm_within_rounding_bound(shape, weighting)
