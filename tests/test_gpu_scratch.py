"""Scratch kept between calls: several threads, each with a stream of its own
and blocks of its own sizes (from below the smallest kept buffer to above the
largest), get the oracle's results; so do calls that follow each other on
changing streams without a synchronisation, and calls after a trim."""

import threading

import numpy as np
import pytest

import oracle
import synth
import paper_2401_13834_amd as tx
from gpu_helpers import device_block

pytestmark = pytest.mark.gpu

SIZES = {"small": (16, 8, 700), "middle": (64, 60, 40000), "large": (64, 400, 30000)}   # channels, trials, samples


def job(name, seed):
    nchan, ndm, nt = SIZES[name]
    f = synth.band_centres(1500.0, 1200.0, nchan)
    dms = np.arange(ndm) * 0.5
    g = 1 if name == "large" else 4
    ref = oracle.make_plan(f, 256e-6, dms, 4, g=g)
    plan = tx.tx_plan(f, 256e-6, dms, 4, dms_per_group=g)
    x = synth.uniform_u8(nchan, nt + ref.overlap, seed)
    return plan, device_block(x), nt, oracle.dedisperse_subband(x, ref, nt)


def test_sizes_span_the_kept_buffers():
    got = [job(name, 1)[0].ws_size(SIZES[name][2]) for name in SIZES]
    assert got[0] < 4 << 20 < got[1] < 64 << 20 < got[2]


def test_threads_and_streams():
    import torch
    jobs = [job(name, 10 + k) for k, name in enumerate(["small", "middle", "large", "small", "middle"])]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        plan, d, nt, want = jobs[k]
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for _ in range(6):
                y = torch.full((plan.ndm, nt), -1, dtype=torch.int32, device="cuda")
                tx.tx_dedisperse(plan, d, nt, y, stream=st)
                st.synchronize()
                if not np.array_equal(y.cpu().numpy(), want):
                    bad.append(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


@pytest.mark.parametrize("trim", [False, True])
def test_changing_streams(trim):
    import torch
    jobs = [job(name, 20 + k) for k, name in enumerate(["small", "middle", "small", "middle"])]
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [torch.full((p.ndm, nt), -1, dtype=torch.int32, device="cuda") for p, _, nt, _ in jobs for _ in range(3)]
    torch.cuda.synchronize()
    if trim:
        tx.tx_pool_trim()
    for k, y in enumerate(outs):
        plan, d, nt, _ = jobs[k // 3]
        tx.tx_dedisperse(plan, d, nt, y, stream=streams[k % 3])
    torch.cuda.synchronize()
    for k, y in enumerate(outs):
        assert np.array_equal(y.cpu().numpy(), jobs[k // 3][3])
