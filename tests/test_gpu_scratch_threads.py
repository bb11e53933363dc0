"""Kept scratch under several threads, each with a stream of its own and
several calls queued on it before it is waited for; a call that fails in a
thread fails the test."""

from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import paper_2401_13834_amd as tx
from test_gpu_scratch import job

pytestmark = pytest.mark.gpu


def test_queued_calls():
    import torch
    jobs = [job(name, 30 + k) for k, name in enumerate(["small", "middle", "small", "middle", "small", "middle"])]
    torch.cuda.synchronize()

    def work(k):
        plan, d, nt, want = jobs[k]
        other = jobs[(k + 2) % len(jobs)]                 # the same kind of block with other samples
        st = torch.cuda.Stream()
        done = 0
        with torch.cuda.stream(st):
            for _ in range(4):
                outs = []
                for p, x, n, w in (jobs[k], other, jobs[k], other):
                    y = torch.full((p.ndm, n), -1, dtype=torch.int32, device="cuda")
                    tx.tx_dedisperse(p, x, n, y, stream=st)
                    outs.append((y, w))
                st.synchronize()
                for y, w in outs:
                    assert np.array_equal(y.cpu().numpy(), w), k
                    done += 1
        return done

    with ThreadPoolExecutor(len(jobs)) as pool:
        assert [f.result() for f in [pool.submit(work, k) for k in range(len(jobs))]] == [16] * len(jobs)
