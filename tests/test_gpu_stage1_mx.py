"""The matrix-core first stage against the oracle, bit for bit, where its tiling
can go wrong: channels per sub-band that are no multiple of 4, coarse trials
around multiples of 4 and 16, block lengths around a tile (1152 outputs) and a
run of tiles, trials spread over one and many 16-byte windows, rows whose last
piece straddles the end of the input, dropped channels, band orders, byte
offsets of a stream, one and two staging buffers."""

import numpy as np
import pytest

import oracle
import synth
import paper_2401_13834_amd as tx

pytestmark = pytest.mark.gpu

# name: (channels, sub-bands, trials, DM step, DMs per group, block, band order, LDS bytes)
CASES = {
    "one channel": (4, 4, 9, 3.0, 2, 1153, "down", 0),
    "m3": (12, 4, 17, 2.0, 1, 1151, "down", 0),
    "m5 one trial": (10, 2, 1, 5.0, 1, 1152, "down", 0),
    "m7 up": (14, 2, 33, 1.0, 2, 2305, "up", 0),
    "m16 coarse": (32, 2, 40, 40.0, 1, 700, "down", 0),
    "m16 mixed": (32, 2, 15, 9.0, 1, 3001, "mixed", 0),
    "m64": (64, 1, 21, 0.3, 1, 1200, "down", 0),
    "m64 one buffer": (64, 1, 21, 0.3, 1, 2500, "down", 13000),
    "m256": (256, 1, 5, 1.5, 1, 1400, "down", 0),
    "long": (8, 2, 6, 1.0, 1, 40001, "down", 0),
    "short": (8, 2, 6, 1.0, 1, 1, "down", 0),
}


def mx_variant():
    return len(tx.tx_tile_variants(1)) - 1


def build(case):
    nchan, nsub, ndm, step, g, nt, order, lds = CASES[case]
    f = synth.band_centres(1500.0, 1200.0, nchan)
    if order == "up":
        f = f[::-1].copy()
    elif order == "mixed":
        f = f[np.random.Generator(np.random.PCG64(3)).permutation(nchan)]
    dms = np.arange(ndm) * step
    ref = oracle.make_plan(f, 256e-6, dms, nsub, g=g)
    plan = tx.tx_plan(f, 256e-6, dms, nsub, dms_per_group=g)
    plan.set_tiles(mx_variant(), lds, -1, 0)
    return ref, plan, nt


def exact_block(x):
    """Device rows whose last row ends with the last valid byte (of a
    16-byte multiple pitch): the input's allocation holds nothing past it."""
    import torch
    nchan, n = x.shape
    pitch = (n + 15) // 16 * 16
    flat = torch.full((nchan * pitch,), 201, dtype=torch.uint8, device="cuda")
    d = torch.as_strided(flat, (nchan, n), (pitch, 1))
    d.copy_(torch.from_numpy(x).to("cuda"))
    return d


@pytest.mark.parametrize("case", list(CASES))
def test_matches_oracle(case):
    import torch
    print(case, flush=True)
    ref, plan, nt = build(case)
    x = synth.uniform_u8(plan.nchan, nt + ref.overlap, 5)
    y = torch.full((plan.ndm, nt + (nt & 1)), -3, dtype=torch.int32, device="cuda")
    tx.tx_dedisperse(plan, exact_block(x), nt, y)
    torch.cuda.synchronize()
    assert plan.resolved_tiles(nt)[0] == mx_variant()
    assert np.array_equal(y.cpu().numpy()[:, :nt], oracle.dedisperse_subband(x, ref, nt))
    # dropped channels, the last one among them
    mask = np.ones(plan.nchan, dtype=np.uint8)
    mask[::3] = 0
    mask[-1] = 0
    plan.set_mask(mask)
    tx.tx_dedisperse(plan, exact_block(x), nt, y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy()[:, :nt], oracle.dedisperse_subband(x * mask[:, None], ref, nt))


@pytest.mark.parametrize("case", ["m3", "m7 up", "m16 coarse"])
def test_stream_offsets(case):
    """Blocks of odd lengths: every push reads its rows at another byte offset
    until the history is full, then the history's own."""
    import torch
    print(case, flush=True)
    ref, plan, nt = build(case)
    total = nt + ref.overlap
    x = synth.uniform_u8(plan.nchan, total, 6)
    want = oracle.dedisperse_subband(x, ref, nt)
    s = tx.Stream(plan, 1003)
    got, at = [], 0
    while at < total:
        n = min(1003 if at % 2 else 997, total - at)
        block = torch.from_numpy(np.ascontiguousarray(x[:, at:at + n])).to("cuda")
        y = torch.empty((plan.ndm, 1004), dtype=torch.int32, device="cuda")
        m = s.push(block, n, y)
        torch.cuda.synchronize()
        got.append(y[:, :m].cpu().numpy())
        at += n
    assert np.array_equal(np.concatenate(got, axis=1), want)


def test_batch_equals_alone():
    import torch
    jobs = []
    b = tx.Batch(4)
    for k, case in enumerate(["m3", "m64", "m16 coarse", "m256"]):
        ref, plan, nt = build(case)
        x = synth.uniform_u8(plan.nchan, nt + ref.overlap, 20 + k)
        d = exact_block(x)
        y = torch.empty((plan.ndm, nt + (nt & 1)), dtype=torch.int32, device="cuda")
        b.add(plan, d, nt, y)
        jobs.append((ref, plan, nt, x, d, y))
    b.launch()
    torch.cuda.synchronize()
    for ref, plan, nt, x, d, y in jobs:
        assert np.array_equal(y.cpu().numpy()[:, :nt], oracle.dedisperse_subband(x, ref, nt))


@pytest.mark.parametrize("order", [("fine", "coarse"), ("coarse", "fine")])
def test_graph_takes_plans_of_either_form(order):
    """A captured batch launched again with a plan that would choose the other
    first stage: DM steps of 0.2 choose the matrix-core form, of 40 the general."""
    import torch
    f = synth.band_centres(1500.0, 1200.0, 32)
    st = torch.cuda.Stream()
    b = tx.Batch(1, graph=True)
    for k, name in enumerate(order):
        dms = np.arange(32) * (0.2 if name == "fine" else 40.0)
        ref = oracle.make_plan(f, 256e-6, dms, 2, g=1)
        plan = tx.tx_plan(f, 256e-6, dms, 2, dms_per_group=1)
        assert (plan.resolved_tiles(1500)[0] == mx_variant()) == (name == "fine")
        x = synth.uniform_u8(32, 1500 + ref.overlap, 40 + k)
        d = exact_block(x)
        y = torch.empty((32, 1500), dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        b.clear()
        b.add(plan, d, 1500, y)
        b.launch(st)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), oracle.dedisperse_subband(x, ref, 1500))
