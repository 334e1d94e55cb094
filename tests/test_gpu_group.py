"""The group-sum forward kernel: what an integer plan runs by default where groups of
neighbouring channels share few delay patterns.  Explicitly chosen tiles run the staged or
direct-read kernel of that shape instead, so every case here is checked both against the
oracle and, bit for bit, against the plan with its own default shape chosen explicitly.
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import oracle_table, plan_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dd():
    import paper_2311_05341_amd as dd
    assert torch.cuda.is_available()
    return dd


def _input(dtype, n_chan, n_samp, seed):
    """Random samples in rows padded to whole 16 bytes; the padding holds the largest value."""
    rng = np.random.default_rng(seed)
    elem = {"u8": np.uint8, "u4": np.uint8, "u16": np.uint16}[dtype]
    n = n_samp // 2 if dtype == "u4" else n_samp
    unit = 16 // np.dtype(elem).itemsize
    x = np.full((n_chan, (n + unit - 1) // unit * unit), np.iinfo(elem).max, dtype=elem)
    x[:, :n] = rng.integers(0, np.iinfo(elem).max + 1, (n_chan, n), dtype=elem)
    return x


# (channels, samples, trials, dm_start, dm_step): rows of whole 16-byte units whose last samples are
# needed, ragged rows, DM blocks with a tail, a partial last group of channels, less than one time
# tile, tiles that start right at a row's end, no delay at all, pattern rows of one to seven chunks
CASES = [(512, 32768, 96, 0.0, 0.5), (512, 32770, 97, 10.0, 0.25), (301, 20032, 33, 0.0, 0.5), (1024, 3000, 130, 0.0, 0.1),
         (257, 1026, 40, 0.0, 0.0), (1024, 40000, 64, 200.0, 1.0), (2048, 16384, 65, 0.0, 2.0), (515, 9216, 200, 0.0, 0.25)]


@pytest.mark.parametrize("dtype", ["u8", "u4", "u16"])
@pytest.mark.parametrize("case", CASES)
def test_default_route_equals_oracle_and_explicit_shape(dd, dtype, case):
    n_chan, n_samp, n_dm, start, step = case
    cfg = dict(dtype=dtype, n_chan=n_chan, n_samp=n_samp, f_high=1500.0, chan_bw=300.0 / n_chan, t_samp=64e-6,
               dm_start=start, dm_step=step, n_dm=n_dm)
    s = oracle_table(cfg)
    x = _input(dtype, n_chan, n_samp, 7)
    want = oracle.forward(x, dtype, n_samp, s)
    plan = plan_for(dd, cfg, in_pitch_bytes=x.strides[0])
    xd = torch.from_numpy(x).cuda()
    out = torch.full((plan.n_dm, plan.out_pitch + 8), -7.0, dtype=torch.float32, device="cuda")
    got = plan.forward(xd, out=out)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), want)
    assert bool((out[:, plan.n_out:] == -7.0).all())  # nothing is written past the row
    t = plan.tiles(0)
    plan.set_tiles(0, t["shape"], t["order"])
    assert np.array_equal(plan.forward(xd).cpu().numpy(), want)


@pytest.mark.parametrize("dtype", ["u8", "u16"])
def test_unordered_frequencies(dd, dtype):
    """Delays that are not monotone in the channel: windows that start before the tile's first sample."""
    rng = np.random.default_rng(3)
    n_chan, n_samp, n_dm = 96, 9000, 50
    freqs = 1500.0 - rng.permutation(n_chan) * (300.0 / n_chan)
    s = oracle.shift_table(n_chan, 1500.0, 0.0, 64e-6, 0.0, 0.03, n_dm, freqs=freqs)
    xp = _input(dtype, n_chan, n_samp, 8)
    plan = dd.Plan(n_chan, n_samp, dtype, 1500.0, 0.0, 64e-6, 0.0, 0.03, n_dm, chan_freq=freqs,
                   in_pitch_bytes=xp.strides[0])
    got = plan.forward(torch.from_numpy(xp).cuda()).cpu().numpy()
    assert np.array_equal(got, oracle.forward(xp, dtype, n_samp, s))


def test_replayed_graph_and_side_stream(dd):
    """Captured calls replay with fresh inputs, and a side stream gives the same bits."""
    cfg = dict(dtype="u8", n_chan=512, n_samp=20000, f_high=1500.0, chan_bw=300.0 / 512, t_samp=64e-6, dm_start=0.0,
               dm_step=0.5, n_dm=64)
    s = oracle_table(cfg)
    x = _input("u8", cfg["n_chan"], cfg["n_samp"], 9)
    plan = plan_for(dd, cfg, in_pitch_bytes=x.strides[0])
    xd = torch.from_numpy(x).cuda()
    out = torch.empty((plan.n_dm, plan.out_pitch), dtype=torch.float32, device="cuda")
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        eager = plan.forward(xd).clone()
    torch.cuda.current_stream().wait_stream(side)
    with torch.cuda.graph(g):
        plan.forward(xd, out=out)
    for k in range(3):
        xd.copy_(torch.from_numpy(np.roll(x, k, axis=1)).cuda())
        g.replay()
        torch.cuda.synchronize()
        want = oracle.forward(np.ascontiguousarray(np.roll(x, k, axis=1)), "u8", cfg["n_samp"], s)
        assert np.array_equal(out[:, : plan.n_out].cpu().numpy(), want)
        if k == 0:
            assert np.array_equal(eager.cpu().numpy(), want)


@pytest.mark.parametrize("dtype", ["u8", "u4", "u16"])
def test_batch_of_group_sum_and_other_beams(dd, dtype):
    """Beams on group sums next to one on its explicitly chosen shape and one whose delays spread too
    wide for group sums: every beam equals the oracle, on every replay."""
    sizes = [(512, 32768, 96, 0.25), (300, 9000, 40, 0.5), (1024, 20000, 33, 0.25), (64, 16384, 64, 30.0)]
    plans, xs, want = [], [], []
    for k, (n_chan, n_samp, n_dm, step) in enumerate(sizes):
        cfg = dict(dtype=dtype, n_chan=n_chan, n_samp=n_samp, f_high=1500.0, chan_bw=300.0 / n_chan, t_samp=64e-6,
                   dm_start=0.0, dm_step=step if k < 3 else 0.7 * step, n_dm=n_dm if k < 3 else 10)
        s = oracle_table(cfg)
        x = _input(dtype, n_chan, n_samp, 20 + k)
        plans.append(plan_for(dd, cfg, in_pitch_bytes=x.strides[0]))
        xs.append(torch.from_numpy(x).cuda())
        want.append(oracle.forward(x, dtype, n_samp, s))
    t = plans[1].tiles(0)
    plans[1].set_tiles(0, t["shape"], t["order"])
    batch = dd.Batch(plans, xs)
    for _ in range(3):
        for o in batch.outputs:
            o.fill_(-1.0)
        for got, w in zip(batch.run(), want):
            assert np.array_equal(got[:, : w.shape[1]].cpu().numpy(), w)
    batch.set_tiles(plans[0].n_shapes - 2)  # one shape for every beam: no group sums
    for got, w in zip(batch.run(), want):
        assert np.array_equal(got[:, : w.shape[1]].cpu().numpy(), w)
