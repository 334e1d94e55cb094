"""Default routes, with the kernel named: ``shares_sums`` tells that a plan, direction or beam runs by
shared sums, and each of these cases does (or does not) before its result is compared.
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import plan_for

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


@pytest.mark.parametrize("dtype", ["u8", "u4", "u16"])
def test_beams_by_shared_sums_and_by_their_shape(dd, dtype):
    """Beams whose plan runs by group sums, whose plan does not (few workgroups) though the beam
    does (not in 16 bits), with explicit tiles, and with delays that no group shares; the same plan twice; then
    one shape for all, and the autotuner."""
    sizes = [(1024, 20000, 130, 0.1), (256, 9000, 64, 0.25), (1024, 20000, 64, 0.1), (64, 16384, 10, 21.0)]
    plans, xs, want = [], [], []
    for k, (n_chan, n_samp, n_dm, step) in enumerate(sizes):
        cfg = dict(dtype=dtype, n_chan=n_chan, n_samp=n_samp, f_high=1500.0, chan_bw=300.0 / n_chan, t_samp=64e-6,
                   dm_start=0.0, dm_step=step, n_dm=n_dm)
        s = oracle.shift_table(n_chan, 1500.0, 300.0 / n_chan, 64e-6, 0.0, step, n_dm)
        x = _input(dtype, n_chan, n_samp, 40 + k)
        plans.append(plan_for(dd, cfg, in_pitch_bytes=x.strides[0]))
        xs.append(torch.from_numpy(x).cuda())
        want.append(oracle.forward(x, dtype, n_samp, s))
    assert [p.shares_sums(0) for p in plans] == [True, False, True, False]
    t = plans[2].tiles(0)
    plans[2].set_tiles(0, t["shape"], t["order"])
    plans.append(plans[0])
    xs.append(xs[0])
    want.append(want[0])
    batch = dd.Batch(plans, xs)

    def check():
        for o in batch.outputs:
            o.fill_(-1.0)
        for got, w in zip(batch.run(), want):
            assert np.array_equal(got[:, : w.shape[1]].cpu().numpy(), w)

    assert [batch.shares_sums(b) for b in range(5)] == [True, dtype != "u16", False, False, True]
    assert not batch.shares_sums(-1) and not batch.shares_sums(5)
    check()
    check()
    for shape in range(plans[0].n_shapes - 2, plans[0].n_shapes):  # direct reads hold every beam
        batch.set_tiles(shape)
        assert not any(batch.shares_sums(b) for b in range(5))
        check()
    rep = batch.autotune()
    print(dtype, rep, [batch.shares_sums(b) for b in range(5)], flush=True)
    assert batch.shares_sums(0) and batch.shares_sums(2)  # also the beam whose tiles were chosen
    check()
