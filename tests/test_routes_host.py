"""Which kernel a plan runs by default, where both were timed (no GPU needed).

``Plan.shares_sums`` tells whether a direction runs by shared sums.  Every row holds a plan, the
measured us by shared sums and by the plan's own shape, and the faster of the two is the default.
"""
import pytest


@pytest.fixture(scope="module")
def dd():
    import paper_2311_05341_amd as dd
    return dd


def _plan(dd, dtype, n_chan, n_samp, n_dm, start, step, f_high, t_us, band=300.0):
    per = {"u4": 0.5, "u8": 1, "u16": 2, "f32": 4}[dtype]
    pitch = (int(n_samp * per) + 15) // 16 * 16
    return dd.Plan(n_chan, n_samp, dtype, f_high, band / n_chan, t_us * 1e-6, start, step, n_dm, in_pitch_bytes=pitch,
                   bind=False)


# (dtype, channels, samples, trials, dm_start, dm_step, f_high, t_us, shared us, own shape's us)
INTEGER = [
    # few workgroups or channels: shared sums start and end slower
    ("u8", 200, 82109, 116, 300.0, 0.25, 1500.0, 64.0, 97.9, 77.7), ("u8", 256, 4418, 49, 0.0, 0.5, 1500.0, 64.0, 79.9, 42.9),
    ("u8", 128, 8002, 154, 800.0, 1.0, 1550.0, 256.0, 44.0, 23.3), ("u8", 256, 7092, 240, 800.0, 2.0, 1550.0, 256.0, 79.7, 43.1),
    ("u4", 160, 17386, 624, 800.0, 0.25, 1550.0, 64.0, 55.3, 40.5), ("u4", 512, 31240, 267, 0.0, 1.0, 1550.0, 128.0, 189.0, 144.4),
    ("u4", 256, 45918, 171, 50.0, 0.25, 1550.0, 128.0, 90.5, 76.0), ("u16", 32, 107844, 1247, 50.0, 0.02, 1550.0, 64.0, 284.4, 205.2),
    ("u16", 64, 154472, 96, 800.0, 0.05, 1550.0, 128.0, 64.9, 53.6),
    # and where they pay
    ("u8", 512, 118615, 251, 0.0, 0.25, 1550.0, 64.0, 293.0, 434.6), ("u8", 1024, 29844, 616, 50.0, 0.25, 1550.0, 64.0, 365.5, 547.2),
    ("u8", 768, 164212, 35, 0.0, 0.1, 1550.0, 256.0, 98.9, 254.2), ("u8", 1024, 49254, 162, 0.0, 1.0, 1550.0, 64.0, 239.4, 491.2),
    ("u4", 200, 48394, 146, 0.0, 0.1, 1500.0, 128.0, 39.1, 59.7), ("u4", 1024, 170480, 175, 50.0, 0.5, 1500.0, 64.0, 615.8, 716.2),
    ("u16", 128, 102299, 77, 300.0, 0.1, 1500.0, 256.0, 56.4, 87.0), ("u16", 512, 14880, 22, 0.0, 0.02, 1550.0, 128.0, 56.7, 220.6),
]


@pytest.mark.parametrize("row", INTEGER, ids=lambda r: "%s-%d-%d-%d" % r[:4])
def test_integer_default_is_the_faster_kernel(dd, row):
    p = _plan(dd, *row[:8])
    assert p.shares_sums(0) == (row[8] < row[9])
    assert not p.shares_sums(1)
    t = p.tiles(0)
    p.set_tiles(0, t["shape"], t["order"])  # an explicit choice runs that shape's kernel
    assert not p.shares_sums(0)


# (channels, samples, trials, dm_start, dm_step, f_high, t_us, direction, shared us, own shape's us)
FLOAT = [
    (200, 28745, 137, 50.0, 1.0, 1550.0, 128.0, 1, 110.0, 94.0), (200, 21952, 258, 800.0, 0.5, 1550.0, 256.0, 1, 187.0, 157.0),
    (128, 21590, 374, 800.0, 0.1, 1500.0, 128.0, 1, 269.0, 240.0),
    (1024, 21994, 79, 0.0, 0.1, 1550.0, 256.0, 0, 118.1, 550.5), (1024, 21994, 79, 0.0, 0.1, 1550.0, 256.0, 1, 70.3, 155.4),
    (512, 44666, 258, 0.0, 1.0, 1550.0, 128.0, 0, 307.0, 560.8), (256, 38454, 246, 50.0, 1.0, 1500.0, 128.0, 1, 236.6, 282.4),
    (1000, 118215, 512, 300.0, 1.0, 1550.0, 64.0, 1, 3585.6, 4169.1),
]


@pytest.mark.parametrize("row", FLOAT, ids=lambda r: "%d-%d-%d-dir%d" % (r[0], r[1], r[2], r[7]))
def test_float_default_is_the_faster_kernel(dd, row):
    p, d = _plan(dd, "f32", *row[:7]), row[7]
    assert p.shares_sums(d) == (row[8] < row[9])
    other = p.shares_sums(1 - d)
    t = p.tiles(d)
    p.set_tiles(d, t["shape"], t["order"])  # that direction only
    assert not p.shares_sums(d) and p.shares_sums(1 - d) == other


@pytest.mark.parametrize("dtype", ["u8", "u4", "u16", "f32"])
@pytest.mark.parametrize("n_dm", [1, 33, 300])
def test_workspace_is_that_of_the_default_shapes(dd, dtype, n_dm):
    """Tables that shared sums take the place of are sized without being filled in."""
    p = _plan(dd, dtype, 512, 40000, n_dm, 0.0, 0.25, 1500.0, 128.0)
    dirs = (0, 1) if dtype == "f32" else (0,)
    assert any(p.shares_sums(d) for d in dirs) or n_dm == 1
    want = p.info.dev_table_bytes
    for d in dirs:
        t = p.tiles(d)
        p.set_tiles(d, t["shape"], t["order"])
        assert p.info.dev_table_bytes == want and p.info.tune_ws_bytes >= want


def test_beams_near_the_line_follow_the_batch(dd):
    """A 4-bit beam that group sums slow down a little (12.7 against 11.7 us in a batch of itself) runs
    by them next to one that they speed up (the two kernels fill each other's waits), else not;
    and never after its plan's tiles were chosen."""
    import ctypes

    lib = ctypes.CDLL(dd.LIB_PATH)
    lib.dd_batch_create.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_int32, ctypes.POINTER(ctypes.c_void_p)]
    lib.dd_batch_shares_sums.argtypes = [ctypes.c_void_p, ctypes.c_int32]
    lib.dd_batch_destroy.argtypes = [ctypes.c_void_p]

    def shares(*plans):
        h = ctypes.c_void_p()
        assert lib.dd_batch_create((ctypes.c_void_p * len(plans))(*[p._h for p in plans]), len(plans), ctypes.byref(h)) == 0
        got = [lib.dd_batch_shares_sums(h, i) for i in range(len(plans))]
        lib.dd_batch_destroy(h)
        return got

    near = _plan(dd, "u4", 128, 42994, 73, 0.0, 0.5, 1500.0, 256.0)
    gains = _plan(dd, "u4", 1024, 40000, 300, 0.0, 0.1, 1500.0, 64.0)
    loses = _plan(dd, "u4", 64, 16384, 10, 0.0, 21.0, 1500.0, 64.0)
    assert shares(near, near) == [0, 0] and shares(near, gains) == [1, 1] and shares(gains, loses, near) == [1, 0, 1]
    t = gains.tiles(0)
    gains.set_tiles(0, t["shape"], t["order"])
    assert shares(near, gains) == [0, 0]
