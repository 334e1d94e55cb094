"""Performance cases: the work that users of this library have it do, through its public entry points.

Every case is a dict of plain values.  ``kind`` names the entry point:

* ``forward``   one ``Plan.forward`` call into a kept output buffer, channel-major filterbank in
                memory (8-, 4-, 16-bit or float samples);
* ``grad``      one autograd step through ``DedisperseFn`` (float): the plane and the input gradient;
* ``batch``     one ``Batch.run`` over many small beams;
* ``survey``    one ``Survey.run``: time-major spectra are turned, binned once per factor and every
                DM range is dedispersed;
* ``corner``    one ``corner_turn`` of time-major spectra;
* ``bin``       one ``bin_time`` call.

Channel c sits at ``f_high - c * band / n_chan``; samples are seeded noise of the kind such backends
deliver: N(128, 16) in 8 bits, uniform 4-bit values, N(32768, 4096) in 16 bits, N(0, 1) floats.
"""
import math
import random

import numpy as np
import torch

import paper_2311_05341_amd as dd

K_DM = 4.148808e3  # s MHz^2 cm^3 / pc
ELEM = {"u8": 1, "u4": 0.5, "u16": 2, "f32": 4}
TORCH = {"u8": torch.uint8, "u4": torch.uint8, "u16": torch.uint16, "f32": torch.float32}


def _forward(name, dtype, n_chan, n_samp, n_dm, dm_step, f_high=1500.0, band=300.0, t_us=64.0, dm_start=0.0, pad=0,
             kind="forward"):
    c = dict(kind=kind, dtype=dtype, n_chan=n_chan, n_samp=n_samp, n_dm=n_dm, dm_step=dm_step, dm_start=dm_start,
             f_high=f_high, band=band, t_us=t_us, pad=pad)
    return dict(c, name=name) if name else c


# The L-band pipeline plan: (dm_start, dm_step, trials, binning factor) per range.
PIPELINE = "0:0.1:1500:1,150:0.2:750:1,300:0.25:800:1,500:0.5:1000:2,1000:1:1000:4,2000:2:500:8"


def listed():
    return [
        # The smallest call: a 128-channel, 2 s filterbank searched over 256 trials (a quick look, a
        # calibration, one block of a stream); launches and the host path count here.
        _forward("small_u8", "u8", 128, 32768, 256, 1.0, band=200.0),
        # An ordinary single beam of a multi-beam search: 1024 channels, about 6.5 s, 700 trials;
        # ragged length and trial count.
        _forward("beam_u8", "u8", 1024, 101_773, 700, 0.5, pad=19),
        # The flagship: 8192 channels x 2^20 samples (67 s) x 4000 trials at L band.
        _forward("headline_u8", "u8", 8192, 1 << 20, 4000, 0.5),
        # Low-frequency array on packed 4-bit samples, 120-190 MHz, fine trials.
        _forward("lowfreq_u4", "u4", 4096, 1 << 19, 2048, 0.1, f_high=190.0, band=70.0, t_us=327.68),
        # L-band backend with 4-bit samples: one 16.8 s block, 500 trials from DM 500.
        _forward("lband_u4", "u4", 8192, 1 << 18, 500, 0.5, dm_start=500.0),
        # Low-frequency array with a coarse trial step: the delay spread of neighbouring trials is
        # hundreds of samples.
        _forward("lowfreq_wide_u8", "u8", 4096, 1 << 20, 1024, 0.5, f_high=190.0, band=70.0, t_us=327.68),
        # L-band backend with 16-bit samples: one 16.8 s block, 500 trials.
        _forward("lband_u16", "u16", 8192, 1 << 18, 500, 0.5),
        # Differentiable use: float samples, forward and backward of one training step.
        _forward("grad_f32", "f32", 1024, 1 << 17, 1024, 1.0, t_us=128.0, kind="grad"),
        # A survey pipeline block from time-major spectra: six ranges up to DM 3000, binned by 1, 2, 4, 8
        # (12.5 s of 4096 channels).
        dict(name="pipeline_u8", kind="survey", dtype="u8", n_chan=4096, n_samp=195_312, f_high=1550.0, band=300.0,
             t_us=64.0, ranges=PIPELINE),
        # Many small beams at once, as a multi-beam receiver delivers them.
        dict(name="batch_u8", kind="batch", dtype="u8", beams=64, beam_seed=4, chan_lo=256, chan_hi=1024,
             samp_lo=1 << 15, samp_hi=1 << 17, dm_lo=64, dm_hi=512, f_high=1500.0, band=300.0, t_us=64.0),
        # Turning the spectra of a 50 s, 4096-channel observation (a filterbank file) channel-major.
        dict(name="corner_u8", kind="corner", dtype="u8", n_chan=4096, n_samp=781_250),
        # Binning that observation by 4 before a high-DM search.
        dict(name="bin_u8", kind="bin", dtype="u8", n_chan=4096, n_samp=781_250, factor=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "forward", "grad", "batch", "survey", "corner", "bin"])
    dtype = rng.choice(["u8", "u8", "u4", "u16", "f32"])
    if kind in ("forward", "grad"):
        if kind == "grad":
            dtype = "f32"
        wide = rng.random() < 0.3  # low-frequency band against L band
        f_high, band, t_us = (190.0, 70.0, 327.68) if wide else (rng.choice([1500.0, 1550.0]), 300.0,
                                                                 rng.choice([64.0, 128.0, 256.0]))
        step = rng.choice([0.1, 0.2, 0.5]) if wide else rng.choice([0.1, 0.25, 0.5, 1.0])
        n_chan = rng.choice([128, 256, 512, 1024, 2048, 4096, 1000, 3000])
        n_dm = _log(rng, 64, 1000)
        start = rng.choice([0.0, 0.0, 50.0, 300.0])
        if dtype == "f32":
            n_chan, n_dm = min(n_chan, 1024), min(n_dm, 512)
        last = start + step * (n_dm - 1)
        delay = K_DM * last * ((f_high - band) ** -2 - f_high ** -2) / (t_us * 1e-6)
        n_samp = int(delay) + _log(rng, 1 << 14, 1 << 18)
        return _forward(None, dtype, n_chan, n_samp + (n_samp & 1 if dtype == "u4" else 0), n_dm, step, f_high, band,
                        t_us, start, rng.choice([0, 0, 16, 33, 96]), kind)
    if kind == "batch":
        return dict(kind="batch", dtype=rng.choice(["u8", "u8", "u4", "u16"]), beams=rng.randint(3, 64),
                    beam_seed=rng.randint(0, 1 << 20), chan_lo=128, chan_hi=1024, samp_lo=1 << 15, samp_hi=1 << 17,
                    dm_lo=64, dm_hi=512, f_high=1500.0, band=300.0, t_us=rng.choice([64.0, 128.0]))
    if kind == "survey":
        n_chan = rng.choice([512, 1024, 2048, 4096])
        return dict(kind="survey", dtype=rng.choice(["u8", "u8", "u4", "u16"]), n_chan=n_chan,
                    n_samp=_log(rng, 60_000, 180_000) // 2 * 2, f_high=1550.0, band=300.0, t_us=64.0,
                    ranges="0:0.2:%d:1,100:0.5:%d:%d,200:1:%d:4" % (rng.randint(100, 500), rng.randint(60, 200),
                                                                    rng.choice([2, 3]), rng.randint(60, 200)))
    n_chan, n_samp = rng.choice([257, 512, 1024, 2048, 4096]), 2 * _log(rng, 10_000, 390_000) + 2 * rng.randint(0, 7)
    c = dict(kind=kind, dtype=dtype, n_chan=n_chan, n_samp=n_samp if dtype != "f32" else n_samp // 4 * 2)
    if kind == "bin":
        c["factor"] = rng.choice([2, 3, 4, 5, 8, 16, 32])
    return c


# ---------------------------------------------------------------- inputs


def _noise(dtype, rows, cols, gen):
    """[rows][cols] noise of an encoding (4-bit: cols bytes of two samples)."""
    out = torch.empty((rows, cols), dtype=TORCH[dtype], device="cuda")
    step = max(1, (1 << 27) // max(1, cols))
    for r in range(0, rows, step):
        n = min(step, rows - r)
        if dtype == "u4":
            out[r:r + n] = torch.randint(0, 256, (n, cols), dtype=torch.uint8, device="cuda", generator=gen)
            continue
        z = torch.randn((n, cols), dtype=torch.float32, device="cuda", generator=gen)
        if dtype == "f32":
            out[r:r + n] = z
        elif dtype == "u8":
            out[r:r + n] = z.mul_(16.0).add_(128.0).round_().clamp_(0.0, 255.0).to(torch.uint8)
        else:
            v = z.mul_(4096.0).add_(32768.0).round_().clamp_(0.0, 65535.0).to(torch.int32)
            out.view(torch.int16)[r:r + n] = (v - 65536 * (v > 32767)).to(torch.int16)
    return out


def _gen(seed, k=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + k) & 0x7fffffffffff)
    return g


def _row_elems(dtype, n_samp, pad=0):
    """Elements of a channel row padded to whole 16 bytes (4-bit: bytes)."""
    n = n_samp // 2 if dtype == "u4" else n_samp
    unit = {"u8": 16, "u4": 16, "u16": 8, "f32": 4}[dtype]
    return (n + pad + unit - 1) // unit * unit


def _row_bytes(dtype, elems):
    return elems * {"u8": 1, "u4": 1, "u16": 2, "f32": 4}[dtype]


def _spectrum_elems(dtype, n_chan):
    n = (n_chan + 1) // 2 if dtype == "u4" else n_chan
    unit = {"u8": 16, "u4": 16, "u16": 8, "f32": 4}[dtype]
    return (n + unit - 1) // unit * unit


def _beams(c):
    """Per-beam sizes of a batch: any length from samp_lo to samp_hi, and an ordinary step."""
    r = random.Random(int(c["beam_seed"]))
    chans = [n for n in (128, 256, 512, 1024) if c["chan_lo"] <= n <= c["chan_hi"]]
    out = []
    for _ in range(c["beams"]):
        out.append(dict(dtype=c["dtype"], n_chan=r.choice(chans), n_samp=r.randint(c["samp_lo"], c["samp_hi"]) // 2 * 2,
                        n_dm=r.randint(c["dm_lo"], c["dm_hi"]), dm_step=r.choice([0.25, 0.5, 1.0]), dm_start=0.0,
                        f_high=c["f_high"], band=c["band"], t_us=c["t_us"], pad=0))
    return out


def _ranges(c):
    return [(float(a), float(b), int(n), int(f)) for a, b, n, f in (r.split(":") for r in c["ranges"].split(","))]


def _plan(c):
    pitch = _row_bytes(c["dtype"], _row_elems(c["dtype"], c["n_samp"], c["pad"]))
    return dd.Plan(c["n_chan"], c["n_samp"], c["dtype"], c["f_high"], c["band"] / c["n_chan"], c["t_us"] * 1e-6,
                   c["dm_start"], c["dm_step"], c["n_dm"], in_pitch_bytes=pitch)


def _input(c, seed, k=0):
    return _noise(c["dtype"], c["n_chan"], _row_elems(c["dtype"], c["n_samp"], c["pad"]), _gen(seed, k))


def _spectra(c, seed):
    return _noise(c["dtype"], c["n_samp"], _spectrum_elems(c["dtype"], c["n_chan"]), _gen(seed))


def prepare(case, seed):
    kind, dtype = case["kind"], case["dtype"]
    if kind == "forward":
        plan = _plan(case)
        out = torch.empty((plan.n_dm, plan.out_pitch), dtype=torch.float32, device="cuda")
        return dict(kind=kind, plan=plan, x=_input(case, seed), out=out)
    if kind == "grad":
        plan = _plan(case)
        x = _input(case, seed)[:, : case["n_samp"]].requires_grad_(True)
        g = torch.randn((plan.n_dm, plan.n_out), dtype=torch.float32, device="cuda", generator=_gen(seed, 1))
        return dict(kind=kind, plan=plan, x=x, g=g)
    if kind == "batch":
        beams = _beams(case)
        plans = [_plan(b) for b in beams]
        return dict(kind=kind, batch=dd.Batch(plans, [_input(b, seed, k) for k, b in enumerate(beams)]))
    if kind == "survey":
        x = _spectra(case, seed)
        sv = dd.Survey(case["n_chan"], case["n_samp"], dtype, case["f_high"], case["band"] / case["n_chan"],
                       case["t_us"] * 1e-6, _ranges(case), in_pitch_bytes=_row_bytes(dtype, x.shape[1]),
                       time_major=True)
        return dict(kind=kind, survey=sv, x=x, outs=sv.empty_outputs())
    if kind == "corner":
        out = torch.zeros((case["n_chan"], _row_elems(dtype, case["n_samp"])), dtype=TORCH[dtype], device="cuda")
        return dict(kind=kind, case=case, x=_spectra(case, seed), out=out)
    if kind == "bin":
        x = _noise(dtype, case["n_chan"], _row_elems(dtype, case["n_samp"]), _gen(seed))
        odt = dd.BIN_OUT[dtype]
        out = torch.zeros((case["n_chan"], _row_elems(odt, case["n_samp"] // case["factor"])), dtype=TORCH[odt],
                          device="cuda")
        return dict(kind=kind, case=case, x=x, out=out)
    raise ValueError(kind)


def run(s):
    kind = s["kind"]
    if kind == "forward":
        return s["plan"].forward(s["x"], out=s["out"])
    if kind == "grad":
        s["x"].grad = None
        y = dd.DedisperseFn.apply(s["x"], s["plan"])
        y.backward(s["g"])
        return y.detach(), s["x"].grad
    if kind == "batch":
        return s["batch"].run()
    if kind == "survey":
        return s["survey"].run(s["x"], s["outs"])
    c = s["case"]
    if kind == "corner":
        y = dd.corner_turn(s["x"], c["dtype"], c["n_chan"], c["n_samp"], out=s["out"])
    else:
        y = dd.bin_time(s["x"], c["dtype"], c["n_samp"], c["factor"], out=s["out"])
    return y.view(torch.int16) if y.dtype == torch.uint16 else y  # the same bits; torch indexes few uint16 tensors


# ---------------------------------------------------------------- work and exact results


def _shifts(c):
    """Delays in samples, [n_dm][n_chan]: floor(DM * K * (f_c^-2 - f_high^-2) / t_samp + 1/2) in float64."""
    f = c["f_high"] - np.arange(c["n_chan"], dtype=np.float64) * (c["band"] / c["n_chan"])
    k = 1.0 / (f * f) - 1.0 / (c["f_high"] * c["f_high"])
    dm = c["dm_start"] + np.arange(c["n_dm"], dtype=np.float64) * c["dm_step"]
    return np.floor(((dm * K_DM)[:, None] * k[None, :]) / (c["t_us"] * 1e-6) + 0.5).astype(np.int64)


def _n_out(c):
    f = c["f_high"] - (c["n_chan"] - 1) * (c["band"] / c["n_chan"])
    dm = c["dm_start"] + (c["n_dm"] - 1) * c["dm_step"]
    k = 1.0 / (f * f) - 1.0 / (c["f_high"] * c["f_high"])
    return c["n_samp"] - int(math.floor(((dm * K_DM) * k) / (c["t_us"] * 1e-6) + 0.5))


def _range_cases(c):
    """Every range of a survey as a forward case on its binned grid."""
    return [dict(c, dm_start=a, dm_step=b, n_dm=n, n_samp=c["n_samp"] // f, t_us=c["t_us"] * f, factor=f)
            for a, b, n, f in _ranges(c)]


def _adds(c):
    return float(c["n_dm"]) * _n_out(c) * c["n_chan"]


def work(case):
    """Inputs once, outputs once; operations are the additions that the transform's definition counts,
    n_dm * n_out * n_chan (one per sample summed)."""
    kind = case["kind"]
    if kind in ("forward", "grad"):
        n_out = _n_out(case)
        b = case["n_chan"] * case["n_samp"] * ELEM[case["dtype"]] + 4.0 * case["n_dm"] * n_out
        return dict(bytes=2 * b, flops=2 * _adds(case)) if kind == "grad" else dict(bytes=b, flops=_adds(case))
    if kind == "batch":
        ws = [work(dict(b, kind="forward")) for b in _beams(case)]
        return dict(bytes=sum(w["bytes"] for w in ws), flops=sum(w["flops"] for w in ws))
    if kind == "survey":
        rs = _range_cases(case)
        return dict(bytes=case["n_chan"] * case["n_samp"] * ELEM[case["dtype"]]
                    + sum(4.0 * r["n_dm"] * _n_out(r) for r in rs), flops=sum(_adds(r) for r in rs))
    n = float(case["n_chan"]) * case["n_samp"]
    if kind == "corner":
        return dict(bytes=2 * n * ELEM[case["dtype"]], flops=0.0)
    return dict(bytes=n * ELEM[case["dtype"]] + n / case["factor"] * ELEM[dd.BIN_OUT[case["dtype"]]], flops=n)


def _values(x, dtype, n):
    """The first n samples of each row as float64."""
    if dtype == "u4":
        y = torch.empty((x.shape[0], 2 * x.shape[1]), dtype=torch.float64, device=x.device)
        y[:, 0::2] = (x & 15).double()
        y[:, 1::2] = (x >> 4).double()
        return y[:, :n]
    if dtype == "u16":
        v = x.view(torch.int16)[:, :n].double()
        return v + 65536.0 * (v < 0)
    return x[:, :n].double()


def _sum64(c, row):
    """The transform in float64: ``row(ch)`` is channel ch's samples."""
    sh = torch.from_numpy(_shifts(c)).cuda()
    n_out = _n_out(c)
    out = torch.zeros((c["n_dm"], n_out), dtype=torch.float64, device="cuda")
    for ch in range(c["n_chan"]):
        out += row(ch).unfold(0, n_out, 1)[sh[:, ch]]
    return out


def _affordable(adds):
    return adds <= 1.1e12


def exact(case, seed):
    kind, dtype = case["kind"], case["dtype"]
    if kind in ("corner", "bin"):
        if kind == "corner":
            return None  # moves of values: whole numbers, compared as they are
        if dd.BIN_OUT[dtype] != "f32" or case["n_chan"] * case["n_samp"] > 1 << 30:
            return None
        x = _noise(dtype, case["n_chan"], _row_elems(dtype, case["n_samp"]), _gen(seed))
        n = case["n_samp"] // case["factor"]
        return _values(x, dtype, n * case["factor"]).reshape(case["n_chan"], n, case["factor"]).sum(2)
    if kind == "forward":
        if not _affordable(_adds(case)):
            return None
        x = _input(case, seed)
        return _sum64(case, lambda ch: _values(x[ch:ch + 1], dtype, case["n_samp"])[0])
    if kind == "grad":
        if not _affordable(2 * _adds(case)):
            return None
        x = _input(case, seed)[:, : case["n_samp"]].double()
        sh, n_out = torch.from_numpy(_shifts(case)).cuda(), _n_out(case)
        g = torch.randn((case["n_dm"], n_out), dtype=torch.float32, device="cuda", generator=_gen(seed, 1)).double()
        y = _sum64(case, lambda ch: x[ch])
        m = case["n_samp"] - n_out
        gp = torch.zeros((case["n_dm"], n_out + 2 * m), dtype=torch.float64, device="cuda")
        gp[:, m:m + n_out] = g
        gx = torch.zeros((case["n_chan"], case["n_samp"]), dtype=torch.float64, device="cuda")
        for d in range(case["n_dm"]):  # g(c, t) = sum_d y(d, t - shift): windows of the padded row
            gx += gp[d].unfold(0, case["n_samp"], 1)[m - sh[d]]
        return y, gx
    if kind == "batch":
        if not _affordable(sum(_adds(b) for b in _beams(case))):
            return None
        out = []
        for k, b in enumerate(_beams(case)):
            x = _input(b, seed, k)
            out.append(_sum64(b, lambda ch, x=x, b=b: _values(x[ch:ch + 1], dtype, b["n_samp"])[0]))
        return out
    rs = _range_cases(case)
    if not _affordable(sum(_adds(r) for r in rs)):
        return None
    v = _values(_spectra(case, seed), dtype, case["n_chan"]).t().contiguous()
    outs = []
    for r in rs:
        f, n = r["factor"], r["n_samp"]
        xb = v[:, : n * f].reshape(case["n_chan"], n, f).sum(2)
        outs.append(_sum64(r, lambda ch, xb=xb: xb[ch]))
    return outs
