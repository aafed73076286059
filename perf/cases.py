"""Performance cases of the correlator: what a program that uses it has it do.

Every case is one integration (or one batch of serving jobs) on device-resident
input, through ``Correlator``, ``aggregate_w16`` and ``Scheduler``, with the
result read out.  The sizes are those of the benchmark and the tests: the
64-input prototype (128 channels, 1000 to 10000 spectra), the 256-input
low-precision configuration, the 512- and 1024-input arrays and the serving
mix, with ragged and tiny calls beside them.

A case has a ``kind``:

* ``x``      samples -> X-engine -> integration dump;
* ``fx``     voltages -> F-stage -> X-engine on the ring -> dump (real samples,
             with or without the filterbank, or the prototype's complex ones,
             16-bit words with the capture-stream aggregation in front);
* ``serve``  a batch of integration jobs through the serving scheduler.
"""
from __future__ import annotations

import math
import time

import torch

from paper_0906_1887_amd import (CORR_DUMP_FOLD, CORR_DUMP_INTEG, CORR_DUMP_LONGRUN, Correlator, Scheduler,
                                 aggregate_w16)

DEV = "cuda:0"


# ------------------------------------------------------------------- cases

def _x(name, engine, sample, n_in, n_ch, n_t, stage=0, host=False):
    c = {"kind": "x", "engine": engine, "sample": sample, "n_in": n_in, "n_ch": n_ch, "n_t": n_t, "stage": stage,
         "host": host}
    return {"name": name, **c} if name else c


def _fx(name, volt, n_in, n_blocks, taps=0, longrun=False, engine="i8"):
    c = {"kind": "fx", "volt": volt, "n_in": n_in, "n_blocks": n_blocks, "taps": taps, "longrun": longrun,
         "engine": engine}
    return {"name": name, **c} if name else c


def listed():
    return [
        # a monitoring snapshot: a handful of inputs, read to host memory; all latency
        _x("snapshot_ci8", "i8", "ci8", 8, 16, 250, host=True),
        # the small-array configuration (64 inputs, 128 channels, 1000 samples), on the FP32 matrix cores
        _x("small_fp32m", "fp32m", "cf32", 64, 128, 1000),
        # a mid-sized array in plain FP32: the precision the method was published with
        _x("mid_fp32", "fp32", "cf32", 128, 96, 2000),
        # an array size that fits no tile and an odd number of samples (rows start on odd sample addresses)
        _x("ragged_ci8", "i8", "ci8", 100, 133, 2001),
        # the full array (512 antennas x 2 polarisations), int8 pairs
        _x("array1024_ci8", "i8", "ci8", 1024, 768, 8000),
        # a 512-input array on packed one-byte samples
        _x("array512_ci4", "i8", "ci4", 512, 256, 8000),
        # 256 inputs of float samples on the FP16 engine (converted as they are loaded) ...
        _x("float256_f16", "f16", "cf32", 256, 512, 4096),
        # ... and on the FP8 engine through its staging buffer
        _x("float256_f8", "f8", "cf32", 256, 512, 4096, stage=4096),
        # a real-voltage stream folded into the long-run sum: resume a run from its checkpoint, add one
        # integration of 10000 blocks and read the sum
        _fx("fx_real_longrun", "r8", 64, 10000, longrun=True),
        # the same stream through the 4-tap filterbank, per-integration dumps
        _fx("fx_filterbank", "r8", 64, 10000, taps=4),
        # one second of the prototype: capture records of 4 streams -> aggregation -> complex F-stage -> X
        _fx("prototype_1s", "cw16", 64, 10000),
        # a batch of small and mid-sized jobs arriving together at the serving scheduler
        {"name": "serve_batch", "kind": "serve", "n_jobs": 12, "mix": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["ci8", "ci8", "ci8", "ci4", "fp32", "fp32m", "f16", "f8", "r8", "pfb", "cw16", "cb8"])
    if family in ("r8", "pfb", "cw16", "cb8"):
        n_blocks = _log_int(rng, 100, 10000)
        if family == "cw16":
            return _fx(None, "cw16", 16 * rng.randint(1, 4), n_blocks)
        n_in = rng.choice([rng.randint(4, 100), 8 * rng.randint(1, 16)])
        if family == "cb8":
            return _fx(None, "cb8", n_in, n_blocks)
        return _fx(None, "r8", n_in, n_blocks, taps=4 if family == "pfb" else 0, longrun=rng.random() < 0.4,
                   engine=rng.choice(["i8", "i8", "fp32"]))
    top = {"ci8": 1024, "ci4": 1024, "fp32": 512, "fp32m": 256, "f16": 512, "f8": 512}[family]
    while True:
        n_in = rng.choice([_log_int(rng, 4, top), 16 * _log_int(rng, 1, top // 16)])
        n_ch, n_t = _log_int(rng, 8, 768), _log_int(rng, 100, 8000)
        # bounded by arithmetic (the float engines are 10 to 20 times slower per product) and by input size
        cmac = n_ch * n_t * n_in * (n_in + 1) / 2
        if cmac > (2e12 if family in ("ci8", "ci4") else 6e10) or n_ch * n_t * n_in > 1.2e9:
            continue
        break
    if family in ("ci8", "ci4"):
        return _x(None, "i8", family, n_in, n_ch, n_t, host=n_ch * n_in * n_in < 1 << 16)
    stage = rng.choice([0, n_t, (n_t + 2) // 3]) if family in ("f16", "f8") else 0
    return _x(None, family, "cf32", n_in, n_ch, n_t + (n_t & 1 if family == "fp32m" else 0), stage=stage)


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _ci8_fill(x, g):
    """Rounded Gaussian levels of rms 2 clipped to +-7 (the 4-bit range) into int8 x, a few channels at a time."""
    step = max(1, (1 << 27) // max(1, x[0].numel()))
    for c in range(0, x.shape[0], step):
        n = torch.randn(x[c:c + step].shape, device=DEV, generator=g)
        x[c:c + step] = n.mul_(2.0).round_().clamp_(-7, 7)
    return x


def _x_samples(case, seed):
    g = _gen(seed)
    n_ch, n_in, n_t = case["n_ch"], case["n_in"], case["n_t"]
    if case["sample"] == "cf32":
        # unit complex noise with per-input gains in [0.5, 2] and a weak signal common to all inputs
        x = torch.randn((n_ch, n_in, n_t, 2), device=DEV, generator=g)
        x += 0.3 * torch.randn((n_ch, 1, n_t, 2), device=DEV, generator=g)
        x *= (0.5 + 1.5 * torch.rand((n_in, 1, 1), device=DEV, generator=g)) * math.sqrt(0.5)
        return x
    x = _ci8_fill(torch.empty((n_ch, n_in, n_t, 2), dtype=torch.int8, device=DEV), g)
    if case["sample"] == "ci4":
        # one byte per sample, re in the high nibble; rows padded to 16 bytes
        b = torch.zeros((n_ch, n_in, (n_t + 15) // 16 * 16), dtype=torch.uint8, device=DEV)
        for c in range(n_ch):
            b[c, :, :n_t] = (((x[c, ..., 0] & 15) << 4) | (x[c, ..., 1] & 15)).view(torch.uint8)
        return b
    return x


def _fx_len(case):
    """DFT length of the case's F-stage."""
    return 256 if case["volt"] == "r8" else 128


def _fx_volts(case, seed):
    """Voltages with a common tone and, on a few inputs, common noise."""
    g = _gen(seed)
    n, n_in = _fx_len(case), case["n_in"]
    rows = (case["n_blocks"] + max(0, case["taps"] - 1)) * n
    k = torch.arange(rows, device=DEV) % n
    if case["volt"] == "r8":
        v = 16.0 * torch.randn((rows, n_in), device=DEV, generator=g)
        v[:, :8] += 5.0 * torch.randn((rows, 1), device=DEV, generator=g)
        v += 2.0 * torch.cos(2 * math.pi * ((37 * k) % n) / n)[:, None]
        return v.round_().clamp_(-128, 127).to(torch.int8)
    bits, sigma = (5, 4.0) if case["volt"] == "cw16" else (4, 2.0)
    z = sigma * math.sqrt(0.5) * torch.randn((rows, n_in, 2), device=DEV, generator=g)
    z[:, :8] += 0.3 * sigma * torch.randn((rows, 1, 2), device=DEV, generator=g)
    ph = 2 * math.pi * ((19 * k) % n) / n
    z += torch.stack([torch.cos(ph), torch.sin(ph)], -1)[:, None]
    m = 1 << (bits - 1)
    z = z.round_().clamp_(-m, m - 1).to(torch.int32)
    if case["volt"] == "cb8":
        return (((z[..., 0] & 15) << 4) | (z[..., 1] & 15)).to(torch.uint8)
    w = ((z[..., 0] & 31) << 5) | (z[..., 1] & 31)
    # records of n_in / 16 capture streams: a counter word, then 16 sample words
    rec = torch.empty((n_in // 16, rows, 17), dtype=torch.int16, device=DEV)
    rec[:, :, 0] = torch.arange(rows, device=DEV).to(torch.int16)
    rec[:, :, 1:] = w.to(torch.int16).view(rows, n_in // 16, 16).transpose(0, 1)
    return rec


def _fx_scale(case):
    """Requantisation scale: the spectra's rms becomes about 2."""
    return 2.0 / (16.0 * math.sqrt(128.0)) if case["volt"] == "r8" else (1.0 / 22.0 if case["volt"] == "cw16" else 1.0 / 11.0)


def _checkpoint(case, seed):
    p = case["n_in"] * (case["n_in"] + 1) // 2
    return torch.randint(-10 ** 6, 10 ** 6, (128, p, 2), device=DEV, generator=_gen(seed + 77)).double()


def _serve_jobs(case):
    """(inputs, channels, samples) of each job: the benchmark's small and middle array sizes."""
    sizes, chans = (16, 64, 128), (64, 256)
    return [(sizes[(k * 5 + case["mix"]) % 3], chans[(k // 3) % 2], 1000 + (k * 1237 + 411 * case["mix"]) % 4001)
            for k in range(case["n_jobs"])]


def _serve_samples(case, seed):
    g = _gen(seed)
    xs = []
    for n_in, n_ch, n_t in _serve_jobs(case):
        # a stream's ring: rows of whole 16-byte pieces
        xs.append(_ci8_fill(torch.empty((n_ch, n_in, (n_t + 7) // 8 * 8, 2), dtype=torch.int8, device=DEV), g))
    return xs


# ------------------------------------------------------------ prepare, run

def prepare(case, seed):
    if case["kind"] == "serve":
        xs = _serve_samples(case, seed)
        dst = [torch.empty((c, n * (n + 1) // 2, 2), dtype=torch.int32, device=DEV) for n, c, _ in _serve_jobs(case)]
        torch.cuda.synchronize()   # the scheduler reads the rings on its own streams
        return {"case": case, "x": xs, "dst": dst, "sched": Scheduler(64 << 20, n_streams=4, device=DEV)}
    n_in = case["n_in"]
    if case["kind"] == "x":
        x = _x_samples(case, seed)
        c = Correlator(n_in, case["n_ch"], engine=case["engine"], sample_type=case["sample"],
                       max_abs=0 if case["sample"] == "cf32" else 7, ring_samples=case["stage"], device=DEV)
        st = {"case": case, "x": x, "plan": c}
    else:
        x = _fx_volts(case, seed)
        c = Correlator(n_in, 128, engine=case["engine"], sample_type="ci8", fft_size=_fx_len(case), max_abs=7,
                       requant_scale=_fx_scale(case), ring_samples=case["n_blocks"], fp64_longrun=case["longrun"],
                       device=DEV, volt_format=case["volt"], pfb_taps=case["taps"])
        st = {"case": case, "x": x, "plan": c, "seq": 0}
        if case["volt"] == "cw16":
            st["agg"] = torch.empty((x.shape[1], n_in), dtype=torch.int16, device=DEV)
            st["bad"] = torch.zeros(1, dtype=torch.uint32, device=DEV)
        if case["longrun"]:
            st["ck"] = _checkpoint(case, seed)
    dt = torch.float64 if case.get("longrun") else (torch.int32 if case["engine"] == "i8" else torch.float32)
    st["out"] = None if case.get("host") else torch.empty((c.n_channels, c.n_products, 2), dtype=dt, device=DEV)
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "serve":
        s = state["sched"]
        ids = [s.submit(n, c, t, d, d_samples=x.data_ptr(), row_stride=x.shape[2])
               for (n, c, t), d, x in zip(_serve_jobs(case), state["dst"], state["x"])]
        while ids:
            ids = [j for j in ids if s.poll(j) is None]
            if ids:
                time.sleep(0.00005)
        return state["dst"]
    c = state["plan"]
    if case["kind"] == "x":
        c.correlate(state["x"], case["n_t"])
        return c.dump(CORR_DUMP_INTEG, out=state["out"], device_out=not case["host"])[0]
    x, what = state["x"], CORR_DUMP_INTEG
    if case["longrun"]:
        c.restore(state["ck"], 10000, state["seq"], True)
        what = CORR_DUMP_FOLD | CORR_DUMP_LONGRUN
    if case["volt"] == "cw16":
        x, _ = aggregate_w16(x, out=state["agg"], bad=state["bad"])
    c.channelise(x, first_seq=state["seq"])
    state["seq"] += case["n_blocks"]
    c.correlate(None)
    return c.dump(what, out=state["out"])[0]


# ------------------------------------------------------------- work, exact

def work(case):
    if case["kind"] == "serve":
        jobs = _serve_jobs(case)
        return {"bytes": sum(c * (n * t * 2 + n * (n + 1) // 2 * 8) for n, c, t in jobs),
                "flops": sum(8 * c * t * n * (n + 1) // 2 for n, c, t in jobs)}
    n_in = case["n_in"]
    p = n_in * (n_in + 1) // 2
    if case["kind"] == "x":
        sb = {"ci8": 2, "ci4": 1, "cf32": 8}[case["sample"]]
        return {"bytes": case["n_ch"] * (n_in * case["n_t"] * sb + p * 8), "flops": 8 * case["n_ch"] * case["n_t"] * p}
    n, nb = _fx_len(case), case["n_blocks"]
    rows = (nb + max(0, case["taps"] - 1)) * n
    read = rows * n_in * {"r8": 1, "cb8": 1, "cw16": 2}[case["volt"]]
    if case["volt"] == "cw16":
        read = read * 17 // 16
    # a real transform of n points: half the 5 n log2 n of a complex one; the taps' multiply-adds
    fft = (2.5 if case["volt"] == "r8" else 5.0) * n * math.log2(n) + 2 * n * case["taps"]
    out = 128 * p * (16 if case["longrun"] else 8) + (128 * p * 16 if case["longrun"] else 0)
    return {"bytes": read + out, "flops": int(nb * n_in * fft) + 8 * 128 * p * nb}


def _triangle(a, b):
    """Packed lower triangle of (a + i b)(a + i b)^H, a and b float64 [inputs][samples]: [products][2]."""
    i, j = torch.tril_indices(a.shape[0], a.shape[0], device=a.device)
    re = a @ a.T + b @ b.T
    m = b @ a.T
    return torch.stack([re[i, j], (m - m.T)[i, j]], -1)


def _sums(x, dtype):
    """x [channels][inputs][samples][2] -> [channels][products][2], in 64 bits channel by channel."""
    return torch.stack([_triangle(x[c, ..., 0].double(), x[c, ..., 1].double()).to(dtype) for c in range(x.shape[0])])


def _dft(case, volts):
    """Requantised spectra, float64 [128][inputs][blocks][2]."""
    n, nb, n_in = _fx_len(case), case["n_blocks"], case["n_in"]
    s = float(torch.tensor(_fx_scale(case), dtype=torch.float32))
    if case["taps"]:
        m = torch.arange(case["taps"] * n, device=DEV, dtype=torch.float64)
        u = (m - (case["taps"] * n - 1) / 2) / n
        h = (0.54 - 0.46 * torch.cos(2 * math.pi * m / (case["taps"] * n - 1))) * torch.sinc(u)
    q = torch.empty((128, n_in, nb, 2), dtype=torch.float64, device=DEV)
    for i in range(n_in):
        if case["volt"] == "r8":
            b = volts[:, i].double().view(-1, n)
            if case["taps"]:
                b = sum(h[p * n:(p + 1) * n] * b[p:p + nb] for p in range(case["taps"]))
            f = torch.fft.fft(b, dim=1)[:, :128]
        else:
            f = torch.fft.fft(torch.complex(volts[:, i, 0], volts[:, i, 1]).view(-1, n), dim=1)
        f = torch.view_as_real(f).permute(1, 0, 2)
        q[:, i] = (f * s).round().clamp(-7, 7)
    return q


def exact(case, seed):
    if case["kind"] == "serve":
        return [_sums(x[:, :, :t], torch.int64) for x, (_, _, t) in zip(_serve_samples(case, seed), _serve_jobs(case))]
    if case["kind"] == "x":
        x = _x_samples(case, seed)
        if case["sample"] == "ci4":
            x = x[:, :, :case["n_t"]].view(torch.int8)
            x = torch.stack([x >> 4, (x << 4) >> 4], -1)
        return _sums(x, torch.int64 if case["engine"] == "i8" else torch.float64)
    v = _fx_volts(case, seed)
    if case["volt"] == "cw16":
        w = v[:, :, 1:].transpose(0, 1).reshape(v.shape[1], -1).to(torch.int32)
        v = torch.stack([(w << 22) >> 27, (w << 27) >> 27], -1).double()
    elif case["volt"] == "cb8":
        w = v.to(torch.int32)
        v = torch.stack([(w << 24) >> 28, (w << 28) >> 28], -1).double()
    if case["longrun"]:
        return _sums(_dft(case, v), torch.float64) + _checkpoint(case, seed)
    return _sums(_dft(case, v), torch.int64 if case["engine"] == "i8" else torch.float64)
