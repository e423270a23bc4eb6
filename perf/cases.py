"""Workloads of the engine's public entry points, with their inputs.

listed() names twelve that a user of the library runs: the X-engine from the
smallest array to the largest, in one call and over several, for input counts
that are and are not a multiple of 16; the batched engine over many arrays and
over the blocks of a serving loop; the F stage's channeliser and equaliser and
the X side's packet ingest.  draw() gives others of the same ranges.

A case is a dict of plain values.  "op" is the path it takes:

    xcorr     one array: `calls` blocks of t samples, the last one dumped in
              the same call (correlate ... correlate_dump)
    dump      the same, with a dump call of its own at the end
    batch     several arrays ("NxFxT;..."), integrated and dumped by one call
    serve     several arrays fed `blocks` blocks each, one call per block,
              every integration dumped with its last block
    chan      channeliser: n real streams -> `spectra` spectra of f channels
    requant   equaliser / 4-bit requantiser over [t][f][n] words
    ingest    packets of `boards` boards -> one block of 8 `blocks` samples
    eqloop    equaliser calibration: requantise a short block, correlate and
              dump it, update the gains from its autocorrelations

Launch choices are the library's own defaults (no tuning cache is loaded).
"""
import math

import torch

from paper_1904_07778_amd import xeng

SIGMA = 2.5          # RMS of the 4-bit data before rounding, the paper's 2-3
CHUNK = 1 << 26      # samples made at a time (bounds the temporaries)


def listed():
    return [
        # 16 dual-polarisation dishes, few channels, short: the smallest call
        # a calibration script makes, where latency and launches count
        {"name": "dish_tiny", "op": "xcorr", "n": 32, "f": 64, "t": 4096, "calls": 1},
        # the dish array's ordinary integration: fed in several calls that add
        # to the accumulator, then dumped
        {"name": "dish_integration", "op": "dump", "n": 32, "f": 1024, "t": 16384, "calls": 4},
        # 96 dual-polarisation cylinder feeds, one integration a call: the
        # benchmark's workload
        {"name": "cylinder", "op": "xcorr", "n": 192, "f": 1024, "t": 8192, "calls": 1},
        # 20 dual-polarisation feeds: an input count between multiples of 16,
        # small enough to be bound by memory
        {"name": "ragged_small", "op": "xcorr", "n": 40, "f": 1024, "t": 8192, "calls": 1},
        # 125 dual-polarisation feeds: the largest arrays, not a multiple of 16
        {"name": "ragged_large", "op": "xcorr", "n": 250, "f": 1024, "t": 4096, "calls": 1},
        # twelve sub-arrays of uneven shape in one call: many bands on one GPU
        {"name": "batch_mixed", "op": "batch",
         "arrays": "32x1024x8192;16x512x4096;32x1024x2048;96x512x8192;32x512x2048;96x1024x2048;"
                   "32x512x8192;32x1024x2048;96x512x4096;96x256x4096;16x512x8192;192x1024x4096"},
        # the serving loop's four resident sub-arrays, a block at a time
        {"name": "serve_blocks", "op": "serve", "arrays": "192x1024;96x1024;32x1024;32x256", "t": 1024, "blocks": 4},
        # F stage of the cylinder array: 96 input pairs, 1024 channels
        {"name": "channelise_cylinder", "op": "chan", "n": 192, "f": 1024, "spectra": 2048},
        # F stage of the dish array on a short capture with 512 channels
        {"name": "channelise_dish", "op": "chan", "n": 32, "f": 512, "spectra": 96},
        # equaliser of the cylinder array
        {"name": "requantise_cylinder", "op": "requant", "n": 192, "f": 1024, "t": 2048},
        # packets of the cylinder array's six boards, 32 channels of a band,
        # out of order and with losses
        {"name": "ingest_cylinder", "op": "ingest", "boards": 6, "f": 32, "blocks": 8192},
        # closing the equaliser loop of the dish array on a short block
        {"name": "equaliser_loop", "op": "eqloop", "n": 32, "f": 512, "t": 512},
    ]


# The largest listed correlation, in complex multiply-accumulates and bytes.
MAX_CMACS = 192 * 193 // 2 * 1024 * 8192
MAX_BYTES = 4 * 16384 * 1024 * 32


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _inputs(rng):
    """Half the arrays have a multiple of 16 inputs (boards of 16 or 32), half any number."""
    return 16 * rng.randint(1, 16) if rng.random() < 0.5 else rng.randint(2, 256)


def _fit(n, f, t, calls=1):
    """t cut so that the correlation is no larger than the largest listed one."""
    t = min(t, MAX_CMACS // (n * (n + 1) // 2 * f * calls), MAX_BYTES // (n * f * calls))
    return max(1, t)


def draw(rng):
    op = rng.choice(["xcorr", "xcorr", "xcorr", "dump", "batch", "serve", "chan", "chan", "requant", "ingest", "eqloop"])
    if op in ("xcorr", "dump"):
        n, f = _inputs(rng), _log(rng, 16, 1024)
        calls = 1 if op == "xcorr" else rng.randint(2, 6)
        return {"op": op, "n": n, "f": f, "t": _fit(n, f, _log(rng, 256, 16384), calls), "calls": calls}
    if op == "batch":
        arrays = []
        for _ in range(rng.randint(2, 12)):
            n, f = rng.choice([16, 32, 40, 48, 64, 96, 192]), _log(rng, 64, 1024)
            arrays.append((n, f, _fit(n, f, _log(rng, 512, 8192), 12)))
        return {"op": "batch", "arrays": ";".join("%dx%dx%d" % a for a in arrays)}
    if op == "serve":
        shapes = [(rng.choice([16, 32, 64, 96, 192]), rng.choice([128, 256, 512, 1024])) for _ in range(rng.randint(1, 5))]
        return {"op": "serve", "arrays": ";".join("%dx%d" % s for s in shapes), "t": 1024, "blocks": rng.randint(2, 5)}
    if op == "chan":
        n, f = 2 * rng.randint(1, 96), 1 << rng.randint(3, 10)
        return {"op": "chan", "n": n, "f": f, "spectra": min(_log(rng, 4, 8192), 192 * 1024 * 2048 // (n * f))}
    if op == "requant":
        n, f = _inputs(rng), _log(rng, 8, 1024)
        return {"op": "requant", "n": n, "f": f, "t": min(_log(rng, 16, 8192), 192 * 1024 * 2048 // (n * f))}
    if op == "ingest":
        boards, f = rng.randint(1, 8), rng.choice([8, 16, 32, 64])
        return {"op": "ingest", "boards": boards, "f": f, "blocks": min(_log(rng, 32, 8192), 6 * 32 * 8192 // (boards * f))}
    n, f = 2 * rng.randint(1, 128), _log(rng, 32, 1024)
    return {"op": "eqloop", "n": n, "f": f, "t": min(_log(rng, 64, 2048), MAX_BYTES // (8 * n * f))}


def _arrays(case):
    """(n, f, t per call) of each array of a correlating case."""
    if case["op"] in ("batch", "serve"):
        shapes = [tuple(int(x) for x in a.split("x")) for a in case["arrays"].split(";")]
        return [a if len(a) == 3 else (*a, case["t"]) for a in shapes]
    return [(case["n"], case["f"], case["t"])]


def _blocks(case):
    return case["blocks"] if case["op"] == "serve" else case.get("calls", 1)


def _voltages(gen, t, f, n):
    """uint8 [t, f, n]: Gaussian noise of each input plus a source that all of
    them see, rounded to the equaliser's -7 .. 7, real part in the high nibble."""
    v = torch.empty((t, f, n), dtype=torch.uint8, device="cuda")
    step = max(1, CHUNK // (f * n))
    for a in range(0, t, step):
        b = min(t, a + step)
        z = torch.randn((2, b - a, f, n), device="cuda", generator=gen).mul_(SIGMA)
        z += 0.5 * SIGMA * torch.randn((2, b - a, f, 1), device="cuda", generator=gen)
        q = z.round_().clamp_(-7, 7).to(torch.int32)
        v[a:b] = ((q[0] << 4) | (q[1] & 15)).to(torch.uint8)
    return v


def _words(gen, t, f, n):
    """int64 [t, f, n]: 18-bit real part in bits 35..18, imaginary in 17..0."""
    w = torch.empty((t, f, n), dtype=torch.int64, device="cuda")
    step = max(1, CHUNK // (f * n))
    for a in range(0, t, step):
        b = min(t, a + step)
        z = torch.randn((2, b - a, f, n), device="cuda", generator=gen).mul_(2.0 ** 14)
        q = z.round_().clamp_(-(1 << 17), (1 << 17) - 1).to(torch.int64) & 0x3FFFF
        w[a:b] = (q[0] << 18) | q[1]
    return w


def _gains(gen, f, n):
    """int32 [f, n]: scale factors that bring a sigma of 2^14 to about 2.5 codes."""
    return (320.0 * (0.8 + 0.4 * torch.rand((f, n), device="cuda", generator=gen))).round().to(torch.int32)


def _packets(gen, case):
    """uint8 [packets, 8 + 256 f]: header (counter, board, band 3) and payload;
    one in a hundred lost, the rest in any order."""
    boards, f, blocks = case["boards"], case["f"], case["blocks"]
    total = boards * blocks
    order = torch.randperm(total, device="cuda", generator=gen)[: total - total // 100]
    pk = torch.empty((order.numel(), 8 + 256 * f), dtype=torch.uint8, device="cuda")
    step = max(1, CHUNK // (256 * f))
    for a in range(0, order.numel(), step):
        b = min(order.numel(), a + step)
        pk[a:b, 8:] = _voltages(gen, b - a, 1, 256 * f).view(b - a, 256 * f)
    mcnt = MCNT0 + order // boards
    for k in range(6):
        pk[:, k] = ((mcnt >> (8 * (5 - k))) & 255).to(torch.uint8)
    pk[:, 6] = (order % boards).to(torch.uint8)
    pk[:, 7] = XID
    return pk


MCNT0, XID = 123456789, 3


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    op = case["op"]
    st = {"case": dict(case)}
    if op == "chan":
        n, f = case["n"], case["f"]
        samples = 2 * f * (case["spectra"] + 3)
        adc = torch.empty((n, samples), dtype=torch.int8, device="cuda")
        for i in range(n):  # a stream at a time: real noise of 20 codes RMS
            adc[i] = torch.randn(samples, device="cuda", generator=gen).mul_(20.0).round_().clamp_(-128, 127).to(torch.int8)
        st["adc"] = adc
        st["out"] = torch.empty((case["spectra"], f, n), dtype=torch.complex64, device="cuda")
        st["tables"] = torch.empty(10 * f, dtype=torch.float32, device="cuda")
        return st
    if op == "requant":
        st["words"] = _words(gen, case["t"], case["f"], case["n"])
        st["gains"] = _gains(gen, case["f"], case["n"])
        st["out"] = torch.empty((case["t"], case["f"], case["n"]), dtype=torch.uint8, device="cuda")
        return st
    if op == "ingest":
        st["packets"] = _packets(gen, case)
        st["out"] = torch.empty((8 * case["blocks"], case["f"], 32 * case["boards"]), dtype=torch.uint8, device="cuda")
        return st
    # the engine's stream, which the program's own calls run on too
    st["stream"] = torch.cuda.Stream()
    arrays = _arrays(case)
    if op == "eqloop":
        n, f, t = arrays[0]
        st["words"] = _words(gen, t, f, n)
        st["gains"] = _gains(gen, f, n)
        st["new_gains"] = torch.empty_like(st["gains"])
        st["volts"] = torch.empty((t, f, n), dtype=torch.uint8, device="cuda")
    else:
        st["blocks"] = [[_voltages(gen, t, f, n) for n, f, t in arrays] for _ in range(_blocks(case))]
    st["plan"] = xeng.Plan(arrays, stream=st["stream"])
    st["vis"] = [st["plan"].new_output(a) for a in range(len(arrays))]
    return st


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "chan":
        return xeng.channelise(st["adc"], case["f"], out=st["out"], tables=st["tables"])
    if op == "requant":
        return xeng.requantize(st["words"], st["gains"], out=st["out"])
    if op == "ingest":
        return list(xeng.ingest(st["packets"], MCNT0, case["blocks"], case["boards"], case["f"], XID, out=st["out"]))
    plan, vis = st["plan"], st["vis"]
    with torch.cuda.stream(st["stream"]):
        if op == "eqloop":
            xeng.requantize(st["words"], st["gains"], out=st["volts"])
            _, n = plan.correlate_dump([st["volts"]], out=vis)
            xeng.eq_update(vis[0], n[0], st["gains"], target_rms=2.5, out=st["new_gains"])
            return [vis[0], st["new_gains"]]
        blocks = st["blocks"]
        for v in blocks[: len(blocks) if op == "dump" else -1]:
            plan.correlate(v)
        if op == "dump":
            _, n = plan.dump(out=vis)
        else:
            _, n = plan.correlate_dump(blocks[-1], out=vis)
        return [*vis, *n]


def work(case):
    op = case["op"]
    if op == "chan":
        n, f, s = case["n"], case["f"], case["spectra"]
        length = 2 * f
        # per pair and spectrum: 4 taps on two streams, one complex transform, the split
        flops = (n // 2) * s * (16 * length + 5 * length * math.log2(length) + 8 * f)
        return {"bytes": n * length * (s + 3) + 8 * n * f * s, "flops": flops}
    if op == "requant":
        samples = case["t"] * case["f"] * case["n"]
        return {"bytes": 9 * samples + 4 * case["f"] * case["n"], "flops": 4 * samples}
    if op == "ingest":
        tile = 256 * case["f"]
        slots = case["boards"] * case["blocks"]
        arrived = slots - slots // 100
        return {"bytes": arrived * (tile + 8) + slots * (tile + 4), "flops": 0}
    bytes_, flops = 0, 0
    for n, f, t in _arrays(case):
        nbl = n * (n + 1) // 2
        bytes_ += t * _blocks(case) * f * n + 8 * f * nbl
        flops += 8 * t * _blocks(case) * f * nbl
        if op == "eqloop":
            bytes_ += 8 * t * f * n + 8 * f * n
            flops += 4 * t * f * n
    return {"bytes": bytes_, "flops": flops}


def exact(case, seed):
    """The channeliser's spectra in 64 bits; every other output is integers."""
    if case["op"] != "chan":
        return None
    st = prepare(case, seed)
    n, f, s = case["n"], case["f"], case["spectra"]
    length = 2 * f
    taps = 4 * length
    m = torch.arange(taps, dtype=torch.float64, device="cuda")
    window = 0.54 - 0.46 * torch.cos(2 * math.pi * m / (taps - 1))
    h = (window * torch.sinc((m - taps / 2) / length)).view(4, length)
    out = torch.empty((s, f, n), dtype=torch.complex128, device="cuda")
    for i in range(n):
        x = st["adc"][i].to(torch.float64).view(s + 3, length)
        v = sum(h[p] * x[p:p + s] for p in range(4))
        out[:, :, i] = torch.fft.fft(v, dim=1)[:, :f]
    return out
