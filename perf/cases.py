"""The framework's work as timed cases: what one call, or one step of calls, of a correlator program does.

listed() names the cases, draw() gives more of the same ranges, prepare() builds on the GPU what a program
holds before the step (samples, geometry, scales, plan, buffers), run() makes one step through the public
entry points, work() counts the bytes and operations the step cannot do without, and exact() computes the
same outputs in 64 bits with plain torch.
"""
import math

import numpy as np
import torch

import paper_0910_1517_amd as corr

FS = 66.666666e6
MAX_DELAY = 16
SIGMA = 12.0  # of the 8-bit voltages
PRECISION = {"fp32": corr.FP32, "int8": corr.INT8, "e4m3": corr.FP8_E4M3}
QMAX = {"int8": 127.0, "e4m3": 448.0}


def listed():
    return [
        # eight signals, 512-point FFT: the smallest correlation, a handful of short launches
        {"name": "fx_fp32_small", "kind": "fx", "S": 8, "N": 512, "T": 1024, "prec": "fp32", "compute": False},
        # GMRT scale in FP32: 32 antennas x 2 polarisations, 512 channels
        {"name": "fx_fp32_gmrt", "kind": "fx", "S": 64, "N": 1024, "T": 16384, "prec": "fp32", "compute": False},
        # the real-time step: int8 with held scales, 2048 channels, a 2 s block of every signal
        {"name": "fx_int8_block", "kind": "fx", "S": 64, "N": 4096, "T": 32768, "prec": "int8", "compute": False},
        # the calibration step that measures the requantisation scales, on an odd-sized array
        {"name": "fx_int8_calibrate", "kind": "fx", "S": 47, "N": 2048, "T": 4000, "prec": "int8", "compute": True},
        # flagged step with the MAD flagger, a 30-signal sub-array, FP32 power cells
        {"name": "flagged_mad", "kind": "flagged", "S": 30, "N": 4096, "T": 4096, "learned": False, "f16": False},
        # flagged step with the learned flagger and its column guard, all signals, FP16 power cells
        {"name": "flagged_learned", "kind": "flagged", "S": 64, "N": 8192, "T": 4096, "learned": True, "f16": True},
        # one training pass (loss and gradient) of the learned flagger on a mini-batch of tiles
        {"name": "flagger_train", "kind": "train", "S": 8, "T": 512, "C": 1024, "tiles": 16},
        # pulsar-gated correlation (on and off pulse) of spectra in hand
        {"name": "gated_int8", "kind": "gated", "S": 64, "N": 4096, "T": 8192, "prec": "int8", "bins": 2},
        # spectra of another channeliser: requantised, corner-turned and correlated in e4m3
        {"name": "external_e4m3", "kind": "external", "S": 30, "N": 2048, "T": 4096, "prec": "e4m3"},
        # phased array: incoherent beam, voltage beam of both polarisations, coherent dedispersion
        {"name": "phased_dedisperse", "kind": "phased", "S": 64, "N": 4096, "T": 8192, "prec": "int8", "n_int": 256},
        # acquisition: four-bit card streams unpacked into rows, then impulsive noise blanked in place
        {"name": "front_end_4bit", "kind": "front", "cards": 16, "n": 8388613, "bits": 4, "block": 4096},
        # six sub-arrays of uneven size as one captured graph
        {"name": "batch_subarrays", "kind": "batch",
         "shapes": "8x256x65536 16x512x32768 30x1024x16384 48x2048x8192 60x4096x2048 64x8192x1024"},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def shape(most, unit=32, min_fft=9):
        """S, N, T (a multiple of unit) with S N T up to `most` samples."""
        S, N = rng.randint(2, 64), 1 << rng.randint(min_fft, 14)
        T = unit * log_int(1, max(1, min(most // (S * N), 65536) // unit))
        return {"S": S, "N": N, "T": T}

    kind = rng.choice(["fx", "fx", "fx", "fx", "flagged", "train", "gated", "external", "phased", "front", "batch"])
    if kind == "fx":
        prec = rng.choice(["fp32", "int8", "int8", "e4m3"])
        compute = prec != "fp32" and rng.random() < 0.3
        return {"kind": kind, **shape(1 << 31), "prec": prec, "compute": compute}
    if kind == "flagged":
        return {"kind": kind, **shape(1 << 30, unit=64), "learned": rng.random() < 0.4, "f16": rng.random() < 0.5}
    if kind == "train":
        return {"kind": kind, "S": rng.randint(1, 16), "T": 64 * rng.randint(2, 16), "C": 256 << rng.randint(0, 3),
                "tiles": log_int(2, 64)}
    if kind == "gated":
        return {"kind": kind, **shape(1 << 29), "prec": rng.choice(["int8", "int8", "fp32", "e4m3"]),
                "bins": rng.choice([2, 2, 3, 8])}
    if kind == "external":
        return {"kind": kind, **shape(1 << 29), "prec": rng.choice(["fp32", "int8", "e4m3"])}
    if kind == "phased":
        N, S = 1 << rng.randint(9, 14), rng.randint(2, 64)
        T = 1 << rng.randint(6, 24 - int(math.log2(N)))
        return {"kind": kind, "S": S, "N": N, "T": T, "prec": rng.choice(["int8", "int8", "e4m3", "fp32"]),
                "n_int": 1 << rng.randint(0, 10)}
    if kind == "front":
        return {"kind": kind, "cards": rng.randint(1, 16), "n": log_int(20000, 1 << 23) | 1,
                "bits": rng.choice([4, 8]), "block": 16 * log_int(16, 2048)}
    shapes = []
    for _ in range(rng.randint(2, 6)):
        s = shape(1 << 28)
        shapes.append("%dx%dx%d" % (s["S"], s["N"] // 2, s["T"]))
    return {"kind": kind, "shapes": " ".join(shapes)}


# ------------------------------------------------------------------ inputs

def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 64 + stream)


def _geometry(S, seed):
    """Delays up to 16 samples, fractions, fringe phases and rates up to 5 Hz, as a host array."""
    g = np.random.default_rng([int(seed), 1])
    return corr.geom_array(g.integers(0, MAX_DELAY + 1, S), g.random(S).astype(np.float32), g.random(S),
                           g.uniform(-5.0, 5.0, S))


def _voltages(S, n, stride, D, seed):
    """int8 rows: Gaussian noise, a common source at the signals' delays (coherence 0.3) and a weak tone."""
    gen = _generator(seed, 0)
    x = torch.zeros(S, stride, dtype=torch.int8, device="cuda")
    common = torch.randn(n + MAX_DELAY, generator=gen, device="cuda").mul_(SIGMA * math.sqrt(0.3))
    tone = (2.0 * torch.cos(2 * math.pi * 37 / 512 * torch.arange(512, device="cuda", dtype=torch.float64))).float()
    common += tone.repeat(-(-common.numel() // 512))[:common.numel()]
    for s in range(S):
        v = torch.randn(n, generator=gen, device="cuda").mul_(SIGMA * math.sqrt(0.7))
        v += common[MAX_DELAY - int(D[s]):][:n]
        x[s, :n] = v.round_().clamp_(-127, 127).to(torch.int8)
    return x


def _bandpass(S, C, seed, level):
    """Per signal and channel values around `level`, as a gain table holds them."""
    return torch.rand(S, C, generator=_generator(seed, 1), device="cuda").mul_(0.4).add_(0.8).mul_(level)


def _rows(case, seed):
    S, N, T = case["S"], case["N"], case["T"]
    geom = _geometry(S, seed)
    stride = (N * T + MAX_DELAY + 255) // 256 * 256
    return _voltages(S, N * T + MAX_DELAY, stride, geom["D"], seed), geom


def _held_scale(case, seed):
    """4 sigma of a component of the channels over the code range."""
    return _bandpass(case["S"], case["N"] // 2, seed, 4 * SIGMA * math.sqrt(case["N"] / 2) / QMAX[case["prec"]])


def _layout_spectra(case, seed):
    """Spectra in the X layout [T/G][C/8][S][8][16 bytes] with a common component, and their scales."""
    S, C, T = case["S"], case["N"] // 2, case["T"]
    gen, fp32 = _generator(seed, 2), case["prec"] == "fp32"
    G = 2 if fp32 else 8
    unit, cell = (2, 2) if fp32 else (2, 8)
    out = torch.empty(T // G, C // 8, S, 8, unit, cell, device="cuda",
                      dtype={"fp32": torch.float32, "int8": torch.int8, "e4m3": torch.float8_e4m3fn}[case["prec"]])
    step = max(1, (1 << 27) // out[0].numel())
    sigma = {"fp32": SIGMA * math.sqrt(C), "int8": 127 / 4, "e4m3": 448 / 4}[case["prec"]]
    for g in range(0, T // G, step):
        part = out[g:g + step]
        v = torch.randn(part.shape, generator=gen, device="cuda")
        v += 0.6 * torch.randn(part[:, :, :1].shape, generator=gen, device="cuda")
        v *= sigma / 1.17
        if case["prec"] == "int8":
            v = v.round_().clamp_(-127, 127)
        elif case["prec"] == "e4m3":
            v = v.clamp_(-448, 448)
        part.copy_(v.to(out.dtype))
    return out.view(torch.uint8).view(-1), None if fp32 else _held_scale(case, seed)


def _layout_to_time(spec, case):
    """X layout -> [S][T][C][2] float32 (codes as their values)."""
    S, C, T = case["S"], case["N"] // 2, case["T"]
    if case["prec"] == "fp32":
        a = spec.view(torch.float32).view(T // 2, C // 8, S, 8, 2, 2).permute(2, 0, 4, 1, 3, 5)
    else:
        dt = torch.int8 if case["prec"] == "int8" else torch.float8_e4m3fn
        a = spec.view(dt).view(T // 8, C // 8, S, 8, 2, 8).float().permute(2, 0, 5, 1, 3, 4)
    return a.reshape(S, T, C, 2)


def _gates(case):
    """uint8 gate of every spectrum from a 1.56 ms pulsar."""
    t = (np.arange(case["T"]) + 0.5) * case["N"] / FS
    phase = np.mod(t / 1.5578e-3, 1.0)
    return torch.from_numpy(np.minimum(phase * case["bins"], case["bins"] - 1).astype(np.uint8)).cuda()


def _network(seed):
    """Weights of the 1 -> 16 -> 16 -> 1 network, with a final bias at which few cells are flagged."""
    g = np.random.default_rng([int(seed), 3])
    parts = []
    for out, inp, bias in ((16, 1, 0.0), (16, 16, 0.0), (1, 16, -2.0)):
        parts += [g.standard_normal(out * inp * 9) * math.sqrt(2.0 / (9 * inp)), np.full(out, bias)]
    return torch.from_numpy(np.concatenate(parts).astype(np.float32)).cuda()


def _power(S, T, C, seed):
    """Dynamic spectra: chi-squared cells over a bandpass, persistent tones and broadband bursts; and labels."""
    gen = _generator(seed, 4)
    p = torch.empty(S, T, C, device="cuda").exponential_(1.0, generator=gen)
    p *= _bandpass(S, C, seed, SIGMA ** 2 * C)[:, None, :]
    tones = torch.rand(S, 1, C, generator=gen, device="cuda") < 0.05
    bursts = torch.rand(S, T, 1, generator=gen, device="cuda") < 0.01
    p *= 1 + 40.0 * tones + 20.0 * bursts
    return p, (tones | bursts).to(torch.uint8)


def _time_spectra(case, seed):
    """FP32 spectra [S][T][C][2] of another channeliser, with a common component."""
    S, C, T = case["S"], case["N"] // 2, case["T"]
    gen = _generator(seed, 5)
    common = torch.randn(T, C, 2, generator=gen, device="cuda")
    v = torch.empty(S, T, C, 2, device="cuda")
    for s in range(S):
        v[s] = (torch.randn(T, C, 2, generator=gen, device="cuda") + 0.6 * common) * (SIGMA * math.sqrt(C) / 1.17)
    return v


def _card_streams(case, seed):
    """Raw card streams uint8 [cards][stride]: Gaussian samples with impulsive bursts on a few of them."""
    cards, n, bits = case["cards"], case["n"], case["bits"]
    gen = _generator(seed, 6)
    stride = (-(-n * bits // 2) + 255) // 256 * 256
    raw = torch.zeros(cards, stride, dtype=torch.uint8, device="cuda")
    sigma, low, high = (1.5, -8, 7) if bits == 4 else (SIGMA, -127, 127)
    for c in range(cards):
        v = torch.randn(n, 4, generator=gen, device="cuda").mul_(sigma)
        v *= 1 + 9.0 * (torch.rand(n, 1, generator=gen, device="cuda") < 0.02)
        v = v.round_().clamp_(low, high).to(torch.int8)
        b = v.view(torch.uint8) if bits == 8 else ((v[:, 0::2] & 15) | ((v[:, 1::2] & 15) << 4)).view(torch.uint8)
        raw[c, :b.numel()] = b.reshape(-1)
    return raw


# ------------------------------------------------------------------ state

def _fx_buffers(plan):
    return {"acc": plan.alloc("acc"), "state": plan.alloc("state"), "vis": plan.alloc("vis")}


def prepare(case, seed):
    return {"kind": case["kind"], **globals()["_prepare_" + case["kind"]](case, seed)}


def _prepare_fx(case, seed):
    x, geom = _rows(case, seed)
    S, N, T, prec = case["S"], case["N"], case["T"], case["prec"]
    plan = corr.Plan(S, N, T, precision=PRECISION[prec], max_delay=MAX_DELAY, sample_rate=FS,
                     scale_mode=corr.SCALE_COMPUTE if case["compute"] else corr.SCALE_HOLD)
    scale = None
    if prec != "fp32":
        scale = torch.zeros(S, N // 2, device="cuda") if case["compute"] else _held_scale(case, seed)
    return {"plan": plan, "x": x, "geom": corr.geom_to_device(geom), "scale": scale, "compute": case["compute"],
            "spec": plan.alloc("spectra", zero=False), **_fx_buffers(plan)}


def _prepare_flagged(case, seed):
    x, geom = _rows(case, seed)
    S, N, T = case["S"], case["N"], case["T"]
    plan = corr.Plan(S, N, T, precision=corr.INT8, max_delay=MAX_DELAY, sample_rate=FS, power_fp16=int(case["f16"]))
    return {"plan": plan, "x": x, "geom": corr.geom_to_device(geom), "scale": _held_scale({**case, "prec": "int8"}, seed),
            "spec": plan.alloc("spectra", zero=False), "power": plan.alloc("power", zero=False).view(S, T, N // 2),
            "flags": plan.alloc("flags", zero=False).view(S, T, N // 2), "keep": plan.alloc("keep", zero=False),
            "counts": torch.zeros(N // 2, plan.P, dtype=torch.int32, device="cuda"),
            "net": _network(seed) if case["learned"] else None, **_fx_buffers(plan)}


def _prepare_train(case, seed):
    S, T, C = case["S"], case["T"], case["C"]
    power, labels = _power(S, T, C, seed)
    n = min(case["tiles"], corr.cnn_tiles(S, T, C))
    tiles = np.random.default_rng([int(seed), 7]).choice(corr.cnn_tiles(S, T, C), n, replace=False)
    return {"net": _network(seed), "power": power, "labels": labels, "cnn": corr.CNN(n),
            "tiles": torch.from_numpy(tiles.astype(np.int32)).cuda(), "loss": torch.zeros(1, device="cuda"),
            "grad": torch.zeros(corr.CNN_PARAMS, device="cuda")}


def _prepare_gated(case, seed):
    spec, scale = _layout_spectra(case, seed)
    plan = corr.Plan(case["S"], case["N"], case["T"], precision=PRECISION[case["prec"]], sample_rate=FS)
    bins = case["bins"]
    acc = torch.zeros(bins, plan.acc_bytes // 4, device="cuda", dtype=torch.int32 if case["prec"] == "int8" else torch.float32)
    return {"plan": plan, "spec": spec, "scale": scale, "gate": _gates(case), "bins": bins, "acc": acc,
            "state": [plan.alloc("state") for _ in range(bins)],
            "vis": torch.zeros(bins, plan.C, plan.P, 2, device="cuda")}


def _prepare_external(case, seed):
    plan = corr.Plan(case["S"], case["N"], case["T"], precision=PRECISION[case["prec"]], sample_rate=FS)
    fp32 = case["prec"] == "fp32"
    codes = None if fp32 else torch.empty(case["S"], case["T"], plan.C, 2, device="cuda",
                                          dtype=torch.int8 if case["prec"] == "int8" else torch.uint8)
    return {"plan": plan, "input": _time_spectra(case, seed), "codes": codes,
            "scale": None if fp32 else _held_scale(case, seed), "spec": plan.alloc("spectra", zero=False),
            **_fx_buffers(plan)}


def _prepare_phased(case, seed):
    spec, scale = _layout_spectra(case, seed)
    S, T, C = case["S"], case["T"], case["N"] // 2
    plan = corr.Plan(S, case["N"], T, precision=PRECISION[case["prec"]], sample_rate=FS)
    ph = 2 * math.pi * torch.rand(S, generator=_generator(seed, 8), device="cuda")
    return {"plan": plan, "spec": spec, "scale": scale, "n_int": case["n_int"],
            "w": torch.rand(S, generator=_generator(seed, 9), device="cuda").add_(0.5),
            "c": torch.stack([ph.cos(), ph.sin()], -1)[None].contiguous(),
            "inc": torch.empty(2, T, C, device="cuda"),
            "coh": torch.empty(1, 2, T, C, dtype=torch.complex64, device="cuda"),
            "work": torch.empty(2, T * C, dtype=torch.complex64, device="cuda"),
            "out": torch.empty(T * C // case["n_int"], device="cuda")}


def _prepare_front(case, seed):
    rows, n = 4 * case["cards"], case["n"]
    table = torch.empty(rows, 1 << 16, device="cuda")
    corr.blank_noise_table(seed, table)
    return {"raw": _card_streams(case, seed), "n": n, "bits": case["bits"], "block": case["block"], "table": table,
            "x": torch.zeros(rows, (n + 255) // 256 * 256, dtype=torch.int8, device="cuda"),
            "counts": torch.zeros(rows, -(-n // case["block"]), dtype=torch.int32, device="cuda")}


def _subarrays(case):
    for k, text in enumerate(case["shapes"].split()):
        S, C, T = (int(v) for v in text.split("x"))
        yield k, {"S": S, "N": 2 * C, "T": T, "prec": "int8", "compute": False}


def _prepare_batch(case, seed):
    subs = list(_subarrays(case))
    batch = corr.Batch([{"n_signals": s["S"], "fft_len": s["N"], "n_spectra": s["T"]} for _, s in subs],
                       sample_rate=FS, max_delay=MAX_DELAY)
    vis = []
    for k, s in subs:
        x, geom = _rows(s, seed + 1000 * k)
        plan = batch.plans[k]
        b = _fx_buffers(plan)
        vis.append(b["vis"].view(plan.C, plan.P, 2))
        batch.set_io(k, x=x, geom=corr.geom_to_device(geom), spec=plan.alloc("spectra", zero=False),
                     scale=_held_scale(s, seed + 1000 * k), flags=corr.DUMP | corr.RESET, **b)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    batch.capture(stream)
    return {"batch": batch, "stream": stream, "vis": vis}


# ------------------------------------------------------------------ one pass

def run(state):
    return globals()["_run_" + state["kind"]](state)


def _integrated(s):
    plan = s["plan"]
    plan.integrate(s["acc"], s["state"], s["vis"], s["scale"], flags=corr.DUMP | corr.RESET)
    return s["vis"].view(plan.C, plan.P, 2)


def _run_fx(s):
    s["plan"].fengine(s["x"], s["geom"], s["spec"], s["scale"])
    s["plan"].xengine(s["spec"], s["acc"])
    vis = _integrated(s)
    return {"vis": vis, "scale": s["scale"]} if s["compute"] else {"vis": vis}


def _run_flagged(s):
    plan = s["plan"]
    plan.fengine(s["x"], s["geom"], s["spec"], s["scale"], power=s["power"])
    if s["net"] is not None:
        corr.cnn_infer(s["net"], s["power"], s["flags"], threshold=0.5, guard=3.0)
    else:
        plan.mad_flag(s["power"], s["flags"], 3.0)
    plan.apply_flags(s["flags"], None, s["keep"])
    s["counts"].zero_()
    plan.xengine(s["spec"], s["acc"], keep=s["keep"], counts=s["counts"])
    return {"vis": _integrated(s), "counts": s["counts"], "flags": s["flags"]}


def _run_train(s):
    s["cnn"].loss_grad(s["net"], s["power"], s["labels"], s["tiles"], s["loss"], s["grad"])
    return {"loss": s["loss"], "grad": s["grad"]}


def _run_gated(s):
    plan = s["plan"]
    plan.xengine_gated(s["spec"], s["gate"], s["bins"], s["acc"])
    for b in range(s["bins"]):
        plan.integrate(s["acc"][b], s["state"][b], s["vis"][b], s["scale"], flags=corr.DUMP | corr.RESET)
    return {"vis": s["vis"]}


def _run_external(s):
    plan = s["plan"]
    if s["codes"] is not None:
        plan.requantize(s["input"], s["scale"], s["codes"])
    plan.xpack(s["input"] if s["codes"] is None else s["codes"], s["spec"])
    plan.xengine(s["spec"], s["acc"])
    return {"vis": _integrated(s)}


def _run_phased(s):
    s["plan"].beamform(s["spec"], s["scale"], w=s["w"], inc=s["inc"], c=s["c"], coh=s["coh"], mode=corr.BEAM_VOLTAGE)
    corr.dedisperse(s["coh"][0], sample_rate=FS, nu0=325e6, dm=71.0, n_int=s["n_int"], work=s["work"], out=s["out"])
    return {"incoherent": s["inc"], "series": s["out"], "voltages": s["work"]}


def _run_front(s):
    corr.adc_unpack(s["raw"], s["x"], bits=s["bits"], n=s["n"])
    corr.blank_voltages(s["x"], s["table"], block=s["block"], M=3.0, counts=s["counts"], n=s["n"])
    return {"rows": s["x"][:, :s["n"]], "counts": s["counts"]}


def _run_batch(s):
    s["batch"].launch(s["stream"])
    return {"vis": s["vis"]}


# ------------------------------------------------------------------ work

CELL_BYTES = {"fp32": 8, "int8": 2, "e4m3": 2}


def _fx_work(S, N, T, cell):
    """Samples in, the spectra buffer written and read, visibilities out; FFT, phase and all products."""
    C, P = N // 2, S * (S + 1) // 2
    nbytes = S * T * N + 2 * S * T * C * cell + 8 * C * P
    return nbytes, S * T * (2.5 * N * math.log2(N) + 6 * C) + 8.0 * P * C * T


def work(case):
    kind = case["kind"]
    if kind == "batch":
        both = [_fx_work(s["S"], s["N"], s["T"], 2) for _, s in _subarrays(case)]
        return {"bytes": sum(b for b, _ in both), "flops": sum(f for _, f in both)}
    if kind == "train":
        cells = 64 * 256 * min(case["tiles"], corr.cnn_tiles(case["S"], case["T"], case["C"]))
        return {"bytes": 5 * cells, "flops": 3.0 * 2 * 2592 * cells}
    if kind == "front":
        n = 4 * case["cards"] * case["n"]
        return {"bytes": n * case["bits"] / 8 + n, "flops": 0}
    S, N, T = case["S"], case["N"], case["T"]
    C, P = N // 2, S * (S + 1) // 2
    cells = S * T * C
    if kind == "fx":
        nbytes, flops = _fx_work(S, N, T, CELL_BYTES[case["prec"]])
        return {"bytes": nbytes, "flops": flops}
    if kind == "flagged":
        nbytes, flops = _fx_work(S, N, T, 2)
        power = 2 if case["f16"] else 4
        return {"bytes": nbytes + cells * (2 * power + 2 + 0.25) + 4 * C * P,
                "flops": flops + 2.0 * P * C * T + (2 * 2592.0 * cells if case["learned"] else 0)}
    if kind == "gated":
        return {"bytes": cells * CELL_BYTES[case["prec"]] + 8 * C * P * case["bins"], "flops": 8.0 * P * C * T}
    if kind == "external":
        codes = 0 if case["prec"] == "fp32" else 4 * cells
        return {"bytes": 8 * cells + codes + (16 if case["prec"] == "fp32" else 2) * cells + 8 * C * P,
                "flops": 8.0 * P * C * T}
    L = T * C
    return {"bytes": cells * CELL_BYTES[case["prec"]] + 8 * L + 2 * 16 * L + 16 * L + 4 * L / case["n_int"],
            "flops": 12.0 * cells + 2 * (5 * L * math.log2(C) + 10 * L * math.log2(L) + 9 * L)}


# ------------------------------------------------------------------ the same outputs in 64 bits

def exact(case, seed):
    return globals()["_exact_" + case["kind"]](case, seed)


def _phase(geom, s, N, m0, T):
    """exp of Eq. 2's phase for spectra m0 .. of signal s, [T][C]."""
    t = (torch.arange(m0, m0 + T, device="cuda", dtype=torch.float64) + 0.5) * (N / FS)
    k = torch.arange(N // 2, device="cuda", dtype=torch.float64)
    cycles = (float(geom["psi0"][s]) + float(geom["rate"][s]) * t)[:, None] + (k * (float(geom["frac"][s]) / N))[None, :]
    return torch.polar(torch.ones_like(cycles), 2 * math.pi * cycles)


def _channels(row, D, N, m0, T):
    """Unrotated complex128 channels [T][C] of spectra m0 .. of one row."""
    w = row[D + m0 * N:D + (m0 + T) * N].view(T, N).double()
    return torch.fft.rfft(w)[:, :N // 2]


def _codes(Y, scale, prec):
    """Requantised components of complex Y as float64 [..][2]."""
    v = torch.view_as_real(Y) / scale.double()[..., None]
    if prec == "int8":
        return v.round_().clamp_(-127, 127)
    return v.clamp_(-448, 448).float().to(torch.float8_e4m3fn).double()


def _visibilities(block, S, C, T, scale):
    """V[k][p] over `block(k0, k1)` -> complex128 [S][T][k1 - k0]; scale [S][C] or None."""
    j, i = torch.tril_indices(S, S, device="cuda")
    out = torch.empty(C, S * (S + 1) // 2, dtype=torch.complex128, device="cuda")
    step = max(1, min(C, (1 << 26) // (S * T)))
    for k in range(0, C, step):
        a = block(k, min(C, k + step)).permute(2, 0, 1).contiguous()
        v = torch.matmul(a, a.conj().transpose(1, 2).contiguous())
        out[k:k + step] = v[:, i, j]
        del a, v
    if scale is not None:
        sc = scale.double()
        out *= (sc[i] * sc[j]).t()
    return torch.view_as_real(out)


def _exact_step(case, seed, flag=None):
    """Visibilities of an F, X and integrate step; flag(power [T][C]) -> cells to leave out, per signal."""
    x, geom = _rows(case, seed)
    S, N, T, prec = case["S"], case["N"], case["T"], case["prec"]
    C, fp32 = N // 2, prec == "fp32"
    scale = None if fp32 or case["compute"] else _held_scale(case, seed)
    if case["compute"]:
        scale = torch.empty(S, C, dtype=torch.float64, device="cuda")
    held = torch.empty(S, T, C, 2, device="cuda", dtype=torch.float64 if fp32 else torch.int8 if prec == "int8" else torch.float32)
    step = max(1, min(T, (1 << 25) // N) // 64 * 64) or T
    for s in range(S):
        D = int(geom["D"][s])
        if case["compute"]:
            total = sum(_channels(x[s], D, N, m, min(step, T - m)).abs().square_().sum(0) for m in range(0, T, step))
            scale[s] = 4 * (total / (2 * T)).sqrt() / QMAX[prec]
        for m in range(0, T, step):
            n = min(step, T - m)
            X = _channels(x[s], D, N, m, n)
            Y = X * _phase(geom, s, N, m, n)
            v = torch.view_as_real(Y) if fp32 else _codes(Y, scale[s], prec)
            if flag is not None:
                v = v * (~flag(X.abs().square_()))[..., None]
            held[s, m:m + n] = v.to(held.dtype)
            del X, Y, v
    del x
    vis = _visibilities(lambda a, b: torch.view_as_complex(held[:, :, a:b].double().contiguous()), S, C, T, scale)
    return vis, scale


def _exact_fx(case, seed):
    vis, scale = _exact_step(case, seed)
    return {"vis": vis, "scale": scale} if case["compute"] else {"vis": vis}


def _middle(v):
    n = v.shape[-1] // 2
    s = v.sort(-1).values
    return 0.5 * (s[..., n - 1:n] + s[..., n:n + 1])


def _outliers(v, M=3.0):
    d = (v - _middle(v)).abs()
    return d > M * _middle(d) / 0.6745


def _tiles(p):
    """[T][C] -> [tiles][64][256]."""
    T, C = p.shape
    return p.view(T // 64, 64, C // 256, 256).transpose(1, 2).reshape(-1, 64, 256)


def _untile(t, T, C):
    return t.view(T // 64, C // 256, 64, 256).transpose(1, 2).reshape(T, C)


def _conv(a, w, b):
    """Same-size 3 x 3 cross-correlation of a [n][I][H][W] with w [O][I][3][3]."""
    n, I, H, W = a.shape
    pad = torch.nn.functional.pad(a.transpose(0, 1), (1, 1, 1, 1))
    out = b[:, None].expand(-1, n * H * W)
    for u in range(3):
        for v in range(3):
            out = out + w[:, :, u, v] @ pad[:, :, u:u + H, v:v + W].reshape(I, -1)
    return out.view(-1, n, H, W).transpose(0, 1)


def _logits(net, tiles):
    """Logits [n][64][256] of power tiles, in the weights' type."""
    level = _middle(tiles.mean(1))[:, :, None]
    a = torch.log1p(tiles / torch.where(level > 0, level, torch.ones_like(level)))[:, None]
    at = 0
    for k, (out, inp) in enumerate(((16, 1), (16, 16), (1, 16))):
        w = net[at:at + out * inp * 9].view(out, inp, 3, 3)
        b = net[at + out * inp * 9:at + out * inp * 9 + out]
        at += out * inp * 9 + out
        a = _conv(a.relu() if k else a, w, b)
    return a[:, 0]


def _exact_flagged(case, seed):
    net = _network(seed).double() if case["learned"] else None

    def flag(p):
        T, C = p.shape
        if case["f16"]:
            p = (p / float(case["N"]) ** 2).half().double()
        found = []
        for t in _tiles(p).split(128):
            f = _outliers(t.mean(1))[:, None, :].expand_as(t)
            f = f | ((_logits(net, t) > 0) if net is not None else _outliers(t.mean(2))[:, :, None])
            found.append(f)
        return _untile(torch.cat(found), T, C)

    return {"vis": _exact_step({**case, "prec": "int8", "compute": False}, seed, flag)[0], "counts": None, "flags": None}


def _exact_train(case, seed):
    state = _prepare_train(case, seed)
    net = state["net"].double().requires_grad_()
    ids = state["tiles"].long()
    both = [torch.stack([_tiles(v) for v in state[k].double()]).view(-1, 64, 256)[ids] for k in ("power", "labels")]
    loss = torch.nn.functional.binary_cross_entropy_with_logits(_logits(net, both[0]), both[1])
    loss.backward()
    return {"loss": loss.detach().view(1), "grad": net.grad}


def _exact_gated(case, seed):
    spec, scale = _layout_spectra(case, seed)
    S, C, T = case["S"], case["N"] // 2, case["T"]
    v, gate = _layout_to_time(spec, case), _gates(case)
    return {"vis": torch.stack([
        _visibilities(lambda a, b: torch.view_as_complex(v[:, gate == k, a:b].double().contiguous()), S, C,
                      T, scale) for k in range(case["bins"])])}


def _exact_external(case, seed):
    v, S, C, T = _time_spectra(case, seed), case["S"], case["N"] // 2, case["T"]
    scale = None if case["prec"] == "fp32" else _held_scale(case, seed)

    def block(a, b):
        y = torch.view_as_complex(v[:, :, a:b].double().contiguous())
        return y if scale is None else torch.view_as_complex(_codes(y, scale[:, None, a:b], case["prec"]))

    return {"vis": _visibilities(block, S, C, T, scale)}


def _exact_phased(case, seed):
    spec, scale = _layout_spectra(case, seed)
    S, C, T = case["S"], case["N"] // 2, case["T"]
    w, c = (_prepare_phased_weights(S, seed))
    codes = _layout_to_time(spec, case)
    inc = torch.zeros(2, T, C, dtype=torch.float64, device="cuda")
    v = torch.zeros(2, T, C, dtype=torch.complex128, device="cuda")
    for s in range(S):
        y = torch.view_as_complex(codes[s].double().contiguous())
        if scale is not None:
            y = y * scale[s].double()
        inc[s % 2] += w[s] * y.abs().square_()
        v[s % 2] += c[s] * y
    L = T * C
    z = (torch.fft.ifft(v) * C).view(2, L)
    f = torch.arange(L, device="cuda", dtype=torch.float64) * (FS / (2 * L))
    turns = 4.148808e15 * 71.0 * f * f / (325e6 ** 2 * (325e6 + f))
    z = torch.fft.ifft(torch.fft.fft(z) * torch.polar(torch.ones_like(f), -2 * math.pi * (turns - turns.floor())))
    series = z.abs().square_().sum(0).view(-1, case["n_int"]).sum(1)
    return {"incoherent": inc, "series": series, "voltages": torch.view_as_real(z).reshape(2, L, 2)}


def _prepare_phased_weights(S, seed):
    ph = 2 * math.pi * torch.rand(S, generator=_generator(seed, 8), device="cuda")
    w = torch.rand(S, generator=_generator(seed, 9), device="cuda").add_(0.5)
    return w.double(), torch.complex(ph.cos().double(), ph.sin().double())


def _exact_front(case, seed):
    return None  # whole numbers


def _exact_batch(case, seed):
    return {"vis": [_exact_step(s, seed + 1000 * k)[0] for k, s in _subarrays(case)]}
