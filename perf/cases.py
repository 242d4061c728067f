"""The workloads the beamformer's speed is judged on, and inputs for them.

Every case goes through the package's public classes (``bf.Plan``,
``bf.Batch``, ``bf.Table``) as a user's program does: plans are made and their
weights set once, and a pass beamforms one block (a tracking pass also sets
the next pointing's weights).  Sizes are those of the repository's own
workloads (``synth.small``, ``paper``, ``precision``, ``serve_block``, the
uneven beam sets of ``synth.batch``), a small quick-look block, and ragged
sizes none of the tile shapes divides.

A case is a dict of plain values: ``kind`` ("run", "tracking", "batch",
"table"), the plan's sizes N (antennas), C (channels), B (beams), T (samples
per block) and I (integration), ``prec``, ``bits`` (8 or 4 per voltage
component) and ``output``.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1412_4907_amd import bf

C0 = 299792458.0


def _case(name, kind="run", N=32, C=1024, B=128, T=65536, I=16, prec="fp16", bits=8,
          output="power", blocks=1, sets=""):
    c = {"kind": kind, "N": N, "C": C, "B": B, "T": T, "I": I, "prec": prec, "bits": bits,
         "output": output, "blocks": blocks, "sets": sets}
    return {"name": name, **c} if name else c


def listed():
    return [
        # quick-look of a few channels and beams: launch latency and host cost
        _case("tiny_fp16", N=16, C=32, B=8, T=512, I=16),
        # the small configuration: 32 antennas, four beams at full time resolution
        _case("small_fp32", N=32, C=128, B=4, T=4096, I=1, prec="fp32"),
        # the paper-scale block, reference precision
        _case("paper_fp32", prec="fp32"),
        # the paper-scale block, the form a deployment runs
        _case("paper_fp16"),
        # many beams at full time resolution from the F-engine's native 4-bit
        # samples: a search back end's input
        _case("search_bf16_in4", N=32, C=128, B=512, T=4096, I=1, prec="bf16", bits=4),
        # one large beam set on a 16x16 array
        _case("large_fp16", N=256, C=1024, B=512, T=8192, I=64),
        # odd everything: 66-byte rows, a partial beam range, decimal integration
        _case("ragged_fp16", N=33, C=256, B=100, T=10000, I=10),
        # integration windows that span two blocks, summed into one output
        _case("span_fp32", N=64, C=256, B=72, T=8192, I=64, prec="fp32", blocks=2),
        # complex beams for a folding stage: few beams, every sample kept
        _case("complex_fp16", N=32, C=512, B=16, T=65536, I=1, output="complex"),
        # tracking beams: a new pointing's weights every block
        _case("tracking_fp16", kind="tracking", N=256, C=256, B=512, T=8192, I=64),
        # uneven sub-arrays and beam sets in one launch (N x C x B x T each)
        _case("batch_fp16", kind="batch", I=16,
              sets="16x512x64x16384;32x1024x128x8192;64x256x256x8192;128x256x1024x8192;"
                   "256x256x100x8192;24x256x16x32768"),
        # serving: several requests' beam sets (beams of each) on one block
        _case("serve_fp16", kind="table", N=256, C=1024, T=8192, I=64, sets="100;300;77;35"),
    ]


# ---- more cases of the same ranges ----

def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _ant(rng, by8, hi=512):
    return min(hi, max(8, 8 * _log(rng, 1, hi // 8))) if by8 else _log(rng, 2, 300)


def _padded_flops(N, C, B, T):
    return 8.0 * C * max(B, 16) * T * max(N, 32)


def _fit(N, C, B, T, I, most=1e11, most_bytes=2e9):
    """Fewer channels, then a shorter block, until a set is small enough."""
    def big():
        return (_padded_flops(N, C, B, T) > most or
                C * T * 2.0 * N + 4.0 * C * B * T / I > most_bytes)
    while big() and C > 1:
        C = max(1, C * 2 // 3)
    while big() and T > I:
        T = max(I, T // 2 // I * I)
    return C, T


def draw(rng):
    kind = rng.choice(["run"] * 7 + ["tracking", "batch", "table"])
    I = rng.choice([1, 1, 2, 4, 5, 8, 10, 16, 16, 25, 32, 64, 64, 100, 128])
    prec = rng.choice(["fp32", "fp16", "bf16"])
    if kind == "batch":
        sets = []
        for _ in range(rng.randint(2, 6)):
            N, C, B = _ant(rng, True, 256), _log(rng, 8, 512), _log(rng, 4, 512)
            T = max(I, _log(rng, 512, 32768) // I * I)
            C, T = _fit(N, C, B, T, I, 2e10, 5e8)
            sets.append(f"{N}x{C}x{B}x{T}")
        return _case("", kind, I=I, prec=prec, sets=";".join(sets))
    N = _ant(rng, kind != "run" or rng.random() < 0.5)
    C, B = _log(rng, 1, 1024), _log(rng, 1, 1024)
    T = max(I, _log(rng, 256, 65536) // I * I)
    bits = 4 if N % 8 == 0 and rng.random() < 0.3 else 8
    if kind == "table":
        beams = [_log(rng, 8, 300) for _ in range(rng.randint(1, 6))]
        C, T = _fit(N, C, sum(beams), T, I)
        return _case("", kind, N=N, C=C, T=T, I=I, prec=prec, bits=bits,
                     sets=";".join(str(b) for b in beams))
    C, T = _fit(N, C, B, T, I)
    output, blocks = "power", 1
    if kind == "run" and I == 1 and rng.random() < 0.4:
        output = "complex"
    elif kind == "run" and rng.random() < 0.15:
        blocks = 2
    return _case("", kind, N=N, C=C, B=B, T=T, I=I, prec=prec, bits=bits, output=output,
                 blocks=blocks)


# ---- inputs ----

def _sets(case):
    """(N, C, B, T) of every beam set of the case."""
    if case["kind"] == "batch":
        return [tuple(int(v) for v in s.split("x")) for s in case["sets"].split(";")]
    if case["kind"] == "table":
        return [(case["N"], case["C"], int(b), case["T"]) for b in case["sets"].split(";")]
    return [(case["N"], case["C"], case["B"], case["T"])]


def _geometry(N, C, B, seed):
    """A square-ish array grid, pointings within 25 degrees of zenith, 16 MHz
    of channels above 400 MHz (numpy, FP64)."""
    g = np.random.default_rng(seed)
    side = int(math.ceil(math.sqrt(N)))
    k = np.arange(N)
    pos = np.stack([10.0 * (k % side), 10.0 * (k // side), np.zeros(N)], axis=1)
    pos += g.normal(0.0, 0.05, pos.shape)
    th = np.deg2rad(25.0) * np.sqrt(g.random(B))
    ph = 2.0 * np.pi * g.random(B)
    d = np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], axis=1)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    freqs = 400e6 + 16e6 * (np.arange(C) + 0.5) / C
    return pos, d, freqs


def _voltages(N, C, T, bits, geo, seed):
    """Receiver noise (16 of 127 levels per component; 2 of 7 in 4 bits) and
    one source of the same strength in the first beam: integer components
    [C][T][N][2] as int8 on the GPU, made a few channels at a time."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    pos, d, freqs = geo
    sigma, lim = (16.0, 127) if bits == 8 else (2.0, 7)
    x = torch.empty((C, T, N, 2), dtype=torch.int8, device="cuda")
    kr = torch.from_numpy(pos @ d[0] / C0).cuda()
    step = max(1, int(1.2e8 / (T * N * 2)))
    for c in range(0, C, step):
        n = min(step, C - c)
        v = torch.randn((n, T, N, 2), generator=g, device="cuda")
        src = torch.randn((n, T, 1, 2), generator=g, device="cuda")
        ph = 2.0 * math.pi * (torch.from_numpy(freqs[c:c + n]).cuda()[:, None] * kr)
        cs, sn = ph.cos().float()[:, None, :], ph.sin().float()[:, None, :]
        v[..., 0] += src[..., 0] * cs - src[..., 1] * sn
        v[..., 1] += src[..., 0] * sn + src[..., 1] * cs
        x[c:c + n] = v.mul_(sigma).round_().clamp_(-lim, lim).to(torch.int8)
    return x


def _pack4(x):
    """Integer components in [-8, 7] -> one byte per sample, real part high."""
    return ((x[..., 0] << 4) | (x[..., 1] & 15)).view(torch.uint8).contiguous()


def _inputs(case, seed):
    """One (geometry, [voltage blocks]) per set; a table's sets share one block."""
    out = []
    for i, (N, C, B, T) in enumerate(_sets(case)):
        geo = _geometry(N, C, B, [seed, i])
        if case["kind"] == "table":
            geo = (_geometry(N, C, 1, [seed, 99])[0],) + geo[1:]
            xs = out[0][1] if out else [_voltages(N, C, T, case["bits"], geo, seed)]
        else:
            xs = [_voltages(N, C, T, case["bits"], geo, seed + 1000003 * (16 * i + k))
                  for k in range(case["blocks"])]
        out.append((geo, xs))
    return out


def _scale(N):
    return 1.0 / (16.0 * math.sqrt(N))


def prepare(case, seed):
    """Plans with their weights set, voltages and output buffers on the GPU."""
    plans, blocks, outs, geos = [], [], [], []
    packed = None
    for (N, C, B, T), (geo, xs) in zip(_sets(case), _inputs(case, seed)):
        plan = bf.Plan(N, C, B, T, case["I"], precision=case["prec"],
                       accumulate=case["blocks"] > 1, input_bits=case["bits"],
                       output=case["output"])
        if case["output"] == "complex":
            plan.set_output_scale(_scale(N))
        plan.set_weights(*geo)
        if case["bits"] == 4:
            if packed is None or case["kind"] != "table":
                packed = [_pack4(x) for x in xs]
            xs = packed
        plans.append(plan)
        blocks.append(xs)
        geos.append(geo)
        outs.append(torch.empty(plan.p_shape, dtype=plan.p_dtype, device="cuda"))
    state = {"kind": case["kind"], "plans": plans, "blocks": blocks, "outs": outs, "geos": geos}
    if case["kind"] == "batch":
        state["batch"] = bf.Batch(plans)
    elif case["kind"] == "table":
        state["table"] = bf.Table(case["N"], case["I"], case["prec"], input_bits=case["bits"])
    elif case["kind"] == "tracking":
        state["side"] = torch.cuda.Stream()
    return state


def run(state):
    """One block of every set (two, summed, where windows span blocks)."""
    plans, outs, kind = state["plans"], state["outs"], state["kind"]
    if kind == "batch":
        state["batch"].run([b[0] for b in state["blocks"]], outs)
    elif kind == "table":
        state["table"].set(plans, [b[0] for b in state["blocks"]], outs)
        state["table"].run()
    elif kind == "tracking":
        plans[0].set_weights_async(*state["geos"][0], stream=state["side"])
        plans[0].run(state["blocks"][0][0], outs[0])
    else:
        xs = state["blocks"][0]
        if len(xs) > 1:
            outs[0].zero_()
        for x in xs:
            plans[0].run(x, outs[0])
    return outs


def work(case):
    """Bytes (voltages, weights and outputs once) and flops (8 per complex
    multiply-accumulate) of one pass."""
    es = 4 if case["prec"] == "fp32" else 2
    nbytes = flops = 0.0
    for i, (N, C, B, T) in enumerate(_sets(case)):
        if case["kind"] != "table" or i == 0:
            nbytes += case["blocks"] * C * T * N * 2.0 * case["bits"] / 8
        nbytes += 2.0 * es * C * B * N + 4.0 * C * B * (T // case["I"])
        flops += 8.0 * case["blocks"] * C * B * T * N
    return {"bytes": nbytes, "flops": flops}


def exact(case, seed):
    """The same outputs in FP64: per channel, the weights from the geometry,
    the complex beams as two real matrix products, power summed over I."""
    res = []
    I = case["I"]
    for (N, C, B, T), ((pos, d, freqs), xs) in zip(_sets(case), _inputs(case, seed)):
        kr = torch.from_numpy(d @ pos.T / C0).cuda()  # [B][N] seconds
        cx = case["output"] == "complex"
        out = torch.zeros((C, B, T, 2) if cx else (C, B, T // I), dtype=torch.float64,
                          device="cuda")
        for c in range(C):
            cyc = float(freqs[c]) * kr
            ph = -2.0 * math.pi * (cyc - cyc.round())
            wr, wi = ph.cos(), ph.sin()
            re_row = torch.stack([wr, -wi], dim=-1).reshape(B, 2 * N)
            im_row = torch.stack([wi, wr], dim=-1).reshape(B, 2 * N)
            for x in xs:
                v = x[c].reshape(T, 2 * N).double().t().contiguous()
                re, im = re_row @ v, im_row @ v  # [B][T]
                if cx:
                    out[c, :, :, 0] = re * _scale(N)
                    out[c, :, :, 1] = im * _scale(N)
                else:
                    out[c] += (re * re + im * im).reshape(B, T // I, I).sum(dim=-1)
        res.append(out)
    return res
