"""The streamed form (any K that fits LDS, any integration, input and output)
and the register-resident form at the sizes where they can go wrong: rows that
are not multiples of 16 bytes (odd N included, with odd block lengths, so
channels start mid-dword), K remainders of a chunk, partial and uneven beam
ranges, window counts that are not multiples of 4 or of 16, integrations that
are not multiples of the row-tile count, accumulation and complex output.

Each is checked against the FP64 oracle to the precision form's tolerance and,
bit for bit, against the general form (tile (4, 8, 2, 0) or (4, 1, 1, 0)), which
accumulates every output over the same K slices and sums windows in the same
order but reads rows byte by byte where they are not 16-byte aligned."""
import numpy as np
import pytest

import oracle
from paper_1412_4907_amd import bf, synth
from tests.gpu_util import assert_parity, run_plan

pytestmark = pytest.mark.gpu
TOL = {"fp32": 1e-5, "fp16": 2e-3, "bf16": 1e-2}

SHAPES = [  # N, C, B, T, I
    (1, 3, 1, 7, 1), (3, 2, 17, 35, 5), (33, 3, 100, 630, 10), (31, 2, 16, 101, 1),
    (65, 2, 33, 198, 2), (2, 3, 5, 64, 4), (10, 2, 72, 51, 3), (36, 2, 130, 272, 16),
    (50, 2, 20, 1017, 9), (64, 2, 144, 1040, 13), (24, 2, 112, 330, 6), (100, 1, 9, 257, 1),
    (32, 2, 96, 1020, 12), (16, 2, 208, 1000, 8), (129, 1, 40, 75, 25), (48, 2, 80, 514, 2),
]


def _case(shape, seed):
    N, C, B, T, I = shape
    g = np.random.default_rng(seed)
    pos = synth.disc_positions(N, 200.0, g)
    dirs = synth.random_dirs(B, g)
    freqs = np.linspace(400e6, 416e6, C)
    x = g.integers(-128, 128, (C, T, N, 2)).astype(np.int8)
    return pos, dirs, freqs, x


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=[f"N{s[0]}C{s[1]}B{s[2]}T{s[3]}I{s[4]}" for s in SHAPES])
def test_forms_against_oracle_and_general(gpu, shape, prec):
    N, C, B, T, I = shape
    print(f"forms {shape} {prec}", flush=True)
    pos, dirs, freqs, x = _case(shape, sum(shape) * 3 + len(prec))
    with bf.Plan(N, C, B, T, I, precision=prec) as plan:
        plan.set_weights(pos, dirs, freqs)
        got = run_plan(plan, x, gpu)
        default = plan.tile()
        outs = []
        for t in plan.tile_candidates():
            if t[3] in (1, -2, -3, -4) and t[0] == 4:
                plan.set_tile(*t, 4)
                outs.append((t, run_plan(plan, x, gpu)))
        assert any(t[3] == -4 for t, _ in outs)
        plan.set_tile(4, 1, 1, 0, 4)
        general = run_plan(plan, x, gpu)
    ref = oracle.beamform(oracle.weights(pos, dirs, freqs), x, I)
    assert_parity(got, ref, TOL[prec], f"{shape} {prec} {default}")
    assert np.array_equal(got, general), (shape, prec, default)
    for t, o in outs:
        assert np.array_equal(o, general), (shape, prec, t)


@pytest.mark.parametrize("shape", [(33, 2, 20, 210, 7), (32, 2, 72, 512, 16), (64, 2, 40, 96, 2),
                                   (5, 2, 9, 45, 1), (32, 2, 40, 66, 1), (40, 1, 8, 84, 4)],
                         ids=lambda s: f"N{s[0]}B{s[2]}T{s[3]}I{s[4]}")
@pytest.mark.parametrize("prec", ["fp32", "fp16"])
def test_accumulate_adds_in_one_rounding(gpu, shape, prec):
    import torch
    N, C, B, T, I = shape
    print(f"forms accumulate {shape} {prec}", flush=True)
    pos, dirs, freqs, x = _case(shape, sum(shape))
    with bf.Plan(N, C, B, T, I, precision=prec) as a, \
            bf.Plan(N, C, B, T, I, precision=prec, accumulate=True) as b:
        a.set_weights(pos, dirs, freqs)
        b.set_weights(pos, dirs, freqs)
        p1 = run_plan(a, x, gpu)
        base = np.random.default_rng(1).random(p1.shape).astype(np.float32) * p1.max()
        for t in [b.tile()] + [c + (4,) for c in b.tile_candidates() if c[3] < -2]:
            b.set_tile(*t)
            acc = torch.from_numpy(base).to(gpu)
            b.run(torch.from_numpy(x).to(gpu), acc)
            torch.cuda.synchronize()
            assert np.array_equal(acc.cpu().numpy(), base + p1), (shape, prec, t)


@pytest.mark.parametrize("shape", [(33, 2, 20, 61), (31, 2, 16, 64), (70, 2, 37, 130), (8, 1, 3, 40)],
                         ids=lambda s: f"N{s[0]}B{s[2]}T{s[3]}")
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_complex_forms(gpu, shape, prec):
    import torch
    N, C, B, T = shape
    print(f"forms complex {shape} {prec}", flush=True)
    pos, dirs, freqs, x = _case(shape + (1,), sum(shape))
    xd = torch.from_numpy(x).to(gpu)
    with bf.Plan(N, C, B, T, 1, precision=prec, output="complex") as plan:
        plan.set_weights(pos, dirs, freqs)
        plan.set_output_scale(1.0 / 16)
        outs = []
        for t in [plan.tile()] + [c + (4,) for c in plan.tile_candidates() if c[3] in (0, -3, -4)]:
            plan.set_tile(*t)
            p = torch.full(plan.p_shape, float("nan"), dtype=torch.float16, device=gpu)
            plan.run(xd, p)
            torch.cuda.synchronize()
            outs.append(p.cpu().numpy())
    for o in outs[1:]:
        assert np.array_equal(outs[0], o)
    ref = oracle.beams(oracle.weights(pos, dirs, freqs), x) / 16
    got = outs[0][..., 0].astype(np.float64) + 1j * outs[0][..., 1]
    rms = np.sqrt(np.mean(np.abs(ref) ** 2, axis=-1, keepdims=True))
    # FP32 weights: FP16 output rounding (2^-11 per component) dominates
    assert np.max(np.abs(got - ref) / (np.abs(ref) + rms)) <= (1e-3 if prec == "fp32" else 1e-2)


@pytest.mark.parametrize("N", [8, 40])
def test_fp32_split_holds_the_fp32_range(gpu, N):
    """FP32 weights travel as three BF16 parts: weights over 30 decades keep
    their FP32 value, and a raw weight beyond the FP32 range is an infinity
    in every part's sum, as in one FP32 product."""
    print(f"fp32 split N={N}", flush=True)
    g = np.random.default_rng(N)
    C, B, T, I = 2, 18, 64, 4
    W = (g.normal(size=(C, B, N)) + 1j * g.normal(size=(C, B, N))) * \
        10.0 ** g.integers(-12, 13, (C, B, 1))
    x = g.integers(1, 128, (C, T, N, 2)).astype(np.int8)
    with bf.Plan(N, C, B, T, I) as plan:
        plan.set_weights_raw(W)
        wq = plan.get_weights()
        assert np.array_equal(wq.real, W.real.astype(np.float32))
        got = run_plan(plan, x, gpu).astype(np.float64)
        ref = oracle.beamform(wq, x, I)
        # accumulation alone: 2N <= 80 products, each sum within 2^-24 of its
        # size per accumulation step, twice in the power
        assert np.max(np.abs(got - ref) / np.mean(ref, axis=-1, keepdims=True)) <= 2e-6
        W[1, 5, 3] = 1e300
        plan.set_weights_raw(W)
        inf = run_plan(plan, x, gpu)
        plan.set_tile(4, 1, 1, 0, 4)
        assert np.array_equal(inf, run_plan(plan, x, gpu))
    assert np.all(np.isinf(inf[1, 5])) and np.all(np.isfinite(inf[0]))
