"""The general form (channels past 2 GiB, byte-load batches, weights too large for
LDS split into their parts): every compiled width against the plan's own form,
batches of antenna counts that are no multiple of 8 against their plans alone,
and channels past 2 GiB against the same samples run as two blocks, which the
pipelined and streamed forms take.  All bit for bit: every form accumulates in
one order."""
import numpy as np
import pytest

import oracle
from paper_1412_4907_amd import bf, synth
from tests.gpu_util import assert_parity, run_plan

pytestmark = pytest.mark.gpu
TOL = {"fp32": 1e-5, "fp16": 2e-3, "bf16": 1e-2}


def _geometry(N, C, B, seed):
    g = np.random.default_rng(seed)
    return (synth.disc_positions(N, 200.0, g), synth.random_dirs(B, g),
            np.linspace(400e6, 416e6, C))


# half chunk alone, one chunk, chunk and half chunk (first and second of a pair
# of fragment buffers), three chunks, 100 beams as 4 + 3 tiles, dummy rows
WIDTHS = [(8, 40, 96, 4), (32, 100, 330, 10), (40, 24, 77, 1), (96, 72, 130, 2), (16, 33, 64, 16),
          (104, 17, 63, 9)]


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("shape", WIDTHS, ids=lambda s: f"N{s[0]}B{s[1]}T{s[2]}I{s[3]}")
def test_every_width_equals_the_default(gpu, shape, prec):
    N, B, T, I = shape
    print(f"general widths {shape} {prec}", flush=True)
    C = 2
    x = np.random.default_rng(N).integers(-128, 128, (C, T, N, 2)).astype(np.int8)
    with bf.Plan(N, C, B, T, I, precision=prec) as plan:
        plan.set_weights(*_geometry(N, C, B, N + B))
        for overflow in (False, True):
            if overflow:  # an infinite weight reaches its own beam and no other
                w = plan.get_weights()
                w[1, 3, N - 1] = 1e300
                plan.set_weights_raw(w)
            want = run_plan(plan, x, gpu)
            assert np.all(np.isinf(want[1, 3]) | np.isnan(want[1, 3])) == overflow
            tiles = [t for t in plan.tile_candidates() if t[3] in (0, -1)]
            wide = (4, 4, 2, 0) if prec == "fp32" else (4, 4, 4, 0)  # passes of two tiles, of four
            assert {wide, (4, 1, 1, 0), (4, 2, 2, -1)} <= set(tiles)
            default = plan.tile()
            for t in tiles:
                plan.set_tile(*t, 8)
                assert np.array_equal(run_plan(plan, x, gpu), want, equal_nan=True), (t, overflow)
            plan.set_tile(*default)


BATCHES = {
    "odd": [(33, 9, 100, 480), (17, 5, 40, 160), (5, 20, 8, 80)],
    "even": [(34, 9, 100, 480), (36, 5, 20, 160), (2, 20, 70, 80)],
    "mixed": [(33, 3, 16, 240), (34, 11, 130, 320), (100, 4, 33, 160)],
}


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("I", [1, 2, 10, 16])
@pytest.mark.parametrize("name", list(BATCHES))
def test_batch_of_short_rows_equals_solo(gpu, name, I, prec):
    import torch
    print(f"general batch {name} I={I} {prec}", flush=True)
    plans, xs, solo = [], [], []
    for k, (N, C, B, T) in enumerate(BATCHES[name]):
        plan = bf.Plan(N, C, B, T, I, precision=prec)
        geo = _geometry(N, C, B, 7 + k)
        plan.set_weights(*geo)
        x = np.random.default_rng(k).integers(-128, 128, (C, T, N, 2)).astype(np.int8)
        solo.append(run_plan(plan, x, gpu))
        ref = oracle.beamform(oracle.weights(geo[0], geo[1], geo[2][:1]), x[:1], I)
        assert_parity(solo[-1][:1], ref, TOL[prec], f"{name} {k}")
        plans.append(plan)
        xs.append(torch.from_numpy(x).to(gpu))
    batch = bf.Batch(plans)
    outs = [torch.full(p.p_shape, float("nan"), device=gpu) for p in plans]
    for _ in range(2):
        batch.run(xs, outs)
        torch.cuda.synchronize()
        for k, o in enumerate(outs):
            assert np.array_equal(o.cpu().numpy(), solo[k]), (name, k)
            o.fill_(float("nan"))
    batch.destroy()


# one channel a little past 2 GiB; T is a multiple of 2 I
FAR = [
    (32, 70, 33_600_000, 16, 8, "power"), (32, 20, 33_600_000, 10, 8, "power"),
    (64, 33, 16_800_000, 2, 8, "power"), (33, 17, 32_640_000, 16, 8, "power"),
    (256, 20, 4_200_000, 1, 8, "power"), (32, 40, 67_200_000, 16, 4, "power"),
    (40, 5, 27_000_000, 1, 8, "complex"), (40, 24, 54_000_000, 3, 4, "power"),
    (32, 20, 33_600_000, 1, 8, "power"),  # 16 output rows past 2 GiB too: general
]


@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("shape", FAR, ids=lambda s: f"N{s[0]}I{s[3]}b{s[4]}{s[5]}")
def test_channel_past_2gib_equals_two_blocks(gpu, shape, prec):
    import torch
    N, B, T, I, bits, output = shape
    print(f"general far {shape} {prec}", flush=True)
    row = N if bits == 4 else 2 * N
    assert T * row > 2 ** 31 and T % (2 * I) == 0
    g = torch.Generator(device=gpu).manual_seed(N)
    geo = _geometry(N, 1, B, N)
    with bf.Plan(N, 1, B, T, I, precision=prec, input_bits=bits, output=output) as far, \
            bf.Plan(N, 1, B, T // 2, I, precision=prec, input_bits=bits, output=output) as half:
        x = torch.randint(0, 256, (T * row,), generator=g, dtype=torch.uint8, device=gpu)
        x = x.view(far.x_dtype).reshape(far.x_shape)
        for p in (far, half):
            p.set_weights(*geo)
            if output == "complex":
                p.set_output_scale(1 / 64)
        got = torch.empty(far.p_shape, dtype=far.p_dtype, device=gpu)
        far.run(x, got)
        streamed = [t for t in far.tile_candidates() if t[3] == -4]
        assert bool(streamed) == (T // I * 4 * min(B, 16) < 2 ** 31 - 256)
        if streamed:  # work units longer than a wave's offsets reach
            far.set_tile(*streamed[-1], 1 << 20)
            longest = torch.empty_like(got)
            far.run(x, longest)
            assert torch.equal(longest, got)
            del longest
        want = torch.empty(half.p_shape, dtype=half.p_dtype, device=gpu)
        n = half.p_shape[2]
        for k in range(2):
            block = x[:, k * (T // 2):(k + 1) * (T // 2)].clone()
            half.run(block, want)
            assert torch.equal(got[:, :, k * n:(k + 1) * n], want), (shape, prec, k)
            del block


@pytest.mark.parametrize("N,prec", [(1121, "fp16"), (1123, "bf16"), (601, "fp32"), (600, "fp16"),
                                    (552, "bf16")])
def test_large_rows_by_default(gpu, N, prec):
    """Arrays whose default is the general form for its weights' size: byte-load
    rows with the weights in device memory, and two beam tiles in LDS."""
    print(f"general large N={N} {prec}", flush=True)
    C, B, T, I = 64, 128, 96, 16  # at least one unit per CU in each form
    geo = _geometry(N, C, B, N)
    x = np.random.default_rng(N).integers(-128, 128, (C, T, N, 2)).astype(np.int8)
    with bf.Plan(N, C, B, T, I, precision=prec) as plan:
        plan.set_weights(*geo)
        assert plan.tile()[3] == (-1 if N % 8 else 0)
        got = run_plan(plan, x, gpu)
        plan.set_tile(4, 1, 1, 0, 4)
        assert np.array_equal(run_plan(plan, x, gpu), got)
    assert_parity(got, oracle.beamform(oracle.weights(*geo), x, I), TOL[prec], f"N={N}")
