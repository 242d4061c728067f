"""Batches that take the eight-wave persistent launch (bf_host.cpp, wide_sets;
tests/host_choice_check.cpp checks on the CPU that these very sets do): all sets
in it, with a voltage block of their own or a shared one, and together with a
four-wave launch behind it.  In every integration class, accumulating sets
included, each set's output equals its plan's alone, bit for bit, over repeated
launches."""
import numpy as np
import pytest

from paper_1412_4907_amd import bf, synth

pytestmark = pytest.mark.gpu

# (antennas, channels, beams, windows, accumulate); the first two ask for the
# eight-wave form by tile, 520 channels of one beam tile being 520 work units
WIDE = [(136, 520, 16, 32, False), (200, 520, 10, 20, True)]
MIXED = WIDE + [(16, 1030, 16, 32, False), (32, 1030, 30, 6, True)]
SHARED = [(136, 520, 16, 32, False), (136, 520, 40, 32, True), (136, 520, 5, 32, False)]
CASES = {"all": WIDE, "mixed": MIXED, "shared": SHARED}


@pytest.mark.parametrize("prec", ["fp16", "bf16", "fp32"])
@pytest.mark.parametrize("I", [1, 2, 10, 16])
@pytest.mark.parametrize("name", list(CASES))
def test_eight_wave_batch_equals_solo(gpu, name, I, prec):
    import torch
    print(f"wide batch {name} I={I} {prec}", flush=True)
    g = np.random.default_rng(31)
    plans, xs, base, want = [], [], [], []
    for k, (N, C, B, W, acc) in enumerate(CASES[name]):
        plan = bf.Plan(N, C, B, W * I, I, precision=prec, accumulate=acc)
        plan.set_weights(synth.disc_positions(N, 150.0, g), synth.random_dirs(B, g),
                         np.linspace(400e6, 416e6, C))
        if N > 64:
            plan.set_tile(4, 1, 1, -3, 4)
        if name == "shared" and k:
            x = xs[0]
        else:
            x = torch.randint(-128, 128, plan.x_shape, dtype=torch.int8, device=gpu,
                              generator=torch.Generator(device=gpu).manual_seed(k))
        start = torch.ones(plan.p_shape, device=gpu) if acc else \
            torch.full(plan.p_shape, float("nan"), device=gpu)
        out = start.clone()
        plan.run(x, out)
        plans.append(plan)
        xs.append(x)
        base.append(start)
        want.append(out)
    batch = bf.Batch(plans)
    for rep in range(3):
        outs = [b.clone() for b in base]
        batch.run(xs, outs)
        torch.cuda.synchronize()
        for k, (o, w) in enumerate(zip(outs, want)):
            assert torch.equal(o, w), (name, I, prec, rep, k)
    batch.destroy()
