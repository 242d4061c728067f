"""FP32 weights down to the smallest normal one, seen through complex output with a
large scale: the weights are 2^-k (1 + 2^-23) and -2^-k on two antennas with equal
voltages, so a beam is the last bit of the first weight times 64, and any bit that
the three BF16 parts of a weight do not hold would show.  The sums are exact in
FP32 (64 is a power of two), the scaled results in FP16: equality is asked for."""
import numpy as np
import pytest

from paper_1412_4907_amd import bf, synth

pytestmark = pytest.mark.gpu


def _run(plan, x, gpu):
    import torch
    p = torch.empty(plan.p_shape, dtype=torch.float16, device=gpu)
    plan.run(torch.from_numpy(x).to(gpu), p)
    torch.cuda.synchronize()
    return p.cpu().numpy()


@pytest.mark.parametrize("N,tile", [(8, None), (40, None), (40, (4, 1, 1, 0)), (40, (4, 2, 2, -1))])
@pytest.mark.parametrize("k", [60, 100, 110, 111, 114, 118, 122, 126])
def test_last_bit_of_small_weights(gpu, k, N, tile):
    print(f"fp32 range 2^-{k} N={N} {tile}", flush=True)
    C, B, T = 2, 20, 64
    w = np.zeros((C, B, N, 2))
    w[:, :, 1, 0] = 2.0 ** -k * (1 + 2.0 ** -23)
    w[:, :, N - 1, 0] = -2.0 ** -k
    x = np.zeros((C, T, N, 2), np.int8)
    x[:, :, 1, 0] = x[:, :, N - 1, 0] = 64
    scale = min(127, k + 17)
    with bf.Plan(N, C, B, T, 1, precision="fp32", output="complex") as plan:
        plan.set_weights_raw(w)
        plan.set_output_scale(2.0 ** scale)
        if tile:
            plan.set_tile(*tile, 4)
        got = _run(plan, x, gpu)
    assert np.all(got[..., 0] == 2.0 ** (6 + scale - k - 23)) and np.all(got[..., 1] == 0)


def test_scale_past_the_line_changes_no_bit(gpu):
    """Scales on both sides of 2^60 differ by the power of two alone; a plan that
    also holds a weight of 2^90 keeps its other beams."""
    print("fp32 range line", flush=True)
    N, C, B, T = 24, 2, 20, 96
    g = np.random.default_rng(3)
    w = (g.normal(size=(C, B, N)) + 1j * g.normal(size=(C, B, N))) * 2.0 ** -62
    x = g.integers(-128, 128, (C, T, N, 2)).astype(np.int8)
    with bf.Plan(N, C, B, T, 1, precision="fp32", output="complex") as plan:
        plan.set_weights_raw(w)
        plan.set_output_scale(2.0 ** 59)
        low = _run(plan, x, gpu)
        plan.set_output_scale(2.0 ** 60)
        high = _run(plan, x, gpu)
        normal = np.abs(low) >= 2.0 ** -13  # of those, doubling is exact in FP16
        assert np.mean(normal) > 0.95
        assert np.array_equal(high[normal], 2 * low[normal])
        big = w.copy()
        big[0, 4, 2] = 2.0 ** 90
        plan.set_weights_raw(big)
        got = _run(plan, x, gpu)
        rest = np.ones((C, B), bool)
        rest[0, 4] = False
        assert np.array_equal(got[rest], high[rest])
        pos = synth.disc_positions(N, 50.0, g)  # new weights: the line holds again
        plan.set_weights(pos, synth.random_dirs(B, g), np.array([401e6, 402e6]))
        plan.set_weights_raw(w)
        assert np.array_equal(_run(plan, x, gpu), high)
