"""Many handles destroyed while their runs are still queued, and as many new ones
of the same sizes made and given other weights at once: every queued run still
reads the memory of its own handle (each output equals the one the run gave
before anything was destroyed)."""
import numpy as np
import pytest

from paper_1412_4907_amd import bf, synth

pytestmark = pytest.mark.gpu
N, C, B, T, I = 16, 4, 20, 256, 4
COUNT = 16


def _weights(plan, seed, stream):
    g = np.random.default_rng(seed)
    plan.set_weights(synth.disc_positions(N, 50.0, g), synth.random_dirs(B, g),
                     np.linspace(401e6, 409e6, C), stream=stream)


def _long_work(torch, gpu, stream):
    """A plan whose 40 runs take about 0.1 s, set up and warmed."""
    n, c, b, t, i = 256, 128, 512, 8192, 64
    plan = bf.Plan(n, c, b, t, i)
    g = np.random.default_rng(2)
    plan.set_weights(synth.disc_positions(n, 50.0, g), synth.random_dirs(b, g),
                     np.linspace(401e6, 409e6, c), stream=stream)
    with torch.cuda.stream(stream):
        x = torch.randint(-128, 128, (c, t, n, 2), dtype=torch.int8, device=gpu)
        p = torch.empty((c, b, t // i), dtype=torch.float32, device=gpu)
    plan.run(x, p, stream=stream)
    stream.synchronize()
    return plan, x, p


@pytest.mark.parametrize("kind", ["plan", "batch", "table"])
def test_queued_runs_outlive_their_handles(gpu, kind):
    import torch
    print(f"lifetime {kind}", flush=True)
    busy, side = torch.cuda.Stream(), torch.cuda.Stream()
    long_plan, lx, lp = _long_work(torch, gpu, busy)
    xs = [torch.from_numpy(np.random.default_rng(k).integers(-128, 128, (C, T, N, 2))
                           .astype(np.int8)).to(gpu) for k in range(COUNT)]
    outs = [torch.empty((C, B, T // I), device=gpu) for _ in range(COUNT)]
    plans = [bf.Plan(N, C, B, T, I, precision="fp16") for _ in range(COUNT)]
    for k, p in enumerate(plans):
        _weights(p, 100 + k, busy)
    batches = [bf.Batch([p]) for p in plans] if kind == "batch" else []
    tables = [bf.Table(N, I, "fp16") for _ in plans] if kind == "table" else []

    def run_all():
        for k, p in enumerate(plans):
            if kind == "batch":
                batches[k].run([xs[k]], [outs[k]], stream=busy)
            elif kind == "table":
                tables[k].set([p], [xs[k]], [outs[k]], stream=busy)
                tables[k].run(stream=busy)
            else:
                p.run(xs[k], outs[k], stream=busy)

    run_all()
    torch.cuda.synchronize()
    want = [o.cpu().numpy() for o in outs]
    for o in outs:
        o.fill_(float("nan"))
    torch.cuda.synchronize()
    for _ in range(40):
        long_plan.run(lx, lp, stream=busy)
    run_all()
    ran = torch.cuda.Event()
    ran.record(busy)
    for h in batches + tables:
        h.destroy()
    if kind != "table":  # a table's launches are not tracked by its plans
        for p in plans:
            p.destroy()
    assert not ran.query(), "a destroy waited for its queued run"
    fresh = [bf.Plan(N, C, B, T, I, precision="fp16") for _ in range(COUNT)]
    handles = []
    for k, p in enumerate(fresh):
        _weights(p, 900 + k, side)
        if kind == "batch":
            handles.append(bf.Batch([p]))
        elif kind == "table":
            handles.append(bf.Table(N, I, "fp16"))
            handles[-1].set([], [], [], stream=side)
    side.synchronize()
    torch.cuda.synchronize()
    for k in range(COUNT):
        assert np.array_equal(outs[k].cpu().numpy(), want[k]), (kind, k)
    for h in handles:
        h.destroy()
