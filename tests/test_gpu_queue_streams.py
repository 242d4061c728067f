"""Runs of one batch or table on several streams: the caller orders nothing, and
the runs share the handle's queue counters, so each has to follow the last one
on the device.  A set that were handed out twice, or not at all, would show in
the accumulating sums.  And launches captured into a graph: replays alternate
with eager runs, each checked against the plan alone."""
import numpy as np
import pytest

from paper_1412_4907_amd import bf, synth

pytestmark = pytest.mark.gpu
SETS = [(32, 300, 40, 1024), (64, 70, 130, 768), (16, 33, 8, 64)]


def _rows(gpu, sets, prec, accumulate):
    import torch
    g = np.random.default_rng(23)
    rows = []
    for N, C, B, T in sets:
        plans = []
        pos, dirs = synth.disc_positions(N, 100.0, g), synth.random_dirs(B, g)
        for acc in (False, accumulate):
            p = bf.Plan(N, C, B, T, 16, precision=prec, accumulate=acc)
            p.set_weights(pos, dirs, np.linspace(401e6, 409e6, C))
            plans.append(p)
        x = torch.from_numpy(g.integers(-128, 128, (C, T, N, 2)).astype(np.int8)).to(gpu)
        want = torch.empty((C, B, T // 16), device=gpu)
        plans[0].run(x, want)
        rows.append((plans[1], x, want))
    torch.cuda.synchronize()
    return rows


@pytest.mark.parametrize("prec", ["fp16", "fp32"])
def test_batch_runs_on_several_streams(gpu, prec):
    import torch
    print(f"queue streams batch {prec}", flush=True)
    rows = _rows(gpu, SETS, prec, accumulate=True)
    batch = bf.Batch([r[0] for r in rows])
    xs = [r[1] for r in rows]
    streams = [torch.cuda.Stream() for _ in range(3)]
    for rep in range(3):
        outs = [[torch.ones_like(r[2]) for r in rows] for _ in streams]
        torch.cuda.synchronize()
        for s, o in zip(streams, outs):
            batch.run(xs, o, stream=s)
        torch.cuda.synchronize()
        for o in outs:
            for got, r in zip(o, rows):
                assert torch.equal(got, 1.0 + r[2]), (prec, rep)
    batch.destroy()


def test_table_runs_on_several_streams(gpu):
    import torch
    print("queue streams table", flush=True)
    N, T = 32, 1024
    rows = _rows(gpu, [(N, 200, 100, T), (N, 9, 33, T)], "fp16", accumulate=True)
    table = bf.Table(N, 16, "fp16")
    outs = [torch.zeros_like(r[2]) for r in rows]
    table.set([r[0] for r in rows], [r[1] for r in rows], outs)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for s in streams:  # each adds the same sums into the same outputs
        table.run(stream=s)
    torch.cuda.synchronize()
    for o, r in zip(outs, rows):
        assert torch.equal(o, r[2] + r[2] + r[2])
    table.destroy()


def test_captured_batch_replays_between_eager_runs(gpu):
    import torch
    print("queue streams capture", flush=True)
    rows = _rows(gpu, SETS, "fp16", accumulate=False)
    batch = bf.Batch([r[0] for r in rows])
    xs = [r[1] for r in rows]
    outs = [torch.empty_like(r[2]) for r in rows]
    eager = [torch.empty_like(r[2]) for r in rows]
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        batch.run(xs, outs, stream=s)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            batch.run(xs, outs, stream=s)
        for rep in range(4):
            for o in outs + eager:
                o.fill_(float("nan"))
            graph.replay()
            batch.run(xs, eager, stream=s)
            if rep % 2:
                graph.replay()
            torch.cuda.synchronize()
            for o, e, r in zip(outs, eager, rows):
                assert torch.equal(o, r[2]) and torch.equal(e, r[2]), rep
    del graph
    batch.run(xs, eager, stream=s)
    torch.cuda.synchronize()
    batch.destroy()
