"""The persistent launches' device queues: every launch leaves its counters
cleared for the next, whatever the launch held -- fewer units than workgroups
or XCDs, an empty table between full ones, a batch whose sets differ by orders
of magnitude -- eagerly, back to back, and replayed from a captured graph."""
import numpy as np
import pytest

from paper_1412_4907_amd import bf, synth

pytestmark = pytest.mark.gpu


def _plans(gpu, shapes, prec, I):
    import torch
    g = np.random.default_rng(17)
    out = []
    for N, C, B, T in shapes:
        plan = bf.Plan(N, C, B, T, I, precision=prec)
        plan.set_weights(synth.disc_positions(N, 100.0, g), synth.random_dirs(B, g),
                         np.linspace(401e6, 409e6, C))
        x = torch.from_numpy(g.integers(-128, 128, (C, T, N, 2)).astype(np.int8)).to(gpu)
        p = torch.empty((C, B, T // I), device=gpu)
        plan.run(x, p)
        out.append((plan, x, p))
    return out


SETS = [
    [(32, 1, 4, 64)],                                        # one unit, one XCD
    [(256, 9, 40, 512), (16, 3, 4, 16), (64, 70, 130, 768)],  # more XCD queues than channels
    [(16, 300, 8, 64), (128, 2, 300, 1600)],                 # many short units, a few long
]


@pytest.mark.parametrize("prec", ["fp16", "fp32"])
@pytest.mark.parametrize("sets", SETS, ids=["one", "mixed", "uneven"])
def test_batch_repeats_equal_solo(gpu, sets, prec):
    import torch
    print(f"queue batch {sets} {prec}", flush=True)
    rows = _plans(gpu, sets, prec, 16)
    batch = bf.Batch([r[0] for r in rows])
    outs = [torch.empty_like(r[2]) for r in rows]
    for rep in range(4):
        for o in outs:
            o.fill_(float("nan"))
        batch.run([r[1] for r in rows], outs)
        batch.run([r[1] for r in rows], outs)
        for o, r in zip(outs, rows):
            assert torch.equal(o, r[2]), (sets, prec, rep)
    batch.destroy()


def test_table_replays_over_empty_and_uneven_tables(gpu):
    import torch
    print("queue table", flush=True)
    rows = _plans(gpu, [(32, 5, 100, 256), (32, 130, 8, 64), (32, 1, 16, 4096)], "fp16", 16)
    outs = [torch.empty_like(r[2]) for r in rows]
    table = bf.Table(32, 16, "fp16")
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        table.set([], [], [], stream=s)
        table.run(stream=s)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            table.run(stream=s)
        for ids in ([0, 1, 2], [], [2], [1, 0], [0], [2, 1]):
            for o in outs:
                o.fill_(float("nan"))
            table.set([rows[i][0] for i in ids], [rows[i][1] for i in ids],
                      [outs[i] for i in ids], stream=s)
            graph.replay()
            table.run(stream=s)
            torch.cuda.synchronize()
            for i, o in enumerate(outs):
                if i in ids:
                    assert torch.equal(o, rows[i][2]), ids
                else:
                    assert bool(torch.isnan(o).all()), ids
    table.destroy()
