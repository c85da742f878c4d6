"""Jobs of a batch above the batched form's sizes, which run beside the batched
launches on streams of the batch's own: more of them than streams, alone and
among others, eager, planned anew and as captured replays with the program's
own work between them, per-kernel timing on, and a job whose bases overflow
their buffer.  Equal to the oracle, element by element."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import oracle
from tests.parity import mismatches
from tests.test_gpu_components import _graph

pytestmark = pytest.mark.gpu

LARGE = [([17_000, 40, 2], [3], 50), ([2] * 17_000, [], 9), ([9_000] * 2, [700], 11),
         ([130] * 140, [], 0), ([3] * 6_000, [5] * 900, 7)]
SMALL = [([40, 3, 2], [5], 30), ([2] * 50, [], 400)]


@pytest.fixture(scope="module")
def graphs():
    gs = [_graph(np.random.default_rng(20 + i), *c) for i, c in enumerate(LARGE + SMALL)]
    assert all(g.m > 32768 for g in gs[:len(LARGE)])
    return [(g, {P: oracle.run(g, P=P, min_reads=2) for P in (5,)}) for g in gs]


def _jobs(cg, graphs, which):
    return [(cg.DeviceGraph(graphs[i][0], "cuda"),
             cg.Outputs(graphs[i][0].n, 5, graphs[i][0].seq_words, "cuda"), 5, 2) for i in which]


def _same(cg, graphs, which, jobs):
    for i, (dg, out, P, _) in zip(which, jobs):
        g, want = graphs[i]
        assert mismatches(cg.to_host(out, g.n), want[P]) == [], i


def _clear(jobs):
    for _, out, _, _ in jobs:
        for t in vars(out).values():
            if isinstance(t, torch.Tensor):
                t.zero_()


@pytest.mark.parametrize("which", [[0], [0, 1], [5, 2, 6], [0, 1, 2, 3, 4, 5, 6]])
def test_eager_and_replayed(graphs, which):
    from paper_2207_04350_amd import cg
    print("external jobs", which, flush=True)
    ctx = cg.Context(0, 0)
    jobs = _jobs(cg, graphs, which)
    b = cg.Batch(ctx, jobs)
    for _ in range(2):
        _clear(jobs)
        b.run()
        _same(cg, graphs, which, jobs)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    b.capture(side)
    for _ in range(3):
        _clear(jobs)
        side.wait_stream(torch.cuda.current_stream())
        b.launch(side)
        torch.cuda.current_stream().wait_stream(side)
        _same(cg, graphs, which, jobs)
    ctx.profile(200)
    _clear(jobs)
    b.run()
    _same(cg, graphs, which, jobs)
    assert ctx.status() == 0
    b.close()
    ctx.close()


def test_planned_anew(graphs):
    from paper_2207_04350_amd import cg
    ctx = cg.Context(0, 0)
    sizes = [(g.n, g.m, 5) for g, _ in graphs]
    lane = cg.Batch.empty(ctx, cg.batch_bytes(sizes))
    for which in ([5, 6], [0, 1, 2, 3, 4, 5, 6], [3], [6, 4]):
        print("planned", which, flush=True)
        jobs = _jobs(cg, graphs, which)
        lane.plan(jobs)
        lane.run()
        _same(cg, graphs, which, jobs)
    assert ctx.status() == 0
    lane.close()
    ctx.close()


def test_overflow_reported(graphs):
    from paper_2207_04350_amd import cg
    ctx = cg.Context(0, 0)
    g = graphs[1][0]
    jobs = [(cg.DeviceGraph(g, "cuda"), cg.Outputs(g.n, 5, 4, "cuda"), 5, 2)] + _jobs(cg, graphs, [0, 5])
    b = cg.Batch(ctx, jobs)
    b.run()
    torch.cuda.synchronize()
    assert ctx.status() & 1  # CG_STATUS_BASES_OVERFLOW
    _same(cg, graphs, [0, 5], jobs[1:])
    b.close()
    ctx.close()
