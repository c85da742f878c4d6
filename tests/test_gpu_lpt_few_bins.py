"""The partition step for few bins, item by item: bin counts and component
counts at the edges of the loop (bins around kLptStepBins and the 32-lane
sort, items around a turn and a wave, the LDS sort's capacity), read and bases
weights, single graph, steps and batched, equal to the oracle.  And its time
does not run away from that of 64 bins: with every item waiting for a round's
tests, 7,000 one-read components took 1,620 us into one to three bins and 126
into 64."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import oracle
import synth
from tests.parity import mismatches

pytestmark = pytest.mark.gpu


def _graph(k, singles, seed, lo=16, hi=900):
    """k components, a share of them of one read, the others of up to six."""
    rng = np.random.default_rng(seed)
    sizes = np.where(rng.random(k) < singles, 1, rng.integers(2, 7, k))
    n = int(sizes.sum())
    ids = rng.permutation(n)
    lens = rng.integers(lo, hi, n)
    last = np.zeros(n, bool)
    last[np.cumsum(sizes) - 1] = True
    at = np.nonzero(~last)[0]
    u, v = ids[at], ids[at + 1]
    bits = rng.integers(0, 2, size=(2, len(u)))
    row_ptr, col, ovl, strand = synth.gen.csr_from_edges(n, u, v, np.full(len(u), 9), bits[0],
                                                         bits[1])
    words = (lens + 15) // 16
    off = np.concatenate([[0], np.cumsum(words)])
    return synth.StringGraph(n=n, m=len(col), row_ptr=row_ptr, col=col, ovl=ovl, strand=strand,
                             read_len=lens.astype(np.uint32),
                             read_off=(16 * off[:-1]).astype(np.uint64),
                             seq=rng.integers(0, 1 << 32, size=int(off[-1]),
                                              dtype=np.uint64).astype(np.uint32))


@pytest.mark.parametrize("P", [1, 2, 3, 15, 16, 17, 32, 33])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 63, 64, 65, 257, 3000, 8193])
def test_few_bins(P, k):
    from paper_2207_04350_amd import cg
    g = _graph(k, 0.4, k)
    dg = cg.DeviceGraph(g, "cuda")
    ctx = cg.Context.for_graph(g.n, g.m, P)
    for weight in ("reads", "bases"):
        print("few bins", P, k, weight, flush=True)
        out = cg.Outputs(g.n, P, g.seq_words, "cuda")
        cg.run_path(ctx, dg, out, P, 1, weight=weight)
        assert mismatches(cg.to_host(out, g.n), oracle.run(g, P=P, min_reads=1, weight=weight)) == []
    assert ctx.status() == 0
    ctx.close()


def test_few_bins_batched():
    from paper_2207_04350_amd import cg
    gs = [_graph(k, 0.4, k) for k in (1, 9, 64, 257, 1023, 1025, 2500)]
    ctx = cg.Context(0, 0)
    for P in (1, 3, 16, 17):
        print("few bins batched", P, flush=True)
        jobs = [(cg.DeviceGraph(g, "cuda"), cg.Outputs(g.n, P, g.seq_words, "cuda"), P, 1,
                 "bases" if i % 2 else "reads") for i, g in enumerate(gs)]
        b = cg.Batch(ctx, jobs)
        b.run()
        torch.cuda.synchronize()
        for i, g in enumerate(gs):
            want = oracle.run(g, P=P, min_reads=1, weight=jobs[i][4])
            assert mismatches(cg.to_host(jobs[i][1], g.n), want) == [], i
        b.close()
    assert ctx.status() == 0
    ctx.close()


@pytest.mark.parametrize("k", [2000, 7000])
def test_few_bins_take_no_multiple_of_many(k):
    from paper_2207_04350_amd import cg
    g = _graph(k, 1.0, k)
    dg = cg.DeviceGraph(g, "cuda")
    us = {}
    for P in (64, 1, 2, 3):
        print("few bins time", k, P, flush=True)
        ctx = cg.Context.for_graph(g.n, g.m, P)
        out, t = cg.Outputs(g.n, P, g.seq_words, "cuda"), []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            cg.run_path(ctx, dg, out, P, 1)
            b.record()
            torch.cuda.synchronize()
            t.append(1e3 * a.elapsed_time(b))
        us[P] = min(t[1:])
        ctx.close()
    assert max(us[P] for P in (1, 2, 3)) < 4 * us[64], us
