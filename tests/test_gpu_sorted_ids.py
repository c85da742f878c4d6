"""Reads numbered along the genome: every kept neighbour is the read before or
after.  Chains and cycles in that order, in runs of it and shuffled are equal
to the oracle in the whole path, the allocation-free call and the steps one by
one, and a step takes no more than a small multiple of its time on a shuffled
chain.  (The walk went through such a chain one read at a time, 65 ms for
12,000 reads where a shuffled one took 0.4; the small graph's climbs took 3.9
ms where a shuffled chain took 0.05, and a sorted cycle's last read climbed all
of it alone, 7.7 ms for 30,000 reads.)"""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import oracle
import synth
from tests.parity import mismatches

pytestmark = pytest.mark.gpu


def _chains(sizes, order, cycles, seed=5):
    """Chains (or cycles) of reads 64 bases long; ids along them, in runs of
    50 along them, or shuffled."""
    rng = np.random.default_rng(seed)
    n = int(sum(sizes))
    ids = np.arange(n)
    if order == "runs":
        blocks = [ids[i:i + 50] for i in range(0, n, 50)]
        ids = np.concatenate([blocks[i] for i in rng.permutation(len(blocks))])
    elif order == "shuffled":
        ids = rng.permutation(n)
    ends = np.cumsum(sizes)
    inner = np.ones(n, bool)
    inner[ends - 1] = False
    u = np.nonzero(inner)[0]
    v = u + 1
    if cycles:
        u, v = np.concatenate([u, ends - 1]), np.concatenate([v, ends - np.asarray(sizes)])
    u, v = ids[u], ids[v]
    bits = rng.integers(0, 2, size=(2, len(u)))
    row_ptr, col, ovl, strand = synth.gen.csr_from_edges(n, u, v, np.full(len(u), 20), bits[0],
                                                         bits[1])
    return synth.StringGraph(n=n, m=len(col), row_ptr=row_ptr, col=col, ovl=ovl, strand=strand,
                             read_len=np.full(n, 64, np.uint32),
                             read_off=64 * np.arange(n, dtype=np.uint64),
                             seq=rng.integers(0, 1 << 32, size=4 * n,
                                              dtype=np.uint64).astype(np.uint32))


def _steps(cg, ctx, dg, out, P):
    cg.mask_branches(ctx, dg, out.flags, out.counts)
    cg.components(ctx, dg, out.flags, out.label)
    cg.partition(ctx, dg, out.flags, out.label, P, 2, out.parts)
    cg.induce(ctx, dg, out.flags, out.label, out.parts, P, out.local)
    cg.assemble(ctx, dg, out.parts, out.local, P, out.contigs)


@pytest.mark.parametrize("order", ["sorted", "runs", "shuffled"])
@pytest.mark.parametrize("cycles", [False, True])
@pytest.mark.parametrize("sizes", [[2000], [12288], [13000], [700] * 30, [5] * 3000],
                         ids=lambda s: "%dx%d" % (len(s), s[0]))
def test_orders_match_the_oracle(sizes, cycles, order):
    from paper_2207_04350_amd import cg
    print("order", sizes[0], cycles, order, flush=True)
    g, P = _chains(sizes, order, cycles), 7
    want = oracle.run(g, P=P, min_reads=2)
    ctx = cg.Context.for_graph(g.n, g.m, P)
    dg = cg.DeviceGraph(g, "cuda")
    for run in (lambda o: cg.run_path(ctx, dg, o, P), lambda o: _steps(cg, ctx, dg, o, P),
                lambda o: cg.contig_generation_noalloc(dg, o, P)):
        out = cg.Outputs(g.n, P, g.seq_words, "cuda")
        run(out)
        assert mismatches(cg.to_host(out, g.n), want) == []
    assert ctx.status() == 0
    ctx.close()


def _us(run):
    t = []
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        run()
        b.record()
        torch.cuda.synchronize()
        t.append(1e3 * a.elapsed_time(b))
    return min(t[1:])


@pytest.mark.parametrize("n", [12000, 30000])
@pytest.mark.parametrize("call", ["components", "assemble", "path"])
@pytest.mark.parametrize("cycle", [False, True])
def test_a_sorted_chain_takes_no_chain_of_steps(n, call, cycle):
    from paper_2207_04350_amd import cg
    P, us = 8, {}
    for order in ("shuffled", "sorted"):
        print("order time", n, call, cycle, order, flush=True)
        g = _chains([n], order, cycle)
        ctx = cg.Context.for_graph(g.n, g.m, P)
        dg, out = cg.DeviceGraph(g, "cuda"), cg.Outputs(g.n, P, g.seq_words, "cuda")
        _steps(cg, ctx, dg, out, P)
        us[order] = _us({
            "components": lambda: cg.components(ctx, dg, out.flags, out.label),
            "path": lambda: cg.run_path(ctx, dg, out, P),
            "assemble": lambda: cg.assemble(ctx, dg, out.parts, out.local, P, out.contigs),
        }[call])
        ctx.close()
    assert us["sorted"] < 8 * us["shuffled"], us
