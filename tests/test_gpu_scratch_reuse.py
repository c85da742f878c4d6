"""The steps one by one on a context that another graph used before: what a
smaller graph's call left in the scratch lies where a larger graph's look-back
words are (its sort keys under words 224 and up, read as published prefixes),
so the assemble step has to clear them itself.  1.9 million one-read contigs
take 232 words.  All reads are 16 bases long, so contig k starts at 16 k."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import synth

pytestmark = pytest.mark.gpu


def _isolated(n):
    return synth.StringGraph(
        n=n, m=0, row_ptr=np.zeros(n + 1, np.int32), col=np.zeros(0, np.int32),
        ovl=np.zeros(0, np.uint32), strand=np.zeros(0, np.uint8),
        read_len=np.full(n, 16, np.uint32), read_off=16 * np.arange(n, dtype=np.uint64),
        seq=np.arange(n, dtype=np.uint32))


def _steps(cg, ctx, g, P):
    dg = cg.DeviceGraph(g, "cuda")
    out = cg.Outputs(g.n, P, g.seq_words, "cuda")
    cg.mask_branches(ctx, dg, out.flags, out.counts)
    cg.components(ctx, dg, out.flags, out.label)
    cg.partition(ctx, dg, out.flags, out.label, P, 1, out.parts)
    cg.induce(ctx, dg, out.flags, out.label, out.parts, P, out.local)
    cg.assemble(ctx, dg, out.parts, out.local, P, out.contigs)
    return dg, out


def test_steps_on_a_smaller_graphs_scratch():
    from paper_2207_04350_amd import cg
    n = 1_900_000
    print("scratch reuse", n, flush=True)
    ctx = cg.Context.for_graph(n, 0, 3000)
    for small in (10, 300, 5000):
        _steps(cg, ctx, _isolated(small), 3000)  # its keys are sorted in the scratch
    dg, out = _steps(cg, ctx, _isolated(n), 3)
    torch.cuda.synchronize()
    assert ctx.status() == 0
    ctx.close()
    assert int(out.n_comp.item()) == n and int(out.total_words.item()) == n
    assert torch.equal(out.c_base_off, 16 * torch.arange(n, device="cuda"))
    # contig k is one read's store word
    assert torch.equal(out.bases[:n], out.layout_vid[:n])
