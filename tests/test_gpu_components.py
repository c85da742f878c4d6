"""The induce and assemble steps at the edges of their kernels: components at
the sizes where a lane, a wave, a workgroup, the sort in LDS and the bitmap
windows, the walk in LDS, with rays in LDS and with rays in global memory take
over from one another,
cycles among them (a cycle moves every later row by two), read ids spread
wider than one bitmap window, and many cycles by rank.  Outputs are integers:
equal to the oracle's, element by element."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import oracle
import synth
from tests.parity import mismatches

pytestmark = pytest.mark.gpu


def _graph(rng, chains, cycles=(), isolated=0):
    """Chains and cycles over randomly numbered reads, `isolated` reads
    between them."""
    n = sum(chains) + sum(cycles) + isolated
    ids = rng.permutation(n).astype(np.int64)
    lens = rng.integers(6, 12, size=n)
    u, v, at = [], [], 0
    for q, cyc in [(q, False) for q in chains] + [(q, True) for q in cycles]:
        grp = ids[at:at + q]
        at += q
        u.append(grp[:-1])
        v.append(grp[1:])
        if cyc:
            u.append(grp[-1:])
            v.append(grp[:1])
    u, v = np.concatenate(u), np.concatenate(v)
    bits = rng.integers(0, 2, size=(2, len(u)))
    row_ptr, col, ovl, strand = synth.gen.csr_from_edges(n, u, v, np.full(len(u), 3), bits[0],
                                                         bits[1])
    return synth.StringGraph(n=n, m=len(col), row_ptr=row_ptr, col=col, ovl=ovl, strand=strand,
                             read_len=lens.astype(np.uint32),
                             read_off=16 * np.arange(n, dtype=np.uint64),
                             seq=rng.integers(0, 1 << 32, size=n, dtype=np.uint64).astype(np.uint32))


CASES = {
    "wave edges": ([2, 3, 63, 64, 65, 127, 128, 129, 130], [3, 64, 65, 128, 129], 40),
    "workgroup edges": ([512, 513, 1024, 1025, 3456, 3457], [511, 3000], 100),
    "sort and bitmap": ([16383, 16384, 16385], [16390, 5], 7),
    "rays apart": ([1025, 3455, 3456, 3457], [7000, 514], 30_000),
    "two windows": ([17000, 40, 2], [16500], 300_000),
    "cycles by rank": ([2] * 3000, [3] * 5000 + [4] * 300, 11),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("min_reads", [1, 2])
def test_component_edges(name, min_reads):
    from paper_2207_04350_amd import cg
    print("component case", name, min_reads, flush=True)
    g = _graph(np.random.default_rng(3), *CASES[name])
    P = 5
    ctx = cg.Context.for_graph(g.n, g.m, P)
    dg = cg.DeviceGraph(g, "cuda")
    out = cg.Outputs(g.n, P, g.seq_words, "cuda")
    cg.run_path(ctx, dg, out, P, min_reads)
    got = cg.to_host(out, g.n)
    assert ctx.status() == 0
    ctx.close()
    assert mismatches(got, oracle.run(g, P=P, min_reads=min_reads)) == []


def test_batched_windows_and_rays():
    """Components above the batched sort's LDS, with ids wider than its bitmap
    windows and with more rays than LDS holds."""
    from paper_2207_04350_amd import cg
    g = _graph(np.random.default_rng(4), [4097, 1100, 513, 9], [700], 60_000)
    ctx = cg.Context(0, 0)
    dg = cg.DeviceGraph(g, "cuda")
    out = cg.Outputs(g.n, 3, g.seq_words, "cuda")
    b = cg.Batch(ctx, [(dg, out, 3, 2)])
    b.run()
    got = cg.to_host(out, g.n)
    assert ctx.status() == 0
    b.close()
    ctx.close()
    assert mismatches(got, oracle.run(g, P=3, min_reads=2)) == []
