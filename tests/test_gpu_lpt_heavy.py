"""The partition step where one component outweighs all others: bases weights
whose largest is too large for narrow keys by the bound on the loads'
differences, but whose total fits (narrow keys all the same), and totals that
do not fit (wide keys, item by item), around one window of bins and above, in
LDS and in global memory, single graph and batched, equal to the oracle.  The
heavy component may not cost a multiple of the others' time: 7,000 components
took 856 us with it and 213 without.  The loop with keys up to the total is
compared with plain LPT on the CPU."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import oracle
import synth
from tests.parity import mismatches
from tests.test_lpt_loop_cpu import PAD, STEP_BINS, _Loop, _bits, _lpt


def _graph(k, heavy_bases, seed, heavy_reads=60):
    """k components of one to six short reads and one of heavy_bases bases."""
    rng = np.random.default_rng(seed)
    sizes = np.concatenate([[heavy_reads], np.where(rng.random(k) < 0.5, 1, rng.integers(2, 7, k))])
    n = int(sizes.sum())
    ids = rng.permutation(n)
    lens = rng.integers(300, 900, n)
    lens[ids[:heavy_reads]] = heavy_bases // heavy_reads
    last = np.zeros(n, bool)
    last[np.cumsum(sizes) - 1] = True
    at = np.nonzero(~last)[0]
    u, v = ids[at], ids[at + 1]
    bits = rng.integers(0, 2, size=(2, len(u)))
    row_ptr, col, ovl, strand = synth.gen.csr_from_edges(n, u, v, np.full(len(u), 99), bits[0],
                                                         bits[1])
    words = (lens + 15) // 16
    off = np.concatenate([[0], np.cumsum(words)])
    return synth.StringGraph(n=n, m=len(col), row_ptr=row_ptr, col=col, ovl=ovl, strand=strand,
                             read_len=lens.astype(np.uint32),
                             read_off=(16 * off[:-1]).astype(np.uint64),
                             seq=rng.integers(0, 1 << 32, size=int(off[-1]),
                                              dtype=np.uint64).astype(np.uint32))


def test_keys_up_to_the_total():
    rng = np.random.default_rng(3)
    for P in (1, 2, 16, 17, 33, 64):
        top = 1 << (32 - _bits(P))
        for share in (0.4, 0.9, 1.0):
            ws = sorted((int(x) for x in rng.integers(1, 5000, 300)), reverse=True)
            ws = [int(share * (top - 2)) - sum(ws)] + ws
            # past the bound on the differences (64 bins: five times the
            # largest), within the bound on the total
            assert ws[0] * ((64 + P - 1) // P + 4) + 1 >= top and sum(ws) + 1 < top
            got = _Loop(ws, P)  # asserts every raised key below the padding
            got = got.few() if P <= STEP_BINS else got.rounds()
            assert (got.out, got.loads()) == _lpt(ws, P) and max(got.key[:P]) < PAD


@pytest.mark.gpu
@pytest.mark.parametrize("P", [1, 16, 17, 64, 65, 256, 1024, 2049])
@pytest.mark.parametrize("k,heavy", [(63, 2_000_000), (400, 18_000_000), (3000, 18_000_000),
                                     (3000, 60_000_000), (9000, 18_000_000), (300, 300_000_000)])
def test_heavy_component(k, heavy, P):
    from paper_2207_04350_amd import cg
    print("heavy", k, heavy, P, flush=True)
    g = _graph(k, heavy, k)
    ctx = cg.Context.for_graph(g.n, g.m, P)
    out = cg.Outputs(g.n, P, g.seq_words, "cuda")
    cg.run_path(ctx, cg.DeviceGraph(g, "cuda"), out, P, 1, weight="bases")
    assert mismatches(cg.to_host(out, g.n), oracle.run(g, P=P, min_reads=1, weight="bases")) == []
    assert ctx.status() == 0
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("P", [16, 64, 256])
def test_heavy_component_batched(P):
    from paper_2207_04350_amd import cg
    print("heavy batched", P, flush=True)
    gs = [_graph(k, h, k) for k, h in ((63, 2_000_000), (800, 18_000_000), (1500, 18_000_000),
                                       (700, 120_000_000))]
    ctx = cg.Context(0, 0)
    jobs = [(cg.DeviceGraph(g, "cuda"), cg.Outputs(g.n, P, g.seq_words, "cuda"), P, 1, "bases")
            for g in gs]
    b = cg.Batch(ctx, jobs)
    b.run()
    torch.cuda.synchronize()
    for g, j in zip(gs, jobs):
        want = oracle.run(g, P=P, min_reads=1, weight="bases")
        assert mismatches(cg.to_host(j[1], g.n), want) == []
    assert ctx.status() == 0
    b.close()
    ctx.close()


@pytest.mark.gpu
def test_a_heavy_component_costs_no_multiple():
    """Times of the partition step alone (the heavy component's own assembly
    is not part of it)."""
    from paper_2207_04350_amd import cg
    P, us = 64, {}
    for heavy in (60_000, 18_000_000):
        print("heavy time", heavy, flush=True)
        g = _graph(7000, heavy, 5)
        dg, ctx = cg.DeviceGraph(g, "cuda"), cg.Context.for_graph(g.n, g.m, P)
        out, t = cg.Outputs(g.n, P, g.seq_words, "cuda"), []
        cg.run_path(ctx, dg, out, P, 1, weight="bases")
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            cg.partition(ctx, dg, out.flags, out.label, P, 1, out.parts, weight="bases")
            b.record()
            torch.cuda.synchronize()
            t.append(1e3 * a.elapsed_time(b))
        us[heavy] = min(t[1:])
        ctx.close()
    assert us[18_000_000] < 2 * us[60_000], us
