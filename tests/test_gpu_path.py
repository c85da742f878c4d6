"""The five steps in one call, in one call without a context, and one by one:
the same outputs as the oracle's, element by element, around the chunk sizes
of the count and compaction (2,048 reads; more rounds per chunk above 2^21
reads), for least sizes that the flags decide and that the counts decide, on
chains whose reads are in random, ascending and descending order (the forest
the unions start from), and again on the same buffers after another graph."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import oracle
from tests.parity import mismatches
from tests.test_gpu_components import _graph

pytestmark = pytest.mark.gpu

CASES = {
    "one read": ([], [], 1),
    "two reads": ([2], [], 0),
    "2047": ([40, 3, 2], [5, 3], 1994),
    "2048": ([500, 2], [3], 1543),
    "2049": ([2] * 1000, [], 49),
    "6145": ([3, 9, 700, 2], [2000], 3431),
    "rounds": ([5000, 17, 2, 2], [3, 40], 2_100_000),
}


class _Ordered:
    """Read ids in order along the components instead of at random."""

    def __init__(self, rng, step):
        self.rng, self.step = rng, step

    def permutation(self, n):
        return np.arange(n)[::self.step]

    def __getattr__(self, name):
        return getattr(self.rng, name)


def _steps(cg, ctx, dg, out, P, min_reads, weight):
    cg.mask_branches(ctx, dg, out.flags, out.counts)
    cg.components(ctx, dg, out.flags, out.label)
    cg.partition(ctx, dg, out.flags, out.label, P, min_reads, out.parts, weight=weight)
    cg.induce(ctx, dg, out.flags, out.label, out.parts, P, out.local)
    cg.assemble(ctx, dg, out.parts, out.local, P, out.contigs)


def _check(g, P, min_reads, weight="reads"):
    from paper_2207_04350_amd import cg
    want = oracle.run(g, P=P, min_reads=min_reads, weight=weight)
    dg = cg.DeviceGraph(g, "cuda")
    ctx = cg.Context.for_graph(g.n, g.m, P)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ways = {
        "path": lambda o: cg.run_path(ctx, dg, o, P, min_reads, weight=weight),
        "path again": lambda o: cg.run_path(ctx, dg, o, P, min_reads, weight=weight),
        "steps": lambda o: _steps(cg, ctx, dg, o, P, min_reads, weight),
    }
    if g.n < 400_000:
        ways["noalloc"] = lambda o: cg.contig_generation_noalloc(dg, o, P, min_reads,
                                                                 weight=weight, d_status=status)
    for name, run in ways.items():
        print("path case", g.n, P, min_reads, name, flush=True)
        out = cg.Outputs(g.n, P, g.seq_words, "cuda")
        run(out)
        got = cg.to_host(out, g.n)
        assert ctx.status() == 0 and int(status.item()) == 0
        assert mismatches(got, want) == [], name
    ctx.close()


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("min_reads", [1, 2, 3, 6])
def test_calls_agree(name, min_reads):
    _check(_graph(np.random.default_rng(2), *CASES[name]) if name != "one read" else _single(),
           7, min_reads, "bases" if min_reads == 3 else "reads")


def _single():
    g = _graph(np.random.default_rng(2), [2], [], 0)
    g.n, g.m = 1, 0
    g.row_ptr = np.zeros(2, dtype=np.int32)
    g.col, g.ovl, g.strand = g.col[:0], g.ovl[:0], g.strand[:0]
    g.read_len, g.read_off = g.read_len[:1], g.read_off[:1]
    return g


@pytest.mark.parametrize("step", [1, -1])
def test_ordered_chains(step):
    rng = _Ordered(np.random.default_rng(6), step)
    _check(_graph(rng, [3000, 2, 65, 129], [700, 3], 100), 5, 2)
