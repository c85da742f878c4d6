"""Offsets and copy of a small graph where the launch changes: no contig, one, a
thread's and a workgroup's worth and one more, as many as one launch takes and
one more, as many reads as it takes and one more; a buffer of the exact size
and one word less.  Equal to the oracle, element by element."""
import numpy as np
import pytest
import torch  # noqa: F401  (before the library, so that both use torch's HIP runtime)

import oracle
from tests.parity import mismatches
from tests.test_gpu_components import _graph

pytestmark = pytest.mark.gpu

# chains, cycles, single reads, min_reads
CASES = {
    "none": ([2], [], 40, 3),
    "one": ([3], [], 0, 2),
    "one read": ([2], [], 1, 1),
    "a thread's": ([2] * 256, [3], 0, 2),
    "two a thread": ([2] * 511, [3] * 2, 0, 2),
    "most contigs": ([2], [], 8190, 1),
    "a contig more": ([2], [], 8192, 1),
    "most reads": ([2] * 8000, [384], 0, 2),
    "a read more": ([2] * 8000, [385], 0, 2),
    "one long": ([9000], [], 0, 2),
}


def _run(cg, g, min_reads, words):
    ctx = cg.Context.for_graph(g.n, g.m, 6)
    dg = cg.DeviceGraph(g, "cuda")
    out = cg.Outputs(g.n, 6, words, "cuda")
    status = []
    for _ in range(2):
        cg.run_path(ctx, dg, out, 6, min_reads)
        status.append(ctx.status())
    got = cg.to_host(out, g.n) if status[-1] == 0 else None
    ctx.close()
    return got, status


@pytest.mark.parametrize("name", sorted(CASES))
def test_edges(name):
    from paper_2207_04350_amd import cg
    print("small copy", name, flush=True)
    g = _graph(np.random.default_rng(31), *CASES[name][:3])
    got, status = _run(cg, g, CASES[name][3], g.seq_words)
    assert status[-1] == 0
    want = oracle.run(g, P=6, min_reads=CASES[name][3])
    assert mismatches(got, want) == []


@pytest.mark.parametrize("name", ["one", "two a thread", "a contig more"])
def test_buffer(name):
    from paper_2207_04350_amd import cg
    print("small copy buffer", name, flush=True)
    g = _graph(np.random.default_rng(32), *CASES[name][:3])
    want = oracle.run(g, P=6, min_reads=CASES[name][3])
    words = int(want["contigs"]["total_words"])
    got, status = _run(cg, g, CASES[name][3], words)
    assert status[-1] == 0 and mismatches(got, want) == []
    _, status = _run(cg, g, CASES[name][3], words - 1)
    assert status == [cg.STATUS_BASES_OVERFLOW] * 2
