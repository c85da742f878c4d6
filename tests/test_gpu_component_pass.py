"""The whole path's component pass where it changes form: a lane, a wave of one
and of two reads a lane, a workgroup in LDS, and above by a bitmap with the
neighbours and the rays in LDS, the rays only, and neither, and without a
bitmap (more ids than it has bits for); paths and cycles of each, as the last
component by rank and before others, with explicit coordinates too.  Equal to
the oracle, element by element."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import oracle
import synth
from tests.parity import mismatches
from tests.test_gpu_components import _graph

pytestmark = pytest.mark.gpu

CASES = {
    "waves": ([2, 63, 64, 65, 127, 128], [3, 64, 65, 128], 9),
    "workgroups": ([129, 511, 512, 513], [129, 512, 513], 9),
    "neighbours apart": ([3711, 3712, 3713, 3714], [3712], 20),
    "rays apart": ([7423, 7424, 7425], [7424], 20),
    "one long path": ([40_000], [], 0),
    "one long cycle": ([], [33_000], 0),
    "ranks above 16 bits": ([65_535, 65_536], [], 3),
    "last id of the bitmap": ([600, 2], [700], 316_769 - 1302),
    "no bitmap": ([600, 2, 8193], [700, 5000], 320_000),
    "many large": ([130] * 700, [131] * 30, 5),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("min_reads", [1, 2])
def test_forms(name, min_reads):
    from paper_2207_04350_amd import cg
    print("component pass case", name, min_reads, flush=True)
    g = _graph(np.random.default_rng(11), *CASES[name])
    ctx = cg.Context.for_graph(g.n, g.m, 6)
    dg = cg.DeviceGraph(g, "cuda")
    out = cg.Outputs(g.n, 6, g.seq_words, "cuda")
    for _ in range(2):
        cg.run_path(ctx, dg, out, 6, min_reads)
    got = cg.to_host(out, g.n)
    assert ctx.status() == 0
    ctx.close()
    assert mismatches(got, oracle.run(g, P=6, min_reads=min_reads)) == []


@pytest.mark.parametrize("extra", [0.0, 0.0005, 0.02])
def test_coordinates(extra):
    from paper_2207_04350_amd import cg
    g = synth.simulate(G=2_000_000, cov=25, mean_len=6_000, sd_len=2_000, err=0.0,
                       extra_rate=extra, seed=77)
    g = synth.with_alignment_ends(g, np.random.default_rng(78), 150)
    print("component pass coordinates", extra, flush=True)
    ctx = cg.Context.for_graph(g.n, g.m, 9)
    dg = cg.DeviceGraph(g, "cuda")
    out = cg.Outputs(g.n, 9, g.seq_words, "cuda")
    cg.run_path(ctx, dg, out, 9, 2)
    got = cg.to_host(out, g.n)
    assert ctx.status() == 0
    ctx.close()
    assert mismatches(got, oracle.run(g, P=9, min_reads=2)) == []
