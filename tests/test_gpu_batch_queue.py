"""The batch's pass over its work queue where its split changes: no, one, a few
and many components above a wave's, fewer and more of them than workgroups,
those above one pass's among them, and grids of two workgroups to all that are
resident.  Equal to the oracle, element by element."""
import numpy as np
import pytest
import torch  # noqa: F401  (before the library, so that both use torch's HIP runtime)

import oracle
from tests.parity import mismatches
from tests.test_gpu_components import _graph

pytestmark = pytest.mark.gpu

HEADS = {
    "none": ([2, 64, 65, 128], [3, 64, 65, 128], 40),
    "one": ([2, 31, 32, 33, 129], [4], 7),
    "two": ([63, 512], [511, 30], 20),
    "above one pass": ([513, 1100, 140, 2], [600, 128, 64], 3),
    "rays in scratch": ([4096, 4097], [3000], 5),
    "many": ([130] * 40 + [2] * 50, [131, 128], 9),
    "only": ([200] * 30, [], 0),
}


@pytest.mark.parametrize("persist", [0, 1, 2, 7])
@pytest.mark.parametrize("which", [*([k] for k in sorted(HEADS)), sorted(HEADS)])
def test_split(which, persist):
    from paper_2207_04350_amd import cg
    print("queue", which, persist, flush=True)
    gs = [_graph(np.random.default_rng(60 + len(k)), *HEADS[k]) for k in which]
    ctx = cg.Context(0, 0)
    jobs = [(cg.DeviceGraph(g, "cuda"), cg.Outputs(g.n, 5, g.seq_words, "cuda"), 5, 2) for g in gs]
    b = cg.Batch(ctx, jobs, persist_blocks=persist)
    for _ in range(2):
        b.run()
    got = [cg.to_host(out, g.n) for g, (_, out, _, _) in zip(gs, jobs)]
    assert ctx.status() == 0
    for g, o in zip(gs, got):
        assert mismatches(o, oracle.run(g, P=5, min_reads=2)) == []
