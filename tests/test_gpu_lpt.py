"""The partition step where whole rounds of equal weights are placed at once,
keys are relative to the least load, components are sorted in global memory
and the (bin, label) order is taken over many workgroups: one-read components
around the LDS sort's capacity, a heavy component that keeps one bin out of
the rounds, bin counts around one window and above the LDS lists, both
weights, single graph and batched.  Outputs are integers: equal to the
oracle's, element by element.  The rule for whole rounds is also compared
with plain LPT on the CPU."""
import heapq

import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import oracle
from tests.parity import mismatches
from tests.test_gpu_components import _graph


def _plain(weights, P):
    h = [(0, b) for b in range(P)]
    out = []
    for w in weights:
        load, b = heapq.heappop(h)
        out.append(b)
        heapq.heappush(h, (load + w, b))
    return out


def _rounds(weights, P, least):
    """LPT with whole rounds of equal weights: the m bins below the least
    loaded one's raised key take an item each, J times over, while all of them
    stay below bin m's key."""
    keys, out, i = [(0, b) for b in range(P)], [], 0
    while i < len(weights):
        w = weights[i]
        R = 1
        while i + R < len(weights) and weights[i + R] == w:
            R += 1
        keys.sort()
        m = sum(1 for k in keys if k < (keys[0][0] + w, keys[0][1]))
        J = R // m
        if m < P:
            # keys as whole numbers, as the kernels hold them
            k = [x[0] * P + x[1] for x in keys]
            J = min(J, (k[m] - 1 - k[m - 1]) // (w * P) + 1)
        if J * m < least:
            J, m = 1, 1
        out += [keys[r % m][1] for r in range(J * m)]
        keys = [(k[0] + J * w, k[1]) if r < m else k for r, k in enumerate(keys)]
        i += J * m
    return out


def test_whole_rounds_match_lpt():
    rng = np.random.default_rng(5)
    for trial in range(300):
        P = int(rng.integers(1, 70))
        head = rng.integers(1, [4, 40, 4000][trial % 3], size=rng.integers(0, 60))
        tail = np.full(rng.integers(0, 900), rng.integers(1, 5))
        w = sorted((int(x) for x in np.concatenate([head, tail])), reverse=True)
        assert _rounds(w, P, int(rng.integers(1, 40))) == _plain(w, P), (trial, P)


SHAPES = {
    # (chains, cycles, one-read components)
    "singles in LDS": ([50, 9, 2, 2], [5], 8000),
    "at the LDS sort": ([700], [], 8191),
    "above the LDS sort": ([3, 2], [4], 8192),
    "heavy component": ([9000, 40], [], 20_001),
    "pairs and singles": ([2] * 9000 + [3] * 5, [3] * 4, 30_011),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(SHAPES))
@pytest.mark.parametrize("P", [1, 7, 64, 65, 1000, 2049])
@pytest.mark.parametrize("weight", ["reads", "bases"])
def test_many_equal_components(name, P, weight):
    from paper_2207_04350_amd import cg
    print("lpt case", name, P, weight, flush=True)
    g = _graph(np.random.default_rng(8), *SHAPES[name])
    ctx = cg.Context.for_graph(g.n, g.m, P)
    dg = cg.DeviceGraph(g, "cuda")
    for min_reads in (1, 2):
        out = cg.Outputs(g.n, P, g.seq_words, "cuda")
        cg.run_path(ctx, dg, out, P, min_reads, weight=weight)
        got = cg.to_host(out, g.n)
        assert ctx.status() == 0
        assert mismatches(got, oracle.run(g, P=P, min_reads=min_reads, weight=weight)) == []
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("P", [7, 64, 300])
def test_many_equal_components_batched(P):
    from paper_2207_04350_amd import cg
    names = sorted(SHAPES)
    gs = [_graph(np.random.default_rng(9), *SHAPES[k]) for k in names]
    ctx = cg.Context(0, 0)
    jobs = [(cg.DeviceGraph(g, "cuda"), cg.Outputs(g.n, P, g.seq_words, "cuda"), P, 1,
             "bases" if i % 2 else "reads") for i, g in enumerate(gs)]
    print("lpt batch", P, flush=True)
    b = cg.Batch(ctx, jobs)
    b.run()
    torch.cuda.synchronize()
    assert ctx.status() == 0
    for i, g in enumerate(gs):
        want = oracle.run(g, P=P, min_reads=1, weight=jobs[i][4])
        assert mismatches(cg.to_host(jobs[i][1], g.n), want) == [], names[i]
    b.close()
    ctx.close()


def _sizes(kind, k, rng):
    if kind == "exponential":
        return np.maximum(2, rng.exponential(18, size=k)).astype(int)
    if kind == "uniform":
        return rng.integers(2, 60, size=k)
    if kind == "powers":
        return 2 ** rng.integers(1, 8, size=k)
    return np.concatenate([rng.integers(2, 5, size=k - 3), [3000, 1500, 700]])  # a few large ones


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["exponential", "uniform", "powers", "few large"])
@pytest.mark.parametrize("k", [257, 1100, 5000, 9000])
def test_rounds_over_the_list(kind, k):
    """Hundreds of bins: rounds over the whole list by all threads, and windows
    where they are short, below and above what the LDS sort holds."""
    from paper_2207_04350_amd import cg
    rng = np.random.default_rng(k)
    g = _graph(rng, [int(x) for x in rng.permutation(_sizes(kind, k, rng))], [], 40)
    dg = cg.DeviceGraph(g, "cuda")
    for P in (63, 64, 255, 256, 300, 1024, 2048):
        for weight in ("reads", "bases"):
            print("lpt rounds", kind, k, P, weight, flush=True)
            ctx = cg.Context.for_graph(g.n, g.m, P)
            out = cg.Outputs(g.n, P, g.seq_words, "cuda")
            cg.run_path(ctx, dg, out, P, 2, weight=weight)
            got = cg.to_host(out, g.n)
            assert ctx.status() == 0
            ctx.close()
            assert mismatches(got, oracle.run(g, P=P, min_reads=2, weight=weight)) == []
