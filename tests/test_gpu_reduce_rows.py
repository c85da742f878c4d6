"""cg_reduce where its passes change shape: row lengths around one and four
rounds of a wave and around what LDS holds, read counts at which a workgroup
takes more rows, a last block that is not full, and blocks enough for the
sums over 64 of them.  Equal to the oracle's, element by element."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import synth
from tests.test_gpu_reduce import cg, check  # noqa: F401  (cg is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 15, 16, 17, 63, 64, 65, 127, 128, 255, 256, 257])
def test_row_lengths(cg, k):  # noqa: F811
    """A hub with k neighbours in a row, every third of them contained in a
    longer read, among reads without entries."""
    rng = np.random.default_rng(k)
    reads = [rng.integers(0, 4, size=60_000).astype(np.uint8)]
    reads += [rng.integers(0, 4, size=10_000).astype(np.uint8) for _ in range(k)]
    inner = list(range(1, k + 1, 3))
    reads += [rng.integers(0, 4, size=12_000).astype(np.uint8) for _ in inner]
    reads += [rng.integers(0, 4, size=50).astype(np.uint8) for _ in range(k % 7)]
    edges = [(0, i, 9_990 - 5 * i, 0, 0) for i in range(1, k + 1)]
    edges += [(i, i + 1, 9_995, 0, 0) for i in range(1, k)]
    edges += [(k + 1 + j, i, 10_000, int(i % 2), 0) for j, i in enumerate(inner)]
    check(cg, synth.graph_from_edges(reads, edges), name="hub%d" % k)


@pytest.mark.parametrize("n", [4095, 8193, 16389, 32771, 65541, 131_075])
def test_read_counts(cg, n):  # noqa: F811
    g = synth.simulate(G=n * 200, cov=15, mean_len=3_000, sd_len=1_000, err=0.0, extra_rate=0.02,
                       seed=n)
    assert g.n == n
    check(cg, synth.overlap_graph(g), 2, name="n%d" % n)


@pytest.mark.parametrize("cov", [6, 45, 90])
def test_few_contained(cg, cov):  # noqa: F811
    """Reads of about one length: hardly any is contained, so that a read has
    up to cov near neighbours on each side: more than the scratch holds for
    every read, and more than LDS does for a row."""
    g = synth.simulate(G=300_000, cov=cov, mean_len=6_000, sd_len=3, err=0.0, extra_rate=0.05,
                       seed=cov)
    r = synth.overlap_graph(g)
    got, out, dg, s = check(cg, r, 1, name="cov%d" % cov)
    assert got["contained"].mean() < 0.2
