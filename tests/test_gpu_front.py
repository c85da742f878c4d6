"""The first half of the path in one workgroup, at the read counts where it
takes another round, another read per thread and gives way to the passes over
the chip: equal to the oracle, element by element, and to the steps one by one,
for every least size, both weights, chains in random and in ascending order,
branch reads among them, and graphs without an entry."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import synth
from tests.test_gpu_components import _graph
from tests.test_gpu_path import _check, _Ordered

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 1023, 1024, 1025, 4095, 4096, 4097, 7168, 7169, 12287, 12288,
                               12289])
@pytest.mark.parametrize("weight", ["reads", "bases"])
def test_read_counts(n, weight):
    rng = np.random.default_rng(n)
    chains = [] if n == 2 else [n // 4, 2, 3, 130, 17] + [2] * (n // 50)
    cycles = [] if n == 2 else [3, n // 8]
    g = _graph(rng, chains or [2], cycles, n - sum(chains or [2]) - sum(cycles))
    assert g.n == n
    for min_reads in (1, 2, 4):
        _check(g, 13, min_reads, weight)


@pytest.mark.parametrize("step", [1, -1])
def test_ordered(step):
    _check(_graph(_Ordered(np.random.default_rng(1), step), [5000, 7, 2], [4000], 11), 3, 2)


@pytest.mark.parametrize("extra", [0.0, 0.02, 0.5])
def test_branches(extra):
    g = synth.simulate(G=4_000_000, cov=20, mean_len=8_000, sd_len=2_500, err=0.0,
                       extra_rate=extra, seed=5)
    for min_reads, weight in ((1, "bases"), (2, "reads"), (3, "bases")):
        _check(g, 33, min_reads, weight)


def test_no_entries():
    g = synth.simulate(G=3_000_000, cov=0.5, mean_len=2_000, sd_len=10, err=0.0, extra_rate=0.0,
                       seed=6)
    for min_reads in (1, 2):
        _check(g, 4, min_reads)
