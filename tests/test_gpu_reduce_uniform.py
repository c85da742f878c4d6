"""cg_reduce on reads of about one length, of which hardly any is contained in
another: rows of 129 to 256 neighbours that stay (and some above), fewer, and
both in one graph.  Equal to the oracle's, element by element; and rows of 150
neighbours do not cost a multiple of what their pairs do (read in place, one
neighbour at a time, they took twice as long as with room in LDS)."""
import numpy as np
import pytest
import torch  # before the library, so that both use torch's HIP runtime

import synth
from tests.test_gpu_reduce import cg, check  # noqa: F401  (cg is a fixture)

pytestmark = pytest.mark.gpu


def _overlaps(G, cov, mean, sd, seed, runs=()):
    """The overlap graph of cov times G bases of reads of mean +- sd bases;
    runs: (start, bases, cov) of further reads there."""
    rng = np.random.default_rng(seed)
    parts = [(0, G, cov)] + list(runs)
    n = [int(round(g * c / mean)) for _, g, c in parts]
    ln = np.maximum(1200, np.rint(rng.normal(mean, sd, sum(n)))).astype(np.int64)
    a = np.concatenate([s + rng.integers(0, g - mean // 2, k) for (s, g, _), k in zip(parts, n)])
    a = np.minimum(a, G - ln)
    rc = rng.integers(0, 2, len(a))
    ids = rng.permutation(len(a))
    order = np.lexsort((ids, -(a + ln), a))
    A, B = a[order], (a + ln)[order]
    us, vs, os_ = [], [], []
    for k in range(1, len(a)):
        ov = np.minimum(B[:-k], B[k:]) - A[k:]
        if not (A[k:] + 1000 <= B[:-k]).any():
            break
        i = np.nonzero((A[k:] + 1000 <= B[:-k]) & (ov >= 1000))[0]
        us.append(order[i])
        vs.append(order[i + k])
        os_.append(ov[i])
    u, v, o = (np.concatenate(x) for x in (us, vs, os_))
    s, d = rc[u], rc[v]
    N = len(a)
    rl = np.empty(N, np.uint32)
    rl[ids] = ln
    row_ptr, col, ovl, strand = synth.gen.csr_from_edges(N, ids[u], ids[v], o, s, d)
    return synth.StringGraph(n=N, m=len(col), row_ptr=row_ptr, col=col, ovl=ovl, strand=strand,
                             read_len=rl, read_off=np.zeros(N, np.uint64),
                             seq=np.zeros(1, np.uint32))


CASES = {
    # reads of one length have about 2 cov (1 - 1000 / mean) neighbours; with few
    # enough entries a read they are not gathered at all
    "short rows": (900_000, 12, 6000, 3, ()),
    "short rows, some contained": (900_000, 12, 6000, 300, ()),
    "rows below 128": (200_000, 55, 6000, 3, ()),
    "rows around 128": (200_000, 75, 6000, 3, ()),
    "rows around 256": (200_000, 150, 6000, 3, ()),
    "spread lengths": (200_000, 120, 6000, 300, ()),
    # mostly short rows, long ones where a repeat gathers reads
    "a few long rows": (4_000_000, 9, 6000, 3, ((300_000, 7_000, 120), (900_000, 7_000, 240))),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("fuzz", [0, 4])
def test_one_length(cg, name, fuzz):  # noqa: F811
    r = _overlaps(*CASES[name][:4], seed=3, runs=CASES[name][4])
    got = check(cg, r, fuzz, name=name)[0]
    left = np.flatnonzero(got["contained"] == 0)
    rows = np.diff(r.row_ptr)[left]
    assert len(left) > 0.5 * r.n or name == "spread lengths"
    if "short" in name or "a few" in name:
        assert r.m < 40 * r.n
    if "long" in name or "128" in name:
        assert rows.min() < 128 < rows.max()
    if "long" in name or "256" in name:
        assert rows.max() > 256


def test_longer_rows_cost_their_pairs(cg):  # noqa: F811
    us, pairs = {}, {}
    for cov in (60, 80):
        r = _overlaps(1_000_000, cov, 12_000, 3, seed=4)
        print("reduce time", cov, r.n, r.m, flush=True)
        ctx, dg, out = cg.Context.for_graph(r.n, r.m, 1), cg.DeviceGraph(r), cg.Reduced(r.n, r.m)
        t = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            cg.reduce(ctx, dg, out)
            b.record()
            torch.cuda.synchronize()
            t.append(1e3 * a.elapsed_time(b))
        ctx.close()
        deg = np.diff(r.row_ptr).astype(np.float64)
        us[cov], pairs[cov] = min(t[1:]), float((deg[r.col]).sum())
    assert us[80] / us[60] < 1.5 * pairs[80] / pairs[60], (us, pairs)


@pytest.mark.parametrize("cov", [160, 200, 330])
def test_rows_of_a_wave(cg, cov):  # noqa: F811
    """Entries per read around those from which the containment pass gives a
    row a whole wave, most reads contained."""
    r = _overlaps(60_000, cov, 3000, 900, seed=cov)
    got = check(cg, r, 2, name="cov%d" % cov)[0]
    assert (r.m >= 256 * r.n) == (cov >= 200) and got["contained"].mean() > 0.5


def _near(r, contained):
    """Near neighbours of every read that stays: those that stay too."""
    u = np.repeat(np.arange(r.n), np.diff(r.row_ptr))
    return np.bincount(u, weights=1 - contained[r.col], minlength=r.n)[contained == 0]


@pytest.mark.parametrize("cov, sd, runs, wide", [
    (90, 30, (), True), (100, 60, (), True), (90, 150, (), False), (130, 120, (), False),
    # few near neighbours but for a repeat's, above 128, which are read in place
    (62, 40, ((60_000, 9_000, 90),), False),
])
def test_wide_rows_by_near_neighbours(cg, cov, sd, runs, wide):  # noqa: F811
    """From 96 entries a read on, both sides of the 96 near neighbours a row that
    give a row room for 256 of them."""
    r = _overlaps(200_000, cov, 6000, sd, seed=cov + sd, runs=runs)
    got = check(cg, r, 3, name="cov%d sd%d" % (cov, sd))[0]
    near = _near(r, got["contained"])
    assert 96 * r.n <= r.m < 256 * r.n
    assert (near.mean() > 96 / 0.93 if wide else near.mean() < 96 * 0.93), near.mean()
    assert not runs or (near > 128).any()
