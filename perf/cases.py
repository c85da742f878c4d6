"""The work users have this library do, as measurable cases.

A case is a dict of plain sizes and options; `prepare` makes what a user's
program holds in device memory before the call (graphs, contexts, output
buffers, planned batches), `run` is one pass through the public entry points
of `paper_2207_04350_amd.cg`, `work` the bytes that pass cannot do without.

Graphs are simulated on the device with the recipe of the repository's
workloads: long reads sampled from a random genome, contained reads without
edges, consecutive remaining reads linked when they overlap by at least 1000
bases, a share of extra overlaps that make branch vertices, vertex ids in file
order.  Every output is a whole number or packed bases, so there is no value
in 64-bit floating point to compare with (`exact` gives none).
"""
from __future__ import annotations

import math
import random

import torch

from paper_2207_04350_amd import cg

MIN_OVERLAP = 1000
MAX_LEN_BITS = 20          # read lengths stay far below 2^20 bases
WORD_CHUNK = 1 << 27       # store words packed at a time


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _path(name, mb, cov, mean, extra, P, min_reads=2, weight="reads", coords=False, kind="path"):
    return dict(name=name, kind=kind, mb=mb, cov=cov, mean=mean, extra=extra, P=P,
                min_reads=min_reads, weight=weight, coords=coords)


def listed():
    return [
        # one bacterial-size graph through the five calls: latency and launches
        _path("path 1 Mbp", 1.0, 10, 10_000, 0.01, 8),
        # one mid-size genome, the single-graph workload of the benchmark
        _path("path 50 Mbp", 50.0, 30, 12_000, 0.02, 64),
        # one GPU's share of a large genome, the largest single graph
        _path("path 1 Gbp", 1000.0, 20, 15_000, 0.01, 1024),
        # every read wanted in a contig, unassembled ones included
        _path("path 50 Mbp all reads", 50.0, 30, 12_000, 0.02, 64, min_reads=1),
        # a clean genome: few branch reads, contigs of hundreds to thousands of reads
        _path("path 50 Mbp long contigs", 50.0, 30, 12_000, 0.0004, 64),
        # without a context or allocation: aligner coordinates per overlap,
        # bins balanced by bases, a bin count that is no power of two
        _path("noalloc 17 Mbp coords", 17.3, 23, 9_000, 0.015, 100, weight="bases", coords=True,
              kind="noalloc"),
        # a few small graphs as one captured launch
        dict(name="batch 8 small", kind="batch", graphs=8, mb_lo=0.2, mb_hi=2.0, cov_lo=10,
             cov_hi=40, mean=10_000, extra=0.015, P=64),
        # the headline batch: 512 independent graphs of 0.2-20 Mbp
        dict(name="batch 512", kind="batch", graphs=512, mb_lo=0.2, mb_hi=20.0, cov_lo=10,
             cov_hi=40, mean=10_000, extra=0.0175, P=64),
        # one wave of a serving loop: resident request graphs planned into a
        # lane's batch memory, run, counted and packed for the download
        dict(name="serving wave 16", kind="wave", graphs=16, mb_lo=1.0, mb_hi=100.0, cov_lo=15,
             cov_hi=30, mean=12_000, extra=0.015, P=64),
        # a graph of an untrusted producer: checked, then the five calls
        _path("checked path 8 Mbp", 8.4, 17, 11_000, 0.01, 33, kind="checked"),
        # pruning and transitive reduction of an overlap graph: small and ordinary
        dict(name="reduce 2 Mbp", kind="reduce", mb=2.0, cov=15, mean=10_000, extra=0.01, fuzz=0),
        dict(name="reduce 50 Mbp", kind="reduce", mb=50.0, cov=30, mean=12_000, extra=0.02,
             fuzz=0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case of the listed ranges: genomes of 1 Mbp to 1 Gbp (log-uniform),
    10-40x of 9-15 kbp reads, clean to branchy graphs, each option."""
    kind = rng.choice(["path", "path", "path", "noalloc", "checked", "batch", "wave", "reduce",
                       "reduce"])
    cov = round(rng.uniform(10, 40), 2)
    mean = rng.randrange(9_000, 15_001)
    extra = round(_log(rng, 0.0004, 0.03), 6)
    if kind == "batch":
        lo = round(_log(rng, 0.2, 2.0), 3)
        graphs = int(_log(rng, 4, 256))
        return dict(kind=kind, graphs=graphs, mb_lo=lo, mb_hi=round(lo * rng.uniform(1.5, 10), 3),
                    cov_lo=10, cov_hi=40, mean=mean, extra=max(extra, 0.005),
                    P=rng.choice([8, 33, 64, 100]))
    if kind == "wave":
        lo = round(_log(rng, 1.0, 10.0), 3)
        return dict(kind=kind, graphs=rng.randrange(1, 17), mb_lo=lo,
                    mb_hi=round(lo * rng.uniform(1.5, 10), 3), cov_lo=15, cov_hi=30, mean=mean,
                    extra=max(extra, 0.01), P=rng.choice([16, 64, 200]))
    if kind == "reduce":
        return dict(kind=kind, mb=round(_log(rng, 1.0, 40.0), 4), cov=min(cov, 32.0), mean=mean,
                    extra=extra, fuzz=rng.choice([0, 0, 10]))
    # one-read contigs are asked for of small and mid-size genomes
    min_reads = 1 if kind == "path" and rng.random() < 0.3 else 2
    top = 30.0 if min_reads == 1 or kind == "noalloc" else 400.0
    P = rng.choice([1, 8, 50, 64, 128, 500, 1024])
    c = _path("", round(_log(rng, 1.0, top), 4), cov, mean, extra, P, min_reads,
              rng.choice(["reads", "reads", "bases"]), rng.random() < 0.3, kind)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Simulated graphs, all jobs of a case at once
# ---------------------------------------------------------------------------

def _sizes(case):
    """(genome bases, coverage) of every graph of the case; the sizes are the
    case's own, the reads come from the seed."""
    if "graphs" not in case:
        return [(int(round(case["mb"] * 1e6)), float(case["cov"]))]
    r = random.Random("%d %s %s" % (case["graphs"], case["mb_lo"], case["mb_hi"]))
    return [(int(round(1e6 * _log(r, case["mb_lo"], case["mb_hi"]))),
             r.uniform(case["cov_lo"], case["cov_hi"])) for _ in range(case["graphs"])]


def _cat0(x):
    """Exclusive prefix sums with the total at the end."""
    return torch.cat([x.new_zeros(1), torch.cumsum(x, 0)])


def _pack_store(start, length, rc, genome_bases, gen, dev):
    """Reads at [start, start + length) of a random genome, stored reverse-
    complemented where rc, 2 bits a base at whole-word offsets: (first word of
    every read + total, the store)."""
    W = (genome_bases + 15) // 16 + 2
    fwd = torch.randint(0, 1 << 32, (W,), generator=gen, device=dev, dtype=torch.int64)
    x = fwd.flip(0)  # the reverse strand: words reversed, fields reversed and complemented
    for s, m in ((2, 0x33333333), (4, 0x0F0F0F0F), (8, 0x00FF00FF), (16, 0x0000FFFF)):
        x = ((x >> s) & m) | ((x & m) << s)
    both = torch.cat([fwd, x ^ 0xFFFFFFFF, fwd[:1]])
    del fwd, x
    both = both[:-1] | (both[1:] << 32)  # a word and the next one, for the unaligned starts
    src = torch.where(rc, 32 * W - (start + length), start)
    words = (length + 15) >> 4
    offw = _cat0(words)
    total = int(offw[-1])
    seq = torch.empty(max(total, 1), dtype=torch.int32, device=dev)
    cuts = torch.searchsorted(offw, torch.arange(0, total, WORD_CHUNK, device=dev)).tolist()
    cuts = sorted(set([0] + cuts + [int(length.numel())]))
    at = [int(v) for v in offw[torch.tensor(cuts, device=dev)].tolist()]
    for (r0, r1), (w0, w1) in zip(zip(cuts[:-1], cuts[1:]), zip(at[:-1], at[1:])):
        w = words[r0:r1]
        pos = torch.repeat_interleave(src[r0:r1] - 16 * offw[r0:r1], w, output_size=w1 - w0)
        pos += 16 * torch.arange(w0, w1, device=dev)
        seq[w0:w1] = (both[pos >> 4] >> (2 * (pos & 15))).to(torch.int32)
        del pos
    # zero the bits past each read's last base
    last, keep = offw[1:] - 1, length - 16 * (words - 1)
    mask = torch.where(keep == 16, torch.full_like(keep, 0xFFFFFFFF),
                       (torch.ones_like(keep) << (2 * keep)) - 1)
    seq[last] = ((seq[last].to(torch.int64) & mask)).to(torch.int32)
    return offw, seq


def _simulate(case, seed, dev="cuda", overlaps=False, store=True):
    """Device graphs of the case as (n, m, tensors, seq words) per graph."""
    sizes = _sizes(case)
    mean, sd, extra = float(case["mean"]), case["mean"] / 3.0, float(case["extra"])
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    i64 = dict(dtype=torch.int64, device=dev)
    G = torch.tensor([g for g, _ in sizes], **i64)
    n_j = torch.tensor([max(2, round(g * c / mean)) for g, c in sizes], **i64)
    job0, base0 = _cat0(n_j), _cat0(G)
    N = int(job0[-1])
    job = torch.repeat_interleave(torch.arange(len(sizes), device=dev), n_j, output_size=N)

    # reads: lognormal lengths, uniform starts, half of them reverse-complemented
    s2 = math.log1p((sd / mean) ** 2)
    z = torch.randn(N, generator=gen, device=dev, dtype=torch.float64)
    length = torch.exp(math.log(mean) - s2 / 2 + math.sqrt(s2) * z).round().to(torch.int64)
    length = torch.minimum(length.clamp(500, (1 << MAX_LEN_BITS) - 1), G[job])
    u = torch.rand(N, generator=gen, device=dev, dtype=torch.float64)
    a = base0[job] + (u * (G[job] - length + 1).to(torch.float64)).to(torch.int64)
    rc = torch.rand(N, generator=gen, device=dev) < 0.5
    # ids are file order; genome order: by (start, longest first)
    order = torch.argsort((a << MAX_LEN_BITS) + ((1 << MAX_LEN_BITS) - 1 - length))
    A, B = a[order], (a + length)[order]
    reach = torch.cummax(B, 0).values
    contained = torch.zeros(N, dtype=torch.bool, device=dev)
    contained[1:] = reach[:-1] >= B[1:]

    if overlaps:  # every pair that overlaps enough, contained reads included
        us, vs, os_ = [], [], []
        k = 1
        while k < N:
            cand = A[k:] + MIN_OVERLAP <= B[:-k]
            ov = torch.minimum(B[:-k], B[k:]) - A[k:]
            i = torch.nonzero(cand & (ov >= MIN_OVERLAP)).flatten()
            if not bool(cand.any()):
                break
            us.append(i)
            vs.append(i + k)
            os_.append(ov[i])
            k += 1
        gu, gv, ov = torch.cat(us), torch.cat(vs), torch.cat(os_)
        n_true = int((~contained).sum())
    else:  # the reduced graph: consecutive reads that are not contained
        keep = torch.nonzero(~contained).flatten()
        ov = B[keep[:-1]] - A[keep[1:]]
        link = ov >= MIN_OVERLAP
        gu, gv, ov = keep[:-1][link], keep[1:][link], ov[link]
        n_true = int(gu.numel())
    tu, tv = order[gu], order[gv]
    s, d = rc[tu].to(torch.int64), rc[tv].to(torch.int64)

    # extra overlaps between distant reads of one genome: branch vertices
    keep = torch.nonzero(~contained).flatten()
    kj = job[order[keep]]
    first = torch.searchsorted(kj, torch.arange(len(sizes) + 1, device=dev))
    want = int(round(extra * n_true))
    x = torch.randint(0, keep.numel(), (want,), generator=gen, device=dev)
    jx = kj[x]
    r = torch.rand(want, generator=gen, device=dev, dtype=torch.float64)
    y = first[jx] + (r * (first[jx + 1] - first[jx]).to(torch.float64)).to(torch.int64)
    far = (x - y).abs() > 64
    x, y = torch.minimum(x, y)[far], torch.maximum(x, y)[far]
    pair = torch.unique(x * keep.numel() + y)
    x, y = order[keep[pair // keep.numel()]], order[keep[pair % keep.numel()]]
    hi = torch.minimum(length[x], length[y]) - 1
    ok = hi >= MIN_OVERLAP
    x, y, hi = x[ok], y[ok], hi[ok]
    k = x.numel()
    r = torch.rand(k, generator=gen, device=dev, dtype=torch.float64)
    xo = MIN_OVERLAP + (r * (hi - MIN_OVERLAP + 1).to(torch.float64)).to(torch.int64)
    xb = torch.randint(0, 2, (2, k), generator=gen, device=dev)
    tu, tv, ov = torch.cat([tu, x]), torch.cat([tv, y]), torch.cat([ov, xo])
    s, d = torch.cat([s, xb[0]]), torch.cat([d, xb[1]])

    # symmetric CSR: the twin of (s, d) is (not d, not s)
    E = tu.numel()
    key = torch.cat([tu * N + tv, tv * N + tu])
    key, at = torch.sort(key)
    src, dst = key // N, key % N
    e, twin = at % max(E, 1), at >= E
    bits = torch.where(twin, (1 - d[e]) | ((1 - s[e]) << 1), s[e] | (d[e] << 1))
    row = torch.searchsorted(src, torch.arange(N + 1, device=dev))
    o = ov[e]
    pre = post = None
    if case.get("coords"):
        # alignments stop short of the overlap's ends by up to 200 bases
        c = torch.rand((2, E), generator=gen, device=dev, dtype=torch.float64)
        c = (c * (torch.clamp((ov - 1) // 2, max=200) + 1).to(torch.float64)).to(torch.int64)
        clip = torch.where(twin, c[1][e], c[0][e])
        lu, lv = length[src], length[dst]
        wp = lu - o + clip - 1
        pre = torch.where((bits & 1) == 0, wp, lu - 1 - wp)
        post = torch.where((bits >> 1) == 0, clip, lv - 1 - clip)

    if store:
        offw, seq = _pack_store(a, length, rc, int(base0[-1]), gen, dev)
    else:
        offw, seq = _cat0((length + 15) >> 4), torch.zeros(1, dtype=torch.int32, device=dev)

    # one set of arrays per graph
    out = []
    j0, e0, w0 = (t.tolist() for t in (job0, row[job0], offw[job0]))
    i32 = torch.int32
    o, dst, bits = o.to(i32), (dst - job0[job[src]]).to(i32), bits.to(torch.uint8)
    ln = length.to(i32)
    for j in range(len(sizes)):
        v0, v1, b, f = j0[j], j0[j + 1], e0[j], e0[j + 1]
        sw = w0[j + 1] - w0[j] if store else 1
        pad = lambda t: t[b:f].clone() if f > b else t.new_zeros(1)
        t = dict(row_ptr=(row[v0:v1 + 1] - b).to(i32), col=pad(dst), ovl=pad(o), strand=pad(bits),
                 read_len=ln[v0:v1].clone(), read_off=16 * (offw[v0:v1] - w0[j]),
                 seq=seq[w0[j]:w0[j + 1]].clone() if len(sizes) > 1 else seq)
        if pre is not None:
            t["pre"], t["post"] = pad(pre.to(i32)), pad(post.to(i32))
        out.append((v1 - v0, f - b, t, sw))
    return out


def _graphs(case, seed, **kw):
    return [cg.DeviceGraph.from_tensors(n, m, t, sw) for n, m, t, sw in _simulate(case, seed, **kw)]


# ---------------------------------------------------------------------------
# State and passes
# ---------------------------------------------------------------------------

def _zero(obj):
    for v in vars(obj).values():
        if isinstance(v, torch.Tensor):
            v.zero_()
    return obj


def _tensors(obj):
    return {k: v for k, v in vars(obj).items() if isinstance(v, torch.Tensor)}


def _word_caps(case):
    """Words of packed contigs per graph: what all of its reads come to, with
    room for the spread of their lengths."""
    return [int(1.1 * max(2, round(g * c / case["mean"])) * (case["mean"] / 16 + 1)) + 4096
            for g, c in _sizes(case)]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "reduce":
        dg = _graphs(case, seed, overlaps=True, store=False)[0]
        cap = int(2.4 * dg.n * case["cov"]) + 1024
        assert dg.m <= cap
        return dict(case=case, g=dg, ctx=cg.Context.for_graph(dg.n, dg.m, 1),
                    out=_zero(cg.Reduced(dg.n, cap)))
    gs = _graphs(case, seed)
    dg = gs[0]
    caps = _word_caps(case)
    if kind in ("path", "checked", "noalloc"):
        st = dict(case=case, g=dg, out=_zero(cg.Outputs(dg.n, case["P"], caps[0])))
        if kind == "noalloc":
            st["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        else:
            st["ctx"] = cg.Context.for_graph(dg.n, dg.m, case["P"])
            st["bad"] = torch.zeros(2, dtype=torch.int64, device="cuda")
        return st
    P = case["P"]
    sizes = [cg.job_outputs_bytes(g.n, P, cap) for g, cap in zip(gs, caps)]
    st = dict(case=case, graphs=gs, caps=caps, sizes=sizes, ctx=cg.Context(0, 0))
    if kind == "wave":
        st["lane"] = cg.Batch.empty(st["ctx"], cg.batch_bytes([(g.n, g.m, P) for g in gs]))
        st["packed"] = torch.cuda.Event()
        # records, layouts and bases of every graph: below a third of the outputs
        st["dst"] = torch.zeros(sum(sizes) // 3, dtype=torch.uint8, device="cuda")
        st["packed"].record()
        return st
    # the planned batch a program keeps, its outputs carved from one buffer,
    # captured once; small batches mix the options
    st["buf"] = torch.zeros(sum(sizes), dtype=torch.uint8, device="cuda")
    jobs, at = [], 0
    mixed = len(gs) <= 64
    for i, (g, nb, cap) in enumerate(zip(gs, sizes, caps)):
        jobs.append((g, cg.CarvedOutputs(st["buf"], at, g.n, P, cap), P,
                     1 if mixed and i % 4 == 3 else 2, "bases" if mixed and i % 3 == 2 else "reads"))
        at += nb
    st["batch"] = cg.Batch(st["ctx"], jobs)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    st["batch"].capture(side)
    torch.cuda.current_stream().wait_stream(side)
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("path", "checked"):
        if kind == "checked":
            cg.validate(state["ctx"], state["g"], state["bad"])
        cg.run_path(state["ctx"], state["g"], state["out"], case["P"], case["min_reads"],
                    weight=case["weight"])
        return dict(_tensors(state["out"]), bad=state["bad"])
    if kind == "noalloc":
        cg.contig_generation_noalloc(state["g"], state["out"], case["P"], case["min_reads"],
                                     weight=case["weight"], d_status=state["status"])
        return dict(_tensors(state["out"]), status=state["status"])
    if kind == "reduce":
        cg.reduce(state["ctx"], state["g"], state["out"], case["fuzz"])
        return _tensors(state["out"])
    if kind == "batch":
        state["batch"].launch(torch.cuda.current_stream())
        return state["buf"].view(torch.int64)  # every output of every graph
    # a serving lane's wave: its memory is planned anew once its last wave's
    # results are out, the counts are read to size the packed download
    state["packed"].synchronize()
    buf = torch.empty(sum(state["sizes"]), dtype=torch.uint8, device="cuda")
    jobs, at = [], 0
    for g, nb, cap in zip(state["graphs"], state["sizes"], state["caps"]):
        jobs.append((g, cg.CarvedOutputs(buf, at, g.n, case["P"], cap), case["P"], 2))
        at += nb
    lane = state["lane"]
    lane.plan(jobs)
    lane.run()
    counts = torch.empty(4 * len(jobs) + 1, dtype=torch.int64, device="cuda")
    lane.counts(counts)
    if int(counts[-1].item()) > state["dst"].numel():
        raise RuntimeError("the wave's results are larger than its download buffer")
    lane.pack(counts, state["dst"])
    state["packed"].record()
    return [counts, state["dst"]]


def exact(case, seed):
    """Every output is a whole number or packed bases."""
    return None


def work(case):
    """Each input read once and each output written once (expected sizes: the
    share of reads that are not contained falls with the coverage)."""
    n_reads = edges = genome = 0.0
    for g, cov in _sizes(case):
        n = max(2, round(g * cov / case["mean"]))
        n_reads += n
        edges += n * min(0.9, 3.7 / cov) * (1 + case["extra"])
        genome += g
    m = 2 * edges
    kind = case["kind"]
    if kind == "reduce":
        cov = case["cov"]
        m = 2 * n_reads * cov * 0.92
        return {"bytes": 4 * n_reads + 9 * m + 4 * n_reads + n_reads + m + 4 * n_reads + 9 * 2 * edges,
                "flops": 0}
    graph = 4 * n_reads + 9 * m + 12 * n_reads + (8 * m if case.get("coords") else 0)
    singles = n_reads - edges if case.get("min_reads") == 1 else 0.0
    in_contigs = edges * (1 - 2 * case["extra"]) + singles
    bases = genome + singles * case["mean"]
    # per read: flags, label, label_comp; per contig read: perm, local CSR row
    # and two entries, layout; packed bases in and out
    outs = 9 * n_reads + in_contigs * (4 + 4 + 16 + 5) + singles * 61
    total = graph - 12 * n_reads + 12 * in_contigs + outs + bases / 2
    if kind == "wave":
        total += bases / 2
    if kind == "checked":
        total += graph
    return {"bytes": total, "flops": 0}
