"""Every kernel of a call is enqueued inside one range of the tracer that names
its step or steps of Algorithm 2, so that a trace shows no launch beside them
(the path's count, compaction, offsets and copy lay outside any)."""
import pytest

from tests.host_trace import trace

M, CC = "cg: BranchRemoval", "cg: ConnectedComponent"
PART, IND, ASM = "cg: GreedyPartitioning", "cg: InducedSubgraph", "cg: LocalAssembly"
PATH = [M + " + ConnectedComponent", PART, IND + " + LocalAssembly", ASM]

CALLS = {
    # (reads, entries, options, ranges)
    "small path": ("cg.run_path(ctx, graph(500, 900), outputs(), 8, 2, S)", PATH),
    "path": ("cg.run_path(ctx, graph(50000, 90000), outputs(), 8, 2, S)", PATH),
    "path, least size": ("cg.run_path(ctx, graph(50000, 90000), outputs(), 8, 3, S)", PATH),
    "path, all reads": ("cg.run_path(ctx, graph(50000, 90000), outputs(), 8, 1, S)", PATH),
    "path, bases": ("cg.run_path(ctx, graph(50000, 90000), outputs(), 8, 2, S, 'bases')", PATH),
    "noalloc": ("cg.contig_generation_noalloc(graph(50000, 90000), outputs(), 8, 2, S)", PATH),
    "steps": ("""
g, o = graph(50000, 90000), outputs()
cg.mask_branches(ctx, g, o.flags, o.counts, S)
cg.components(ctx, g, o.flags, o.label, S)
cg.partition(ctx, g, o.flags, o.label, 8, 1, o.parts, S, 'bases')
cg.induce(ctx, g, o.flags, o.label, o.parts, 8, o.local, S)
cg.assemble(ctx, g, o.parts, o.local, 8, o.contigs, S)
""", [M, CC, PART, IND, ASM]),
    "validate": ("cg.validate(ctx, graph(500, 900), outputs().flags, S)", ["cg: validate"]),
    "batch": ("""
b = cg.Batch(cg.Context(0, 0), [(graph(500, 900), outputs(), 8, 2, w) for w in ('reads', 'bases')],
             persist_blocks=1024)
mark(b"go")
b.run(S)
""", ["cg_batch: BranchRemoval + ConnectedComponent",
      "cg_batch: GreedyPartitioning, InducedSubgraph, LocalAssembly"]),
}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_every_launch_lies_in_a_range(name, tmp_path):
    call, want = CALLS[name]
    events, _ = trace("ctx = cg.Context(0, 64 << 20)\n%s\n" % call, tmp_path)
    if ("mark", "go") in events:
        events = events[events.index(("mark", "go")) + 1:]
    seen, depth, outside, inside = [], 0, [], 0
    for what, arg in events:
        if what == "push":
            assert depth == 0, "a range inside another"
            depth, seen = 1, seen + ([arg] if not seen or seen[-1] != arg else [])
        elif what == "pop":
            depth = 0
        elif what == "launch":
            inside += depth
            outside += [] if depth else [arg]
    assert outside == [] and depth == 0 and inside >= len(want)
    assert seen == want
