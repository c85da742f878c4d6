"""When a batch makes the streams that its large jobs run on: a lane of a
serving loop at its creation, so that no wave waits for it (on a new lane the
first wave took 680 us where the second took 596, and the process's first lane
7 ms more), a batch of known jobs only if one of them is large."""
from tests.host_trace import trace

SNIPPET = """
ctx = cg.Context(0, 0)
large, small = graph(50000, 40000), graph(500, 900)
job = lambda g: (g, outputs(), 8, 2)
need = 64 << 20
mark(b"create")
lane = cg.Batch.empty(ctx, need, persist_blocks=1024)
for wave in ([small], [large, small], [large] * 5):
    mark(b"plan")
    lane.plan([job(g) for g in wave], S)
    mark(b"run")
    lane.run(S)
mark(b"small batch")
b = cg.Batch(ctx, [job(small)], persist_blocks=1024)
mark(b"large batch")
c = cg.Batch(ctx, [job(small), job(large)], persist_blocks=1024)
mark(b"end")
"""


def test_streams_are_made_at_creation(tmp_path):
    events, _ = trace(SNIPPET, tmp_path)
    made, at = {}, None
    for what, arg in events:
        if what == "mark":
            at = arg
        elif what in ("stream", "event"):
            made[at] = made.get(at, 0) + (what == "stream")
    assert made == {"create": 3, "large batch": 3}, made
