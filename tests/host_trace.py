"""The host side of the library without a GPU: a snippet runs in a process of
its own over a stand-in for the HIP runtime (host_trace.cpp), which takes down
launches, ranges, streams and events in order and runs nothing."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes
from paper_2207_04350_amd import cg

L = cg.lib()
mark = ctypes.CDLL(None).hostTraceMark


class S:
    cuda_stream = 0


# stands for every device buffer: never read by the host
BUF = ctypes.create_string_buffer(1 << 12)
P = ctypes.c_void_p((ctypes.addressof(BUF) + 255) // 256 * 256)


def graph(n, m):
    g = cg.CgGraph(n, m, P, P, P, P, P, P, P, n + 1, None, None)
    return type("G", (), dict(n=n, m=m, struct=g, seq_words=n + 1))


def outputs():
    o = type("O", (), {})()
    for k in ("flags", "counts", "label"):
        setattr(o, k, type("T", (), dict(data_ptr=lambda self: P.value))())
    o.parts, o.local = cg.CgParts(*[P] * 9), cg.CgLocal(*[P] * 6)
    o.contigs = cg.CgContigs(*[P] * 11, 1 << 20, P)
    return o
"""


def trace(snippet, tmp_path):
    """The events of the snippet as (what, argument) pairs; a snippet may
    print, which comes back as its second part."""
    so, log = os.path.join(str(tmp_path), "host_trace.so"), os.path.join(str(tmp_path), "log")
    if not os.path.exists(so):
        subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-std=c++17",
                               os.path.join(HERE, "host_trace.cpp"), "-o", so])
    preload = " ".join([so] + os.environ.get("LD_PRELOAD", "").split())
    env = dict(os.environ, HOST_TRACE=log, LD_PRELOAD=preload, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", PRELUDE + snippet], env=env, cwd=ROOT,
                       stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(log) as f:
        return [tuple(line.rstrip("\n").split(" ", 1)) for line in f], r.stdout
