"""The per-kernel timing names a kernel as it is written, also one whose
template arguments hold a comma (those kept the parentheses that the launch
macro takes them in), and the benchmark's phases and bytes know every kernel of
the path (a pass over the reads was in no phase, and some were priced as kernels
that are gone)."""
import glob
import os
import re

import pytest

import bench
from tests.host_trace import ROOT, trace

PATHS = {
    "small path": "cg.run_path(ctx, graph(500, 900), outputs(), 8, 2, S)",
    "path": "cg.run_path(ctx, graph(50000, 90000), outputs(), 8, 2, S)",
    "all reads": "cg.run_path(ctx, graph(50000, 90000), outputs(), 8, 1, S, 'bases')",
    "batch": "cg.Batch(ctx, [(graph(500, 900), outputs(), 8, 2, w) for w in ('reads', 'bases')],"
             " persist_blocks=1024).run(S)",
}
SIZES = dict(N=1000, m=1800, m_nb=1700, n_e=990, m_e=1600, n_comp=40, contig_bases=10 ** 6,
             words=63000)


@pytest.mark.parametrize("name", sorted(PATHS))
def test_a_profile_names_kernels_that_the_benchmark_knows(name, tmp_path):
    _, out = trace("""
ctx = cg.Context(0, 64 << 20)
ctx.profile(64)
%s
for k in ctx.profile_read():
    print(k)
""" % PATHS[name], tmp_path)
    names = out.split("\n")[:-1]
    assert len(names) >= 3
    for k in names:
        assert re.fullmatch(r"kb?_\w+(<.+>)?", k), k
    ms = bench.phase_ms({k: (1, 2.0) for k in names})
    assert sum(ms.values()) == 2.0 * len(names)
    assert all(bench.kernel_bytes(k, SIZES) >= 0 for k in names)


def test_the_benchmark_lists_the_kernels_that_are_there():
    src = "".join(open(f).read() for f in glob.glob(os.path.join(ROOT, "paper_2207_04350_amd",
                                                                 "csrc", "*.hip")))
    there = {k for k in re.findall(r"CG_LAUNCH\([\w>.-]+, \(?(\w+)", src)
             if not re.match(r"k_red_|k_val_|kb_counts|kb_pack", k)}  # other entry points'
    listed = [k for ks in bench.PHASES.values() for k in ks]
    assert sorted(listed) == sorted(there)
    for k in there:
        assert bench.kernel_bytes(k, SIZES) is not None
    assert set(bench.BATCHED_AS) <= there


def test_a_kernel_that_no_phase_lists_is_an_error():
    with pytest.raises(KeyError):
        bench.phase_ms({"k_mask<1>": (1, 1.0), "k_gone": (1, 1.0)})
    with pytest.raises(KeyError):
        bench.kernel_bytes("k_gone", SIZES)


@pytest.mark.parametrize("row, kernel, found", [
    ("cg::k_comp(cg::CompArgs)", "k_comp", True),
    ("void cg::k_red_trans<128>(int, int const*)", "k_red_trans<128>", True),
    ("void cg::k_mask<false>(int)", "k_mask<true>", True),
    ("cg::k_comp_more(int)", "k_comp", False),
])
def test_traffic_is_found_under_a_template_name(row, kernel, found, tmp_path, monkeypatch):
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "p.md").write_text(
        "csrc sha256: abc\n| kernel | F | W | MB |\n| `%s` | 1 | 2 | 3.5 |\n" % row)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "csrc_digest", lambda: "abc")
    assert bench.profiled_traffic(kernel, "p.md") == (3.5e6 if found else None)
