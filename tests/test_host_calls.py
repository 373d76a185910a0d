"""The library's host code on a stand-in for the HIP runtime (tests/fake_hip.cpp): no device, no
kernels, but the allocations that the calls make and the launches that they queue, in order."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(ROOT, "paper_0910_0121_amd")


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    import paper_0910_0121_amd as t
    t.lib()  # built
    exe = str(tmp_path_factory.mktemp("fake") / "fake_hip")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([gxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-rdynamic",
                    "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(PKG, "csrc"), os.path.join(HERE, "fake_hip.cpp"),
                    os.path.join(PKG, "libtreepm.so"), f"-Wl,-rpath,{PKG}",
                    f"-Wl,-rpath,{rocm}/lib", f"-L{rocm}/lib", "-lpthread", "-o", exe], check=True)

    def call(*args):
        r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, (args, r.returncode, r.stdout[-2000:], r.stderr[-2000:])
        return r.stdout.splitlines()
    return call


@pytest.mark.parametrize("groups", [1, 1024, 1025, 16384, 16385, 200000])
def test_walk_returns_after_its_last_launch(run, groups):
    """The walk's results reach the host only once everything that it leaves for the force has
    been written: whatever publishes them is the last launch."""
    lines = run("walk", groups)
    assert lines[-1] == "returned 1000000"
    assert lines[-2] == "published"
    assert sum("k_walk_results" in l or "k_class_scatter" in l for l in lines) == 1


@pytest.mark.parametrize("more", range(18))
def test_a_failed_allocation_of_the_groups_leaves_no_half_of_them(run, more):
    """A build whose group arrays cannot all be allocated fails; the same build afterwards
    launches the group kernels on whole arrays."""
    lines = run("groups", more)
    assert lines[0] == "failed -3"  # TREEPM_ERR_OOM
    assert lines[-1] == "built"
    assert any("k_group_bbox" in l for l in lines)
    assert not [l for l in lines if "too small" in l]


def _field(lines, name):
    return [int(l.split()[1]) for l in lines if l.startswith(name + " ")]


@pytest.mark.parametrize("groups,longest,mean", [(1500, 3700, 1170), (14197, 3940, 1180),
                                                 (64, 310, 280), (60000, 5000, 1250)])
def test_slots_take_about_four_times_the_lists(run, groups, longest, mean):
    """From its second walk on a context holds at most about four times the packed lists of the
    first (with the eighth that every allocation adds, and blocks of 2 MiB)."""
    lines = run("slots", groups, longest, mean)
    packed, held = 4 * groups * mean, _field(lines, "held")
    assert len(held) == 3
    for h in held[1:]:
        assert h - held[0] <= 3 * packed * 9 // 8 + (4 << 20)
    assert held[1] == held[2]
    # and they are slots: one traversal
    assert sum("k_walk<0, 0>" in l for l in lines) == 1


@pytest.mark.parametrize("n,groups,longest,mean", [(200000, 4000, 4000, 1000),
                                                   (400000, 7781, 4600, 1190),
                                                   (30000, 500, 4000, 1200)])
def test_a_server_keeps_a_box_within_what_it_admitted(run, n, groups, longest, mean):
    """Repeated requests on one box of ordinary lists: the server holds no more than its estimate
    for the box (320 bytes a particle and 64 MiB), which is what it asked its budget for."""
    lines = run("server", n, groups, longest, mean, 4, n * 320 + (64 << 20))
    resident = _field(lines, "resident")
    assert sum(l == "served 0" for l in lines) == 4 and len(resident) == 4 and max(resident) <= n * 320 + (64 << 20)


def test_a_server_serves_a_box_that_outgrew_its_budget(run):
    """Lists several times as long as the estimate allows for: the box counts more than the
    budget after its first request, and its later requests are still served."""
    n = 100000
    lines = run("server", n, 20000, 9000, 3000, 3, n * 330 + (64 << 20))
    assert max(_field(lines, "resident")) > n * 330 + (64 << 20)
    assert sum(l == "served 0" for l in lines) == 3


@pytest.mark.parametrize("pairs,table", [(34_000_000, False), ((1 << 28) - 1, False),
                                         (1 << 28, True), (1 << 33, True)])
def test_fp64_table_only_where_it_pays(run, pairs, table):
    """A small box's first FP64 force does not make a table on the host, which takes longer than
    all of its call."""
    lines = run("force", 1, pairs, 0)
    assert [l for l in lines if f"k_force_f64<{str(table).lower()}>" in l]
    assert not [l for l in lines if f"k_force_f64<{str(not table).lower()}>" in l]


@pytest.mark.parametrize("precision,pairs,rows", [(0, 1000000, 0), (0, 1000000, 300000),
                                                  (1, 1000000, 300000), (1, 1 << 30, 0)])
def test_force_takes_no_memory(run, precision, pairs, rows):
    """With device outputs the force uses what the build and the walk allocated."""
    assert "allocations 0" in run("force", precision, pairs, rows)


@pytest.mark.parametrize("ratio,rc", [("0.0001220703125", 0), ("0.016666666666666666", 0), ("1", 0),
                                      ("7.9", 0), ("7.9999999999999", 0),
                                      ("7.99999999999999911", 0), ("8", -1), ("9", -1)])
def test_fp32_softening_range(run, ratio, rc):
    """FP32 boxes have a table for every eps / r_cut in [2^-13, 8), to the last bit."""
    assert f"force {rc}" in run("force", 0, 1000000, 0, ratio)
