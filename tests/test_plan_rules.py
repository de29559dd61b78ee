"""The host-side rules that shape the launches (plans, split lengths, grids and
scratch), through a small program linked with the library: no GPU needed."""
import os
import subprocess

import pytest

import paper_1504_03687_amd as nb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_1504_03687_amd")
CXX = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not os.path.exists(CXX), reason="ROCm toolchain not available")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """rules("plan 1024 1024 0", ...) -> one list of numbers per query."""
    nb.lib()   # built
    exe = str(tmp_path_factory.mktemp("rules") / "plan_rules")
    r = subprocess.run(
        [CXX, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
         "-I", os.path.join(ROOT, "include"), "-I", os.path.join(LIB_DIR, "csrc"),
         os.path.join(ROOT, "tests", "plan_rules_driver.cpp"), "-o", exe,
         os.path.join(LIB_DIR, "libnbreg.so"), "-L/opt/rocm/lib", "-lamdhip64",
         f"-Wl,-rpath,{LIB_DIR}", "-Wl,-rpath,/opt/rocm/lib"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def ask(*queries):
        r = subprocess.run([exe], input="\n".join(queries) + "\n", capture_output=True, text=True,
                           timeout=60)
        assert r.returncode == 0, (queries, r.stdout, r.stderr)
        out = [[int(v) for v in line.split()] for line in r.stdout.splitlines()]
        assert len(out) == len(queries)
        return out

    return ask


def test_refinement_grid_of_small_calls(rules):
    """Calls of up to 1024 rows launch half of the refinement's work-groups."""
    for n, n_i, per in ((524288, 64, 2), (262144, 1024, 2), (1 << 20, 41, 1)):
        grid, groups = rules(f"redo {n} {n_i} {per}")[0]
        assert grid == groups // 2
    assert rules("redo 1048576 1025 2")[0] == [2048, 2048]
    assert rules("redo 1024 300 2")[0] == [300, 2048]      # a work-group per row
    assert rules("redo 2049 1 2")[0] == [2, 2048]          # two chunks of one row


def test_short_splits_of_long_ranges(rules):
    """Small blocks: splits of 64 bodies up to 131072 bodies, of 128 above."""
    for n, n_i, length in ((131072, 41, 64), (131072, 64, 64), (131073, 41, 128),
                           (200000, 64, 128), (262144, 100, 128), (262144, 41, 128),
                           (1 << 20, 64, 256)):
        for mixed in (0, 1):
            mapping, rows, splits, got = rules(f"plan {n} {n_i} {mixed}")[0]
            assert (mapping, rows, got) == (3, 1, length)
            assert splits == -(-n // length)


def test_even_splits_of_packed_blocks(rules):
    """Packed launches: at most 64 splits where 512 bodies a split give no more,
    but 256 bodies a split where even that leaves a CU few work-groups."""
    for n, n_i, splits, length in ((30000, 10000, 59, 512), (32768, 16384, 64, 512),
                                   (24576, 4099, 96, 256), (30000, 2500, 118, 256),
                                   (16384, 9000, 64, 256), (131072, 4099, 187, 704)):
        for mixed in (0, 1):
            assert rules(f"plan {n} {n_i} {mixed}")[0] == [1, 1, splits, length]
