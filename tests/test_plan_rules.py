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
    # lengths between are multiples of 64
    assert rules("plan 262144 300 1")[0] == [3, 1, 1366, 192]


def test_even_splits_of_packed_blocks(rules):
    """Packed launches: at most 64 splits where 512 bodies a split give no more,
    but 256 bodies a split where even that leaves a CU few work-groups."""
    for n, n_i, splits, length in ((30000, 10000, 59, 512), (32768, 16384, 64, 512),
                                   (24576, 4099, 96, 256), (30000, 2500, 118, 256),
                                   (16384, 9000, 64, 256), (131072, 4099, 187, 704)):
        for mixed in (0, 1):
            assert rules(f"plan {n} {n_i} {mixed}")[0] == [1, 1, splits, length]


def _up(a, b):
    return -(-a // b)


def _coarse_bytes(n, n_i, mixed):
    """Scratch of splits of 512 bodies (128 in one-wave work-groups), at most 64
    (16) work-groups per CU: what a call may always be given instead of its
    plan's."""
    if n_i <= 40:
        return None
    u1, u3 = _up(n_i, 256), _up(n_i, 64)
    narrow = u1 * 256 * 5 > u3 * 64 * 6
    unit = 64 if narrow else 256
    s = min(_up(4096, u3), _up(n, 128)) if narrow else min(_up(16384, u1), _up(n, 512))
    k = _up(n, _up(_up(n, unit), s) * unit)
    slots = 0 if k == 1 else sum(_up(k * n_i * b, 256) * 256 for b in (64, 4, 384))
    return slots + (3 * _up(4 * n_i, 256) * 256 if mixed else 0)


def test_scratch_fits_a_small_budget(rules):
    """Every block runs in the scratch of the coarse splits, with the most splits
    that fit; with less than that it is refused."""
    cases = [(n, n_i, mixed, _coarse_bytes(n, n_i, mixed))
             for n in (300, 512, 1024, 3001, 8192, 16384, 65537, 131072, 200000, 1 << 20)
             for n_i in (41, 64, 130, 300, 520, 777, 1024, 4099, 8192, n) if 40 < n_i <= n
             for mixed in (0, 1)]
    at = [rules(*[f"fit {n} {n_i} {m} {budget(room)} 0" for n, n_i, m, room in cases])
          for budget in (lambda room: room, lambda room: 1 << 50, lambda room: 4096)]
    for case, coarse, free, none in zip(cases, *at):
        assert coarse[2] <= case[3] and coarse[0] <= free[0], case
        if case[3] > 8 * 4096:
            assert none[4] and none[2] > 4096, case
    # most splits that fit: 8192 of 8192 in 64 MiB, 452 bytes a row and split
    splits, _, total, _, _ = rules(f"fit 8192 8192 0 {64 << 20} 0")[0]
    assert 16 <= splits <= 18 and total <= 64 << 20


def test_fixed_workspace_plans(rules):
    """In the 64 MiB of the allocation-free call the splits fill the CUs evenly, and
    the refinement leaves them most of the room."""
    ws = nb.fixed_workspace_bytes()
    for n, n_i in ((131072, 1024), (65536, 2048), (262144, 1024), (16384, 16384),
                   (1 << 20, 1272), (100003, 1500), (131072, 4099)):
        for mixed in (0, 1):
            splits, length, total, packed, _ = rules(f"fit {n} {n_i} {mixed} {ws} 1")[0]
            most = ws // (452 * n_i)
            assert total <= ws and splits >= 0.8 * most
            groups = _up(n_i, 256) * splits
            assert groups / 256 > 0.85 * _up(groups, 256), (n, n_i, splits)


def test_adjoint_panels_fill_the_chip(rules):
    """Gradients in several panels keep the launches of one: about 24 work-groups
    per CU; the entries stay within 1 GiB next to the row sums."""
    for n, n_i in ((65536, 65536), (1 << 18, 1 << 18), (1 << 19, 1 << 19), (1 << 20, 1 << 20),
                   (1 << 21, 1 << 21), (1 << 20, 5000), (1 << 22, 1 << 16), (64, 1 << 25),
                   (1000, 1 << 24)):
        block, tile, length, panel, in_gm, total = rules(f"adjoint {n} {n_i} 0")[0]
        assert total <= (1 << 30) + 2 * (48 * n_i + 256) and not in_gm
        items = min(panel, _up(n_i, block)) * _up(n, length)
        assert items >= 20 * 256 or length == tile, (n, n_i)
        assert items * 256 < 1 << 32 and panel * block <= 1 << 25
    # a million rows of few bodies are one panel
    assert rules(f"adjoint 64 {1 << 20} 0")[0][3] == (1 << 20) // 256
    # the least: 7 n + 12 n_i values
    for n, n_i in ((3000, 2000), (9000, 5000), (1 << 18, 1 << 18)):
        room = 8 * (7 * n + 12 * n_i) + 768
        _, _, _, panel, _, total = rules(f"adjoint {n} {n_i} {room}")[0]
        assert panel == 1 and total <= room


def test_tuner_times_the_automatic_plan(rules):
    """The automatic plan is the first candidate, for every size and precision."""
    for n, n_i in ((64, 1), (1024, 64), (16384, 4096), (131072, 4096), (1 << 20, 65536)):
        for mixed in (0, 1):
            count, first, automatic = rules(f"tune {n} {n_i} {mixed}")[0]
            assert count > 1 and first == 0 and automatic == 1
