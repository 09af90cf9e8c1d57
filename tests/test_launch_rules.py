"""Rules that size and choose launches, checked on the host over every size they serve: tests/launch_rules.hip is
compiled against the library's internal header (host code only) and prints what the rules give."""
import os
import subprocess

import pytest

from paper_1403_4099_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
MAX_LDS = 65536                                   # bytes a workgroup may allocate


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    r = subprocess.run([build.HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-w",
                        os.path.join(HERE, "launch_rules.hip"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(what):
        p = subprocess.run([exe, what], capture_output=True, text=True, timeout=60)
        assert p.returncode == 0
        return [line.split() for line in p.stdout.splitlines()]
    return run


def test_breed_launches_ask_for_the_lds_that_their_largest_instance_uses(rules):
    rows = [tuple(map(int, r)) for r in rules("breed_lds")]
    assert len(rows) == 8 * 4096
    for inds, n, asked, used in rows:
        assert asked == used, (inds, n)
        assert asked + 4096 <= MAX_LDS, (inds, n)          # 4096: the ranking's, beside it


def test_the_fp64_row_walk_stays_inside_the_matrix(rules):
    """Every load of the walk is inside C, and a row above the column (its value counts) is read itself."""
    rows = [tuple(map(int, r)) for r in rules("fp64_rows")]
    assert [r[0] for r in rows] == list(range(1, 4097))
    for n, loads, outside, other in rows:
        blocks = (n + 63) // 64
        assert loads == 4 * blocks + 64 * blocks * (blocks + 1) // 2
        assert outside == 0 and other == 0, n
