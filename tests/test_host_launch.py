"""CPU tests of the rules that shape launches: no grid reaches 2^32 threads in x, which HIP refuses."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_16864_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("launch") / "host_launch")
    cmd = ["g++", "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           os.path.join(ROOT, "tests", "host_launch_main.cpp"), os.path.join(CSRC, "jenga_plan.cpp"),
           os.path.join(CSRC, "jenga_host.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _run(driver, rows):
    lines = "".join(" ".join(str(x) for x in row) + "\n" for row in rows)
    r = subprocess.run([driver], input=lines, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return [line.split() for line in r.stdout.strip().split("\n")]


# Blocks of 32 tokens: 512 threads a query block at head dim 64, 256 at 128; few and many blocks a head, text or none.
def test_attention_launches_stay_below_the_grid_limit(driver):
    rows = [(1, 1, 32 * m_v - 3, n_text, 1, heads, d, 32, 0.3, 0.3, 512 if d == 64 else 256)
            for m_v in (1, 7, 64, 128, 129, 300, 2000) for n_text in (0, 40) for heads in (1, 24, 5000, 65535) for d in (64, 128)]
    cut = 0
    for row, got in zip(rows, _run(driver, rows)):
        pairs, some, wgs_all, wgs_some = [int(x) for x in got]
        threads = row[-1]
        assert pairs == row[5] and 1 <= some <= pairs
        assert wgs_some * threads < 1 << 32, row
        if wgs_all * threads < 1 << 32:
            assert some == pairs, row
        else:
            cut += 1
    assert cut > 4      # e.g. 65535 heads of 129 blocks at head dim 64
