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


def _run(driver, rows, *args):
    lines = "".join(" ".join(str(x) for x in row) + "\n" for row in rows)
    r = subprocess.run([driver, *args], input=lines, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, rows[r.stdout.count("\n")], r.stderr)
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


# Every query block is dealt out once, and text blocks to XCDs that work on their head: alone on another XCD a row that
# sees every block finds no key in its L2.
def test_work_mapping(driver):
    rows = [(1, 1, block * m_v - 3, n_text, 1, heads, d, block, 0.3, p)
            for block in (32, 64, 128) for d in (64, 128) for m_v in (1, 7, 8, 31, 64, 129, 300) for n_text in (0, 3, 300)
            for heads in (1, 2, 3, 8, 13, 24, 80) for p in (0.3, 0.9)]
    shares = set()
    for row, got in zip(rows, _run(driver, rows, "work")):
        least, most, share, apart = [int(x) for x in got]
        assert (least, most) == (1, 1), row
        shares.add(share)
        if row[2] > 8 * row[7]:           # a vision block for every XCD of a head
            assert apart == 0, (row, share)
    assert shares == {1, 2, 4, 8}


# Every part of every list is dealt out once and has a slot of its own, which is where the merge looks for it.
def test_positions_cover_every_part_once(driver):
    rows = [(1, 1, block * m_v - 3, n_text, 1, heads, d, block, topk, p)
            for block in (64, 128) for d in (64, 128) for m_v, heads in ((31, 27), (49, 16), (80, 12), (137, 8), (257, 9), (300, 24))
            for n_text in (0, 3, 300) for topk, p in ((0.3, 0.3), (0.1, 0.3), (0.25, 0.9))]
    text, tails = set(), 0
    for row, got in zip(rows, _run(driver, rows, "deal")):
        text_parts, tail, least, most, used, slots = [int(x) for x in got[:6]]
        assert (least, most) == (0, 0) and used <= slots, row
        text.add(text_parts)
        tails += tail > 0
    assert len(text) > 3 and tails > 10


# The same where text blocks outnumber vision blocks, down to a single one: the lists cut at the end are vision lists, of which
# an XCD then has fewer than it has places for.
@pytest.mark.parametrize("flags", [0, 4, 5, 7, 15])
def test_positions_cover_every_part_once_with_more_text_than_vision(driver, flags):
    rows = [(1, 1, block * m_v - 3, block * m_c - 7, 1, heads, d, block, topk, p)
            for block in (64, 128) for d in (64, 128) for m_c in (36, 77, 120, 500, 1064)
            for m_v in sorted({min(2048 - m_c, max(1, m_c * part // 100)) for part in (0, 3, 7, 17, 40, 100)})
            for heads in (1, 4, 7, 12, 24) for topk, p in ((0.05, 0.5), (0.2, 0.5), (0.3, 0.3), (0.25, 0.9))]
    rows += [(1, 1, 6754, 16434, 1, 4, 128, 64, 0.05, 0.5), (1, 1, 2333, 9726, 1, 7, 128, 64, 0.1, 0.5),
             (1, 1, 2560, 13824, 1, 12, 128, 128, 0.2, 0.5), (1, 1, 46327, 136099, 1, 1, 128, 128, 0.05, 0.5),
             (1, 1, 1024, 15360, 1, 8, 128, 128, 0.2, 0.5), (1, 1, 3840, 15360, 1, 8, 128, 128, 0.2, 0.5)]
    both = 0
    for row, got in zip(rows, _run(driver, rows, "deal", str(flags))):
        text_parts, tail, least, most, used, slots, _, _ = [int(x) for x in got]
        assert (least, most) == (0, 0) and used <= slots, row
        both += tail > 0 and text_parts > 1
    assert both > 0


# Results of parts take 129 MiB of the workspace at most, also of text rows, of which there may be tens of thousands.
@pytest.mark.parametrize("flags", [0, 7, 15])
def test_parts_of_text_rows_are_bounded(driver, flags):
    rows = [(1, 1, vision, n_text, batch, heads, d, block, topk, p)
            for block in (64, 128) for d in (64, 128) for n_text in (10000, 27348, 64000, 109477, 128000)
            for vision in (100, 893, 2068, 15000) for batch, heads in ((1, 1), (1, 3), (1, 14), (2, 40))
            for topk, p in ((0.05, 0.0), (0.05, 0.5), (0.3, 0.2), (0.2, 0.9))
            if -(-vision // block) + -(-n_text // block) <= 2048]
    rows += [(1, 1, 8330, 9838, 1, 8, 128, 128, 0.05, 0.5), (33, 45, 80, 256, 1, 24, 128, 128, 0.1, 0.3)]
    cut = 0
    for row, got in zip(rows, _run(driver, rows, "deal", str(flags))):
        assert int(got[7]) <= 129 << 20, (row, got)
        cut += int(got[0]) > 1
    assert cut > 0


# Blocks of 64 tokens at head dim 128 take steps of 32 keys only where the chip is full of them and no whole text row runs on alone: in
# a call that may cut lists, and in the packed entry, which cuts nothing.
@pytest.mark.parametrize("blocks,heads,text,topk,p,cuts,whole", [
    (8, 2, 1, 0.25, 0.3, 0, 0), (41, 8, 1, 0.25, 0.3, 0, 0), (84, 10, 1, 0.25, 0.3, 0, 0), (150, 6, 1, 0.25, 0.3, 0, 0),
    (145, 2, 2, 0.25, 0.3, 0, 0), (120, 6, 1, 0.25, 0.3, 1, 0), (305, 2, 0, 0.3, 0.5, 1, 0), (76, 6, 1, 0.2, 0.9, 1, 0), (40, 24, 0, 0.25, 0.3, 0, 0),
    (62, 20, 0, 0.25, 0.3, 1, 1), (120, 12, 0, 0.25, 0.3, 1, 1), (120, 12, 1, 0.25, 0.3, 1, 0), (30, 40, 1, 0.25, 0.3, 1, 0),
    (40, 40, 0, 0.25, 0.3, 0, 0), (62, 28, 0, 0.25, 0.3, 0, 0), (120, 14, 0, 0.25, 0.3, 1, 0), (62, 40, 0, 0.25, 0.3, 1, 1),
    (62, 24, 1, 0.1, 0.3, 0, 0), (62, 32, 1, 0.25, 0.3, 0, 0), (92, 24, 1, 0.25, 0.3, 0, 0), (222, 40, 2, 0.05, 0.3, 0, 0),
    (222, 8, 2, 0.25, 0.3, 1, 0), (222, 12, 2, 0.25, 0.3, 1, 0), (222, 24, 2, 0.25, 0.3, 1, 1), (492, 24, 4, 0.3, 0.3, 1, 1),
    (40, 40, 1, 0.25, 0.9, 0, 0), (138, 10, 1, 0.25, 0.9, 1, 1), (150, 12, 1, 0.1, 0.5, 0, 0), (222, 12, 1, 0.25, 0.9, 1, 1),
    (220, 40, 0, 0.1, 0.3, 0, 0), (94, 16, 0, 0.1, 0.3, 1, 1), (220, 24, 0, 0.2, 0.5, 0, 0), (222, 24, 2, 0.25, 0.9, 1, 1),
    (444, 24, 4, 0.25, 0.9, 0, 0), (700, 12, 4, 0.1, 0.9, 0, 0)])
def test_steps_of_32_keys(driver, blocks, heads, text, topk, p, cuts, whole):
    row = (1, 1, 64 * (blocks - text) - 3, 64 * text, 1, heads, 128, 64, topk, p)
    assert _run(driver, [row], "keys") == [[str(cuts), str(whole)]]
    for head_dim, block in ((64, 64), (128, 128), (64, 128), (128, 32)):
        assert _run(driver, [(1, 1, block * (blocks - text) - 3, 64 * text, 1, heads, head_dim, block, topk, p)],
                    "keys") == [["0", "0"]]


# Text rows of such calls are cut into parts that a call with short lists of its own does not wait for: no longer than they were in steps
# of 64 keys, which take three quarters of the time a block, where one generation has room for them.
@pytest.mark.parametrize("blocks,heads,text,topk,parts", [
    (120, 9, 1, 0.25, 5), (222, 8, 2, 0.25, 5), (222, 12, 2, 0.25, 4), (300, 5, 1, 0.25, 5), (222, 16, 2, 0.2, 3), (160, 9, 2, 0.25, 4),
    (222, 24, 2, 0.25, 2), (492, 24, 4, 0.3, 2), (62, 60, 1, 0.25, 1), (120, 13, 1, 0.1, 1)])
def test_parts_of_text_rows_in_steps_of_32_keys(driver, blocks, heads, text, topk, parts):
    row = (1, 1, 64 * (blocks - text) - 3, 64 * text, 1, heads, 128, 64, topk, 0.3)
    assert int(_run(driver, [row], "deal", "7")[0][0]) == parts


# Planes of a stage switch: 2^24 of them are more than one grid takes with a workgroup each.
def test_stage_switch_launches_stay_below_the_grid_limit(driver):
    rows = [(channels, t, h, w, t, h, w, 1) for channels in (1, 16, 1 << 20, (1 << 24) - 1, 1 << 24, (1 << 31) - 1)
            for t in (1, 33) for h, w in ((1, 1), (1, 4), (3, 7), (68, 120), (45, 79))]
    for row, (tiled, rows_per_wg, _) in zip(rows, _run(driver, rows, "switch")):
        assert not int(tiled) or row[0] * row[4] * 256 < 1 << 32, row
        assert not int(tiled) or -(-row[5] // int(rows_per_wg)) <= 65535
    assert all(int(got[0]) for row, got in zip(rows, _run(driver, rows, "switch")) if row[0] == 16 and row[2] > 9)


# Small planes off the 16-byte grid are not worth a workgroup each; rows on it are staged as long as they fit.
@pytest.mark.parametrize("shape_in,shape_out,tiled", [
    ((8, 1, 1), (8, 1, 1), 0), ((8, 2, 5), (8, 3, 7), 0), ((61, 3, 3), (60, 5, 5), 0), ((8, 11, 21), (8, 11, 21), 0),
    ((8, 7, 13), (8, 14, 26), 0), ((8, 7, 13), (8, 10, 18), 0), ((8, 11, 21), (8, 15, 29), 1), ((8, 17, 31), (8, 17, 31), 0),
    ((33, 45, 79), (33, 67, 117), 1), ((33, 91, 161), (11, 30, 53), 1), ((8, 25, 45), (8, 35, 63), 1),
    ((8, 2, 4), (8, 3, 6), 1), ((33, 68, 120), (33, 90, 160), 1), ((8, 9, 16), (8, 2, 4), 1)])
def test_stage_switch_small_planes_are_not_staged(driver, shape_in, shape_out, tiled):
    for channels in (1, 16, 4096):
        assert int(_run(driver, [(channels, *shape_in, *shape_out, 1)], "switch")[0][0]) == tiled


def _window(o, n_in, n_out):
    return o * n_in // n_out, -(-(o + 1) * n_in // n_out)


# Every workgroup's input rows fit the tile that the launch asks for: up, down, same size, rows on and off the 16-byte grid.
def test_stage_switch_tiles_hold_what_is_staged(driver):
    sizes = [(1, 1), (1, 3), (2, 2), (3, 2), (4, 9), (9, 4), (13, 18), (20, 20), (33, 10), (68, 90), (45, 67), (120, 7)]
    rows = [(2, ti, hi, wi, to, ho, wo, 1) for hi, ho in sizes for wi, wo in sizes + [(120, 160), (1031, 1033), (2048, 2560)]
            for ti, to in ((1, 1), (3, 3), (5, 4), (4, 9), (9, 2))]
    tiled = 0
    for (_, ti, hi, wi, to, ho, wo, _), got in zip(rows, _run(driver, rows, "switch")):
        per_wg, floats = int(got[1]), int(got[2])
        if not int(got[0]):
            continue
        tiled += 1
        assert floats * 4 <= 48 << 10
        cells_t = max(b - a for a, b in (_window(t, ti, to) for t in range(to)))
        cells_h = max(_window(min(h + per_wg, ho) - 1, hi, ho)[1] - _window(h, hi, ho)[0] for h in range(0, ho, per_wg))
        pitch = cells_h * wi if wi % 4 == 0 else (cells_h * wi + 6) // 4 * 4
        assert cells_t * pitch <= floats, (ti, hi, wi, to, ho, wo)
    assert tiled > 300


# Rows on the 16-byte grid need no room for a boundary below them: tiles of exactly 48 KB are staged.
@pytest.mark.parametrize("shape_in,shape_out,rows", [((33, 8, 2048), (33, 8, 2048), 1), ((33, 12, 2048), (33, 15, 2560), 1),
                                                     ((5, 96, 256), (5, 72, 64), 16)])
def test_stage_switch_tiles_up_to_the_limit(driver, shape_in, shape_out, rows):
    tiled, per_wg, floats = [int(x) for x in _run(driver, [(16, *shape_in, *shape_out, 1)], "switch")[0]]
    assert tiled and floats <= 12288 and per_wg == rows
