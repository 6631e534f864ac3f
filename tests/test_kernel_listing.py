"""Static check of the attention kernel's generated code (CPU only: hipcc cross-compiles to assembly).

attn_h_kernel issues its LDS fragment reads and the wait for them as separate asm statements so that the reads
of one group of fragments fly under the MFMAs of the previous group.  That is only correct if the compiler leaves
the destination registers of an issued read alone until the wait: this test reads the listing of the built code
and fails if any instruction between a `ds_read_b128` of the main loop and the next `s_waitcnt lgkmcnt(0)`
touches a register that read is still writing.  It also fails on register spills inside the main loop of an attention kernel."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_16864_amd", "csrc")


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("isa") / "jenga_attn.s")
    cmd = ["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-S", "--cuda-device-only",
           "-o", out, os.path.join(CSRC, "jenga_attn.hip")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return open(out).read()


def _regs(text):
    """Set of VGPR numbers named in an operand string."""
    regs = set()
    for a, b in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        regs.update(range(int(a), int(b) + 1))
    for a in re.findall(r"\bv(\d+)\b", text):
        regs.add(int(a))
    return regs


def _kernel_bodies(listing, name):
    for m in re.finditer(r"^(_Z\w*%s\w*):.*?^\.Lfunc_end" % name, listing, re.S | re.M):
        yield m.group(1), m.group(0)


def test_fragment_registers_untouched_between_read_and_wait(listing):
    checked = 0
    for sym, body in _kernel_bodies(listing, "attn_h_kernel"):
        pending = set()
        for line in body.split("\n"):
            ins = line.split(";")[0].strip()
            if not ins or ins.endswith(":") or ins.startswith("."):
                continue
            op, _, rest = ins.partition(" ")
            if op == "s_waitcnt" and "lgkmcnt(0)" in rest:
                pending.clear()
                continue
            if op == "ds_read_b128":
                dst, _, addr = rest.partition(",")
                assert not (_regs(dst) & pending), "%s: %s overwrites a fragment still being read" % (sym, ins)
                assert not (_regs(addr) & pending), "%s: %s" % (sym, ins)
                pending |= _regs(dst)
                checked += 1
                continue
            assert not (_regs(rest) & pending), "%s: `%s` touches a fragment register before the wait" % (sym, ins)
    assert checked >= 2 * (32 + 16)   # fragment reads per step: 32 at head dim 128, 16 at head dim 64; two walks each


# The same for V read in place, by columns: 16 or 32 reads a step and kernel at head dim 64 or 128.
def test_column_registers_untouched_between_read_and_wait(listing):
    checked = {}
    for sym, body in _kernel_bodies(listing, "attn_h_kernel"):
        pending = set()
        checked[sym] = 0
        for line in body.split("\n"):
            ins = line.split(";")[0].strip()
            op, _, rest = ins.partition(" ")
            if op == "s_waitcnt" and "lgkmcnt(0)" in rest:
                pending.clear()
            elif ins and not ins.endswith(":") and not ins.startswith("."):
                assert not (_regs(rest) & pending), "%s: `%s` touches a column register before the wait" % (sym, ins)
                if op == "ds_read_b64_tr_b16":
                    pending |= _regs(rest.partition(",")[0])
                    checked[sym] += 1
    for block, d, paced, cut, rows in ATTN_H:
        name = "attn_h_kernelILi%dELi%dELb%dELb%dELb%dEEE" % (block, d, paced, cut, rows)
        assert [n for sym, n in checked.items() if name in sym] == [rows * d // 4], name


def _step_loop(body, mfmas):
    """Text of the smallest loop with at least `mfmas` MFMAs in it, from its label to the last backward branch to it."""
    best = ""
    for m in re.finditer(r"^(\.LBB\d+_\d+):", body, re.M):
        label = m.group(1)
        back = [b.end() for b in re.finditer(r"s_cbranch_\w+ %s\b|s_branch %s\b" % (re.escape(label), re.escape(label)),
                                             body[m.end():])]
        if back:
            span = body[m.end(): m.end() + back[-1]]
            if span.count("v_mfma") >= mfmas and (not best or len(span) < len(best)):
                best = span
    return best


# block, head dim, paced, cut, K in place
ATTN_H = [(block, d, paced, cut, rows) for block in (128, 64) for d in (128, 64) for paced in (0, 1) for cut in (0, 1)
          for rows in (0, 1) if not (paced and (block == 64 or (rows and not cut)))]


def _attention_kernels(listing):
    """Symbol -> (MFMAs in the code of a step, register limit, body) of every attention kernel there has to be."""
    bodies = {}
    for block, d, paced, cut, rows in ATTN_H:
        # S = K Q^T stands in the code of a step twice (without and with the row maximum), O += V P once; 64 keys a step,
        # so d / 16 x 2 and d / 32 x 4 MFMAs.  Wavefronts per SIMD: three at head dim 128, four at 64.
        name = "attn_h_kernelILi%dELi%dELb%dELb%dELb%dEEE" % (block, d, paced, cut, rows)
        bodies[name] = (2 * (d // 8) + d // 8, 168 if d == 128 else 128)
    for d, ns in ((128, 4), (64, 8)):
        for ranges in (0, 1):   # 32 keys a step
            bodies["attn_kernelILi%dELi%dELb%dEEE" % (d, ns, ranges)] = (d // 16 + d // 16, 256 if d == 128 else 128)
    found = {}
    for sym, body in list(_kernel_bodies(listing, "attn_h_kernel")) + list(_kernel_bodies(listing, "attn_kernel")):
        names = [n for n in bodies if n in sym]
        assert len(names) == 1, sym
        found[names[0]] = (sym, *bodies[names[0]], body)
    assert set(found) == set(bodies)
    return found


def test_attention_step_loops_do_not_spill(listing):
    for sym, mfmas, _, body in _attention_kernels(listing).values():
        loop = _step_loop(body, mfmas)
        assert loop.count("v_mfma") == mfmas, (sym, loop.count("v_mfma"))
        assert "scratch_" not in loop, "%s: register spill inside the loop over the keys" % sym


def test_attention_kernels_keep_their_occupancy(listing):
    limits = {sym: (name, regs) for name, (sym, _, regs, _) in _attention_kernels(listing).items()}
    seen = set()
    for b in re.split(r"\n  - \.agpr_count", listing):
        m = re.search(r"\.name:\s+(\S+)", b)
        if not m or m.group(1) not in limits:
            continue
        name, regs = limits[m.group(1)]
        seen.add(name)

        def of(key):
            return int(re.search(r"\.%s:\s+(\d+)" % key, b).group(1))
        assert of("vgpr_count") <= regs, name
        # a few values that only the epilogue needs may sit in scratch over the loop; none is touched inside it
        assert of("vgpr_spill_count") <= (4 if "ILi128E" in name else 0), name
        # Blocks of 64 tokens copy with a 64-bit scalar base for each of twice as many copies as a wavefront of 128 has:
        # some of those go to lanes of a vector register.  No other kernel is short of scalar registers.
        assert of("sgpr_spill_count") <= (33 if "ILi64ELi128E" in name else 17 if "ILi64ELi64E" in name else 0), name
    assert len(seen) == len(limits)


# Rows for the token order are stored by instances of their own: the others store a row of results once and read no table for it.
def test_only_kernels_with_token_order_rows_store_rows_twice(listing):
    for suffix, copies in (("", 1), ("_thw", 2)):
        seen = set()
        for sym, body in _kernel_bodies(listing, "attn_h%s_kernel" % suffix):
            d = int(re.search(r"ILi\d+ELi(\d+)E", sym).group(1))
            assert body.count("global_store_dwordx2") == copies * d // 8, sym
            seen.add(sym)
        assert len(seen) == len(ATTN_H), suffix


# The instances that store rows of both orders run the same loops: nothing spilled there, and the registers leave as many wavefronts.
def test_kernels_with_token_order_rows_keep_their_loops(listing):
    seen = 0
    for sym, body in list(_kernel_bodies(listing, "attn_h_thw_kernel")) + list(_kernel_bodies(listing, "attn_32_thw_kernel")):
        d = int(re.findall(r"Li(\d+)E", sym)["attn_h" in sym])
        mfmas, limit = (3 * (d // 8), 168 if d == 128 else 128) if "attn_h" in sym else (d // 8, 256 if d == 128 else 128)
        loop = _step_loop(body, mfmas)
        assert loop.count("v_mfma") == mfmas and "scratch_" not in loop, sym
        meta = re.search(r"\.name:\s+%s\n.*?\.vgpr_count:\s+(\d+)" % re.escape(sym), listing, re.S)
        assert int(meta.group(1)) <= limit, sym
        seen += 1
    assert seen == len(ATTN_H) + 2


# Blocks of 64 tokens at head dim 128 in steps of 32 keys: the same rules as for the other attention kernels, and LDS for six
# workgroups on a CU (160 KB, given out in pieces of 1280 bytes).
def test_steps_of_32_keys_keep_the_rules(listing):
    kernels = [s for n in ("attn_keys32_kernel", "attn_keys32_thw_kernel") for s in _kernel_bodies(listing, n)]
    assert len(kernels) == 8
    for sym, body in kernels:
        pending = set()
        for line in body.split("\n"):
            ins = line.split(";")[0].strip()
            op, _, rest = ins.partition(" ")
            if op == "s_waitcnt" and "lgkmcnt(0)" in rest:
                pending.clear()
            elif ins and not ins.endswith(":") and not ins.startswith("."):
                assert not (_regs(rest) & pending), "%s: `%s` touches a register before the wait" % (sym, ins)
                if op in ("ds_read_b64_tr_b16", "ds_read_b128"):
                    pending |= _regs(rest.partition(",")[0])
        loop = _step_loop(body, 48)   # two steps: S = K Q^T twice each, O += V P
        assert loop.count("v_mfma") == 48 and "scratch_" not in loop, sym
        block = next(b for b in re.split(r"\n  - \.agpr_count", listing) if re.search(r"\.name:\s+%s\n" % re.escape(sym), b))
        assert int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1)) <= 168, sym
        lds = int(re.search(r"\.group_segment_fixed_size:\s+(\d+)", block).group(1))
        assert 6 * (-(-lds // 1280) * 1280) <= 160 << 10, (sym, lds)
