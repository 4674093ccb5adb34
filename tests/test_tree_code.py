"""The compiled code of the tree descent (gfx950 assembly; no GPU needed)."""
import os
import re
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, ".."))
from paper_2301_00806_amd import build as BLD  # noqa: E402

SRC = os.path.join(BLD.CSRC, "tree.hip")


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    if not os.path.exists(BLD.HIPCC):
        pytest.skip("hipcc not installed")
    out = tmp_path_factory.mktemp("asm") / "tree.s"
    cmd = ([BLD.HIPCC, "-O3", "-std=c++17"] + BLD.DEVICE + BLD.EXTRA.get("tree.hip", []) +
           ["--cuda-device-only", "-S", SRC, "-o", str(out)])
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


def test_results_are_counted_in_64_bits(asm):
    # An instance's results are counted over all the items that a workgroup
    # takes in a row, which can hold more than 2^32 of them: a wave adds those
    # of each check to a 64-bit word, and those past the ridges to another.  (A
    # third 64-bit LDS atomic returns the place in the block of record slots.)
    assert len(re.findall(r"\bds_add_u64\b", asm)) == 2


def meta(asm):
    return {k: int(re.search(r"\." + k + r":\s+(\d+)", asm).group(1))
            for k in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size", "group_segment_fixed_size")}


def test_register_budget_and_no_scratch(asm):
    # compiled for 7 waves per SIMD: at most 72 of the 512 VGPRs a lane has
    m = meta(asm)
    assert m["vgpr_count"] <= 72, m
    assert m["vgpr_spill_count"] == 0 and m["private_segment_fixed_size"] == 0, m
    assert not re.search(r"^\s*(scratch_|buffer_store|buffer_load)", asm, re.M)


def test_lds_for_seven_workgroups(asm):
    # 256 threads, rows of 44 words, 36 rows: seven workgroups, as many as the
    # registers allow, fit the 160 KB of a compute unit
    def tree_lds_bytes(max_kp, max_row_words, wg):
        nw, up = wg // 64, max(max_kp - 17, 0)
        return 4 * (nw * (192 + 64) + 56 * 16 + up * 20 + (56 + nw) * (max_row_words | 4))
    with open(os.path.join(BLD.CSRC, "tree_kernel.h")) as f:
        src = f.read()
    for text in ("TREE_LIST = 192", "CHILD_LIST = 128", "LVT_WORDS = 16", "DLV_WORDS = 20", "WIN_BITS = 21",
                 "return RS | 4;"):
        assert text in src, text
    assert 7 * (tree_lds_bytes(36, 44, 256) + meta(asm)["group_segment_fixed_size"]) <= 160 * 1024
