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
