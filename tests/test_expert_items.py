"""The order in which a bf16 expert launch deals its work to the XCDs (csrc/expert_items.h), on the CPU:
host_stub/items_test.cpp walks the workgroups of launches with 1 to 384 segments and 1 to 128 columns."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = os.path.join(ROOT, "tests", "host_stub")


def test_every_item_once_and_equal_shares(tmp_path):
    exe = str(tmp_path / "items_test")
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-I", STUB, "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2503_09304_amd", "csrc"), os.path.join(STUB, "items_test.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "all item checks passed" in r.stdout, r.stdout[-2000:]
