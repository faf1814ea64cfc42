"""The order in which a bf16 expert launch deals its work to the XCDs (csrc/expert_items.h), on the CPU:
host_stub/items_test.cpp walks the workgroups of launches with 1 to 384 segments and 1 to 128 columns.  The columns of its gate-up waves."""
import os
import subprocess

from test_gpu_fragments import WAVE_COLUMNS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STUB = os.path.join(ROOT, "tests", "host_stub")


def items_test(tmp_path, *args):
    exe = str(tmp_path / "items_test")
    cmd = ["g++", "-std=c++17", "-O1", "-Wall", "-I", STUB, "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2503_09304_amd", "csrc"), os.path.join(STUB, "items_test.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]
    return r.stdout


def test_every_item_once_and_equal_shares(tmp_path):
    assert "all item checks passed" in items_test(tmp_path)


def test_wave_columns_that_the_gpu_cases_take(tmp_path):
    """Each case of test_wave_columns_of_the_rule runs with the width it is listed for, and every width is among them."""
    args = []
    for fmt, E, H, F, rows, width in WAVE_COLUMNS:
        args += [("rowmajor", "packed", "mxfp4").index(fmt), (rows + 31) // 32, E, F]
    widths = [int(v) for v in items_test(tmp_path, *args).split()]
    assert widths == [case[-1] for case in WAVE_COLUMNS]
    for fmt in ("rowmajor", "packed"):
        assert {w for case, w in zip(WAVE_COLUMNS, widths) if case[0] == fmt} == {16, 20, 24, 28, 32}


def test_few_tokens_split_the_down_projection_by_the_experts_they_reach():
    """down_ksplit = 0: the K ranges follow from the experts that max_tokens tokens reach, not from all E;
    the workspace size shows the choice."""
    import paper_2503_09304_amd as q

    def picks(E, k, H, F, tokens):
        size = {ks: q.moe_workspace_bytes(q.MoeConfig(E, k, H, F, q.MOE_BF16, 256, tokens, ks)) for ks in (0, 1, 2, 4) if ks < 2 or F % (64 * ks) == 0}
        return [ks for ks in size if ks and size[ks] == size[0]][0]

    assert [picks(8, 2, 4096, 14336, n) for n in (1, 2, 5, 8, 512)] == [4, 4, 4, 2, 2]
    assert [picks(64, 8, 2048, 1536, n) for n in (1, 2, 3, 8)] == [4, 4, 2, 1]
    assert picks(64, 8, 2048, 1408, 1) == 2          # F is a multiple of 128, not of 256


def test_the_benchmark_prices_the_planes_that_the_library_chose():
    import paper_2503_09304_amd as q
    from bench import k_ranges

    def of(tokens, ks=0, E=8, k=2, H=4096, F=14336, dtype=q.MOE_BF16):
        return k_ranges(q.MoeConfig(E, k, H, F, dtype, 256, tokens, ks))

    assert [of(n) for n in (1, 5, 8, 512, 3584)] == [4, 4, 2, 2, 1]
    assert of(64, ks=4) == 4 and of(3584, ks=2) == 2
    assert of(3, E=64, k=8, H=2048, F=1536) == 2 and of(64, E=4, H=128, F=256, dtype=q.MOE_F32) == 1
