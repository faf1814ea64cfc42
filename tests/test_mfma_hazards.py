"""CPU check of the built bf16 expert kernels' instructions.  Their MFMAs stand in inline assembly, where the compiler does
not insert the matrix unit's wait states, so the built code has to keep them by itself: a vector instruction that
writes an MFMA's weight or token operand at least two wait states before it, nothing but MFMAs on the same accumulator within
eight wait states of an MFMA's write.  The kernels also keep their arguments and accumulators in registers (no scratch) and
load from global memory without the detour that waits for LDS (no flat loads)."""
import os
import re
import subprocess

import pytest

from paper_2503_09304_amd import build

LLVM = "/opt/rocm/llvm/bin"
REG = re.compile(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def regs(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        lo, hi = (int(lo), int(hi)) if lo else (int(one), int(one))
        out.update((kind, i) for i in range(lo, hi + 1))
    return out


def kernels(name, tmp):
    """[(kernel, [instructions])] of one object file of the build."""
    obj = os.path.join(build.OBJ, name + ".hip.o")
    if not os.path.exists(obj):
        build.build()
    fat, dev = str(tmp / "fat"), str(tmp / "dev")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, str(tmp / "copy.o")], check=True, timeout=60)
    listed = subprocess.run([f"{LLVM}/clang-offload-bundler", "--list", "--type=o", f"--input={fat}"], capture_output=True, text=True, check=True, timeout=60)
    target = next(t for t in listed.stdout.split() if "gfx950" in t)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--targets={target}", f"--output={dev}"], check=True, timeout=60)
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", dev], capture_output=True, text=True, check=True, timeout=300).stdout
    out = []
    for line in text.splitlines():
        m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
        if m:
            out.append((m.group(1), []))
        elif out and line.startswith("\t"):
            out[-1][1].append(line.split("//")[0].strip())
    return [(k, i) for k, i in out if any("v_mfma" in x for x in i)]


def waits(ins):
    return int(ins.split()[1], 0) + 1 if ins.startswith("s_nop") else 1


@pytest.mark.parametrize("name", ["experts_bf16_w%d_%s" % (w, k) for w in (0, 1, 2) for k in ("gate_up", "down")])
def test_mfma_wait_states(name, tmp_path):
    found = kernels(name, tmp_path)
    # five sizes with 4-bit weights, else four; streaming or not; the narrow down projection
    assert len(found) == (10 if "_w2_" in name else 8) + name.endswith("_down")
    for kernel, ins in found:
        assert not [x for x in ins if x.startswith(("scratch_", "flat_"))], kernel
        assert sum("v_mfma_f32_16x16x32_bf16" in x for x in ins) == sum("v_mfma" in x for x in ins)
        for at, x in enumerate(ins):
            if not x.startswith("v_mfma"):
                continue
            dst, w, t, c = (regs(p) for p in x.split(None, 1)[1].split(", "))
            assert dst == c and len(dst) == 4 and all(k == "a" for k, _ in dst), x
            left, i = 2, at - 1
            while left > 0 and i >= 0:
                y = ins[i]
                if y.startswith("v_") and not y.startswith("v_mfma"):
                    parts = y.split(None, 1)[1].split(", ")
                    written = regs(parts[0]) | (regs(parts[1]) if "swap" in y else set())
                    assert not written & (w | t | c), (kernel, y, x)
                left -= waits(y)
                i -= 1
            left, i = 8, at + 1
            while left > 0 and i < len(ins):
                y = ins[i]
                if y.startswith("v_mfma"):
                    break                                    # it and those after it are looked at in their turn: 4 cycles each and more
                assert not regs(y) & dst, (kernel, x, y)
                left -= waits(y)
                i += 1


@pytest.mark.parametrize("name", ["experts_bf16_w2_gate_up", "experts_bf16_w2_down"])
def test_conversions_stand_between_mfmas(name, tmp_path):
    """4-bit weights: at most 12 conversions between one MFMA and the next.  16 of them in a row (all of an MFMA step's, as in
    front of a variant's first iteration) leave the matrix unit idle where a workgroup has a CU to itself."""
    for kernel, ins in kernels(name, tmp_path):
        tcap = re.search(r"expert_bf16ILi(\d)E", kernel)
        variants = {1: 2, 2: 3, 4: 7, 6: 11, 8: 15}[int(tcap.group(1))] if tcap else 2      # copies of the loop: 1, 2, 4, 5 .. 2 * tcap fragments
        gaps, run = [], 0
        for x in ins:
            if x.startswith("v_mfma"):
                gaps.append(run)
                run = 0
            run += x.startswith("v_cvt_scalef32_pk_bf16_fp4")
        assert max(gaps) <= 16 and sum(g > 12 for g in gaps) <= variants, (kernel, sorted(gaps)[-variants - 3:])
