"""CPU check of the built bf16 expert kernels' instructions.  Their MFMAs stand in inline assembly, where the compiler does
not insert the matrix unit's wait states, so the built code has to keep them by itself, along every path: a vector
instruction that writes an MFMA's operand at least two wait states before it, nothing but MFMAs on the same accumulator within
eight wait states of an MFMA's write (an MFMA in between counts as the four that it takes).  The kernels also keep their
arguments and accumulators in registers (no scratch) and load from global memory without the detour that waits for LDS (no
flat loads)."""
import functools
import glob
import os
import re
import subprocess

import pytest

from paper_2503_09304_amd import build

LLVM = "/opt/rocm/llvm/bin"
REG = re.compile(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+)\b)")


@functools.lru_cache(maxsize=None)
def regs(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        lo, hi = (int(lo), int(hi)) if lo else (int(one), int(one))
        out.update((kind, i) for i in range(lo, hi + 1))
    return frozenset(out)


def built(name, tmp):
    """The object of the build, or one of its own if a source is newer."""
    obj, src = os.path.join(build.OBJ, name + ".hip.o"), os.path.join(build.CSRC, name + ".hip")
    read = [src] + glob.glob(os.path.join(build.CSRC, "*.h")) + glob.glob(os.path.join(build.ROOT, "include", "*.h"))
    if os.path.exists(obj) and os.path.getmtime(obj) >= max(os.path.getmtime(f) for f in read):
        return obj
    obj = str(tmp / "own.o")
    subprocess.run([build.HIPCC, *build.FLAGS, "-c", src, "-o", obj], check=True, capture_output=True, timeout=600)
    return obj


def listing(text):
    """{kernel: [(instruction, index of the branch's target or None)]} of a disassembly."""
    out, at, here = {}, {}, None
    for line in text.splitlines():
        m = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
        if m:
            here = out.setdefault(m.group(1), [])
            base = None
        elif here is not None and line.startswith("\t") and "//" in line:
            ins, _, note = line.partition("//")
            addr = int(note.split(":")[0], 16)
            base = addr if base is None else base
            at[id(here), addr - base] = len(here)
            to = re.search(r"\+0x([0-9a-f]+)>", note) if ins.strip().startswith(("s_branch", "s_cbranch")) else None
            here.append((ins.strip(), (id(here), int(to.group(1), 16)) if to else None))
    return {k: [(i, at[t] if t else None) for i, t in v] for k, v in out.items()}


def kernels(name, tmp):
    """[(kernel, [(instruction, branch target)])] of the kernels with MFMAs of one object."""
    obj, fat, dev = built(name, tmp), str(tmp / "fat"), str(tmp / "dev")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, str(tmp / "copy.o")], check=True, timeout=60)
    listed = subprocess.run([f"{LLVM}/clang-offload-bundler", "--list", "--type=o", f"--input={fat}"], capture_output=True, text=True, check=True, timeout=60)
    target = next(t for t in listed.stdout.split() if "gfx950" in t)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--targets={target}", f"--output={dev}"], check=True, timeout=60)
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", dev], capture_output=True, text=True, check=True, timeout=300).stdout
    return [(k, i) for k, i in listing(text).items() if any("v_mfma" in x for x, _ in i)]


def waits(ins, mfma):
    return int(ins.split()[1], 0) + 1 if ins.startswith("s_nop") else mfma if ins.startswith("v_mfma") else 1


def within(code, at, states, mfma):
    """Indices of the instructions fewer than `states` wait states behind instruction `at`, along every path; an MFMA counts as
    `mfma` of them."""
    todo, best = [(at, states)], {}
    while todo:
        i, left = todo.pop()
        ins, target = code[i]
        if i != at:
            left -= waits(ins, mfma)
        if left <= 0 or ins.startswith("s_endpgm"):
            continue
        for j in ([] if ins.startswith("s_branch") else [i + 1]) + ([target] if target is not None else []):
            if j < len(code) and best.get(j, 0) < left:
                best[j] = left
                todo.append((j, left))
    return best


def operands(ins):
    return [regs(p) for p in ins.split(None, 1)[1].split(", ")]


def violations(code):
    out = []
    for at, (x, _) in enumerate(code):
        if x.startswith("v_mfma"):
            dst, w, t, c = operands(x)
            assert dst == c and len(dst) == 4 and all(k == "a" for k, _ in dst), x
            for j in within(code, at, 8, 4):
                y = code[j][0]
                if regs(y) & dst and not (y.startswith("v_mfma") and operands(y)[0] == dst):
                    out.append((x, y))
        elif x.startswith("v_"):
            parts = operands(x) if " " in x else []
            written = (parts[0] | (parts[1] if "swap" in x else frozenset())) if parts else frozenset()
            for j in within(code, at, 2, 1) if written else ():
                y = code[j][0]
                if y.startswith("v_mfma") and written & regs(y):
                    out.append((x, y))
    return out


@pytest.mark.parametrize("name", ["experts_bf16_w%d_%s" % (w, k) for w in (0, 1, 2) for k in ("gate_up", "down")])
def test_mfma_wait_states(name, tmp_path):
    found = kernels(name, tmp_path)
    # five sizes with 4-bit weights, else four; streaming or not; the narrow down projection
    assert len(found) == (10 if "_w2_" in name else 8) + name.endswith("_down")
    for kernel, code in found:
        assert not [x for x, _ in code if x.startswith(("scratch_", "flat_"))], kernel
        assert sum("v_mfma_f32_16x16x32_bf16" in x for x, _ in code) == sum("v_mfma" in x for x, _ in code)
        assert not violations(code), (kernel, violations(code)[:3])


MFMA = ["v_mfma_f32_16x16x32_bf16 a[%d:%d], v[0:3], v[4:7], a[%d:%d]" % (n, n + 3, n, n + 3) for n in (0, 4, 8)]


@pytest.mark.parametrize("good,lines", [
    (True, [MFMA[0], MFMA[0], "s_nop 7", "v_accvgpr_read_b32 v20, a0"]),
    (False, [MFMA[0], "s_nop 6", "v_accvgpr_read_b32 v20, a0"]),
    (False, [MFMA[0], MFMA[1], "v_accvgpr_read_b32 v20, a0"]),                    # behind another MFMA
    (True, [MFMA[0], MFMA[1], MFMA[2], "v_accvgpr_read_b32 v20, a0"]),
    (False, ["v_accvgpr_read_b32 v20, a0", "s_nop 0", MFMA[0], "s_cbranch_scc1 -4 @0"]),     # across a loop's end
    (False, [MFMA[0], "s_branch 1 @3", "s_nop 7", "ds_write_b32 v9, a3"]),
    (False, [MFMA[0], "v_mfma_f32_16x16x32_bf16 a[2:5], v[0:3], v[4:7], a[2:5]"]),   # an accumulator that overlaps
    (False, ["v_mov_b32_e32 v5, v9", "s_nop 0", MFMA[0]]),
    (True, ["v_mov_b32_e32 v5, v9", "s_nop 1", MFMA[0]]),
    (False, ["v_permlane16_swap_b32_e32 v9, v2", MFMA[0]]),
    (False, ["v_mov_b32_e32 v5, v9", "s_cbranch_scc1 1 @3", "s_nop 7", MFMA[0]]),           # along the jump alone
])
def test_scan_finds_planted_hazards(good, lines):
    text = "0000000000001000 <k>:\n" + "".join(
        "\t%-58s // %012X:%s\n" % (x.split(" @")[0], 0x1000 + 4 * i, " <k+0x%x>" % (4 * int(x.split(" @")[1])) if " @" in x else "") for i, x in enumerate(lines))
    assert (not violations(listing(text)["k"])) == good


@pytest.mark.parametrize("name", ["experts_bf16_w2_gate_up", "experts_bf16_w2_down"])
def test_conversions_stand_between_mfmas(name, tmp_path):
    """4-bit weights: at most 12 conversions between one MFMA and the next.  16 of them in a row (all of an MFMA step's, as in
    front of a variant's first iteration) leave the matrix unit idle where a workgroup has a CU to itself."""
    for kernel, code in kernels(name, tmp_path):
        tcap = re.search(r"expert_bf16ILi(\d)E", kernel)
        variants = {1: 2, 2: 3, 4: 7, 6: 11, 8: 15}[int(tcap.group(1))] if tcap else 2      # copies of the loop: 1, 2, 4, 5 .. 2 * tcap fragments
        gaps, run = [], 0
        for x, _ in code:
            if x.startswith("v_mfma"):
                gaps.append(run)
                run = 0
            run += x.startswith("v_cvt_scalef32_pk_bf16_fp4")
        assert max(gaps) <= 16 and sum(g > 12 for g in gaps) <= variants, (kernel, sorted(gaps)[-variants - 3:])
