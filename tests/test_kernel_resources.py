"""Registers and LDS of kernels whose speed rests on how many workgroups share a CU, as the compiler reports them."""
import os
import re
import subprocess

from paper_2503_09304_amd import build


def usage(src, tmp_path):
    """{mangled kernel name: (vector registers, bytes of LDS)}"""
    cmd = [build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(build.CSRC, src), "-o", str(tmp_path / "kernels.o")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    out = {}
    for part in r.stderr.split("Function Name: ")[1:]:
        regs = [int(re.search(rf"\b{what}: (\d+)", part).group(1)) for what in ("VGPRs", "AGPRs")]
        out[part.split()[0]] = sum(regs), int(re.search(r"LDS Size \[bytes/block\]: (\d+)", part).group(1))
    return out


def test_two_router_workgroups_share_a_cu(tmp_path):
    """512 threads are 2 waves on each SIMD of 512 registers: two workgroups need at most 128 registers and 80 KB of LDS."""
    seen = 0
    for name, (regs, lds) in usage("route.hip", tmp_path).items():
        nb = re.search(r"gate_topk_bf16ILi(\d+)E", name)
        if nb and int(nb.group(1)) <= 8:
            seen += 1
            assert regs <= 128 and lds <= 80 * 1024, (name, regs, lds)
    assert seen == 4
