"""test_compiled_backward_kernels.py with the planned kernels, and where the D = 128 loops of 32-row waves start.  (The 64-row
kernels: test_bwd_wide_loop.py.)"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_registers_and_loop_starts_of_the_planned_kernels_too(tmp_path):
    from paper_2512_18134_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    out = str(tmp_path / "bwd.s")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([hipcc] + flags + ["-S", "--cuda-device-only", "-o", out,
                                      os.path.join(ROOT, "paper_2512_18134_amd", "csrc", "attn_bwd.hip")],
                   check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    text = open(out).read()
    seen = []
    for block in text[text.index("amdhsa.kernels:"):].split("  - .agpr_count:")[1:]:
        m = re.search(r"\.name:\s+\S*attn_bwd_asm_(?:planned_)?kernelILi(\d+)E", block)
        if not m:
            continue
        value = lambda key: int(re.search(r"\.%s:\s+(\d+)" % key, block).group(1))
        assert value("private_segment_fixed_size") == 0 and value("vgpr_spill_count") == 0, block[:400]
        assert value("vgpr_count") <= (256 if m.group(1) == "64" else 512)     # VGPRs and AGPRs together
        seen.append(m.group(1))
    # with a plan or without, causal or not, element type
    assert seen.count("64") == seen.count("128") == 8
    # the loops of 32-row waves at D = 128 start 12 bytes behind a multiple of 32 (gen_attn_bwd_loop.py)
    loops = 0
    for m in re.finditer(r"^_ZN4attn\d+attn_bwd_asm_(?:planned_)?kernelILi128E\S+:(.*?)^\.Lfunc_end", text, re.M | re.S):
        lines = [l.strip() for l in m.group(1).split("\n") if l.strip()]
        for i in [i for i, l in enumerate(lines) if re.match(r"BODY0_\d+:", l)]:
            assert lines[i - 4:i] == [".p2align 5"] + 3 * ["s_nop 0"], lines[i - 5:i + 1]
            loops += 1
    assert loops == 16        # two sweeps a kernel
    assert re.search(r"\.p2align\s+8.*\n(.*\n){0,3}_ZN4attn\d+attn_bwd_asm_planned_kernelILi128E", text)
