"""What the hand-scheduled backward kernels need of the compiler (hipcc -S of csrc/attn_bwd.hip): no vector register in
scratch memory, and at D = 64 no more than 256 registers a wave, so that two workgroups share a CU."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_registers_of_the_hand_scheduled_sweeps(tmp_path):
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
    seen = 0
    for block in text[text.index("amdhsa.kernels:"):].split("  - .agpr_count:")[1:]:
        m = re.search(r"\.name:\s+\S*attn_bwd_asm_kernelILi(\d+)E", block)
        if not m:
            continue
        value = lambda key: int(re.search(r"\.%s:\s+(\d+)" % key, block).group(1))
        assert value("private_segment_fixed_size") == 0 and value("vgpr_spill_count") == 0
        assert value("vgpr_count") <= (256 if m.group(1) == "64" else 512)     # VGPRs and AGPRs together
        seen += 1
    assert seen == 8          # D, causal, element type
