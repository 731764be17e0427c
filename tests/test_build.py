"""What the compiler reports of a kernel's registers, what the build refuses, and what the compiler makes of loops that must stay whole."""
import os
import re
import subprocess

import pytest

from paper_2605_11335_amd import build

REMARK = "csrc/k.hip:1:0: remark: {} [-Rpass-analysis=kernel-resource-usage]"


def usage(scratch=0, sgpr=0, vgpr=0):
    lines = ["Function Name: some_kernel", "    VGPRs: 256", f"    ScratchSize [bytes/lane]: {scratch}", f"    SGPRs Spill: {sgpr}", f"    VGPRs Spill: {vgpr}"]
    return build._resource_usage([REMARK.format(line) for line in lines])


def test_spilled_vector_registers_and_scratch_memory_fail_the_build():
    build._check_usage("k.hip", usage())
    build._check_usage("k.hip", usage(sgpr=12))        # scalar registers go to lanes of a vector register
    for bad in (dict(vgpr=2), dict(scratch=16), dict(scratch=16, vgpr=4)):
        with pytest.raises(RuntimeError, match="some_kernel"):
            build._check_usage("k.hip", usage(**bad))


def test_copies_of_parts_that_meet_are_not_looped_over_lanes(tmp_path):
    """Buffer accesses whose descriptor or scalar offset ends up in vector registers become loops over the lanes' values (16 of them in a main loop
    made two layers of 192x256 tiles 182 us instead of 134)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path / "gemm_meet.asm"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-pthread") and not f.startswith("-Rpass")]
    subprocess.run([hipcc] + flags + ["--cuda-device-only", "-S", "-c", os.path.join(build.CSRC, "gemm_meet.hip"), "-o", str(out)], check=True, capture_output=True)
    kernels = re.split(r"^(?=_ZN\w*kernel\w*:)", out.read_text(), flags=re.M)[1:]
    assert len(kernels) == 9 and all("v_mfma" in k for k in kernels)         # six tiles alone, three of 128 and more features in pairs
    for k in kernels:
        blocks = re.split(r"^(\.LBB\w+):", k, flags=re.M)
        loops = [label for label, body in zip(blocks[1::2], blocks[2::2]) if f"s_cbranch_execnz {label}\n" in body and "v_readfirstlane" in body]
        assert not loops, (k[:80], len(loops))
