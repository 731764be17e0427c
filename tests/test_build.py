"""What the compiler reports of a kernel's registers, and what the build refuses."""
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
