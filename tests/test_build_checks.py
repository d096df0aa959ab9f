"""The build's register check: what the compiler reports of each kernel, and which reports it takes."""
from paper_1912_09327_amd import build as B

REPORT = """x.hip:1:0: remark: Function Name: _ZN4lbt1{name} [-Rpass-analysis=kernel-resource-usage]
x.hip:1:0: remark:     ScratchSize [bytes/lane]: {scratch} [-Rpass-analysis=kernel-resource-usage]
x.hip:1:0: remark:     SGPRs Spill: {sgpr} [-Rpass-analysis=kernel-resource-usage]
x.hip:1:0: remark:     VGPRs Spill: {vgpr} [-Rpass-analysis=kernel-resource-usage]
"""
FP64_MARCH = "13k_step3_marchILi0ELi27ELb1ELi0ELi2ELi7ELi2ELi0EEEvNS_9Step3ArgsENS_9March3MapE"
FP32_MARCH = FP64_MARCH.replace("ILi0ELi27E", "ILi1ELi27E")


def _bad(name, scratch=0, sgpr=0, vgpr=0):
    (k, v), = B._resources(REPORT.format(name=name, scratch=scratch, sgpr=sgpr, vgpr=vgpr)).items()
    return B.spills(k, v)


def test_every_kernel_source_is_checked():
    assert {s for s, _ in B.UNITS} - set(B.CHECKED) == {"lbt1_runtime.hip", "lbt1_batch.hip", "lbt1_probe.hip"}


def test_what_the_check_refuses():
    for name in (FP32_MARCH, "11k_step_tileILi1E"):
        assert not _bad(name) and _bad(name, scratch=4) and _bad(name, sgpr=1) and _bad(name, vgpr=1)
    assert not _bad(FP64_MARCH, sgpr=48)
    assert _bad(FP64_MARCH, sgpr=49) and _bad(FP64_MARCH, sgpr=1, vgpr=1) and _bad(FP64_MARCH, scratch=4)
