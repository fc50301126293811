"""The build refuses kernels that spill vector registers or use scratch memory."""
import pytest

from paper_2605_08699_amd import build

LINE = "csrc/kernels.hip:{n}:1: remark:     {text} [-Rpass-analysis=kernel-resource-usage]\n"


def _report(*kernels):
    out = ""
    for n, (name, scratch, sgpr, vgpr) in enumerate(kernels):
        for text in ("Function Name: " + name, "TotalSGPRs: 40", "VGPRs: 64", "AGPRs: 0",
                     f"ScratchSize [bytes/lane]: {scratch}", "Occupancy [waves/SIMD]: 8", f"SGPRs Spill: {sgpr}",
                     f"VGPRs Spill: {vgpr}", "LDS Size [bytes/block]: 3392"):
            line = LINE.format(n=n, text=text)
            out += line.replace("remark:     Function", "remark: Function") if text.startswith("Function") else line
        out += "\n"
    return out


@pytest.mark.parametrize("scratch,vgpr", [(0, 0), (8, 0), (0, 2), (16, 4)])
def test_kernels_with_spills_or_scratch_are_named(scratch, vgpr):
    report = _report(("k_a", 0, 0, 0), ("k_b", scratch, 19, vgpr), ("k_c", 0, 0, 0))
    bad, n = build.spilling_kernels(report)
    assert n == 3
    assert bad == ([("k_b", scratch, vgpr)] if scratch or vgpr else [])


def test_a_report_without_kernels_is_noticed():
    assert build.spilling_kernels("warning: something else\n") == ([], 0)


def test_sources_are_built_with_the_report_and_the_flags_of_the_kernels():
    assert build.REPORT == ["-Rpass-analysis=kernel-resource-usage"]
    assert "-packed-fp32-ops" in build.FLAGS and "-ffp-contract=off" in build.FLAGS
