"""The build's check of the compiler's resource report."""
import pytest

from paper_2211_01185_amd import build

REPORT = """\
csrc/dem_kernels.hip:876:0: remark: Function Name: _ZN6cfddem10force_kickIfLb1EEEvNS_3DevE [-Rpass-analysis=kernel-resource-usage]
csrc/dem_kernels.hip:876:0: remark:     TotalSGPRs: 100 [-Rpass-analysis=kernel-resource-usage]
csrc/dem_kernels.hip:876:0: remark:     VGPRs: 128 [-Rpass-analysis=kernel-resource-usage]
csrc/dem_kernels.hip:876:0: remark:     ScratchSize [bytes/lane]: {scratch} [-Rpass-analysis=kernel-resource-usage]
csrc/dem_kernels.hip:876:0: remark:     SGPRs Spill: 3 [-Rpass-analysis=kernel-resource-usage]
csrc/dem_kernels.hip:876:0: remark:     VGPRs Spill: {spill} [-Rpass-analysis=kernel-resource-usage]
csrc/couple_kernels.hip:963:0: remark: Function Name: _ZN6cfddem15couple_occupiedIdEEvNS_3DevE [-Rpass-analysis=kernel-resource-usage]
csrc/couple_kernels.hip:963:0: remark:     VGPRs Spill: 74 [-Rpass-analysis=kernel-resource-usage]
"""


def test_spilled_force_kernels_fail_the_build():
    text = REPORT.format(scratch=0, spill=0)
    r = build.kernel_resources(text)["_ZN6cfddem10force_kickIfLb1EEEvNS_3DevE"]
    assert r["VGPRs"] == 128 and r["ScratchSize"] == 0 and r["SGPRs Spill"] == 3 and r["VGPRs Spill"] == 0
    assert build.check_resources(text) == 1  # the other element kernels may spill
    with pytest.raises(RuntimeError, match="1 vector registers spilled"):
        build.check_resources(REPORT.format(scratch=8, spill=1))
    with pytest.raises(RuntimeError, match="unknown"):
        build.check_resources("\n".join(text.splitlines()[:4]))
    assert build.check_resources("") == 0
