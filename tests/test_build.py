"""The build's check for spilled registers, on the compiler's own remarks."""
from paper_2603_16644_amd.build import spills

REPORT = """
csrc/x.hip:10:1: remark: Function Name: _Z1av [-Rpass-analysis=kernel-resource-usage]
csrc/x.hip:10:1: remark:     VGPRs: 256 [-Rpass-analysis=kernel-resource-usage]
csrc/x.hip:10:1: remark:     SGPRs Spill: 17 [-Rpass-analysis=kernel-resource-usage]
csrc/x.hip:10:1: remark:     VGPRs Spill: {a} [-Rpass-analysis=kernel-resource-usage]
csrc/x.hip:20:1: remark: Function Name: _Z1bv [-Rpass-analysis=kernel-resource-usage]
csrc/x.hip:20:1: remark:     VGPRs Spill: {b} [-Rpass-analysis=kernel-resource-usage]
"""


def test_spills_are_found():
    assert spills(REPORT.format(a=0, b=0)) == []
    assert spills(REPORT.format(a=75, b=0)) == [("_Z1av", 75)]
    assert spills(REPORT.format(a=0, b=2)) == [("_Z1bv", 2)]
    assert spills("") == []
