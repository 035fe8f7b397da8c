"""The build refuses subset-tree kernels that use scratch."""
import pytest

from paper_2010_15595_amd import build

REPORT = """csrc/a.hip:1:0: remark: Function Name: _ZN3gbs15charpoly_kernelE [-Rpass-analysis=kernel-resource-usage]
csrc/a.hip:1:0: remark:     ScratchSize [bytes/lane]: 16 [-Rpass-analysis=kernel-resource-usage]
csrc/a.hip:9:0: remark: Function Name: _ZN3gbs15tree_sub_kernelILi28EEEv [-Rpass-analysis=kernel-resource-usage]
csrc/a.hip:9:0: remark:     VGPRs: 256 [-Rpass-analysis=kernel-resource-usage]
csrc/a.hip:9:0: remark:     ScratchSize [bytes/lane]: {} [-Rpass-analysis=kernel-resource-usage]
"""


def test_scratch_in_a_tree_kernel_fails_the_build():
    build.check_tree_scratch(REPORT.format(0), "a.hip")
    with pytest.raises(RuntimeError, match="tree_sub_kernel"):
        build.check_tree_scratch(REPORT.format(88), "a.hip")
    with pytest.raises(RuntimeError, match="tree_sub_kernel"):
        build.check_tree_scratch(REPORT.format(""), "a.hip")
