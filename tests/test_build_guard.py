"""The build refuses kernels whose values in inactive lanes the register
allocator could lose: accumulator registers or spilled vector registers in the
compiler's resource remarks."""
import os

import pytest

from paper_2210_12859_amd import build

KERNEL = """kd_packet.hip:268:1: remark: Function Name: {name} [-Rpass-analysis=kernel-resource-usage]
  268 | __global__ void knn_packet(PacketArgs a) {{
      | ^
kd_packet.hip:268:1: remark:     TotalSGPRs: 106 [-Rpass-analysis=kernel-resource-usage]
kd_packet.hip:268:1: remark:     VGPRs: 97 [-Rpass-analysis=kernel-resource-usage]
kd_packet.hip:268:1: remark:     AGPRs: {agprs} [-Rpass-analysis=kernel-resource-usage]
kd_packet.hip:268:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]
kd_packet.hip:268:1: remark:     SGPRs Spill: 8 [-Rpass-analysis=kernel-resource-usage]
kd_packet.hip:268:1: remark:     VGPRs Spill: {spill} [-Rpass-analysis=kernel-resource-usage]
"""


@pytest.mark.parametrize("agprs,spill,ok", [(0, 0, True), (4, 0, False), (0, 1, False)])
def test_resource_remarks(agprs, spill, ok):
    text = KERNEL.format(name="first", agprs=0, spill=0) + KERNEL.format(name="second", agprs=agprs, spill=spill)
    if ok:
        assert build.check_lane_state(text) == 2
    else:
        with pytest.raises(RuntimeError, match="second"):
            build.check_lane_state(text)


def test_no_remarks_is_no_pass():
    with pytest.raises(RuntimeError):
        build.check_lane_state("warning: nothing\n")


def test_kernels_with_lane_state_are_checked():
    """Every source that reads a wave's value from a lane by number."""
    found = {f for f in os.listdir(build.CSRC)
             if f.endswith(".hip") and "readlane(stack" in open(os.path.join(build.CSRC, f)).read()}
    assert found and found <= set(build.LANE_STATE)
