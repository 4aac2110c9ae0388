"""The fp32 scan that keeps its queries in registers uses nearly all of them: nothing of it may end up in scratch, where a
reload waits for all loads of the stages on their way.  Needs no GPU: the assembly of the build is read."""
import os
import re

from paper_2110_08919_amd import build as lpq_build


def test_resident_scan_keeps_nothing_in_scratch():
    lpq_build.build()
    asm = open(lpq_build.device_asm(os.path.join(lpq_build.CSRC, "search_mfma_f32.hip"))).read()
    found = re.findall(r"\.name: +\S*resident_scan_kernel\S*\n((?:.*\n)*?.*\.vgpr_spill_count: \d+)", asm)
    assert len(found) == 1
    private = re.search(r"\.private_segment_fixed_size: (\d+)", found[0])
    assert private and int(private[1]) == 0 and found[0].endswith(".vgpr_spill_count: 0")
