"""The selection kernels' register use, from the assembly hipcc writes for
them (CPU; compiles one file).  Each keeps 32 keys a thread in registers;
anything beyond them that lives through the radix passes spills, and the
passes then run from scratch memory or through lane reads.
"""
import os
import re
import subprocess

import pytest

from paper_2511_06029_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")


def test_selection_kernels_spill_nothing(tmp_path):
    asm = tmp_path / "select.s"
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-I", build.INCLUDE, "-I", build.CSRC,
                    "-ffp-contract=fast"] + build.DEVICE_FLAGS +
                   ["-x", "hip", "--offload-device-only", "-S", os.path.join(build.CSRC, "select.hip"), "-o",
                    str(asm)], check=True, capture_output=True)
    text = asm.read_text()
    meta = text[text.index("amdhsa.kernels:"):]
    names = re.findall(r"\.name:\s+(\S*select_kernel\S*)", meta)
    assert len(names) >= 3, names
    for field in ("sgpr_spill_count", "vgpr_spill_count", "private_segment_fixed_size"):
        values = [int(v) for v in re.findall(r"\.%s:\s+(\d+)" % field, meta)]
        assert len(values) == len(names)
        assert dict(zip(names, values)) == dict.fromkeys(names, 0), field
