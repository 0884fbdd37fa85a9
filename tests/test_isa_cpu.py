"""Buffer loads straight into LDS are inline assembly, which the compiler's hazard pass does not look into: five wait states
have to pass between a vector write of a scalar register and a buffer instruction that reads it.  Checked in the
compiled kernels: no lane read into a load's descriptor (v_readfirstlane, or the reload of a spilled scalar) close before it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_12131_amd import build as bld

LOAD = re.compile(r"buffer_load_dword(?:x4)? v\d+, s\[(\d+):(\d+)\], 0 offen lds")
LANE_READ = re.compile(r"v_(?:readlane|readfirstlane)_b32 s(\d+),")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("src", ["gemm_ring32.hip", "gemm_ring64.hip", "gemm_ring64x128.hip", "gemm_ring128.hip", "gemm_joint.hip",
                                 "gemm_rows16.hip", "attention.hip"])
def test_descriptors_of_inline_loads_are_settled(src, tmp_path):
    out = tmp_path / "k.s"
    subprocess.run(["hipcc", *bld.FLAGS, "-S", "--offload-device-only", os.path.join(bld.CSRC, src), "-o", str(out)], check=True,
                   capture_output=True)
    text = out.read_text()
    code = [ln.strip() for ln in text.splitlines() if re.match(r"\s+[vsdgb][a-z]*_", ln)]
    loads = 0
    for i, ln in enumerate(code):
        m = LOAD.match(ln)
        if not m:
            continue
        loads += 1
        states = 0
        for prev in reversed(code[:i]):
            states += int(prev.split()[1]) + 1 if prev.startswith("s_nop") else 1
            lane = LANE_READ.match(prev)
            assert not (lane and int(m[1]) <= int(lane[1]) <= int(m[2]) and states <= 5), f"{src}: {prev} before {ln}"
            if states > 5:
                break
    assert loads > 0
