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


@pytest.fixture(scope="module")
def kernels_256(tmp_path_factory):
    """Name -> assembly lines of the 256-row GEMM kernels."""
    out = tmp_path_factory.mktemp("isa") / "k.s"
    subprocess.run(["hipcc", *bld.FLAGS, "-S", "--offload-device-only", os.path.join(bld.CSRC, "gemm_bf16.hip"), "-o", str(out)], check=True,
                   capture_output=True)
    return {m[1]: m[0].split("\n")
            for m in re.finditer(r"^(_ZN\S*gemm_bf16_kernel\S*):\s.*?^\.Lfunc_end\d+:", out.read_text(), re.S | re.M)}


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_slices_of_the_256_row_tiles_need_few_scalar_instructions(kernels_256):
    """The loop over 64-wide slices (32 MFMAs of a 256 x 256 tile's wavefront).  Scalar instructions issue in order and 9 cycles apart where
    they depend on each other: with 79 to 90 of them per slice (descriptors whose base advances) launches were 2 % slower than with 54 to 74."""
    for name, body in kernels_256.items():
        labels = {m[1]: i for i, ln in enumerate(body) if (m := re.match(r"(\.LBB\S+):", ln))}
        loops = []                        # (of a branch that leads back around the loop as well, the shorter way counts)
        for i, ln in enumerate(body):
            m = re.match(r"\ts_c?branch\S*\s+(\.LBB\S+)", ln)
            if not m or labels.get(m[1], i) >= i:
                continue
            ops = [b.split()[0] for b in body[labels[m[1]]:i] if re.match(r"\t[vsdgb][a-z]*_", b)]
            if sum(op.startswith("v_mfma") for op in ops) == 32:
                loops.append(sum(op.startswith("s_") and op not in ("s_waitcnt", "s_barrier", "s_nop") for op in ops))
        assert loops and min(loops) <= 76, f"{name}: {loops}"
    assert len(kernels_256) >= 20


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_down_epilogue_waits_for_none_of_the_next_tile(kernels_256):
    """The epilogue of the down-projection reads one scalar per row.  Asked for pass by pass, behind stores that a branch may leave out, the
    waits for them could not be counted and were for every load in flight, the next tile's two slices included."""
    found = 0
    for name, body in kernels_256.items():
        if not re.search(r"TileILi256ELi256E\S*EELi1ELb0ELb0E", name):        # EPI_DOWN, no gathered statistic, k-contiguous
            continue
        first = next(i for i, ln in enumerate(body) if "v_permlane16_swap" in ln)
        last = max(i for i, ln in enumerate(body) if "buffer_store" in ln)
        waits = [int(m[1]) for ln in body[first:last] if (m := re.match(r"\ts_waitcnt.*vmcnt\((\d+)\)", ln))]
        assert waits and min(waits) >= 7, waits
        found += 1
    assert found == 1


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_256_row_tiles_ask_for_all_lines_of_their_arguments_at_once(kernels_256):
    """Six cache lines of arguments; each that is asked for later is a wait of its own before a workgroup's first loads."""
    for name, body in kernels_256.items():
        first = next(i for i, ln in enumerate(body) if re.match(r"\ts_waitcnt.*lgkmcnt", ln))
        lines = {int(m[1], 16) // 64 for ln in body[:first] if (m := re.match(r"\ts_load_dword\S* \S+, s\[0:1\], (0x[0-9a-f]+)", ln))}
        assert lines == set(range(6)), f"{name}: {sorted(lines)}"
