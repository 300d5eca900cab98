"""Host-side guard on the generated code of the hot kernels (needs hipcc, no GPU).

The tiled kernel's main loop keeps its DMA queue full only as long as the compiler reloads no
spilled register inside it (it cannot see the inline-assembly loads and drains the queue
before any scratch access it schedules there).  A spill costs 5 to 14 % without failing any
parity test (the integer re-bias at 128 rows: six registers, 340 us instead of 298 at
512 x 22016 x 8192), so every instantiation of the kernel is held to a scratch size of zero."""
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2312_08583_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _kernel_field(source: str, field: str) -> dict:
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        flags = [f for f in B.FLAGS if f not in ("-fPIC",)]
        subprocess.run(["hipcc", *flags, "-S", "--cuda-device-only", os.path.join(B.CSRC, source), "-o", out],
                       check=True, stderr=subprocess.DEVNULL)
        text = open(out).read()
    return {m.group(1): int(m.group(2)) for m in re.finditer(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.%s:\s+(\d+)" % field, text)}


def _scratch_sizes(source: str) -> dict:
    return _kernel_field(source, "private_segment_fixed_size")


# the FP6 kernels; those of the ablations, fine-grained scales, FP5 and plane layout 2; those of bf16
@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("source,kernels", [("fp6_gemm.hip", 7), ("fp6_gemm_variants.hip", 22), ("fp6_gemm_bf16.hip", 6)])
def test_tiled_kernels_do_not_spill(source, kernels):
    sizes = {k: v for k, v in _scratch_sizes(source).items() if "gemm_kernel" in k}
    assert len(sizes) == kernels and all(v == 0 for v in sizes.values()), sizes


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_decode_kernels_do_not_spill():
    sizes = {k: v for k, v in _scratch_sizes("fp6_decode.hip").items() if "decode" in k}
    assert sizes and all(v == 0 for v in sizes.values()), sizes


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_short_forms_of_several_row_blocks_leave_room_for_two_wavefronts():
    """More than 256 of a SIMD's 512 registers, and workgroups past the 256th wait for a compute unit (1.2 of the time at 300 of them)."""
    regs = _kernel_field("fp6_decode.hip", "vgpr_count")
    short = {k: v for k, v in regs.items() if re.search(r"decode_kernelILi4ELi[34]ELi0ELb0ELi\dELi[24]ELb0E", k)}
    assert len(short) == 5 and all(v <= 256 for v in short.values()), short


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_the_ablations_have_the_stream_of_the_method():
    """Both forms of the stream for each unpack: the ablations are timed against the method, and the unpack is to be the only difference."""
    forms = set(re.findall(r"decode_kernelILi4ELi4ELi(\d)ELb0ELi6ELi1ELb(\d)E", " ".join(_kernel_field("fp6_decode.hip", "vgpr_count"))))
    assert forms == {(dq, exact) for dq in "012" for exact in "01"}
