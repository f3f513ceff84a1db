"""Build switches of the kernels, read from the assembly of the 3-D step kernels at
radius 1 (compiled here, no device)."""
import os
import subprocess

import pytest

from paper_1912_08063_amd import build


def _asm(out, *flags):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not available")
    subprocess.run([build.HIPCC] + build.COMMON + build.DEVICE_FLAGS +
                   ["-DFWI_STEP3D_M=1", *flags, "-x", "hip", "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "fwi_step3d.hip"), "-o", out],
                   check=True, capture_output=True)
    return [l.split(";")[0].split() for l in open(out) if "buffer_" in l]


def test_stream_cached(tmp_path):
    """FWI_STREAM_CACHED: the fields that a step reads or writes once go through the
    caches instead of past them (nt)."""
    nt = lambda lines: sum("nt" in l for l in lines)
    plain = _asm(str(tmp_path / "plain.s"))
    cached = _asm(str(tmp_path / "cached.s"), "-DFWI_STREAM_CACHED")
    assert nt(plain) > 0 and len(cached) > 0
    assert nt(cached) == 0
