"""The wavefront sums refuse, at compile time, workgroups whose last segment is not whole (no GPU).

A shuffle from a lane that the workgroup does not have is undefined, so a butterfly over it is too."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0906_4548_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")


def _compiles(tmp_path, width, threads, kind):
    src = tmp_path / "sum.hip"
    src.write_text('#include "control.h"\n__global__ void k(%s* x) { x[threadIdx.x] = dgp::wave_sum<%d, %d>(x[threadIdx.x]); }\n'
                   % (kind, width, threads))
    r = subprocess.run([HIPCC, "-fsyntax-only", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature",
                        "-Xclang", "-packed-fp32-ops", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-x", "hip",
                        str(src)], capture_output=True, text=True)
    assert r.returncode == 0 or "every segment must be whole" in r.stderr, r.stderr
    return r.returncode == 0


@pytest.mark.skipif(not HIPCC, reason="needs hipcc")
@pytest.mark.parametrize("kind", ["double", "int"])
def test_wave_sum_needs_whole_segments(tmp_path, kind):
    assert _compiles(tmp_path, 64, 192, kind) and _compiles(tmp_path, 8, 8, kind) and _compiles(tmp_path, 32, 96, kind)
    for width, threads in ((64, 24), (64, 48), (64, 96), (48, 48)):
        assert not _compiles(tmp_path, width, threads, kind)
