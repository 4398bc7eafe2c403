"""A launch that fails is reported: every launch of the split transforms returns the
error of the runtime (host_launch_errors.cpp, linked with the library, in place of
the runtime's launch functions)."""
import os
import shutil
import subprocess

import pytest

from paper_2204_12201_amd import fhe

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_split_launches_report_errors(tmp_path):
    if shutil.which(HIPCC) is None:
        pytest.skip("no hipcc")
    if not os.path.exists(fhe.LIBPATH):
        from paper_2204_12201_amd import build
        build.build(verbose=False)
    exe = str(tmp_path / "host_launch_errors")
    subprocess.run([HIPCC, "--offload-host-only", "--offload-arch=gfx950", "-x", "hip", "-w", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2204_12201_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host_launch_errors.cpp"), "-x", "none", fhe.LIBPATH, "-rdynamic", "-o", exe,
                    "-Wl,-rpath," + os.path.dirname(fhe.LIBPATH)], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
