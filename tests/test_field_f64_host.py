"""The floating-point field of the split transforms (csrc/ntt_field.hpp) built for
the host and run on the CPU: its own passes, reductions, products (of unreduced
operands where the field takes them) and key sums of 1 to 16 digits, against the
same transforms in integers, with congruent values pushed to the ends of the ranges
that the header derives (host_field_f64.cpp)."""
import os
import shutil
import subprocess

import pytest

from oracle import bfv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_field_at_its_bounds(tmp_path):
    if shutil.which(HIPCC) is None:
        pytest.skip("no hipcc")
    exe = str(tmp_path / "host_field_f64")
    subprocess.run([HIPCC, "--offload-host-only", "--offload-arch=gfx950", "-x", "hip", "-w", "-O2", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2204_12201_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host_field_f64.cpp"), "-o", exe], check=True)
    # the largest primes of both classes: below 2^47, and below 2^50
    ps = [q for bits in (47, 50) for q in bfv.ntt_primes(16384, bits, 2)]
    assert [q >> 47 for q in ps] == [0, 0, 7, 7]
    r = subprocess.run([exe, *map(str, ps)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
