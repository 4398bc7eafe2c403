"""Scratch of the kernels that full batches spend their time in, from the metadata of
the built library: registers that no longer fit go to memory on every call."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2204_12201_amd import fhe

READOBJ = shutil.which("llvm-readobj", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))


def code_objects(data):
    """The device code objects of a fat binary (uncompressed offload bundles)."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        off = at + len(magic)
        (count,) = struct.unpack_from("<Q", data, off)
        off += 8
        for _ in range(count):
            start, size, length = struct.unpack_from("<QQQ", data, off)
            name = data[off + 24:off + 24 + length]
            off += 24 + length
            if b"gfx950" in name and size:
                yield data[at + start:at + start + size]
        at = data.find(magic, off)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    if READOBJ is None:
        pytest.skip("no llvm-readobj")
    if not os.path.exists(fhe.LIBPATH):
        from paper_2204_12201_amd import build
        build.build(verbose=False)
    out = {}
    path = str(tmp_path_factory.mktemp("co") / "x.co")
    for co in code_objects(open(fhe.LIBPATH, "rb").read()):
        open(path, "wb").write(co)
        notes = subprocess.run([READOBJ, "--notes", path], capture_output=True, text=True, check=True).stdout
        for m in re.finditer(r"\.name:\s+(_Z\S+)\s.*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            out[m.group(1)] = int(m.group(2))
    assert out
    return out


@pytest.mark.parametrize("kernel,most", [
    ("k_relin_fusedILi14ELb1ELb1E", 24),   # five values at the 128-register cap
    ("k_relin_fusedILi14ELb1ELb0E", 24),
    ("k_square_tensorILi14E", 0),
    ("k_mul_tensorILi14E", 0),
])
def test_scratch(scratch, kernel, most):
    found = {k: v for k, v in scratch.items() if kernel in k}
    assert found
    assert all(v <= most for v in found.values()), found
