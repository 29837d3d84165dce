"""Register use of kernels whose speed hangs on how many wavefronts share a SIMD, read from the
metadata of the built library (a SIMD of gfx950 has 512 vector registers per lane, so two
wavefronts take at most 256 each)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1211_0540_amd import bz


def _readelf():
    for p in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf"), "llvm-readelf"):
        if shutil.which(p):
            return p
    pytest.skip("llvm-readelf is not installed")


def _code_objects(path):
    """The gfx950 code objects of every offload bundle in the library."""
    data, magic, at, out = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", 0, []
    while (at := data.find(magic, at)) >= 0:
        (n,), p = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in triple and size:
                out.append(data[at + off:at + off + size])
        at += len(magic)
    return out


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: vector registers} of the library's kernels."""
    tool, co, found = _readelf(), tmp_path_factory.mktemp("co") / "k.co", {}
    for obj in _code_objects(bz.LIBPATH):
        co.write_bytes(obj)
        text = subprocess.run([tool, "--notes", str(co)], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"\n  - (?=\.)", text)[1:]:
            sym, vgpr = re.search(r"\.symbol:\s+(\S+)", block), re.search(r"\.vgpr_count:\s+(\d+)", block)
            if sym and vgpr:
                found[sym.group(1)] = int(vgpr.group(1))
    assert found
    return found


def test_fp64_batches_of_n16_keep_two_wavefronts_per_simd(kernels):
    """The kernels that hold whole 64-cell groups of the N = 16 mesh."""
    n16 = {k: v for k, v in kernels.items() if re.search(r"k_conv_cells_f64ILi16E(Li[01]E)?E", k)}
    assert n16
    assert all(v <= 256 for v in n16.values()), n16
