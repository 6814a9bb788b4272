"""Registers spilled to scratch, read from the code objects of the built library:
no form of the panel and direct-B kernels does but the ones named here."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2606_21023_amd import build as hbuild

READELF = "/opt/rocm/llvm/bin/llvm-readelf"

# The forms that spill, and at most how many VGPRs: the panel kernel's template
# arguments are INT16, alpha, chunks of K, steps in flight, rows, ragged rows of
# C; the direct-B kernel's begin with the product (0 HEAL-Base, 1 HEAL-Full, 3
# pre-split, 4 bf16x3), B's source (0 packed, 1 N x K, 2 K x N), the 16-row blocks
# of a wave and waves along M, and end with the K tail.
KNOWN = {
    "gemm_panel_kernel<false, false, 4, 1, 128, false>": 2,
    "gemm_panel_kernel<false, false, 4, 1, 32, true>": 9,
    "gemm_panel_kernel<false, true, 4, 1, 32, true>": 9,
    # 128 x 256
    "gemm_direct_kernel<0, 0, 8, 1, 4, 4, 1, 2, 4, 2, false, false, false>": 11,
    "gemm_direct_kernel<0, 0, 8, 1, 4, 4, 1, 2, 4, 2, false, false, true>": 18,
    "gemm_direct_kernel<1, 0, 8, 1, 4, 4, 1, 2, 4, 2, false, false, false>": 12,
    "gemm_direct_kernel<1, 0, 8, 1, 4, 4, 1, 2, 4, 2, false, false, true>": 20,
    "gemm_direct_kernel<3, 0, 8, 1, 4, 4, 1, 2, 4, 2, false, false, false>": 44,
    "gemm_direct_kernel<3, 0, 8, 1, 4, 4, 1, 2, 4, 2, false, false, true>": 58,
    # 96 x 256
    "gemm_direct_kernel<3, 0, 6, 1, 4, 4, 1, 2, 4, 4, false, false, true>": 10,
    # 64 x 64
    "gemm_direct_kernel<4, 2, 4, 1, 1, 4, 4, 4, 4, 2, true, false, true>": 4,
}


def code_objects(path):
    """The device code objects of a library's offload bundles."""
    data, magic = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + ln].decode()
            p += 24 + ln
            if "gfx950" in triple:
                yield data[at + off:at + off + size]
        at = data.find(magic, at + 24)


def spills(tmp_path):
    """VGPRs spilled by every kernel: {demangled name: count}."""
    out = {}
    for i, obj in enumerate(code_objects(hbuild.LIBRARY)):
        f = tmp_path / ("%d.co" % i)
        f.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n  - \.a", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            out[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    names = subprocess.run(["c++filt"], input="\n".join(out), text=True, capture_output=True, check=True).stdout
    return dict(zip(names.split("\n"), out.values()))


def test_only_the_named_forms_spill(tmp_path):
    if not (os.path.exists(hbuild.LIBRARY) and os.path.exists(READELF) and shutil.which("c++filt")):
        pytest.skip("libheal.so, llvm-readelf or c++filt not available")
    found = {}
    total = 0
    for name, n in spills(tmp_path).items():
        m = re.search(r"(gemm_(?:panel|direct)_kernel<.*>)\(", name)
        total += m is not None
        if m and n:
            found[m.group(1)] = n
    assert total > 100, "kernels not found in the library"
    assert {k: n for k, n in found.items() if n > KNOWN.get(k, 0)} == {}
