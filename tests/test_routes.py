"""Which kernel an automatic call takes: the host's choice alone, no GPU needed.

Every kernel gives the same bits, so a wrong choice shows in the time only; the
times behind each case are measured ones (us on one MI355X)."""
import os
import shutil
import subprocess

import pytest

from paper_2606_21023_amd import build as hbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BASE, FULL, I16, PRESPLIT, KN, NK = range(6)


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(hbuild.LIBRARY):
        pytest.skip("g++ or libheal.so not available")
    exe = str(tmp_path_factory.mktemp("routes") / "routes")
    libdir = os.path.dirname(hbuild.LIBRARY)
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", hbuild.INCLUDE, "-I", hbuild.CSRC,
                    "-I", "/opt/rocm/include", os.path.join(ROOT, "tests", "c", "routes.cpp"), "-L", libdir,
                    "-lheal", "-Wl,-rpath," + libdir, "-o", exe], check=True)

    def ask(calls):
        """One route per call: (kind, M, N, K, batch, extra elements per row of A, B
        and C, bytes off 16-byte alignment of A, B and C), all from `batch` optional."""
        full = [c + (1, 0, 0, 0, 0, 0, 0)[len(c) - 4:] for c in calls]
        r = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in full), text=True,
                           capture_output=True, check=True)
        out = r.stdout.splitlines()
        assert len(out) == len(full)
        return out
    return ask


def test_batches_take_the_large_tiles_that_the_plan_finds_fastest(routes):
    """One round of 256 x 256 tiles takes a batch whose entries are small; the
    size of one entry would choose 128 x 128 ones (64 x 512 x 512 x 4096 K x N:
    354 us, 535 on the 128 x 128 ones; 16 x 1024 x 1024 x 4096 298, 450, N x K 297, 453)."""
    calls = [(KN, 512, 512, 4096, 64), (KN, 1024, 1024, 4096, 16), (NK, 1024, 1024, 4096, 16)]
    assert routes(calls) == ["large"] * 3
