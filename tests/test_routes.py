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


# (call, the fast kernels, us on the one taken, us on the one taken before the
# estimates were fitted to shallow products, part rounds and rows of C of any length)
ESTIMATES = [
    ((KN, 155, 11932, 52, 3), ("large", "medium"), 18.3, 35.1),
    ((KN, 228, 10939, 24), ("medium", "direct 64128"), 13.3, 19.8),
    ((PRESPLIT, 265, 11216, 64), ("large", "medium", "direct 96256"), 10.0, 15.0),
    ((PRESPLIT, 83, 22080, 128), ("medium", "direct 64192"), 8.3, 12.4),
    ((PRESPLIT, 259, 26368, 384), ("large", "direct 64192"), 31.5, 46.9),
    ((NK, 65, 4748, 168, 7), ("large", "medium"), 18.4, 34.5),
    ((NK, 73, 17152, 192), ("direct 96128",), 9.7, 15.9),
    ((BASE, 69, 22060, 784), ("direct 64192", "medium"), 13.2, 16.8),
]


def test_the_fastest_tiles_are_found_off_the_deep_whole_products(routes):
    for got, (call, want, now, before) in zip(routes([e[0] for e in ESTIMATES]), ESTIMATES):
        assert got in want, (call, got)


def test_deep_products_keep_their_tiles(routes):
    calls = [(KN, 8192, 8192, 8192), (BASE, 2048, 14336, 4096), (PRESPLIT, 1531, 4096, 14336),
             (FULL, 256, 4096, 4096), (NK, 200, 6144, 4096), (KN, 1001, 1003, 999), (BASE, 512, 6144, 4096),
             (FULL, 1024, 4096, 4096), (FULL, 1536, 4096, 4096), (BASE, 2048, 4096, 4096)]
    assert routes(calls) == ["large", "large", "direct 96256", "direct 32128", "direct 64128", "direct 64064",
                             "direct 64192", "direct 64256", "direct 96256", "direct 128256"]


def test_few_rows_read_by_element_keep_their_strips_where_they_are_faster(routes):
    """Up to 64 rows whose operands are not whole 16-byte units (us on the strips,
    on the direct-B tile that all of them took)."""
    strips = [(BASE, 5, 4, 11216, 1, 1),          # 23.4, 42.7
              (BASE, 3, 1842, 10253),             # 22.9, 40.6
              (PRESPLIT, 3, 8, 16080, 1, 1),      # 51.2, 86.4
              (PRESPLIT, 1, 275, 11419),          # 37.7, 62.8
              (KN, 2, 8951, 5, 130),              # 45.6, 199
              (KN, 1, 26914, 24, 4, 0, 1, 0),     # 7.8, 20.6
              (NK, 2, 4, 62), (NK, 9, 15, 61)]    # 3.0, 4.4 and 3.1, 4.5
    assert routes(strips) == ["skinny"] * len(strips)
    direct = [(KN, 16, 1003, 999), (NK, 16, 1003, 999), (BASE, 64, 4093, 999), (FULL, 33, 2050, 1001)]
    assert all(r.startswith("direct") for r in routes(direct))


def test_shallow_products_of_few_rows_keep_the_skinny_kernel(routes):
    """17 to 64 rows inside the windows of the direct-B kernel but less than 512 deep
    (wide ones less than 2048): us on the skinny kernel, on the direct-B one."""
    skinny = [(FULL, 40, 64, 396),         # 5.5, 6.6
              (BASE, 40, 192, 280),        # 4.3, 5.0
              (BASE, 41, 88568, 288),      # 15.3, 18.4
              (FULL, 51, 66444, 324),      # 17.8, 22.0
              (BASE, 60, 85184, 676)]      # 27.6, 30.2
    assert routes(skinny) == ["skinny"] * len(skinny)
    direct = [(FULL, 64, 8192, 4096), (BASE, 64, 8192, 512), (PRESPLIT, 64, 14336, 4096), (BASE, 64, 65536, 4096)]
    assert all(r.startswith("direct") for r in routes(direct))


# attention scores off the large batches (us on the kernel named, on the panel
# kernel that all of them had been sent to)
OFF_THE_PANEL = [
    ((NK, 138, 8608, 128), 11.7, 25.4),      # one panel, 32 workgroups
    ((NK, 83, 9824, 128, 1, 0, 0, 1), 10.8, 16.0),
    ((NK, 200, 64, 128), 7.6, 11.7),
    ((NK, 288, 247, 128), 4.3, 13.5),
    ((NK, 1, 6720, 128), 3.4, 5.3),
    ((NK, 10, 288, 128), 3.7, 5.2),
    ((NK, 22, 11673, 128), 4.9, 6.0),
    ((NK, 2, 352, 128, 4), 3.7, 5.2),
    ((NK, 9, 749, 128, 169, 1, 8, 0), 23.3, 30.8),
    ((I16, 21, 64, 128, 2), 4.0, 5.0),
    ((I16, 54, 32, 128, 21), 5.1, 5.6),
    ((I16, 105, 18, 128, 19), 7.2, 8.1),
]
# and where it is the faster one (us on the other kernels, on the panel kernel)
ON_THE_PANEL = [
    ((NK, 2048, 2048, 128, 32), 0, 0), ((NK, 1531, 1531, 128, 32), 276.8, 130.5),
    ((NK, 4, 16384, 128, 64), 168, 99), ((NK, 50, 50, 64, 32), 6.9, 5.1),
    ((NK, 126, 267, 128, 115), 25.9, 15.8), ((NK, 24, 4352, 128, 5), 9.7, 7.0),
    ((NK, 60, 368, 128, 13), 12.6, 6.7), ((NK, 7, 4588, 28), 5.0, 3.3),
    ((I16, 1, 3001, 128, 32), 44.6, 8.6), ((I16, 1531, 1531, 128, 32), 172.7, 114.7),
    ((I16, 4, 16384, 128, 64), 0, 54.9), ((I16, 41, 480, 128, 11), 9.0, 5.8),
    ((I16, 66, 4868, 96), 7.5, 6.4),
    # codes whose rows lie so far apart that 256 of them pass 2^31 bytes, 128 do not
    ((I16, 128, 256, 128, 1, 4999872, 0, 0), 0, 0), ((NK, 64, 256, 64, 2, 2499936, 0, 0), 0, 0),
]


def test_scores_take_the_panel_kernel_where_it_is_faster(routes):
    assert "panel" not in routes([e[0] for e in OFF_THE_PANEL])
    assert set(routes([e[0] for e in ON_THE_PANEL])) == {"panel"}


def test_benchmark_labels_follow_the_choice(routes):
    """bench.py names the kernel of a product: its copy of the panel kernel's rules,
    and the library's direct-B tile, against the choice itself."""
    import random
    import bench
    rng = random.Random(17)
    methods = {"f16_base": BASE, "f16_full": FULL, "i16_scores": I16, "presplit": PRESPLIT}
    calls, names = [], []
    for _ in range(4000):
        method = rng.choice(list(methods) + ["bf16x3"] * 3)
        M, N = int(2048 ** rng.random()), int(4 * 4096 ** rng.random())
        K = 8 * rng.randint(1, 16) if rng.random() < 0.7 else 64 * rng.randint(1, 40)
        trans_b = rng.random() < 0.7
        batch = rng.choice((1, 3, 32, 100)) if method in ("bf16x3", "i16_scores") else 1
        calls.append((methods.get(method, NK if trans_b else KN), M, N, K, batch))
        names.append((method, M, N, K, trans_b, batch))
    for call, got in zip(names, routes(calls)):
        tile = bench.direct_tile(*call)
        if got == "panel":
            assert bench.panel_rows(*call), call
        elif got.startswith("direct"):
            assert tile and "direct %d%03d" % tile == got, call
        else:
            assert bench.panel_rows(*call) is None and tile is None, (call, got)
