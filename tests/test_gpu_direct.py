"""The direct-B kernel (heal_gemm_direct.hip), which most products of 65 and
more rows take by themselves: every tile configuration against the tiled
kernels of the forced instances, bit for bit, at tile edges, K tails of every
remainder and rows of every alignment.  The forced instances are checked
against the oracle elsewhere; every instance sums in one order, so no tolerance
is needed."""
import pytest
import torch

import paper_2606_21023_amd as heal
from gpu_util import announce, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

# rows x columns x depth; on 256 CUs the comment's tiles (packed B / FP32 B)
SHAPES = [
    (65, 5, 4),          # smallest: one quad of K
    (65, 4, 7),          # K tail of 3
    (100, 33, 1001),     # 32 x 32; odd in every size
    (128, 257, 66),      # one column past a tile, K tail of 2
    (97, 1030, 129),     # 32 x 32 / 32 x 64, K tail of 1 past a whole chunk
    (200, 2050, 260),    # 32 x 64 ... 64 x 64
    (256, 4096, 128),    # 32 x 128 / 64 x 64, whole stages
    (257, 4093, 190),    # one row and three columns short of whole tiles
    (512, 4096, 96),     # 64 x 128, an odd number of stages
    (513, 4099, 36),     # ... ragged
    (768, 4096, 64),     # 96 x 128
    (1000, 4090, 100),   # 128 x 128, ragged
    (2048, 4000, 72),    # 128 x 256 (HEAL-Full)
]


def _rand(shape, seed, pad=0):
    """N(0,1) on the GPU, rows `pad` elements apart from contiguous."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(shape[:-1] + (shape[-1] + pad,), generator=g, device="cuda")
    return x[..., :shape[-1]]


def _same(a, b, what):
    assert torch.equal(a.contiguous().view(torch.int32), b.contiguous().view(torch.int32)), what


def _out(M, N, pad):
    """Output rows `pad` apart, every element (padding too) a marker."""
    buf = torch.full((M, N + pad), 12345.0, device="cuda")
    return buf, buf[:, :N]


@pytest.mark.parametrize("pad", [0, 1, 2], ids=["whole", "pad1", "pad2"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_bf16x3_both_layouts(shape, pad):
    M, N, K = shape
    A, W = _rand((M, K), 1, pad), _rand((N, K), 2, pad)
    B = W.t().contiguous() if pad == 0 else _rand((K, N), 3, pad)
    for trans_b, Bm in ((False, B), (True, W)):
        announce("direct bf16x3 %s pad %d trans_b %s" % (shape, pad, trans_b))
        ref = heal.heal_gemm_f32_instance(heal.INSTANCE_MEDIUM, A, Bm, alpha=0.75, trans_b=trans_b)
        buf, C = _out(M, N, pad)
        heal.heal_gemm_f32_instance(heal.INSTANCE_AUTO, A, Bm, alpha=0.75, trans_b=trans_b, out=C)
        torch.cuda.synchronize()
        _same(C, ref, "trans_b %s" % trans_b)
        assert bool((buf[:, N:] == 12345.0).all()), "padding of C written"


@pytest.mark.parametrize("pad", [0, 3], ids=["whole", "pad3"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_packed_products(shape, pad):
    M, N, K = shape
    A, W = _rand((M, K), 4, pad), _rand((N, K), 5)
    W16, Bp = heal.heal_pack_f16_weight(W, 11), heal.heal_presplit_b(W, trans_b=True)
    calls = [("base", lambda i, o: heal.heal_gemm_f16w(A, W16, N, 11, 1, out=o, instance=i)),
             ("full", lambda i, o: heal.heal_gemm_f16w(A, W16, N, 11, 2, out=o, instance=i)),
             ("presplit", lambda i, o: heal.heal_gemm_f32_presplit(A, Bp, N, out=o, instance=i))]
    for name, call in calls:
        announce("direct %s %s pad %d" % (name, shape, pad))
        ref = call(heal.INSTANCE_MEDIUM, None)
        buf, C = _out(M, N, pad)
        call(heal.INSTANCE_AUTO, C)
        torch.cuda.synchronize()
        _same(C, ref, name)
        assert bool((buf[:, N:] == 12345.0).all()), "padding of C written by " + name


@pytest.mark.parametrize("trans_b", [False, True])
def test_batched(trans_b):
    A = _rand((3, 130, 203), 6)
    B = _rand((3, 301, 203) if trans_b else (3, 203, 301), 7)
    announce("direct batched trans_b %s" % trans_b)
    C = heal.heal_gemm_f32_strided_batched(A, B, alpha=0.5, trans_b=trans_b)
    ref = heal.heal_gemm_f32_instance(heal.INSTANCE_MEDIUM, A, B, alpha=0.5, trans_b=trans_b)
    torch.cuda.synchronize()
    _same(C, ref, "batched")


def test_more_batch_entries_than_the_grid_has():
    """65537 entries: some workgroups take two, one after the other."""
    A, B = _rand((65537, 3, 5), 12), _rand((65537, 5, 5), 13)
    announce("direct batch 65537")
    C = heal.heal_gemm_f32_strided_batched(A, B)
    ref = heal.heal_gemm_f32_instance(heal.INSTANCE_SKINNY, A, B)
    torch.cuda.synchronize()
    _same(C, ref, "batch 65537")


def test_non_finite_rows_stay_apart():
    """Rows, columns and K positions past the edges hold zeros, so a NaN or an
    infinity in one row or column reaches its own results only."""
    A, B = _rand((70, 130), 8).clone(), _rand((130, 45), 9).clone()
    A[69, 129], B[129, 44] = float("nan"), float("inf")
    announce("direct non-finite")
    C = heal.heal_gemm_f32(A, B)
    torch.cuda.synchronize()
    bad = ~torch.isfinite(C)
    assert bool(bad[69].all()) and bool(bad[:, 44].all())
    assert not bool(bad[:69, :44].any())


# up to 64 rows: unaligned sizes of any row count, and the row counts and widths
# from which the direct-B kernel takes over from the skinny ones
FEW_ROWS = [(1, 7, 5), (16, 1003, 999), (17, 130, 77), (33, 1024, 256), (64, 4096, 320),
            (32, 8192, 256), (32, 16000, 260), (33, 15364, 256), (64, 61440, 256),
            (40, 10240, 512), (64, 8192, 300)]


@pytest.mark.parametrize("shape", FEW_ROWS, ids=lambda s: "x".join(map(str, s)))
def test_few_rows(shape):
    M, N, K = shape
    A, W = _rand((M, K), 10), _rand((N, K), 11)
    W16, Bp = heal.heal_pack_f16_weight(W, 11), heal.heal_presplit_b(W, trans_b=True)
    B = W.t().contiguous()
    calls = [("kn", lambda i: heal.heal_gemm_f32_instance(i, A, B)),
             ("nk", lambda i: heal.heal_gemm_f32_instance(i, A, W, trans_b=True)),
             ("base", lambda i: heal.heal_gemm_f16w(A, W16, N, 11, 1, instance=i)),
             ("full", lambda i: heal.heal_gemm_f16w(A, W16, N, 11, 2, instance=i)),
             ("presplit", lambda i: heal.heal_gemm_f32_presplit(A, Bp, N, instance=i))]
    for name, call in calls:
        announce("few rows %s %s" % (name, shape))
        C, ref = call(heal.INSTANCE_AUTO), call(heal.INSTANCE_SKINNY)
        torch.cuda.synchronize()
        _same(C, ref, name)


# the tiles of 192 and 256 columns (packed B): rows, columns, depth, tile and the
# products that take it; whole and ragged, with a K tail inside a chunk and an odd
# number of chunks
WIDE = [(512, 6144, 1280, 64192, (0, 1, 3)), (509, 6100, 610, 64192, (0, 1, 3)),
        (1024, 4096, 1280, 64256, (1,)), (1021, 4090, 1280, 64256, (0, 1)), (1021, 4090, 706, 64256, (0, 1)),
        (1536, 4096, 640, 96256, (0, 1, 3)), (1530, 4001, 999, 96256, (0, 1, 3)),
        (1500, 4090, 608, 96256, (0, 1, 3)), (2048, 4096, 1536, 128256, (0, 1)), (2048, 4096, 2560, 128256, (3,)),
        (2045, 4093, 1001, 128256, (0, 3)), (2045, 4093, 1056, 128256, (0, 1, 3))]


@pytest.mark.parametrize("shape", WIDE, ids=lambda s: "x".join(map(str, s[:3])))
def test_wide_tiles(shape):
    M, N, K, tile, kinds = shape
    for kind in kinds:
        assert heal.lib().heal_gemm_direct_tile(kind, 0, M, N, K, 1) == tile, kind
    test_packed_products(shape[:3], 3)
