"""The direct-B kernel (heal_gemm_direct.hip), which most products of 65 and
more rows take by themselves, against the tiled kernels of the forced instances,
bit for bit: at tile edges, K tails of every remainder and rows of every
alignment, and every tile configuration of every product, with and without a K
tail, by name (TILES).  The forced instances are checked against the oracle
elsewhere; every instance sums in one order, so no tolerance is needed."""
import pytest
import torch

import paper_2606_21023_amd as heal
from gpu_util import announce, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

# rows x columns x depth (which tiles they take is the plan's business: TILES below)
SHAPES = [
    (65, 5, 4),          # smallest: one quad of K
    (65, 4, 7),          # K tail of 3
    (100, 33, 1001),     # odd in every size
    (128, 257, 66),      # one column past a tile, K tail of 2
    (97, 1030, 129),     # K tail of 1 past a whole chunk
    (200, 2050, 260),
    (256, 4096, 128),    # whole stages
    (257, 4093, 190),    # one row and three columns short of whole tiles
    (512, 4096, 96),     # an odd number of stages
    (513, 4099, 36),     # ... ragged
    (768, 4096, 64),
    (1000, 4090, 100),
    (2048, 4000, 72),
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
        # (the medium instance takes the panel kernel for such a K, as the call itself does)
        tiled = heal.INSTANCE_SKINNY if trans_b and K <= 128 else heal.INSTANCE_MEDIUM
        ref = heal.heal_gemm_f32_instance(tiled, A, Bm, alpha=0.75, trans_b=trans_b)
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


# up to 64 rows: unaligned sizes of any row count, and the row counts, widths and
# depths around which the direct-B kernel takes over from the skinny ones
FEW_ROWS = [(33, 1024, 512), (64, 4096, 516), (32, 8192, 512), (33, 15364, 512), (64, 61440, 2048),
            (1, 7, 5), (16, 1003, 999), (17, 130, 77), (33, 1024, 256), (64, 4096, 320),
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


# Every tile configuration of every product (0 HEAL-Base, 1 HEAL-Full, 3 pre-split,
# 4 and 5 bf16x3 with B stored K x N and N x K), whole stages of K and K tails, one
# or few stages and many: rows, columns, depth and the tile that the plan takes.
# (64 x 256 tiles are not built for the pre-split product, and 128 x 128 ones with an
# FP32 B have no K-tail form.)  N x K is deeper than the panel kernel reaches.
TILES = {
    0: [
        (77, 9, 64, 32032), (35, 13, 512, 32032), (18, 8, 5, 32032), (19, 8, 409, 32032),
        (5086, 33, 64, 32064), (4978, 34, 448, 32064), (18, 10391, 5, 32064), (17, 9, 821, 32064),
        (72, 9984, 64, 32128), (6016, 68, 448, 32128), (34, 15643, 5, 32128), (17, 23310, 402, 32128),
        (7779, 225, 64, 64128), (72, 16320, 448, 64128), (7560, 200, 35, 64128), (6893, 129, 426, 64128),
        (74, 23810, 64, 64192), (72, 18624, 448, 64192), (67, 19195, 5, 64192), (8306, 137, 410, 64192),
        (136, 16576, 64, 64256), (136, 16512, 448, 64256), (8415, 212, 5, 64256), (65, 25444, 437, 64256),
        (70, 24059, 1344, 96128), (70, 24984, 2740, 96128), (134, 23099, 32, 96256), (136, 22144, 448, 96256),
        (8240, 268, 6, 96256), (148, 22046, 463, 96256), (2174, 1894, 128, 128128), (2138, 1886, 576, 128128),
        (8318, 315, 191, 128128), (8368, 311, 459, 128128), (8178, 513, 32, 128256), (8186, 567, 416, 128256),
        (346, 18336, 57, 128256), (8489, 610, 428, 128256)],
    1: [
        (7986, 12, 64, 32032), (7554, 8, 768, 32032), (18, 8, 5, 32032), (73, 8, 64, 32064),
        (43, 9, 576, 32064), (17, 8, 91, 32064), (17, 8, 425, 32064), (7768, 66, 64, 32128),
        (40, 11520, 512, 32128), (8163, 68, 5, 32128), (34, 12045, 477, 32128), (104, 16128, 256, 64128),
        (104, 14016, 448, 64128), (8061, 210, 525, 64128), (97, 18418, 64, 64192), (8280, 192, 448, 64192),
        (5439, 282, 5, 64192), (8284, 148, 429, 64192), (136, 16640, 64, 64256), (80, 25024, 448, 64256),
        (2543, 754, 5, 64256), (8321, 219, 483, 64256), (72, 24832, 1280, 96128), (67, 25689, 6578, 96128),
        (130, 21802, 32, 96256), (200, 17152, 448, 96256), (8282, 294, 6, 96256), (8427, 387, 441, 96256),
        (3483, 1138, 192, 128128), (6176, 563, 1024, 128128), (8267, 260, 305, 128128),
        (5941, 557, 411, 128128), (8229, 539, 32, 128256), (318, 16922, 416, 128256), (8377, 574, 5, 128256),
        (6556, 854, 421, 128256)],
    3: [
        (1485, 26, 64, 32032), (392, 128, 448, 32032), (20, 8, 5, 32032), (8194, 8, 508, 32032),
        (66, 10, 64, 32064), (33, 9, 512, 32064), (19, 8, 153, 32064), (18, 8, 441, 32064),
        (67, 6654, 384, 32128), (40, 9344, 512, 32128), (34, 9512, 191, 32128), (36, 8274, 406, 32128),
        (6431, 203, 128, 64128), (72, 11072, 512, 64128), (34, 24792, 138, 64128), (34, 22300, 401, 64128),
        (66, 20345, 64, 64192), (72, 17408, 448, 64192), (67, 18767, 5, 64192), (65, 16983, 417, 64192),
        (280, 10855, 192, 96128), (8320, 256, 448, 96128), (71, 24855, 142, 96128), (72, 25034, 404, 96128),
        (129, 19352, 32, 96256), (174, 17982, 416, 96256), (134, 18020, 5, 96256), (141, 16929, 449, 96256),
        (2322, 1439, 64, 128128), (197, 12617, 448, 128128), (86, 25556, 5, 128128), (197, 12725, 403, 128128),
        (1673, 3717, 160, 128256), (1283, 4695, 416, 128256), (8390, 671, 432, 128256)],
    4: [
        (21, 9, 64, 32032), (29, 10, 448, 32032), (34, 9, 5, 32032), (18, 8, 427, 32032),
        (72, 3008, 64, 32064), (6621, 8, 576, 32064), (7545, 36, 5, 32064), (7751, 8, 844, 32064),
        (45, 10997, 256, 64064), (40, 12352, 512, 64064), (33, 11529, 360, 64064), (34, 13372, 415, 64064),
        (39, 14801, 64, 64128), (44, 15069, 448, 64128), (66, 9169, 5, 64128), (66, 8587, 416, 64128),
        (8387, 150, 64, 96128), (72, 17600, 448, 96128), (70, 18564, 5, 96128), (66, 16667, 415, 96128),
        (97, 20263, 64, 128128), (112, 16832, 448, 128128)],
    5: [
        (94, 8, 192, 32032), (73, 12, 512, 32032), (17, 8, 137, 32032), (21, 8, 426, 32032),
        (5218, 39, 192, 32064), (5743, 33, 448, 32064), (33, 7576, 143, 32064), (17, 10663, 471, 32064),
        (72, 7872, 256, 64064), (72, 6144, 512, 64064), (34, 13474, 162, 64064), (33, 8803, 425, 64064),
        (72, 7744, 192, 64128), (72, 7744, 448, 64128), (34, 13983, 137, 64128), (17, 23857, 413, 64128),
        (70, 16817, 192, 96128), (72, 17600, 448, 96128), (69, 16749, 138, 96128), (65, 16614, 416, 96128),
        (115, 18926, 256, 128128), (104, 17664, 448, 128128)],
}
TILE_CASES = [(kind,) + case for kind in TILES for case in TILES[kind]]


@pytest.mark.parametrize("case", TILE_CASES, ids=lambda c: "%d-%dx%dx%d-%d" % c)
def test_every_tile(case):
    kind, M, N, K, tile = case
    assert heal.lib().heal_gemm_direct_tile(min(kind, 4), 1 if kind == 5 else 0, M, N, K, 1) == tile
    announce("direct tile %s" % (case,))
    A, W = _rand((M, K), 20), _rand((N, K), 21)
    if kind == 4:
        B = W.t().contiguous()
        call = lambda i, o: heal.heal_gemm_f32_instance(i, A, B, alpha=0.75, out=o)
    elif kind == 5:
        call = lambda i, o: heal.heal_gemm_f32_instance(i, A, W, alpha=0.75, trans_b=True, out=o)
    elif kind == 3:
        Bp = heal.heal_presplit_b(W, trans_b=True)
        call = lambda i, o: heal.heal_gemm_f32_presplit(A, Bp, N, out=o, instance=i)
    else:
        W16 = heal.heal_pack_f16_weight(W, 11)
        call = lambda i, o: heal.heal_gemm_f16w(A, W16, N, 11, kind + 1, out=o, instance=i)
    buf = torch.full((M * N + 64,), 12345.0, device="cuda")
    C = buf[:M * N].view(M, N)
    call(heal.INSTANCE_AUTO, C)
    ref = call(heal.INSTANCE_MEDIUM, None)
    torch.cuda.synchronize()
    _same(C, ref, "tile %d" % tile)
    assert bool((buf[M * N:] == 12345.0).all()), "written past C"


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


# the largest byte offsets that the plan accepts: A's rows, B's rows (N x K) and all
# of B (K x N) end just below 2^31 bytes, and just above, where another kernel runs
def _rows_apart(M, K, pitch, seed):
    x = torch.empty(M * pitch, device="cuda").as_strided((M, K), (pitch, 1))
    return x.copy_(_rand((M, K), seed))


@pytest.mark.parametrize("over", [0, 1], ids=["below", "above"])
def test_offset_bounds(over):
    lim = 0x7fffffff
    M, N, K = 128, 300, 196
    pitch = (lim // 4 - K - 128) // 127 + over
    A, W = _rows_apart(M, K, pitch, 30), _rand((N, K), 31)
    near = A.contiguous()
    W16 = heal.heal_pack_f16_weight(W, 11)
    announce("A's rows %d apart" % pitch)
    C, ref = heal.heal_gemm_f16w(A, W16, N, 11, 2), heal.heal_gemm_f16w(near, W16, N, 11, 2)
    C3, ref3 = heal.heal_gemm_f32(A, W.t().contiguous()), heal.heal_gemm_f32(near, W.t().contiguous())
    torch.cuda.synchronize()
    _same(C, ref, "HEAL-Full")
    _same(C3, ref3, "bf16x3 K x N")
    del A
    pitch = (lim // 4 - K - 128) // 255 + over
    A, W = _rand((M, K), 32), _rows_apart(N, K, pitch, 33)
    near = W.contiguous()
    announce("B's rows %d apart" % pitch)
    C = heal.heal_gemm_f32_instance(heal.INSTANCE_AUTO, A, W, trans_b=True)
    ref = heal.heal_gemm_f32_instance(heal.INSTANCE_AUTO, A, near, trans_b=True)
    torch.cuda.synchronize()
    _same(C, ref, "bf16x3 N x K")
    del W
    M, N = 70, 4096
    K = lim // (4 * N) - 128 + over
    A, B = _rand((M, K), 34), _rand((K, N), 35)
    announce("K x N of %d bytes" % (4 * K * N))
    C = heal.heal_gemm_f32(A, B)
    ref = heal.heal_gemm_f32_instance(heal.INSTANCE_MEDIUM, A, B)
    torch.cuda.synchronize()
    _same(C, ref, "bf16x3 K x N")
