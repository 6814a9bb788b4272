"""The panel kernel on few rows and on outputs of any row length and alignment,
and the one-workgroup INT16 quantization.

Each output is compared bit for bit with the tiled kernels, which other tests
hold to the oracle: the skinny instance for bf16x3, and for the INT16 scores the
same codes behind a row pitch that is not a multiple of eight codes."""
import numpy as np
import pytest
import torch

import paper_2606_21023_amd as heal
from gpu_util import announce, needs_gpu, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]

# batch x rows x columns x depth: panels of 16, 32, 64, 128 and 256 rows, at
# their edges; columns of every remainder of 4, within and across 128-column
# steps, and fewer than one step; one to four chunks of depth with tails
SHAPES = [(3, 1, 3001, 128), (2, 16, 514, 40), (2, 17, 515, 96), (1, 32, 257, 64),
          (2, 33, 1023, 72), (1, 64, 130, 128), (2, 65, 129, 24), (1, 128, 131, 128),
          (2, 129, 383, 120), (2, 300, 301, 128), (1, 257, 5, 8), (1, 5, 4, 8)]


def _codes(rng, shape, pitch):
    x = torch.zeros(shape[:-1] + (pitch,), dtype=torch.int16, device="cuda")[..., :shape[-1]]
    x.copy_(to_dev(rng.integers(-32767, 32768, size=shape).astype(np.int16)))
    return x


def _bits(a, b, what):
    assert torch.equal(a.contiguous().view(torch.int32), b.contiguous().view(torch.int32)), what


@pytest.mark.parametrize("pad", [0, 3], ids=["whole", "pad3"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_scores(shape, pad):
    bat, M, N, K = shape
    rng = np.random.default_rng(M + 5 * N + 11 * K)
    Q, Kt = _codes(rng, (bat, M, K), K), _codes(rng, (bat, N, K), K)
    mq, mk = torch.tensor([3.5], device="cuda"), torch.tensor([0.625], device="cuda")
    Qp = torch.zeros((bat, M, K + 1), dtype=torch.int16, device="cuda")[:, :, :K]
    Qp.copy_(Q)
    announce("ragged scores %s pad %d" % (shape, pad))
    buf = torch.full((bat, M, N + pad), 777.0, device="cuda")
    heal.heal_scores_i16(Q, Kt, mq, mk, 0.125, out=buf[:, :, :N])
    ref = heal.heal_scores_i16(Qp, Kt, mq, mk, 0.125)
    torch.cuda.synchronize()
    _bits(buf[:, :, :N], ref, "scores")
    assert bool((buf[:, :, N:] == 777.0).all()), "padding of S written"


@pytest.mark.parametrize("pad", [0, 1], ids=["whole", "pad1"])
@pytest.mark.parametrize("shape", SHAPES + [(2, 4, 256, 128), (1, 40, 512, 36)],
                         ids=lambda s: "x".join(map(str, s)))
def test_bf16x3(shape, pad):
    bat, M, N, K = shape
    g = torch.Generator(device="cuda").manual_seed(M + N)
    A = torch.randn((bat, M, K), generator=g, device="cuda")
    B = torch.randn((bat, N, K), generator=g, device="cuda")
    announce("ragged bf16x3 %s pad %d" % (shape, pad))
    buf = torch.full((bat, M, N + pad), 777.0, device="cuda")
    heal.heal_gemm_f32_strided_batched(A, B, alpha=0.25, trans_b=True, out=buf[:, :, :N])
    ref = heal.heal_gemm_f32_instance(heal.INSTANCE_SKINNY, A, B, alpha=0.25, trans_b=True)
    torch.cuda.synchronize()
    _bits(buf[:, :, :N], ref, "bf16x3")
    assert bool((buf[:, :, N:] == 777.0).all()), "padding of C written"


@pytest.mark.parametrize("n", [1, 3, 4, 1023, 4096, 16381, 16384, 16385, 16388])
def test_quantize_at_the_one_workgroup_limit(orc, n):
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n).astype(np.float32)
    x[n // 2] = -7.0 if n % 2 else 7.0               # the maximum, of either sign
    announce("quantize n=%d" % n)
    q, m = heal.heal_quantize_i16(to_dev(x))
    qo, mo = orc.quantize_i16(x)
    assert np.array_equal(q.cpu().numpy(), qo) and m.item() == mo


def test_rows_of_codes_far_apart():
    """128 rows 5 000 000 codes apart: the panel's byte offsets reach 1.27 GB."""
    pitch = 5000000 - 5000000 % 8
    rng = np.random.default_rng(6)
    Q, Kt = _codes(rng, (1, 128, 128), 128), _codes(rng, (1, 256, 128), 128)
    far = torch.zeros((1, 128, pitch), dtype=torch.int16, device="cuda")[:, :, :128]
    far.copy_(Q)
    mq, mk = torch.tensor([3.5], device="cuda"), torch.tensor([0.625], device="cuda")
    announce("scores, rows far apart")
    S = heal.heal_scores_i16(far, Kt, mq, mk, 0.125)
    ref = heal.heal_scores_i16(Q, Kt, mq, mk, 0.125)
    torch.cuda.synchronize()
    _bits(S, ref, "scores")
