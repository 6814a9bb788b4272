"""The work that the speed of this library is measured on.

Every case is one call, or the two or three calls of one layer, through the
Python entry points of ``paper_2606_21023_amd``, at sizes of a Llama-3.1-8B
layer (hidden 4096, MLP 14336, 32 heads of 128, vocabulary 128256), the
library's own workloads, or generic ones:

  kn, nk      the bf16x3 product of FP32 activations with an FP32 matrix stored
              K x N (``heal_gemm_f32``) or N x K, as a linear layer keeps it
              (``heal_gemm_f32_strided_batched`` with ``trans_b``);
  presplit    the same product with B split and packed once, at model load;
  full, base  HEAL-Full and HEAL-Base on a packed FP16 weight;
  scores      attention scores of FP32 queries and keys, one product per head;
  i16         attention scores from INT16 codes: a prompt quantizes its queries
              and keys and multiplies them (``cached`` false); a decode step
              quantizes the new queries and meets the codes of its KV cache
              (``cached`` true).

Activations are N(0,1) with 0.1% of the channels scaled by 50, weights are
N(0, 0.02^2), queries and keys N(0,1).
"""
import torch

import paper_2606_21023_amd as heal

LINEAR = ("kn", "nk", "presplit", "full", "base")


def _linear(name, kind, M, N, K):
    return {"name": name, "kind": kind, "M": M, "N": N, "K": K}


def listed():
    return [
        # the smallest product of the library's own workloads: latency counts
        _linear("square-256", "kn", 256, 256, 256),
        # one decode step of 16 sequences through a 4096-wide projection
        _linear("decode-kn", "kn", 16, 4096, 4096),
        # decode of a full batch (256 sequences) with the packed FP16 weight
        _linear("batch-full", "full", 256, 4096, 4096),
        # a ragged batch of 200 tokens through the fused QKV projection,
        # weight as a linear layer stores it
        _linear("batch-nk", "nk", 200, 6144, 4096),
        # logits of 64 sequences: the widest weight there is
        _linear("lm-head-full", "full", 64, 128256, 4096),
        # a prompt chunk of 2048 tokens through the MLP up-projection
        _linear("prefill-base", "base", 2048, 14336, 4096),
        # a ragged prompt through the MLP down-projection, B packed at load
        _linear("prefill-presplit", "presplit", 1531, 4096, 14336),
        # a general matrix product whose sizes divide by nothing
        _linear("odd-kn", "kn", 1001, 1003, 999),
        # attention scores of a 2048-token prompt
        {"name": "prompt-scores", "kind": "scores", "heads": 32, "M": 2048, "N": 2048, "d": 128},
        # INT16 attention of a prompt of odd length, quantization included
        {"name": "prompt-i16", "kind": "i16", "heads": 32, "M": 1531, "N": 1531, "d": 128,
         "cached": False},
        # INT16 attention of one decode step against 3001 cached keys
        {"name": "decode-i16", "kind": "i16", "heads": 32, "M": 1, "N": 3001, "d": 128,
         "cached": True},
        # the largest product of the library's own workloads
        _linear("square-8192", "kn", 8192, 8192, 8192),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    """One more case: rows 1 to 8192 (any number), widths and depths 256 to
    16384 (multiples of 64, as layers have them, and vocabularies up to 131072
    for at most 64 rows), general products of any odd size, and attention of 8
    to 64 heads over 16 to 4096 tokens, or 64 to 16384 cached keys."""
    kind = rng.choice(LINEAR + ("odd", "scores", "i16", "cached"))
    if kind == "odd":
        # as the general product: no size a multiple of anything
        return {"kind": "kn", "M": _log_int(rng, 64, 4096), "N": _log_int(rng, 64, 4096),
                "K": _log_int(rng, 64, 4096)}
    if kind in LINEAR:
        M = _log_int(rng, 1, 8192)
        N = 64 * _log_int(rng, 4, 2048 if M <= 64 and rng.random() < 0.3 else 256)
        K = 64 * _log_int(rng, 4, 256)
        while N * K > 128256 * 4096:
            K = max(256, K // 2 // 64 * 64)
        M = min(M, 8192 ** 3 // (N * K))
        return {"kind": kind, "M": M, "N": N, "K": K}
    heads, d = rng.choice((8, 16, 32, 64)), rng.choice((64, 128))
    if kind == "cached":
        return {"kind": "i16", "heads": heads, "M": rng.randint(1, 8),
                "N": _log_int(rng, 64, 16384), "d": d, "cached": True}
    M = _log_int(rng, 16, 4096)
    while heads * M * M > 32 * 2048 * 2048:
        heads //= 2
    case = {"kind": kind, "heads": heads, "M": M, "N": M, "d": d}
    if kind == "i16":
        case["cached"] = False
    return case


def _activations(g, M, K):
    A = torch.randn((M, K), generator=g, device="cuda")
    channels = torch.randperm(K, generator=g, device="cuda")[:max(1, round(0.001 * K))]
    A[:, channels] *= 50.0
    return A


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] in ("scores", "i16"):
        q = torch.randn((case["heads"], case["M"], case["d"]), generator=g, device="cuda")
        k = torch.randn((case["heads"], case["N"], case["d"]), generator=g, device="cuda")
        return q, k
    M, N, K = case["M"], case["N"], case["K"]
    A = _activations(g, M, K)
    shape = (K, N) if case["kind"] == "kn" else (N, K)
    return A, torch.randn(shape, generator=g, device="cuda").mul_(0.02)


def _exponent(W):
    return heal.heal_f16_weight_exponent(heal.heal_maxabs_f32(W).item())


def prepare(case, seed):
    kind = case["kind"]
    A, B = _inputs(case, seed)
    s = {"kind": kind, "A": A, "alpha": case["d"] ** -0.5 if "d" in case else 1.0}
    if kind == "kn":
        s["B"] = B
    elif kind == "nk":
        s["A"], s["B"] = A.unsqueeze(0), B.unsqueeze(0)
    elif kind == "presplit":
        s["B"], s["N"] = heal.heal_presplit_b(B, trans_b=True), case["N"]
    elif kind in ("full", "base"):
        s["e"] = _exponent(B)
        s["B"], s["N"] = heal.heal_pack_f16_weight(B, s["e"]), case["N"]
    elif kind == "scores":
        s["B"] = B
    else:
        s["cached"] = case["cached"]
        s["B"] = heal.heal_quantize_i16(B) if case["cached"] else B
    return s


def run(s):
    kind = s["kind"]
    if kind == "kn":
        return heal.heal_gemm_f32(s["A"], s["B"])
    if kind == "nk":
        return heal.heal_gemm_f32_strided_batched(s["A"], s["B"], trans_b=True)
    if kind == "presplit":
        return heal.heal_gemm_f32_presplit(s["A"], s["B"], s["N"])
    if kind in ("full", "base"):
        return heal.heal_gemm_f16w(s["A"], s["B"], s["N"], s["e"], 2 if kind == "full" else 1)
    if kind == "scores":
        return heal.heal_gemm_f32_strided_batched(s["A"], s["B"], alpha=s["alpha"], trans_b=True)
    q, mq = heal.heal_quantize_i16(s["A"])
    if s["cached"]:
        k, mk = s["B"]
        return {"S": heal.heal_scores_i16(q, k, mq, mk, s["alpha"]), "q": q, "mq": mq}
    k, mk = heal.heal_quantize_i16(s["B"])
    return {"S": heal.heal_scores_i16(q, k, mq, mk, s["alpha"]), "q": q, "mq": mq, "k": k, "mk": mk}


def work(case):
    """Bytes: each operand read once as it is stored, each output written once
    (codes are written, and read by the product).  Operations: the 16-bit
    matrix products the method consists of, 2MNK each."""
    kind = case["kind"]
    products = {"kn": 3, "nk": 3, "presplit": 3, "scores": 3, "full": 2, "base": 1, "i16": 4}[kind]
    M, N = case["M"], case["N"]
    if kind in LINEAR:
        K = case["K"]
        b = 2 if kind in ("full", "base") else 4
        return {"bytes": 4 * M * K + b * N * K + 4 * M * N, "flops": products * 2 * M * N * K}
    h, d = case["heads"], case["d"]
    flops = products * 2 * h * M * N * d
    if kind == "scores":
        return {"bytes": 4 * h * (M * d + N * d + M * N), "flops": flops}
    quantized = M * d if case["cached"] else M * d + N * d
    return {"bytes": h * (6 * quantized + 2 * (M * d + N * d) + 4 * M * N), "flops": flops}


def tolerance(case):
    """FP32 sums of exact 16-bit products: about four times what the path is
    off its own products summed in 64 bits (at most 1.4e-6, at 14336 deep; the
    largest single difference 1.2e-5 of the result's root mean square).  Codes
    are whole numbers and agree."""
    return {"rel": 5e-6, "max": 5e-5}


def _split(x, dtype, shift=1.0):
    """x as the 16-bit head and the (shifted) 16-bit residual, both in 64 bits."""
    hi = x.to(dtype).float()
    return hi.double(), ((x - hi) * shift).to(dtype).double() / shift


def exact(case, seed):
    """The method's products of the 16-bit parts, summed in 64 bits."""
    kind = case["kind"]
    A, B = _inputs(case, seed)
    if kind == "i16":
        def codes(x):
            m = x.abs().max()
            return torch.round(x.double() * 32767.0 / m.double()), m.reshape(1)
        (q, mq), (k, mk) = codes(A), codes(B)
        # heads one after another: float64 on the whole batch at once is not needed
        S = torch.stack([a @ b.t().contiguous() for a, b in zip(q, k)])
        alpha = torch.tensor(case["d"] ** -0.5, dtype=torch.float32).double().item()
        S *= alpha * mq.double().item() * mk.double().item() / 32767.0 ** 2
        out = {"S": S, "q": q.to(torch.int16), "mq": mq}
        return out if case["cached"] else dict(out, k=k.to(torch.int16), mk=mk)
    if kind == "base" or kind == "full":
        e = 0
        m = B.abs().max().item()
        while m * 2.0 ** (e + 1) <= 65504.0:
            e += 1
        W = (B * 2.0 ** e).to(torch.float16).double().t().contiguous()
        hi, lo = _split(A, torch.float16, 1024.0)
        return ((hi @ W) if kind == "base" else (hi + lo) @ W) * 2.0 ** -e
    if kind == "scores":
        alpha = torch.tensor(case["d"] ** -0.5, dtype=torch.float32).double().item()
        pairs = zip(A, B.transpose(1, 2).contiguous())
        return torch.stack([_products(a, b) for a, b in pairs]) * alpha
    if kind != "kn":
        B = B.t().contiguous()
    S = _products(A, B)
    return S.unsqueeze(0) if kind == "nk" else S


def _products(A, B):
    (ah, al), (bh, bl) = _split(A, torch.bfloat16), _split(B, torch.bfloat16)
    return ah @ (bh + bl) + al @ bh
