"""Layers of few tokens: the one launch gives the bits of the quantizer and the GEMM called one after the other."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vq():
    import paper_2406_02540_amd as vq
    return vq


def _layer(vq, producer, M, K, N, bits, seed):
    """The layer against its two calls.  Whether it was one launch: that leaves the workspace as it was."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def n(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    x = (n(M, K) * torch.exp(n(K))).half()
    x[M // 2] = 0                                # a token whose scale is zero
    w, ws = vq.vq_quantize_weight(n(N, K) * 0.02, None, bits)
    b = (n(N) * 0.01).half()
    T = (M + 1) // 2
    B = (M + T - 1) // T
    cm, sc, sh, y_in = torch.exp(n(K) * 0.3), n(B, K) * 0.2, n(B, K) * 0.5, n(M, K).half()
    gemm = vq.vq_gemm_w8a8 if bits == 8 else vq.vq_gemm_w4a8
    wk = torch.full((vq.vq_linear_workspace_bytes(M, N, K, bits),), 0xA5, dtype=torch.uint8, device="cuda")
    if producer in ("plain", "balanced"):
        c = cm if producer == "balanced" else None
        one, q = vq.vq_linear(x, c, w, bits, ws, b, None, wk), vq.vq_quantize_per_token(x, c)
    elif producer == "layernorm":
        one = vq.vq_layernorm_linear(x, w, bits, ws, sc, sh, T, 1e-6, cm, b, None, wk)
        q = vq.vq_layernorm_quantize(x, sc, sh, T, 1e-6, cm)
    elif producer == "layernorm_bare":
        one = vq.vq_layernorm_linear(x, w, bits, ws, None, None, None, 1e-6, None, b, None, wk)
        q = vq.vq_layernorm_quantize(x, None, None, None, 1e-6, None)
    elif producer in ("gelu", "gelu_erf"):
        t = producer == "gelu"
        one, q = vq.vq_gelu_linear(x, w, bits, ws, t, cm, b, None, wk), vq.vq_gelu_quantize(x, t, cm)
    elif producer == "residual":
        r1, one = vq.vq_residual_linear(x, y_in, w, bits, ws, sc, T, None, cm, b, None, wk)
        r, *q = vq.vq_residual_quantize(x, y_in, sc, T, None, cm)
        assert torch.equal(r1, r)
    else:
        one, q = vq.vq_hadamard_linear(x, cm, w, bits, ws, b, None, wk), vq.vq_hadamard_quantize(x, cm)
    two = gemm(q[0], q[1], w, ws, b)
    torch.cuda.synchronize()
    assert np.array_equal(one.cpu().numpy().view(np.uint16), two.cpu().numpy().view(np.uint16))
    return bool((wk == 0xA5).all())


PRODUCERS = ("plain", "balanced", "layernorm", "layernorm_bare", "gelu", "gelu_erf", "residual", "hadamard")


# one token, a tile of tokens and one past it, partly filled channel tiles and rows of any alignment, K of one
# chunk group and up to the longest row; the last four lie past the rule, LayerNorm is not in it (two launches on both sides)
@pytest.mark.parametrize("producer", PRODUCERS)
@pytest.mark.parametrize("M,K,N", [(1, 128, 1), (8, 1152, 64), (9, 1152, 65), (3, 256, 2304), (30, 1024, 510), (4, 1536, 72),
                                   (61, 512, 300), (2, 1664, 72), (250, 1152, 1100), (40, 4608, 1152), (2, 8192, 64)])
@pytest.mark.parametrize("bits", [8, 4])
def test_one_launch_gives_the_bits_of_two(vq, producer, M, K, N, bits):
    print(f"small layer {producer} {M}x{K}->{N} w{bits}", flush=True)
    past = (M, K, N) in ((2, 1664, 72), (250, 1152, 1100), (40, 4608, 1152), (2, 8192, 64))
    assert _layer(vq, producer, M, K, N, bits, 9000 + M + K + N) == (not producer.startswith("layernorm") and not past)


# near the rule's lines: a workgroup on nearly every CU, in two bands of token tiles and in sixteen, the last one of
# partial height; rows above 1152 channels where tiles x K ends the rule (208 tiles; 216 are past it)
@pytest.mark.parametrize("producer", PRODUCERS)
@pytest.mark.parametrize("M,K,N", [(100, 1152, 1152), (1001, 1152, 100), (100, 1408, 1000), (24, 1408, 4608)])
@pytest.mark.parametrize("bits", [8, 4])
def test_one_launch_fills_the_chip(vq, producer, M, K, N, bits):
    print(f"small layer {producer} {M}x{K}->{N} w{bits}", flush=True)
    assert _layer(vq, producer, M, K, N, bits, 9700 + M + K + N) == (not producer.startswith("layernorm") and (M, N) != (24, 4608))


# K that is no multiple of the stage, of a chunk group or (8 bits) of 32
@pytest.mark.parametrize("producer", [p for p in PRODUCERS if p != "hadamard"])
@pytest.mark.parametrize("K,bits", [(16, 8), (512, 8), (1008, 8), (1168, 8), (1520, 8), (32, 4), (544, 4), (1184, 4), (1504, 4)])
def test_one_launch_k_tails(vq, producer, K, bits):
    print(f"small layer {producer} 21x{K}->100 w{bits}", flush=True)
    assert _layer(vq, producer, 21, K, 100, bits, 9500 + K) == (not producer.startswith("layernorm"))


def test_outputs_over_inputs_take_two_launches(vq):
    # y in the memory of x, the residual sum in place: what the two launches allow
    x = torch.randn((64, 256), device="cuda").half()
    y_in = torch.randn((64, 256), device="cuda").half()
    w, ws = vq.vq_quantize_weight(torch.randn((256, 256), device="cuda") * 0.02, None, 8)
    want = vq.vq_linear(x, None, w, 8, ws)
    over = x.clone()
    vq.vq_linear(over, None, w, 8, ws, None, over)
    r, y = vq.vq_residual_linear(x, y_in, w, 8, ws)
    inplace = x.clone()
    _, y2 = vq.vq_residual_linear(inplace, y_in, w, 8, ws, r=inplace)
    torch.cuda.synchronize()
    assert torch.equal(over, want) and torch.equal(inplace, r) and torch.equal(y2, y)


@pytest.mark.parametrize("vector", ["chan_mul", "gate"])
def test_output_over_a_vector_of_the_quantizer_takes_two_launches(vq, vector):
    # the quantizer is through with its vectors when the GEMM writes y: y may take their memory.  (In one launch the
    # workspace is left alone.)
    M, K, N = 16, 512, 64
    g = torch.Generator(device="cuda").manual_seed(77)
    x, y_in = torch.randn((M, K), generator=g, device="cuda").half(), torch.randn((M, K), generator=g, device="cuda").half()
    w, ws = vq.vq_quantize_weight(torch.randn((N, K), generator=g, device="cuda") * 0.02, None, 8)
    v = torch.exp(torch.randn(K, generator=g, device="cuda") * 0.3)

    def call(vec, y, wk):
        if vector == "chan_mul":
            return vq.vq_linear(x, vec, w, 8, ws, None, y, wk)
        return vq.vq_residual_linear(x, y_in, w, 8, ws, vec.view(1, K), M, None, None, None, y, wk)[1]

    apart = torch.full((vq.vq_linear_workspace_bytes(M, N, K, 8),), 0xA5, dtype=torch.uint8, device="cuda")
    shared = apart.clone()
    want = call(v, None, apart)
    over = v.clone()
    got = call(over, over.view(torch.float16)[: M * N].view(M, N), shared)
    torch.cuda.synchronize()
    assert (apart == 0xA5).all() and (shared != 0xA5).any()
    assert torch.equal(got, want)
