"""The binding's own work: argument checks with their exception types, outputs given or allocated,
the stream that a call is enqueued on."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_02540_amd as pkg
    from paper_2406_02540_amd import binding
    binding.lib()
    return pkg


def _layer(M=37, K=256, N=72, bits=8):
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((M, K), generator=g, device="cuda").half()
    w = torch.randint(-7, 8, (N, K), generator=g, device="cuda", dtype=torch.int8)
    if bits == 4:
        w = ((w[:, ::2] & 15) | ((w[:, 1::2] & 15) << 4)).view(torch.uint8).contiguous()
    return x, torch.rand(K, generator=g, device="cuda") + 0.5, w, torch.rand(N, generator=g, device="cuda"), \
        torch.randn(N, generator=g, device="cuda").half()


@pytest.mark.parametrize("bits", [8, 4])
def test_given_and_allocated_outputs(vq, bits):
    x, cm, w, ws, b = _layer(bits=bits)
    y = torch.empty((37, 72), dtype=torch.float16, device="cuda")
    wk = torch.empty(vq.vq_linear_workspace_bytes(37, 72, 256, bits), dtype=torch.uint8, device="cuda")
    assert vq.vq_linear(x, cm, w, bits, ws, b, y, wk) is y
    assert torch.equal(vq.vq_linear(x, cm, torch.nn.Parameter(w, requires_grad=False), bits, ws, bias=b), y)
    q, s = vq.vq_quantize_per_token(x, cm)
    gemm = vq.vq_gemm_w8a8 if bits == 8 else vq.vq_gemm_w4a8
    y2, acc = gemm(q, s, w, ws, b, return_acc=True)
    assert torch.equal(y2, y) and acc.dtype == torch.int32
    r = torch.empty_like(x)
    got = vq.vq_residual_linear(x, x, w, bits, ws, r=r, workspace=wk)
    assert isinstance(got, tuple) and got[0] is r and torch.equal(r, x + x)
    assert vq.vq_linear(x[:0], None, w, bits, ws).shape == (0, 72)


def test_argument_errors(vq):
    x, cm, w, ws, b = _layer()
    for bad, exc in (((x.float(), cm, w, 8, ws), TypeError), ((x.cpu(), cm, w, 8, ws), TypeError),
                     ((x[:, ::2], None, w, 8, ws), ValueError), ((x[0], None, w, 8, ws), ValueError),
                     ((None, None, w, 8, ws), AttributeError), ((x, cm[:8], w, 8, ws), ValueError),
                     ((x, cm, w[:, :128].contiguous(), 8, ws), ValueError), ((x, cm, w, 4, ws), TypeError),
                     ((x, cm, w, 8, ws[:5]), ValueError), ((x, cm, w, 8, ws, b[:3]), ValueError),
                     ((x, cm, w, 8, ws, b, x), ValueError)):
        with pytest.raises(exc):
            vq.vq_linear(*bad)
    with pytest.raises(vq.VqError) as e:
        vq.vq_linear(x, cm, w, 5, ws)
    assert e.value.status == 7 and "VQ_ERR_BITS" in str(e.value)
    with pytest.raises(vq.VqError) as e:
        vq.vq_linear(x, cm, w, 8, ws, workspace=torch.empty(64, dtype=torch.uint8, device="cuda"))
    assert e.value.status == 4
    with pytest.raises(ValueError):
        vq.vq_layernorm_quantize(x, torch.zeros((2, 256), device="cuda"), None, 37)
    with pytest.raises(ValueError):
        vq.vq_residual_quantize(x, x[:3])
    with pytest.raises(ValueError):
        vq.vq_channel_absmax(x, accumulate=True)
    with pytest.raises(TypeError):
        vq.vq_channel_absmax(w)


def test_stream_argument(vq):
    x, cm, w, ws, b = _layer()
    want = vq.vq_linear(x, cm, w, 8, ws, b)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    by_argument = vq.vq_linear(x, cm, w, 8, ws, b, stream=s)
    with torch.cuda.stream(s):
        by_context = vq.vq_linear(x, cm, w, 8, ws, b)
    torch.cuda.synchronize()
    assert torch.equal(by_argument, want) and torch.equal(by_context, want)
