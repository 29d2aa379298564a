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


def test_memory_taken_for_a_call_on_another_stream(vq):
    # Scratch and outputs that the call allocates belong to the stream that it runs on: held back behind a wait, two
    # streams' layers (two launches each, through the scratch) and the current stream's allocations of the same sizes
    # stay apart, and an output that the current stream reads is not handed out while it does.
    M, K, N = 700, 1152, 520
    x0, cm, w, ws, b = _layer(M, K, N)
    xs = [x0 * f for f in (1.0, 2.0, -3.0, 0.5)]
    want = [vq.vq_linear(x, cm, w, 8, ws, b) for x in xs]
    size = vq.vq_linear_workspace_bytes(M, N, K, 8)
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for s in streams:
        with torch.cuda.stream(s):
            torch.cuda._sleep(2000000)
    got, between = [], []
    for i, x in enumerate(xs):
        got.append(vq.vq_linear(x, cm, w, 8, ws, b, stream=streams[i % 2]))
        between += [torch.full((size,), 77, dtype=torch.uint8, device="cuda"),
                    torch.full((M, N), 7.0, dtype=torch.float16, device="cuda")]
    torch.cuda.synchronize()
    for i in range(4):
        assert torch.equal(got[i], want[i])
    assert all((t == (77 if t.dtype == torch.uint8 else 7.0)).all() for t in between)
    owner = {}
    for seg in torch.cuda.memory_snapshot():
        for y in got:
            if seg["address"] <= y.data_ptr() < seg["address"] + seg["total_size"]:
                owner[y.data_ptr()] = seg["stream"]
    for i, y in enumerate(got):
        assert owner[y.data_ptr()] == streams[i % 2].cuda_stream
    # an output let go of while the current stream still has to read it
    s = streams[0]
    y = vq.vq_linear(xs[0], cm, w, 8, ws, b, stream=s)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda._sleep(2000000)
    copy = y.clone()
    del y
    again = [vq.vq_linear(x, cm, w, 8, ws, b, stream=s) for x in xs]
    torch.cuda.synchronize()
    assert torch.equal(copy, want[0]) and all(torch.equal(a, t) for a, t in zip(again, want))
    # a stream known by its handle only, and the current one given
    class Handle:
        cuda_stream = s.cuda_stream

    by_handle = vq.vq_linear(xs[1], cm, w, 8, ws, b, stream=Handle())
    by_current = vq.vq_linear(xs[2], cm, w, 8, ws, b, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert torch.equal(by_handle, want[1]) and torch.equal(by_current, want[2])
