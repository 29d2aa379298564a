"""Problems whose launches come near 2^32 threads, which HIP refuses: they run, and their last rows are right."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_02540_amd as pkg
    return pkg


@pytest.fixture
def room():
    """Device memory for a test of so many bytes, given back afterwards."""
    def ask(need):
        torch.cuda.empty_cache()
        if torch.cuda.mem_get_info()[0] < need + (4 << 30):
            pytest.skip(f"needs {need >> 30} GiB of device memory")
    yield ask
    torch.cuda.empty_cache()


# few channels, little K: tiles of 32 tokens at 192 threads each would be 4.5e9 threads at 750 million tokens; from
# 2^30 tokens on only the persistent kernel is below 2^32
@pytest.mark.parametrize("M", [750_000_000, 1_074_000_001])
def test_gemm_of_very_many_tokens(vq, room, M):
    N, K = 3, 16
    room(M * (K + 4 + 2 * N))
    print(f"gemm w8a8 M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    part = 4096 + 77
    xq = torch.zeros((M, K), dtype=torch.int8, device="cuda")
    xs = torch.full((M,), 2.0 ** -9, device="cuda")
    spots = [0, M // 2 - part, M - part]
    for at in spots:
        xq[at:at + part] = torch.randint(-127, 128, (part, K), generator=g, device="cuda", dtype=torch.int8)
        xs[at:at + part] = torch.exp2(torch.randint(-12, -8, (part,), generator=g, device="cuda").float())
    wq = torch.randint(-127, 128, (N, K), generator=g, device="cuda", dtype=torch.int8)
    ws = torch.exp2(torch.randint(-8, -4, (N,), generator=g, device="cuda").float())
    b = torch.randn(N, generator=g, device="cuda").half()
    y = torch.full((M, N), 7.0, dtype=torch.float16, device="cuda")
    vq.vq_gemm_w8a8(xq, xs, wq, ws, b, y=y)
    for at in spots:
        acc = xq[at:at + part].double() @ wq.double().t()
        want = (acc * xs[at:at + part].double()[:, None] * ws.double()[None] + b.double()).half()
        assert torch.equal(y[at:at + part], want), at
    # every other row is the bias: so many of them equal it
    assert all(int((y[:, n] == b[n]).sum()) >= M - 3 * part for n in range(N))


# more channels than four times as many fit an int: the scales' bytes and their places are counted in more
def test_gemm_of_very_many_channels(vq, room):
    M, N, K = 3, 600_000_003, 16
    room(N * (K + 4 + 2 + 2 * M + 3))
    print(f"gemm w8a8 M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    part = 4096 + 77
    xq = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    xs = torch.exp2(torch.randint(-12, -8, (M,), generator=g, device="cuda").float())
    wq = torch.zeros((N, K), dtype=torch.int8, device="cuda")
    ws = torch.full((N,), 2.0 ** -9, device="cuda")
    b = torch.full((N,), 0.5, dtype=torch.float16, device="cuda")
    spots = [0, (1 << 29) - part // 2, N - part]
    for at in spots:
        wq[at:at + part] = torch.randint(-127, 128, (part, K), generator=g, device="cuda", dtype=torch.int8)
        ws[at:at + part] = torch.exp2(torch.randint(-8, -4, (part,), generator=g, device="cuda").float())
        b[at:at + part] = torch.randn(part, generator=g, device="cuda").half()
    y = torch.full((M, N), 7.0, dtype=torch.float16, device="cuda")
    vq.vq_gemm_w8a8(xq, xs, wq, ws, b, y=y)
    for at in spots:
        acc = xq.double() @ wq[at:at + part].double().t()
        want = (acc * xs.double()[:, None] * ws[at:at + part].double()[None] + b[at:at + part].double()).half()
        assert torch.equal(y[:, at:at + part], want), at
    # every other output is its bias
    assert all(int((y[m] == b).sum()) >= N - 3 * part for m in range(M))


# 2^35 elements and a few rows, in place: one launch would be 2^32 threads.  Rows at both ends and where the second
# launch begins, against the same rows rotated by themselves
def test_rotation_of_a_very_large_weight(vq, room):
    K, N = 8192, (1 << 22) + 37
    room(N * K * 4)
    print(f"rotate weight {N} x {K} in place", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    s = torch.exp(torch.randn(K, generator=g, device="cuda") * 0.3)
    w = torch.empty((N, K), device="cuda")
    spots = [0, N // 2, (1 << 22) - 5, N - 8]
    want = []
    for at in spots:
        w[at:at + 8] = torch.randn((8, K), generator=g, device="cuda")
        want.append(vq.vq_rotate_weight(w[at:at + 8].clone(), s))
    vq.vq_rotate_weight(w, s, w)
    for at, rows in zip(spots, want):
        assert torch.equal(w[at:at + 8], rows), at
