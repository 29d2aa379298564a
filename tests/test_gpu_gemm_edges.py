"""GEMM kernels at the edges of their tiles and of rows that end inside a vector store: every
output against the exact integer sums, and nothing written outside the output."""
import pytest

from gemm_shapes import EIGHT_BIT_TILES, EVERY_TILE_CASES

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


def check_gemm(vq, bits, M, N, K, seed=3, at=0):
    """Integer sums from float64 products (exact: |sum| <= K * 127^2 < 2^53), outputs from them in
    float64 rounded once: the dequantization is one rounding of an exact multiply-add."""
    print(f"w{bits}a8 M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(seed)
    qmax = 127 if bits == 8 else 7
    xq = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    wq = torch.randint(-qmax, qmax + 1, (N, K), generator=g, device="cuda", dtype=torch.int8)
    w = wq if bits == 8 else ((wq[:, ::2] & 15) | ((wq[:, 1::2] & 15) << 4)).view(torch.uint8).contiguous()
    # power-of-two scales: their product and its product with the sum are exact in fp32
    xs = torch.exp2(torch.randint(-12, -8, (M,), generator=g, device="cuda").float())
    ws = torch.exp2(torch.randint(-8, -4, (N,), generator=g, device="cuda").float())
    b = torch.randn(N, generator=g, device="cuda").half()
    acc = xq.double() @ wq.double().t()
    want = (acc * xs.double()[:, None] * ws.double()[None] + b.double()).half()
    gemm = vq.vq_gemm_w8a8 if bits == 8 else vq.vq_gemm_w4a8
    guard = 64
    buf = torch.full((at + M * N + guard,), 7.0, dtype=torch.float16, device="cuda")
    y = buf[at:at + M * N].view(M, N)
    gemm(xq, xs, w, ws, b, y=y)
    assert torch.equal(y, want), (y != want).sum().item()
    assert (buf[at + M * N:] == 7.0).all() and (buf[:at] == 7.0).all()
    y2, acc2 = gemm(xq, xs, w, ws, b, return_acc=True)
    assert torch.equal(y2, want) and torch.equal(acc2.double(), acc)


# rows of Y that start at any even address (one of them, N % 8 = 4, on dwords): tiles of 256 x 192 in one round (the
# first three) and in two, of 256 x 256 in two rounds and in three, of 128 x 256
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", [(2891, 2817, 160), (2900, 3075, 128), (2305, 4612, 288), (4999, 3075, 160),
                                   (5003, 4999, 96), (5003, 4993, 160), (9000, 4095, 96), (5003, 1151, 96)])
def test_unaligned_output_rows(vq, bits, M, N, K):
    check_gemm(vq, bits, M, N, K)


# ... over stages enough for the persistent kernel's steady loop, in tiles of 256 x 256, with an odd last channel in lanes of one
# and of three channels
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", [(5003, 4999, 1152), (5003, 4993, 1184)])
def test_unaligned_output_rows_over_many_stages(vq, bits, M, N, K):
    assert tile_picked(bits, M, N, K) == (256, 256, 0)
    check_gemm(vq, bits, M, N, K)


# rows of whole 16-byte chunks that do not start on 64-byte boundaries, by N or by Y's address: tiles of 256 x 192
# and of 256 x 256 in one round and in several, full and ragged
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K,at", [(2891, 2824, 160, 0), (2304, 4616, 288, 0), (5003, 5000, 96, 0), (9000, 4104, 96, 0),
                                      (8192, 1152, 128, 8), (5003, 3456, 160, 8)])
def test_output_rows_of_whole_chunks(vq, bits, M, N, K, at):
    check_gemm(vq, bits, M, N, K, at=at)


# ... and rows of whole dwords
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K,at", [(2891, 2820, 160, 0), (8192, 1154, 128, 8), (5003, 3458, 160, 0), (5003, 4994, 96, 0),
                                      (9000, 4098, 128, 8), (260, (1 << 21) - 2, 32, 0)])   # (the last N that is taken there)
def test_output_rows_of_whole_dwords(vq, bits, M, N, K, at):
    check_gemm(vq, bits, M, N, K, at=at)


# every kernel by the tile that it is picked with (test_gemm_choice.py asks whether it still is): ragged last tiles, K of
# one stage, of a few and of many, and a tail
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("tile,M,N,K", EVERY_TILE_CASES)
def test_every_tile(vq, bits, tile, M, N, K):
    check_gemm(vq, bits, M, N, K)


# 256 x 192 keeps two stages of activations in LDS to four stages of K and three from there on: both sides of the line, several
# rounds of tiles, rows of each kind
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", [(9001, 2304, 512), (9001, 2304, 544), (9001, 2306, 480), (9001, 2306, 640), (9001, 2303, 512),
                                   (9001, 2303, 544), (9001, 2304, 128), (9001, 2304, 256)])
def test_stages_of_activations(vq, bits, M, N, K):
    assert tile_picked(bits, M, N, K) == (256, 192, 0)
    check_gemm(vq, bits, M, N, K)


# the tiles whose outputs leave from the registers, by how they write rows (0: on 64-byte boundaries, 1: whole dwords, 2: any
# row): whole and ragged tiles of tokens and channels, with a tail of K and without.  (128 x 64 with 4-bit weights goes through
# LDS and knows one way only: its rows below are stores that end inside a row of eight channels, or don't.)
ROWS_OF_TILES = [((128, 64, 0), 0, 1401, 1856, 128), ((128, 64, 0), 0, 809, 2240, 160), ((128, 64, 0), 1, 982, 2728, 128),
                 ((128, 64, 0), 1, 658, 2392, 416), ((128, 64, 0), 1, 982, 2730, 128), ((128, 64, 0), 1, 658, 2390, 416),
                 ((128, 64, 0), 2, 982, 2729, 128), ((128, 64, 0), 2, 658, 2391, 416), ((128, 128, 0), 0, 2376, 1632, 128),
                 ((128, 128, 0), 0, 490, 4160, 672), ((128, 128, 0), 1, 1541, 1720, 384), ((128, 128, 0), 1, 2790, 984, 160),
                 ((128, 128, 0), 1, 1541, 1722, 384), ((128, 128, 0), 1, 2790, 986, 160), ((128, 128, 0), 2, 1541, 1721, 384),
                 ((128, 128, 0), 2, 2790, 985, 160), ((128, 256, 0), 0, 1175, 3680, 128), ((128, 256, 0), 0, 1911, 2464, 160),
                 ((128, 256, 0), 1, 1417, 3304, 128), ((128, 256, 0), 1, 931, 4656, 160), ((128, 256, 0), 1, 1417, 3306, 128),
                 ((128, 256, 0), 1, 931, 4654, 160), ((128, 256, 0), 2, 1417, 3305, 128), ((128, 256, 0), 2, 931, 4655, 160)]


def tile_picked(bits, M, N, K):
    import ctypes

    from paper_2406_02540_amd import binding
    choice = (ctypes.c_int * 3)()
    binding.lib().vq_internal_gemm_choice(bits, M, N, K, 256, choice)
    return tuple(choice)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("tile,rows,M,N,K", ROWS_OF_TILES)
def test_tiles_write_rows_by_alignment(vq, bits, tile, rows, M, N, K):
    from paper_2406_02540_amd import binding
    assert tile_picked(bits, M, N, K) == tile
    if bits == 8 or tile != (128, 64, 0):
        assert binding.lib().vq_internal_gemm_out(N, None, None) == rows
    check_gemm(vq, bits, M, N, K)


# ... and rows of N % 32 == 0 where Y itself begins off a 64-byte boundary: whole dwords
@pytest.mark.parametrize("bits,tile,M,N,K", [(8, (128, 64, 0), 1401, 1856, 128), (8, (128, 64, 0), 809, 2240, 160)] + [
    (bits, *case) for bits in (8, 4) for case in [((128, 128, 0), 2376, 1632, 128), ((128, 128, 0), 490, 4160, 672),
                                                  ((128, 256, 0), 1175, 3680, 128), ((128, 256, 0), 1911, 2464, 160)]])
def test_tiles_write_rows_by_address(vq, bits, tile, M, N, K):
    import ctypes

    from paper_2406_02540_amd import binding
    assert tile_picked(bits, M, N, K) == tile
    assert [binding.lib().vq_internal_gemm_out(N, ctypes.c_void_p(at), None) for at in (4096, 4096 + 16)] == [0, 1]
    check_gemm(vq, bits, M, N, K, at=8)


# the sums leave these tiles in pairs of channels: an odd last channel alone, rows at any multiple of four bytes, and
# nothing written behind the last one
@pytest.mark.parametrize("bits,tile,M,N,K", [(8, (128, 64, 0), 1153, 2041, 128), (8, (128, 64, 0), 1153, 2042, 128)] + [
    (bits, *case) for bits in (8, 4) for case in [((128, 128, 0), 1926, 1455, 160), ((128, 128, 0), 2153, 1630, 128),
                                                  ((128, 256, 0), 1314, 4057, 128), ((128, 256, 0), 1001, 4608, 160)]])
def test_sums_of_one_tile_per_workgroup(vq, bits, tile, M, N, K):
    import ctypes

    from paper_2406_02540_amd import binding
    assert tile_picked(bits, M, N, K) == tile
    print(f"sums w{bits}a8 M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(11)
    xq = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    wq = torch.randint(-7, 8, (N, K), generator=g, device="cuda", dtype=torch.int8)
    w = wq if bits == 8 else ((wq[:, ::2] & 15) | ((wq[:, 1::2] & 15) << 4)).view(torch.uint8).contiguous()
    ones = torch.ones(max(M, N), device="cuda")
    y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    sums = torch.full((M * N + 64,), 77, dtype=torch.int32, device="cuda")
    gemm = binding.lib().vq_gemm_w8a8 if bits == 8 else binding.lib().vq_gemm_w4a8
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert gemm(p(xq), p(ones), p(w), p(ones), None, p(y), p(sums), M, N, K, stream) == 0
    assert torch.equal(sums[:M * N].view(M, N).double(), xq.double() @ wq.double().t())
    assert (sums[M * N:] == 77).all()


@pytest.mark.parametrize("tile,M,N,K", EIGHT_BIT_TILES)
def test_tiles_of_eight_bit_weights(vq, tile, M, N, K):
    check_gemm(vq, 8, M, N, K)


# one tile per workgroup at the edges of sizes: one token, one channel, one more and one less than a tile's, single
# stages and long K; in tiles whose wavefronts divide K and in shared ones of 32 x 32 to 128 x 256
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", [(1, 8, 32), (1, 1, 32), (31, 33, 64), (33, 31, 4608), (65, 129, 1152), (32, 32, 1024),
                                   (63, 4607, 96), (300, 2000, 1152), (256, 4608, 512),
                                   (1001, 1160, 1152), (1001, 1157, 416),
                                   (1100, 2050, 320), (1500, 2000, 1152), (2000, 1999, 4608),
                                   (1001, 4609, 1152), (1030, 4600, 128), (1025, 4097, 96)])
def test_one_tile_per_workgroup(vq, bits, M, N, K):
    check_gemm(vq, bits, M, N, K)


# wavefronts that divide K (32 x 32 with three, six and eight of them, 48 x 48; a few of the shapes run in shared tiles, and 64 x 32
# and 64 x 64 have theirs in EVERY_TILE): fewer lines of K than wavefronts, a line more than they share evenly, tails of a line, ragged last tiles
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", [(100, 1000, 160), (100, 1001, 512), (1000, 200, 800), (999, 31, 4608), (16, 1152, 4608),
                                   (61, 1001, 1184), (500, 4607, 512), (300, 1152, 4096), (257, 1149, 4128),
                                   (239, 2301, 4000), (240, 2304, 4096), (257, 2300, 2080)])
def test_wavefronts_divide_k(vq, bits, M, N, K):
    check_gemm(vq, bits, M, N, K)
