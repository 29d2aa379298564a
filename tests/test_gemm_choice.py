"""Which GEMM kernel a problem reaches: the choice is made on the host and needs no GPU."""
import ctypes
import os

import pytest

from paper_2406_02540_amd import binding, build
from gemm_shapes import EIGHT_BIT_TILES, EVERY_TILE, EVERY_TILE_CASES, ONE_OF_EACH_TILE

CUS = 256   # of an MI355X


@pytest.fixture(scope="module", autouse=True)
def built():
    if not (os.path.exists(binding.LIB_PATH) and os.path.exists(binding.EXT_PATH)):
        build.build(verbose=False)


def choice(bits, M, N, K):
    """(tokens, channels, wavefronts that divide K or 0) of the tile that launch_gemm takes."""
    out = (ctypes.c_int * 3)()
    binding.lib().vq_internal_gemm_choice(bits, M, N, K, CUS, out)
    return tuple(out)


# few channels, few sums and very many tokens (or the other way round): the tiles that divide K take 192 threads for 32 tokens
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N", [(700_000_000, 8), (750_000_000, 8), (1_000_000_000, 32), (1_100_000_000, 1),
                                 (1, 700_000_000), (1, 750_000_000)])
def test_launch_stays_below_2_to_32_threads(bits, M, N):
    t, c, waves = choice(bits, M, N, 32)
    if waves or t != 256:   # (the persistent kernel has a workgroup per CU)
        tiles = -(-M // t) * -(-N // c)
        assert -(-tiles // 8) * 8 * (64 * waves or 512) < 2 ** 32


# how the persistent kernel writes rows, of int8, packed and fp16 operands alike: those of whole chunks never as any row
@pytest.mark.parametrize("N,at,sums,want", [(1152, 0, 0, 0), (32, 64, 0, 0), (1152, 16, 0, 1), (1160, 0, 0, 1), (8, 0, 0, 1),
                                            (3464, 48, 0, 1), (1153, 0, 0, 2), (1152, 0, 1, 2),
                                            ((1 << 21) - 8, 0, 0, 1), (1 << 21, 0, 0, 2)])
def test_rows_of_whole_chunks_go_out_in_chunks(N, at, sums, want):
    assert binding.lib().vq_internal_gemm_out(N, ctypes.c_void_p(4096 + at), ctypes.c_void_p(4096 if sums else None)) == want


# ... and stores are of dwords, so that rows of whole dwords (Y itself is 16-byte aligned) are none either
@pytest.mark.parametrize("N,at,sums,want", [(1156, 0, 0, 1), (1154, 16, 0, 1), (2, 0, 0, 1), ((1 << 21) - 2, 0, 0, 1), (1, 0, 0, 2),
                                            (1154, 0, 1, 2)])
def test_rows_of_whole_dwords_go_out_in_dwords(N, at, sums, want):
    assert binding.lib().vq_internal_gemm_out(N, ctypes.c_void_p(4096 + at), ctypes.c_void_p(4096 if sums else None)) == want


# what the GPU tests run to reach each kernel reaches it, in both widths, with whole lines of K and with a tail
def test_shapes_reach_their_tiles():
    for tile, M, N, K in EVERY_TILE_CASES + [(tuple(c[:3]), *c[3:]) for c in ONE_OF_EACH_TILE]:
        for bits in (8, 4):
            assert choice(bits, M, N, K) == tile, (bits, M, N, K)
    for tile, M, N, K in EIGHT_BIT_TILES:
        assert choice(8, M, N, K) == tile, (M, N, K)
    assert {tuple(c[:3]) for c in ONE_OF_EACH_TILE} == set(EVERY_TILE)
    for tile, shapes in EVERY_TILE.items():
        assert {K % 128 != 0 for _, _, K in shapes} == {True, False}, tile


# ... and no kernel is left out: what is picked over a spread of problems
def test_every_tile_has_shapes():
    steps = (1, 7, 33, 64, 129, 256, 300, 500, 700, 1001, 1500, 2100, 3000, 5003, 9000)
    picked = {choice(bits, M, N, K) for bits in (8, 4) for M in steps for N in steps for K in (32, 128, 512, 1152, 2080, 4096)}
    assert picked == set(EVERY_TILE)


# many tokens and few channels: memory sets the time, and tiles that ask for the same activations several times over, or
# few of them at a time, take a quarter to two fifths longer
@pytest.mark.parametrize("bits,M,N,K,tile", [(8, 17964, 88, 3744, (128, 128, 0)), (8, 19294, 78, 2080, (128, 128, 0)),
                                             (8, 35115, 136, 3216, (256, 192, 0)), (4, 22909, 643, 4000, (256, 192, 0)),
                                             (8, 14654, 48, 4608, (64, 64, 0)), (4, 23559, 64, 2848, (128, 64, 0))])
def test_many_tokens_and_few_channels(bits, M, N, K, tile):
    assert choice(bits, M, N, K) == tile
