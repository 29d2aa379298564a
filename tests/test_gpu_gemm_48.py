"""The GEMM's tiles of 48 x 48, which take the place of some of 64 tokens: which problems reach them (decided on the host), and
every output and sum exactly."""
import ctypes
import os

import pytest

from paper_2406_02540_amd import binding, build
from test_gpu_gemm_edges import check_gemm, vq  # noqa: F401  (a fixture)

# a token or channel more and less than tiles hold, as many tiles as CUs, K of a line more than the wavefronts share evenly,
# tails of a line; the divided 64 x 64 tile's place, the shared one's and 64 x 32's
TAKEN = [(240, 2304, 4096), (239, 2303, 4000), (760, 746, 4096), (768, 768, 3104), (769, 720, 4128), (1514, 366, 4000),
         (97, 4033, 2080), (192, 3000, 2048), (500, 1040, 3168), (1034, 495, 1568), (1491, 336, 1824)]
NOT_TAKEN = [(310, 2001, 4096), (769, 769, 4096), (16, 1152, 4608), (256, 1152, 1152), (360, 1504, 576), (41, 4192, 2016),
             (8192, 1152, 4608)]
# ... and in the shared 64 x 64 tile's place not below twelve lines of K, eight wavefronts' second turn: 1.07 of its time at nine
SHARED_STAYS = [(432, 1283, 1152), (588, 890, 1152), (824, 641, 1152), (2358, 216, 1184), (621, 892, 1280), (1205, 421, 1376)]


def taken(bits, M, N, K):
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    choice = (ctypes.c_int * 3)()
    binding.lib().vq_internal_gemm_choice(bits, M, N, K, 256, choice)
    return tuple(choice) == (48, 48, 8)


def test_which_problems_take_them():
    for M, N, K in NOT_TAKEN:
        assert not taken(8, M, N, K) and not taken(4, M, N, K), (M, N, K)
    for M, N, K in SHARED_STAYS:
        assert not taken(8, M, N, K), (M, N, K)
    for M, N, K in TAKEN:
        assert taken(8, M, N, K), (M, N, K)
        assert -(-M // 48) * -(-N // 48) <= 256
    assert sum(taken(4, M, N, K) for M, N, K in TAKEN) >= 9


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,N,K", TAKEN)
def test_outputs(vq, bits, M, N, K):  # noqa: F811
    check_gemm(vq, bits, M, N, K)
