"""The streaming kernels with more weight rows than a round of four tiles a wave takes: five to seven tiles, and rounds of four and of three."""
import pytest
import torch

from paper_2601_07475_amd import binding as B
from test_gpu_ragged import operand
from test_gpu_rounds import streamed

pytestmark = pytest.mark.gpu


# first and last weight rows of every number of tiles, in one round and in two; one group per wave and several, left-over chunks, odd block counts; the weight
# tiles a wave takes, and those of a wave behind the first round
NVFP4 = [(1, 16385, 32, 5, 5), (16, 17407, 257, 5, 5), (32, 20480, 129, 5, 5), (16, 20481, 255, 6, 6), (17, 24576, 192, 6, 6),
         (7, 24577, 353, 7, 7), (16, 28672, 529, 7, 7), (32, 28672, 160, 7, 7), (18, 28671, 353, 7, 7), (32, 24577, 384, 4, 3),
         (31, 28672, 385, 4, 3), (20, 26000, 529, 4, 3), (2, 32769, 64, 5, 5), (32, 40960, 71, 5, 5), (16, 40961, 65, 6, 6),
         (24, 57344, 33, 7, 7), (16, 57344, 97, 7, 7), (32, 57344, 385, 4, 4), (16, 57345, 64, 4, 4), (32, 16400, 1, 5, 5)]


@pytest.mark.parametrize("M,N,nb,tiles,behind", NVFP4)
def test_more_weight_tiles_a_wave(M, N, nb, tiles, behind):
    route = B.arcq_gemm_route(M, N, nb * 16)
    assert route[:4] == (B.ROUTE_STREAM, 16 if M <= 16 else 32, 64, 1) and B.arcq_gemm_rest(M, N, nb * 16) is None
    assert B.arcq_gemm_stream_tiles(M, N, nb * 16) == (tiles, behind)
    streamed(M, N, nb, 16, lambda a, w, y: B.arcq_gemm(*a, 1.0, *w, 1.0, y=y))


# K' in the order of four tiles a wave: the bits that the first round of weight rows has by itself
@pytest.mark.parametrize("M,N,nb", [(16, 20480, 255), (16, 24576, 140), (16, 28672, 280), (32, 20000, 200), (32, 24576, 264), (32, 28672, 264), (32, 28672, 529)])
def test_more_weight_tiles_a_wave_are_the_same_sum(M, N, nb):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, w = operand(g, M, nb, 16), operand(g, N, nb, 16)
    y = B.arcq_gemm(*a, 1.0, *w, 1.0, out_dtype=torch.float32)
    for first in (0, N - 12300):
        part = B.arcq_gemm(*a, 1.0, w[0][first:first + 12300], w[1][first:first + 12300], 1.0, out_dtype=torch.float32)
        assert torch.equal(y[:, first:first + 12300], part)


MX = [(1, 16385, 16, 5, 5), (16, 17407, 129, 5, 5), (32, 20480, 67, 5, 5), (16, 20481, 131, 6, 6), (17, 24576, 130, 4, 2),
      (7, 24577, 145, 7, 7), (16, 28672, 66, 7, 7), (32, 28672, 50, 4, 3), (18, 28671, 67, 4, 3), (32, 20481, 32, 4, 2),
      (20, 26000, 35, 4, 3), (2, 32769, 33, 4, 4), (2, 32785, 33, 5, 5), (32, 40960, 66, 5, 5), (16, 40961, 65, 6, 6), (24, 36000, 17, 5, 5),
      (16, 57344, 50, 7, 7), (16, 57345, 33, 4, 4), (32, 16400, 1, 5, 5)]


@pytest.mark.parametrize("M,N,nb,tiles,behind", MX)
def test_more_mx_weight_tiles_a_wave(M, N, nb, tiles, behind):
    route = B.arcq_mx_gemm_route(M, N, nb * 32)
    assert route[:4] == (B.ROUTE_STREAM, 16 if M <= 16 else 32, 64, 1) and B.arcq_mx_gemm_rest(M, N, nb * 32) is None
    assert B.arcq_mx_gemm_stream_tiles(M, N, nb * 32) == (tiles, behind)
    streamed(M, N, nb, 32, lambda a, w, y: B.arcq_mx_gemm(*a, *w, y=y))


@pytest.mark.parametrize("M,N,nb", [(16, 20480, 127), (16, 24576, 140), (16, 28672, 140), (32, 20000, 100), (32, 24576, 132), (32, 28672, 68)])
def test_more_mx_weight_tiles_a_wave_are_the_same_sum(M, N, nb):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, w = operand(g, M, nb, 32), operand(g, N, nb, 32)
    y = B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32)
    for first in (0, N - 12300):
        part = B.arcq_mx_gemm(*a, w[0][first:first + 12300], w[1][first:first + 12300], out_dtype=torch.float32)
        assert torch.equal(y[:, first:first + 12300], part)
