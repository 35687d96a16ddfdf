"""The streaming kernels with more weight rows than a round of four tiles a wave takes: five to seven tiles, and rounds of four and of three."""
import pytest
import torch

from paper_2601_07475_amd import binding as B
from test_gpu_ragged import operand
from test_gpu_rounds import streamed

pytestmark = pytest.mark.gpu


# first and last weight rows of every number of tiles, in one round and in two; one group per wave and several, left-over chunks, odd block counts
@pytest.mark.parametrize("M,N,nb", [(1, 16385, 32), (16, 17407, 257), (32, 20480, 129), (16, 20481, 255), (17, 24576, 192), (7, 24577, 353), (16, 28672, 529),
                                    (32, 28672, 160), (18, 28671, 353), (32, 24577, 384), (31, 28672, 385), (20, 26000, 529), (2, 32769, 64),
                                    (32, 40960, 71), (16, 40961, 65), (24, 57344, 33), (16, 57344, 97), (32, 57344, 385), (16, 57345, 64), (32, 16400, 1)])
def test_more_weight_tiles_a_wave(M, N, nb):
    route = B.arcq_gemm_route(M, N, nb * 16)
    assert route[:4] == (B.ROUTE_STREAM, 16 if M <= 16 else 32, 64, 1) and B.arcq_gemm_rest(M, N, nb * 16) is None
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


@pytest.mark.parametrize("M,N,nb", [(1, 16385, 16), (16, 17407, 129), (32, 20480, 67), (16, 20481, 131), (17, 24576, 130), (7, 24577, 145), (16, 28672, 66),
                                    (32, 28672, 50), (18, 28671, 67), (32, 20481, 32), (20, 26000, 35), (2, 32769, 33), (32, 40960, 66), (16, 40961, 65),
                                    (24, 36000, 17), (16, 57344, 50), (16, 57345, 33), (32, 16400, 1)])
def test_more_mx_weight_tiles_a_wave(M, N, nb):
    route = B.arcq_mx_gemm_route(M, N, nb * 32)
    assert route[:4] == (B.ROUTE_STREAM, 16 if M <= 16 else 32, 64, 1) and B.arcq_mx_gemm_rest(M, N, nb * 32) is None
    streamed(M, N, nb, 32, lambda a, w, y: B.arcq_mx_gemm(*a, *w, y=y))


@pytest.mark.parametrize("M,N,nb", [(16, 20480, 127), (16, 24576, 140), (16, 28672, 140), (32, 20000, 100), (32, 24576, 132), (32, 28672, 68)])
def test_more_mx_weight_tiles_a_wave_are_the_same_sum(M, N, nb):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, w = operand(g, M, nb, 32), operand(g, N, nb, 32)
    y = B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32)
    for first in (0, N - 12300):
        part = B.arcq_mx_gemm(*a, w[0][first:first + 12300], w[1][first:first + 12300], out_dtype=torch.float32)
        assert torch.equal(y[:, first:first + 12300], part)
