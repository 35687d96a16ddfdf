"""GPU: how the tiles of a GEMM are dealt to workgroups."""
import pytest
import torch

from paper_2601_07475_amd import binding as B
from test_gpu_ragged import dequantize, operand, worst

pytestmark = pytest.mark.gpu


# fewer tiles than XCDs, one more than a multiple of 8, tile rows in one, two and three groups of unequal height
@pytest.mark.parametrize("tiles_m,tiles_n", [(1, 1), (1, 7), (3, 3), (9, 1), (9, 5), (11, 3), (17, 2), (19, 7)])
def test_every_tile_is_computed(tiles_m, tiles_n):
    M, N = 128 * tiles_m - 5, 128 * tiles_n - 3
    for block, gemm in ((16, lambda a, w: B.arcq_gemm(*a, 1.0, *w, 1.0, out_dtype=torch.float32)),
                        (32, lambda a, w: B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32))):
        g = torch.Generator(device="cuda").manual_seed(tiles_m + tiles_n)
        a, w = operand(g, M, 512 // block, block), operand(g, N, 512 // block, block)
        assert worst(gemm(a, w), dequantize(*a, block) @ dequantize(*w, block).t()) <= (2e-5 if block == 16 else 5e-3)
