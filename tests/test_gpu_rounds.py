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


# Rows of y of any length, at 4-byte aligned starts, with a stride of their own: vector stores at addresses that are multiples of a value
# only; nothing is written between the rows.  A shape for every kernel with an epilogue of its own: k pairs, tiles, k split, 128 x 128.
@pytest.mark.parametrize("M,N,nb", [(2047, 4093, 32), (767, 14333, 18), (190, 4091, 34), (300, 261, 22)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("pad", [0, 2, 5])
def test_rows_of_y_at_any_address(M, N, nb, dtype, pad):
    for block, gemm in ((16, lambda a, w, y: B.arcq_gemm(*a, 2.0 ** -12, *w, 1.0, y=y)), (32, lambda a, w, y: B.arcq_mx_gemm(*a, *w, y=y))):
        g = torch.Generator(device="cuda").manual_seed(M + N + nb)
        a, w = operand(g, M, nb, block), operand(g, N, nb, block)
        raw = torch.full((M * (N + pad) + 16,), 777.0, dtype=dtype, device="cuda")
        rows = raw[2:2 + M * (N + pad)].view(M, N + pad)
        gemm(a, w, rows[:, :N])
        ref = torch.full((M, N), 555.0, dtype=dtype, device="cuda")
        gemm(a, w, ref)
        assert torch.equal(rows[:, :N], ref) and bool((rows[:, N:] == 777.0).all())
        assert bool((raw[:2] == 777.0).all()) and bool((raw[2 + M * (N + pad):] == 777.0).all())
        out = dequantize(*a, block) @ dequantize(*w, block).t() * (2.0 ** -12 if block == 16 else 1.0)
        fits = out.abs() < 60000.0 if dtype == torch.float16 else torch.ones_like(out, dtype=torch.bool)
        assert worst(torch.where(fits, ref.double(), 0.0), torch.where(fits, out, 0.0)) <= 5e-3
