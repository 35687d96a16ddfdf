"""GPU: the tiled MXFP4 GEMM where its scale bytes are copied for several units of 256 k at once.

Rows of scale bytes that start on dwords come in chunks of two or four units, others in windows of one or three; numbers of units around those, a last
unit of every length, last bytes of the operand that are no whole word, runs of K' that begin anywhere.  Operands lie in front of poison (scale
bytes that decode to NaN).  Reference: the packed bytes' definition in 64 bits.
"""
import pytest
import torch

from paper_2601_07475_amd import binding as B
from test_gpu_ragged import dequantize, operand, worst

pytestmark = pytest.mark.gpu

TILES = {(128, 128): (300, 261), (192, 128): (1277, 4090), (128, 256): (2047, 4093), (192, 256): (767, 14333), (256, 256): (1022, 14331)}
# K' in runs: of units off the chunks' boundaries, and of single ones
RUNS = [(8, 300, 261, 128), (6, 300, 261, 129), (6, 300, 261, 131), (5, 100, 100, 120), (8, 100, 100, 122), (8, 100, 100, 255), (8, 100, 100, 300)]
CASES = [(*tile, 1, M, N, nb) for tile, (M, N) in TILES.items() for nb in (4, 8, 12, 20, 28, 32, 36, 64, 68, 76, 17, 23, 25, 33, 47, 49, 51, 71, 73)] + \
        [(128, 128, *run) for run in RUNS]


@pytest.mark.parametrize("rows,cols,runs,M,N,nb", CASES)
def test_scale_bytes_of_several_units(rows, cols, runs, M, N, nb):
    """The scaled matrix instruction keeps fewer bits inside one instruction: 1.5e-4 of the product's 2-norm."""
    assert B.arcq_mx_gemm_route(M, N, nb * 32, True)[:4] == (B.ROUTE_TILES, rows, cols, runs)
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 32), operand(g, N, nb, 32)
    ref = dequantize(*a, 32) @ dequantize(*w, 32).t()
    ws = torch.empty(max(B.arcq_mx_gemm_workspace_size(M, N, nb * 32), 256), dtype=torch.uint8, device="cuda")
    y = B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32, workspace=ws)
    assert float((y.double() - ref).norm() / ref.norm()) <= 6e-4 and worst(y, ref) <= 5e-3
    assert torch.equal(B.arcq_mx_gemm(*a, *w, workspace=ws), y.half())
    for _ in range(3):                                  # the same bits whenever it runs
        assert torch.equal(B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32, workspace=ws), y)


@pytest.mark.parametrize("rows,cols,runs,M,N,nb", CASES)
def test_every_scale_byte_counts(rows, cols, runs, M, N, nb):
    """Scales of 1/2 to 4: every product is a multiple of 1/16 and every sum, of up to 9600 products of at most 576 at random signs, far below 2^20, so that
    24 bits hold all of them and the result is exact.  One scale byte that is lost or from another place shows in its row."""
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 32), operand(g, N, nb, 32)
    for _, scales in (a, w):
        scales.copy_(torch.randint(126, 130, scales.shape, generator=g, device="cuda", dtype=torch.uint8))
    ref = dequantize(*a, 32) @ dequantize(*w, 32).t()
    assert float(ref.abs().max()) < 2 ** 20
    ws = torch.empty(max(B.arcq_mx_gemm_workspace_size(M, N, nb * 32), 256), dtype=torch.uint8, device="cuda")
    assert torch.equal(B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32, workspace=ws).double(), ref)
