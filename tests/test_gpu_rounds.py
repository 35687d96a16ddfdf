"""GPU: how the tiles of a GEMM are dealt to workgroups and launches, and how they reach y."""
import pytest
import torch

from paper_2601_07475_amd import binding as B
from test_gpu_ragged import dequantize, operand, worst

pytestmark = pytest.mark.gpu


def every_tile(M, N, block):
    gemm = (lambda a, w: B.arcq_gemm(*a, 1.0, *w, 1.0, out_dtype=torch.float32)) if block == 16 else (lambda a, w: B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32))
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, w = operand(g, M, 512 // block, block), operand(g, N, 512 // block, block)
    assert worst(gemm(a, w), dequantize(*a, block) @ dequantize(*w, block).t()) <= (2e-5 if block == 16 else 5e-3)


# MXFP4, 128 x 128 tiles: fewer tiles than XCDs, one more than a multiple of 8, tile rows in one, two and three groups of unequal height, and
# row by row.  (The NVFP4 problems of these sizes run other tiles.)
@pytest.mark.parametrize("tiles_m,tiles_n", [(1, 1), (1, 7), (3, 3), (9, 1), (9, 5), (11, 3), (17, 2), (19, 7), (20, 7), (23, 3), (33, 5)])
def test_every_tile_is_computed(tiles_m, tiles_n):
    M, N = 128 * tiles_m - 5, 128 * tiles_n - 3
    assert B.arcq_mx_gemm_route(M, N, 512)[:4] == (B.ROUTE_TILES, 128, 128, 1)
    for block in (16, 32):
        every_tile(M, N, block)


# the same of NVFP4 tiles, whose kernels are two more
@pytest.mark.parametrize("kernel,rows,cols,tiles_m,tiles_n", [
    (2, 128, 128, 2, 1), (2, 128, 128, 9, 17), (2, 128, 128, 17, 9), (2, 128, 128, 23, 7), (1, 64, 32, 3, 11), (1, 64, 32, 9, 5), (1, 64, 32, 17, 3),
    (1, 64, 32, 25, 3), (1, 64, 64, 9, 15), (1, 64, 64, 33, 5), (1, 96, 64, 9, 19), (1, 96, 64, 27, 7), (1, 64, 128, 9, 17), (1, 64, 128, 31, 5),
    (2, 192, 128, 11, 17), (2, 128, 256, 17, 12), (2, 192, 256, 15, 12)])
def test_every_nvfp4_tile_is_computed(kernel, rows, cols, tiles_m, tiles_n):
    M, N = rows * tiles_m - 5, cols * tiles_n - 3
    assert B.arcq_gemm_route(M, N, 512)[:4] == (kernel, rows, cols, 1) and B.arcq_gemm_rest(M, N, 512) is None
    every_tile(M, N, 16)


# Rows of y of any length, at 4-byte aligned starts, with a stride of their own: vector stores at addresses that are multiples of a value
# only; nothing is written between the rows.  A shape for every kernel with an epilogue of its own: k pairs, tiles, k split, 128 x 128.
@pytest.mark.parametrize("route,M,N,nb", [((2, 128, 256), 2047, 4093, 32), ((2, 192, 256), 767, 14333, 18), ((1, 64, 64), 190, 4091, 34),
                                          ((2, 128, 128), 300, 261, 22)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("pad", [0, 2, 5])
def test_rows_of_y_at_any_address(route, M, N, nb, dtype, pad):
    assert B.arcq_gemm_route(M, N, nb * 16)[:3] == route and B.arcq_gemm_rest(M, N, nb * 16) is None
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


# whole rounds of large tiles and, in a second launch, the columns (rows) behind them: every kernel that may take those, K' on and off the
# grid of 64, the last rows of both operands (whose windows of scale bytes come from the patch) in either launch
TWO = [((1, 128, 128), (0, 16, 48), 392, 8329, 155), ((1, 128, 128), (1, 64, 32), 497, 9199, 249), ((1, 128, 128), (1, 96, 128), 647, 10877, 219),
       ((2, 192, 256), (2, 128, 128), 1335, 12144, 81), ((2, 192, 256), (2, 128, 256), 1580, 12643, 75), ((2, 256, 256), (0, 16, 64), 1287, 12320, 69),
       ((2, 256, 256), (1, 64, 128), 1196, 14070, 73), ((2, 256, 256), (1, 64, 64), 1155, 13815, 82), ((2, 256, 256), (1, 64, 64), 2914, 5838, 82),
       ((2, 256, 256), (1, 96, 64), 1373, 12706, 79), ((2, 256, 256), (1, 128, 64), 2797, 6547, 98), ((2, 256, 256), (2, 192, 128), 1393, 15585, 100),
       ((2, 256, 256), (1, 128, 128), 2118, 8529, 106), ((2, 256, 256), (2, 192, 256), 2643, 14915, 71)]


@pytest.mark.parametrize("first,rest,M,N,nb", TWO)
def test_two_launches(first, rest, M, N, nb):
    assert B.arcq_gemm_route(M, N, nb * 16)[:3] == first and B.arcq_gemm_rest(M, N, nb * 16)[2] == rest
    assert B.arcq_gemm_workspace_size(M, N, nb * 16) == 0
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 16), operand(g, N, nb, 16)
    ref = dequantize(*a, 16) @ dequantize(*w, 16).t()
    for dtype, tol in ((torch.float32, 2e-5), (torch.float16, 1e-3)):
        scale = 2.0 ** -12 if dtype == torch.float16 else 1.0        # keeps fp16 results finite; exact
        raw = torch.full((M, N + 3), 777.0, dtype=dtype, device="cuda")
        B.arcq_gemm(*a, scale, *w, 1.0, y=raw[:, :N])
        assert worst(raw[:, :N], ref * scale) <= tol, dtype
        assert bool((raw[:, N:] == 777.0).all())
        y = torch.empty((M, N), dtype=dtype, device="cuda")
        B.arcq_gemm_noalloc(*a, scale, *w, 1.0, y)
        assert torch.equal(y, raw[:, :N])
    # codes at their minimum alignment; scale bytes at odd addresses (the rule's kernel, in one launch)
    for lead, code_lead in ((0, 8), (1, 0)):
        a1 = operand(torch.Generator(device="cuda").manual_seed(M + N + nb), M, nb, 16, lead=lead, code_lead=code_lead)
        assert worst(B.arcq_gemm(*a1, 1.0, *w, 1.0, out_dtype=torch.float32), ref) <= 2e-5


# one launch that the modelled times prefer to the rule: k-split tiles in several rounds, tiles in rounds of another height
@pytest.mark.parametrize("route,M,N,nb", [((1, 128, 128), 2917, 1071, 245), ((1, 96, 128), 387, 6429, 98), ((2, 128, 256), 992, 5520, 90),
                                          ((2, 128, 128), 1634, 7280, 160), ((2, 192, 128), 1152, 27152, 116)])
def test_one_launch_by_time(route, M, N, nb):
    assert B.arcq_gemm_route(M, N, nb * 16)[:3] == route and B.arcq_gemm_rest(M, N, nb * 16) is None
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 16), operand(g, N, nb, 16)
    assert worst(B.arcq_gemm(*a, 1.0, *w, 1.0, out_dtype=torch.float32), dequantize(*a, 16) @ dequantize(*w, 16).t()) <= 2e-5


# 65 to 128 rows with odd weight rows: k-split tiles, and the streaming kernel where scale bytes lie at odd addresses
@pytest.mark.parametrize("M,N,nb", [(75, 7103, 111), (112, 23375, 77), (128, 9998, 66), (80, 24001, 48)])
def test_odd_weight_rows_on_tiles(M, N, nb):
    assert B.arcq_gemm_route(M, N, nb * 16)[0] == B.ROUTE_KSPLIT
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 16), operand(g, N, nb, 16)
    ref = dequantize(*a, 16) @ dequantize(*w, 16).t()
    for lead, code_lead in ((0, 0), (0, 8), (1, 0)):
        a1 = operand(torch.Generator(device="cuda").manual_seed(M + N + nb), M, nb, 16, lead=lead, code_lead=code_lead)
        assert worst(B.arcq_gemm(*a1, 1.0, *w, 1.0, out_dtype=torch.float32), ref) <= 2e-5


# the streaming kernels with more weight rows than a round takes: one and two tiles a wave behind it, ragged rows and edges
def streamed(M, N, nb, block, gemm):
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, block), operand(g, N, nb, block)
    ref = dequantize(*a, block) @ dequantize(*w, block).t()
    raw = torch.full((M, N + 3), 777.0, dtype=torch.float32, device="cuda")
    gemm(a, w, raw[:, :N])
    assert worst(raw[:, :N], ref) <= (2e-5 if block == 16 else 5e-3) and bool((raw[:, N:] == 777.0).all())
    a1 = operand(torch.Generator(device="cuda").manual_seed(M + N + nb), M, nb, block, lead=1)
    y = torch.empty((M, N), dtype=torch.float32, device="cuda")
    gemm(a1, w, y)
    assert worst(y, ref) <= (2e-5 if block == 16 else 5e-3)


@pytest.mark.parametrize("M,N,nb", [(1, 17408, 256), (16, 20479, 258), (13, 17500, 257), (32, 20481, 385), (7, 24576, 384), (31, 24571, 386)])
def test_streaming_in_two_launches(M, N, nb):
    cols = 16 if N - 16384 <= 4096 else 32
    assert B.arcq_gemm_rest(M, N, nb * 16) == (M, N - 16384, (B.ROUTE_STREAM, 16 if M <= 16 else 32, cols))
    streamed(M, N, nb, 16, lambda a, w, y: B.arcq_gemm(*a, 1.0, *w, 1.0, y=y))


# (32 x 20481 over 12832 streams only where no workspace lets tiles split K')
@pytest.mark.parametrize("M,N,nb", [(1, 17408, 128), (16, 20479, 129), (13, 17500, 257), (7, 24576, 192), (16, 24571, 193), (17, 17500, 128),
                                    (20, 20480, 175), (32, 20479, 129), (32, 20481, 401)])
def test_mx_streaming_in_two_launches(M, N, nb):
    cols = 16 if N - 16384 <= 4096 else 32
    assert B.arcq_mx_gemm_rest(M, N, nb * 32) == (M, N - 16384, (B.ROUTE_STREAM, 16 if M <= 16 else 32, cols))
    streamed(M, N, nb, 32, lambda a, w, y: B.arcq_mx_gemm(*a, *w, y=y))


# two left-over chunks of K' and more: an output's sum has the order, and so the bits, that it has in one launch of four tiles a wave
@pytest.mark.parametrize("M,N,Kp", [(1, 18432, 4352), (16, 20480, 4480), (16, 20480, 8448), (16, 22000, 6400), (17, 17500, 4352), (32, 20480, 4480), (32, 24576, 6400)])
@pytest.mark.parametrize("block", [16, 32])
def test_streaming_in_two_launches_is_the_same_sum(M, N, Kp, block):
    gemm, rest = ((lambda a, w: B.arcq_gemm(*a, 1.0, *w, 1.0, out_dtype=torch.float32), B.arcq_gemm_rest) if block == 16 else
                  (lambda a, w: B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32), B.arcq_mx_gemm_rest))
    whole = 24640
    if block == 32:                     # longer ones run tiles
        Kp, N = (min(Kp, 6400), N) if M <= 16 else (min(Kp, 4480), min(N, 20480))
    assert rest(M, N, Kp)[2][0] == B.ROUTE_STREAM and rest(M, whole, Kp) is None
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a, w = operand(g, M, Kp // block, block), operand(g, whole, Kp // block, block)
    assert torch.equal(gemm(a, (w[0][:N], w[1][:N])), gemm(a, w)[:, :N])
