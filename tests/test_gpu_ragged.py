"""GPU: the tiled GEMMs over K' that is a multiple of one block only, where rows of scale bytes start at any address.

Operands are random packed bytes placed right in front of poison (scale bytes that decode to NaN), so a scale byte from
behind a row or an operand that enters the product shows.  Reference: the packed bytes' definition in 64 bits.
"""
import pytest
import torch

from paper_2601_07475_amd import binding as B

pytestmark = pytest.mark.gpu

E2M1 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]


def operand(g, rows, nb, block, lead=0, code_lead=0):
    """(codes, scales) uint8 with poison behind both, scale bytes `lead` bytes off a 4-byte boundary, codes `code_lead` off 16."""
    def place(rows, width, values, lead):
        n = rows * width
        raw = torch.full((n + lead + 64,), 0xFF, dtype=torch.uint8, device="cuda")
        out = raw[lead:lead + n].view(rows, width)
        out.copy_(values)
        return out
    codes = torch.randint(0, 256, (rows, nb * block // 2), generator=g, device="cuda", dtype=torch.uint8)
    if block == 16:
        sc = torch.randint(0, 0x50, (rows, nb), generator=g, device="cuda", dtype=torch.uint8)
    else:
        sc = torch.randint(118, 134, (rows, nb), generator=g, device="cuda", dtype=torch.uint8)
    return place(rows, nb * block // 2, codes, code_lead), place(rows, nb, sc, lead)


def dequantize(codes, scales, block):
    grid = torch.tensor(E2M1 + [-v for v in E2M1], dtype=torch.float64, device="cuda")
    v = torch.stack([grid[(codes & 15).long()], grid[(codes >> 4).long()]], dim=-1).flatten(1)
    s = scales.long()
    if block == 16:
        val = torch.where(s < 8, s.double() / 512, (1 + (s & 7).double() / 8) * torch.exp2(((s >> 3) - 7).double()))
    else:
        val = torch.exp2((s - 127).double())
    return v * val.repeat_interleave(block, dim=1)


def worst(y, ref):
    rms = ref.square().mean().sqrt()
    return float(((y.double() - ref).abs() / ref.abs().clamp(min=rms)).max())


# Shapes with ragged edges for every tile, under the tile's rows and columns (asserted: a changed rule cannot empty a list).  Rows of
# 16 blocks (two stages) and more; block counts that are multiples of four run the direct copies, the others the windows.
STAGED = {
    (128, 128): [(300, 261, b) for b in (16, 17, 22, 31)],
    (192, 128): [(1277, 4090, b) for b in (19, 24, 26)] + [(150, 28600, b) for b in (33, 40)],
    (128, 256): [(2047, 4093, b) for b in (17, 20, 23, 30)],
    (192, 256): [(767, 14333, b) for b in (18, 20, 21, 25)],
    (256, 256): [(1022, 14331, b) for b in (17, 27, 28)],
}
# k quarters inside the workgroup, rows of 32 blocks (two stages) and more; values stored by fours and one by one
KSPLIT = {
    (64, 32): [(130, 1021, b) for b in (33, 36, 46, 63)],
    (64, 64): [(190, 4091, b) for b in (34, 49)] + [(301, 3070, b) for b in (35, 48, 61)],
    (96, 64): [(147, 5629, b) for b in (33, 46)] + [(65, 8920, b) for b in (36, 39, 50)] + [(509, 2555, 62)],
    (64, 128): [(510, 4090, b) for b in (32, 47, 50)] + [(61, 20475, b) for b in (33, 40, 46)] + [(194, 4249, 36)] + [(509, 2555, 37)],
    (128, 64): [(582, 3260, b) for b in (34, 37, 47, 48)] + [(1256, 1565, b) for b in (42, 55)],
    (96, 128): [(335, 6140, b) for b in (36, 47, 53)] + [(130, 11013, b) for b in (57, 60, 70)],
    (128, 128): [(198, 8692, b) for b in (33, 36, 46)] + [(212, 8221, b) for b in (188, 191)],
}
# 128 x 128 tiles with K' in this many runs across workgroups
RUNS = {2: [(257, 131, 66)], 7: [(300, 77, 257), (140, 260, 259)], 8: [(256, 500, 577), (140, 260, 300)]}
NVFP4 = [(B.ROUTE_TILES, *tile, 1, *shape) for tile, shapes in STAGED.items() for shape in shapes] + \
        [(B.ROUTE_KSPLIT, *tile, 1, *shape) for tile, shapes in KSPLIT.items() for shape in shapes] + \
        [(B.ROUTE_TILES, 128, 128, runs, *shape) for runs, shapes in RUNS.items() for shape in shapes]


@pytest.mark.parametrize("kernel,rows,cols,runs,M,N,nb", NVFP4)
def test_nvfp4_any_number_of_blocks(kernel, rows, cols, runs, M, N, nb):
    assert B.arcq_gemm_route(M, N, nb * 16)[:4] == (kernel, rows, cols, runs)
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 16), operand(g, N, nb, 16)
    ref = dequantize(*a, 16) @ dequantize(*w, 16).t()
    for dtype, tol in ((torch.float32, 2e-5), (torch.float16, 1e-3)):
        scale = 2.0 ** -12 if dtype == torch.float16 else 1.0        # keeps fp16 results finite; exact
        y = B.arcq_gemm(*a, scale, *w, 1.0, out_dtype=dtype)
        assert worst(y, ref * scale) <= tol, dtype
    # scale bytes at odd addresses go through registers: the same products (no 256 x 256 tiles there: a smaller one)
    a1 = operand(torch.Generator(device="cuda").manual_seed(M + N + nb), M, nb, 16, lead=1)
    assert torch.equal(a1[0], a[0]) and torch.equal(a1[1], a[1])
    assert worst(B.arcq_gemm(*a1, 1.0, *w, 1.0, out_dtype=torch.float32), ref) <= 2e-5


# whole rows of blocks, but codes that are not on 16-byte boundaries: windows whose row ends with a stage
@pytest.mark.parametrize("M,N,nb", [shapes[0][:2] + (nb,) for shapes in STAGED.values() for nb in (16, 24)] +
                         [shapes[0][:2] + (nb,) for shapes in KSPLIT.values() for nb in (32, 40, 48)])
def test_nvfp4_codes_at_their_minimum_alignment(M, N, nb):
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 16, code_lead=8), operand(g, N, nb, 16, code_lead=8)
    assert a[0].data_ptr() % 16 == 8
    assert worst(B.arcq_gemm(*a, 1.0, *w, 1.0, out_dtype=torch.float32), dequantize(*a, 16) @ dequantize(*w, 16).t()) <= 2e-5


# the same for the scaled FP4 instruction; runs of K': six of which the last holds one unit and a ragged one, eight of two units each,
# where the last run begins with the first unit whose windows may pass the operand's end (units 14 and 15 of 121 and 127 blocks)
MX = {
    (128, 128, 1): [(300, 261, b) for b in (16, 17, 22, 31, 67)],
    (128, 128, 6): [(300, 261, 130)],
    (128, 128, 8): [(100, 100, 121), (300, 77, 127)],
    (192, 128, 1): [(1277, 4090, b) for b in (19, 26)] + [(150, 28600, b) for b in (16, 21)],
    (128, 256, 1): [(2047, 4093, b) for b in (17, 20, 23, 30)],
    (192, 256, 1): [(767, 14333, b) for b in (18, 21, 25)],
    (256, 256, 1): [(1022, 14331, b) for b in (17, 27, 28, 31)],
}


@pytest.mark.parametrize("rows,cols,runs,M,N,nb", [(*tile, *shape) for tile, shapes in MX.items() for shape in shapes])
def test_mxfp4_any_number_of_blocks(rows, cols, runs, M, N, nb):
    """The scaled matrix instruction keeps fewer bits inside one instruction: 1.5e-4 of the product's 2-norm."""
    assert B.arcq_mx_gemm_route(M, N, nb * 32, True)[:4] == (B.ROUTE_TILES, rows, cols, runs)
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 32), operand(g, N, nb, 32)
    ref = dequantize(*a, 32) @ dequantize(*w, 32).t()
    need = B.arcq_mx_gemm_workspace_size(M, N, nb * 32)
    assert need == (runs * M * N * 4 if runs > 1 else 0)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    a1 = operand(torch.Generator(device="cuda").manual_seed(M + N + nb), M, nb, 32, lead=1)   # through registers
    for case in (a, a1):
        for workspace in (None, ws):
            y = B.arcq_mx_gemm(*case, *w, out_dtype=torch.float32, workspace=workspace)
            assert float((y.double() - ref).norm() / ref.norm()) <= 6e-4 and worst(y, ref) <= 5e-3
    y = B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32)
    h = B.arcq_mx_gemm(*a, *w)
    assert torch.equal(h, y.half())


@pytest.mark.parametrize("M,N,nb", [shapes[0][:2] + (nb,) for shapes in MX.values() for nb in (16, 24)])
def test_mxfp4_codes_at_their_minimum_alignment(M, N, nb):
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 32, code_lead=4), operand(g, N, nb, 32, code_lead=4)
    assert a[0].data_ptr() % 16 == 4
    ref = dequantize(*a, 32) @ dequantize(*w, 32).t()
    y = B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32)
    assert float((y.double() - ref).norm() / ref.norm()) <= 6e-4 and worst(y, ref) <= 5e-3


# weight-streaming kernels: groups of four chunks (512 k) dealt to eight waves: none, one per wave, one or two, two, more; with and
# without chunks and blocks behind the last group; one to four weight tiles per wave, one to four row tiles
STREAM = [(M, N, nb) for M, N in ((1, 250), (16, 4100), (13, 8200), (16, 12300), (32, 4090), (24, 5000), (29, 8200), (32, 12300), (17, 300), (48, 300),
                                  (64, 300), (64, 5000))
          for nb in (31, 256, 295, 471, 512, 557)]


@pytest.mark.parametrize("M,N,nb", STREAM)
def test_streaming_groups(M, N, nb):
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 16), operand(g, N, nb, 16)
    y = B.arcq_gemm(*a, 1.0, *w, 1.0, out_dtype=torch.float32)
    assert worst(y, dequantize(*a, 16) @ dequantize(*w, 16).t()) <= 2e-5
    nb = nb // 2 + nb % 2                            # 512 k are 16 blocks of 32
    a, w = operand(g, M, nb, 32), operand(g, N, nb, 32)
    ref = dequantize(*a, 32) @ dequantize(*w, 32).t()
    y = B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32)
    assert float((y.double() - ref).norm() / ref.norm()) <= 6e-4 and worst(y, ref) <= 5e-3
