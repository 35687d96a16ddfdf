"""GPU: the tiled GEMMs over K' that is a multiple of one block only, where rows of scale bytes start at any address.

Operands are random packed bytes placed right in front of poison (scale bytes that decode to NaN), so a scale byte from
behind a row or an operand that enters the product shows.  Reference: the packed bytes' definition in 64 bits.
"""
import pytest
import torch

from paper_2601_07475_amd import binding as B

pytestmark = pytest.mark.gpu

E2M1 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]


def operand(g, rows, nb, block, lead=0):
    """(codes, scales) uint8 with poison behind both, scale bytes `lead` bytes off a 4-byte boundary."""
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
    return place(rows, nb * block // 2, codes, 0), place(rows, nb, sc, lead)


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


# one shape of each tile: 128 x 128, 192 x 128, 128 x 256 in wave pairs, 192 x 256, 256 x 256, all with ragged edges; rows of
# 16 blocks (two stages) and more, every residue of the block count modulo 8 with odd and even counts on each tile
STAGED = [(300, 261, b) for b in (16, 17, 22, 31)] + [(1277, 4090, b) for b in (19, 24, 26)] + \
         [(2047, 4093, b) for b in (17, 20, 23, 30)] + [(767, 14333, b) for b in (18, 21, 25)] + [(1022, 14331, b) for b in (17, 27, 28)]
# k quarters inside the workgroup: 64 x 32, 64 x 64, 96 x 64, 128 x 64, 128 x 128, 64 x 128, 96 x 128
KSPLIT = [(130, 1021, b) for b in (33, 46, 63)] + [(190, 4091, b) for b in (34, 49)] + [(301, 3070, b) for b in (35, 48, 61)] + \
         [(509, 2555, b) for b in (37, 62)] + [(510, 4090, b) for b in (32, 47, 50)] + \
         [(150, 28600, b) for b in (33, 40)] + [(61, 20475, b) for b in (33, 40, 46)] + [(335, 6140, b) for b in (36, 47, 53)]


@pytest.mark.parametrize("M,N,nb", STAGED + KSPLIT)
def test_nvfp4_any_number_of_blocks(M, N, nb):
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 16), operand(g, N, nb, 16)
    ref = dequantize(*a, 16) @ dequantize(*w, 16).t()
    for dtype, tol in ((torch.float32, 2e-5), (torch.float16, 1e-3)):
        scale = 2.0 ** -12 if dtype == torch.float16 else 1.0        # keeps fp16 results finite; exact
        y = B.arcq_gemm(*a, scale, *w, 1.0, out_dtype=dtype)
        assert worst(y, ref * scale) <= tol, dtype
    # scale bytes at odd addresses go through registers: the same products
    a1 = operand(torch.Generator(device="cuda").manual_seed(M + N + nb), M, nb, 16, lead=1)
    assert torch.equal(a1[0], a[0]) and torch.equal(a1[1], a[1])
    assert worst(B.arcq_gemm(*a1, 1.0, *w, 1.0, out_dtype=torch.float32), ref) <= 2e-5


# one shape of each tile: 128 x 128 (the longer ones cut K' into runs of two and more units), 192 x 128, 128 x 256, 192 x 256, 256 x 256
MX = [(300, 261, b) for b in (16, 17, 22, 31, 67, 130)] + [(1277, 4090, b) for b in (19, 26)] + \
     [(2047, 4093, b) for b in (17, 20, 23, 30)] + [(767, 14333, b) for b in (18, 21, 25)] + [(1022, 14331, b) for b in (17, 27, 28, 31)] + [(150, 28600, b) for b in (16, 21)]


@pytest.mark.parametrize("M,N,nb", MX)
def test_mxfp4_any_number_of_blocks(M, N, nb):
    """The scaled matrix instruction keeps fewer bits inside one instruction: 1.5e-4 of the product's 2-norm."""
    g = torch.Generator(device="cuda").manual_seed(M + N + nb)
    a, w = operand(g, M, nb, 32), operand(g, N, nb, 32)
    ref = dequantize(*a, 32) @ dequantize(*w, 32).t()
    need = B.arcq_mx_gemm_workspace_size(M, N, nb * 32)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    a1 = operand(torch.Generator(device="cuda").manual_seed(M + N + nb), M, nb, 32, lead=1)   # through registers
    for case in (a, a1):
        for workspace in (None, ws):
            y = B.arcq_mx_gemm(*case, *w, out_dtype=torch.float32, workspace=workspace)
            assert float((y.double() - ref).norm() / ref.norm()) <= 6e-4 and worst(y, ref) <= 5e-3
    y = B.arcq_mx_gemm(*a, *w, out_dtype=torch.float32)
    h = B.arcq_mx_gemm(*a, *w)
    assert torch.equal(h, y.half())


# weight-streaming kernels: groups of four chunks (512 k) dealt to eight waves: none, one per wave, one or two, two, more; with and
# without chunks and blocks behind the last group; one to four weight tiles per wave, one to four row tiles
STREAM = [(M, N, nb) for M, N in ((1, 250), (16, 4100), (13, 8200), (16, 12300), (32, 4090), (29, 8200), (32, 12300), (17, 300), (48, 300), (64, 5000))
          for nb in (31, 256, 295, 512, 557)]


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
