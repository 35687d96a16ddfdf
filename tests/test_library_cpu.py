"""No-GPU checks of the C-ABI library: it loads, exports every declared symbol, and rejects
bad arguments before any HIP call (so these run on a machine without a GPU)."""
import ctypes
import math
import os
import random
import re
import types

import pytest
import torch

from paper_2601_07475_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADERS = [os.path.join(ROOT, "include", h) for h in ("arcq.h", "arcq_bench.h")]

pytestmark = pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libarcq.so not built")


def declared_symbols():
    text = "".join(open(h).read() for h in HEADERS)
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(arcq_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported_and_bound():
    names = declared_symbols()
    assert "arcq_quantize_act" in names and "arcq_pack_weight" in names and "arcq_gemm" in names
    handle = ctypes.CDLL(B.LIB_PATH)
    for n in names:
        assert hasattr(handle, n), n
    assert sorted(B.SIGNATURES) == names
    assert B.arcq_version() >= 100


def test_packed_sizes():
    assert B.arcq_packed_sizes(16, 512, 32) == (16 * 544 // 2, 16 * 544 // 16)
    assert B.arcq_packed_sizes(0, 512, 0) == (0, 0)
    for K, S in ((0, 0), (24, 0), (512, 8), (512, 528), (512, -16), (B.MAX_K + 16, 0)):
        with pytest.raises(B.ArcqError) as e:
            B.arcq_packed_sizes(4, K, S)
        assert e.value.status == B.BAD_SHAPE


FAKE = ctypes.c_void_p(0x10000)       # never dereferenced: every call below must fail validation first
ODD = ctypes.c_void_p(0x10004)


def q(fn, x=FAKE, rows=4, K=512, ld=512, perm=FAKE, S=32, sT=1.0, codes=FAKE, scales=FAKE):
    return getattr(B.lib(), fn)(x, rows, K, ld, perm, S, sT, codes, scales, None)


@pytest.mark.parametrize("fn", ["arcq_quantize_act", "arcq_pack_weight"])
def test_quantizer_argument_errors(fn):
    assert q(fn, K=500) == B.BAD_SHAPE
    assert q(fn, S=24) == B.BAD_SHAPE
    assert q(fn, S=1024) == B.BAD_SHAPE
    assert q(fn, rows=-1) == B.BAD_SHAPE
    assert q(fn, ld=496) == B.BAD_SHAPE
    assert q(fn, K=B.MAX_K + 16, ld=B.MAX_K + 16) == B.BAD_SHAPE
    for bad in (0.0, -1.0, float("inf"), float("nan"), 2.0 ** -70, 2.0 ** 70):
        assert q(fn, sT=bad) == B.INVALID_ARG
    assert q(fn, x=None) == B.INVALID_ARG
    assert q(fn, perm=None) == B.INVALID_ARG
    assert q(fn, codes=None) == B.INVALID_ARG
    assert q(fn, scales=None) == B.INVALID_ARG
    assert q(fn, x=ODD) == B.BAD_ALIGN
    assert q(fn, ld=516) == B.BAD_ALIGN
    assert q(fn, codes=ODD) == B.BAD_ALIGN
    assert b"aligned" in B.lib().arcq_last_error()
    assert q(fn, perm=ODD) == B.BAD_ALIGN and q(fn, perm=ctypes.c_void_p(0x10008)) == B.BAD_ALIGN    # read as 16-byte vectors
    assert b"perm" in B.lib().arcq_last_error()
    assert q(fn, rows=0, x=None, perm=None, codes=None, scales=None) == B.OK      # empty input: nothing to do
    assert B.lib().arcq_last_error() == b""


def qn(x=FAKE, rows=4, K=512, ld=512, gamma=FAKE, eps=1e-5, perm=FAKE, S=32, sT=1.0, codes=FAKE, scales=FAKE):
    return B.lib().arcq_rmsnorm_quantize_act(x, rows, K, ld, gamma, eps, perm, S, sT, codes, scales, None)


def test_rmsnorm_quantizer_argument_errors():
    assert qn(K=500) == B.BAD_SHAPE
    assert qn(S=24) == B.BAD_SHAPE
    assert qn(ld=496) == B.BAD_SHAPE
    assert qn(sT=0.0) == B.INVALID_ARG
    for bad in (-1e-6, float("inf"), float("nan")):
        assert qn(eps=bad) == B.INVALID_ARG
    assert b"eps" in B.lib().arcq_last_error()
    assert qn(gamma=None) == B.INVALID_ARG
    assert qn(x=None) == B.INVALID_ARG
    assert qn(gamma=ctypes.c_void_p(0x10008)) == B.BAD_ALIGN
    assert qn(x=ODD) == B.BAD_ALIGN
    assert qn(codes=ODD) == B.BAD_ALIGN
    assert qn(rows=0, x=None, gamma=None, perm=None, codes=None, scales=None) == B.OK


def g(ac=FAKE, asc=FAKE, sa=1.0, wc=FAKE, wsc=FAKE, sw=1.0, M=4, N=8, Kp=64, y=FAKE, dt=0, ldy=8, ws=None, wsb=0):
    return B.lib().arcq_gemm(ac, asc, sa, wc, wsc, sw, M, N, Kp, y, dt, ldy, ws, wsb, None)


def test_gemm_argument_errors():
    assert g(Kp=0) == B.BAD_SHAPE
    assert g(Kp=40) == B.BAD_SHAPE
    assert g(M=-1) == B.BAD_SHAPE
    assert g(ldy=4) == B.BAD_SHAPE
    assert g(dt=7) == B.INVALID_ARG
    assert g(sa=0.0) == B.INVALID_ARG
    assert g(sw=float("nan")) == B.INVALID_ARG
    assert g(ac=None) == B.INVALID_ARG
    assert g(y=None) == B.INVALID_ARG
    assert g(wc=ODD) == B.BAD_ALIGN
    assert g(y=ctypes.c_void_p(0x10002)) == B.BAD_ALIGN
    assert g(M=0, ac=None, asc=None, y=None) == B.OK
    assert g(N=0, wc=None, wsc=None, y=None) == B.OK
    n = ctypes.c_size_t(123)
    assert B.lib().arcq_gemm_workspace_size(4, 8, 64, ctypes.byref(n)) == B.OK
    assert B.lib().arcq_gemm_workspace_size(4, 8, 40, ctypes.byref(n)) == B.BAD_SHAPE
    # few tiles and a long reduction: split into several runs (at most 8), fp32 partial results in the workspace
    assert B.lib().arcq_gemm_workspace_size(256, 512, 14592, ctypes.byref(n)) == B.OK
    assert n.value % (256 * 512 * 4) == 0 and 2 <= n.value // (256 * 512 * 4) <= 8
    assert g(M=256, N=512, Kp=14592, ldy=512) == B.WORKSPACE_TOO_SMALL
    assert g(M=256, N=512, Kp=14592, ldy=512, ws=FAKE, wsb=1024) == B.WORKSPACE_TOO_SMALL
    assert g(M=256, N=512, Kp=14592, ldy=512, ws=ctypes.c_void_p(0x10010), wsb=1 << 30) == B.BAD_ALIGN
    assert B.lib().arcq_gemm_workspace_size(2048, 4096, 4352, ctypes.byref(n)) == B.OK and n.value == 0


def test_gemm_noalloc_argument_errors_and_scratch_limit():
    """The entry point for callers that cannot allocate: the rules of arcq_gemm, and shapes whose partial results
    exceed the built-in scratch are turned away before anything touches the GPU."""
    ga = lambda ac=FAKE, M=4, N=8, Kp=64, y=FAKE, dt=0, ldy=8, sa=1.0: B.lib().arcq_gemm_noalloc(
        ac, FAKE, sa, FAKE, FAKE, 1.0, M, N, Kp, y, dt, ldy, None)
    assert ga(Kp=40) == B.BAD_SHAPE and ga(M=-1) == B.BAD_SHAPE and ga(ldy=4) == B.BAD_SHAPE
    assert ga(dt=7) == B.INVALID_ARG and ga(sa=0.0) == B.INVALID_ARG and ga(ac=None) == B.INVALID_ARG
    assert ga(ac=ODD) == B.BAD_ALIGN and ga(y=ctypes.c_void_p(0x10002)) == B.BAD_ALIGN
    assert ga(M=0, ac=None, y=None) == B.OK
    n = ctypes.c_size_t(0)
    # a few hundred rows against a few hundred weight rows over a very long reduction: K' split seven times
    assert B.lib().arcq_gemm_workspace_size(896, 640, 14592, ctypes.byref(n)) == B.OK
    assert n.value > B.NOALLOC_SCRATCH_BYTES == 8 << 20
    assert ga(M=896, N=640, Kp=14592, ldy=640) == B.WORKSPACE_TOO_SMALL
    assert b"built-in" in B.lib().arcq_last_error()


def random_sizes(seed, count, block):
    rng = random.Random(seed)
    log = lambda a, b: int(math.exp(rng.uniform(math.log(a), math.log(b))))
    return [(log(1, 9000), log(1, 60000), block * log(1, 65536 // block)) for _ in range(count)]


def occupied_without_scratch(M, N, Kp):
    """Some tile with the k split inside the workgroup covers the problem with 144 to 256 workgroups, or the smallest
    (64 x 32) an eighth of the chip over a short K'; the weight-streaming kernel serves up to 64 rows."""
    if M <= 64:
        return True
    t = lambda bm, bn: -(-M // bm) * -(-N // bn)
    return Kp >= 512 and (any(144 <= t(*tile) <= 256 for tile in ((64, 32), (64, 64), (96, 64), (128, 64), (128, 128))) or
                          (Kp <= 8704 and 32 <= t(64, 32) <= 256))


def test_gemm_needs_no_workspace_where_a_tile_occupies_the_chip():
    """Such problems run from a null workspace and leave the built-in scratch of arcq_gemm_noalloc alone, whichever of the
    paths the modelled times prefer."""
    shapes = [(68, 5664, 14544), (103, 2336, 20000), (476, 256, 8464), (443, 197, 7104), (893, 67, 7488), (3907, 1, 8560)]
    shapes += random_sizes(5, 40000, 16)
    checked = 0
    for M, N, Kp in shapes:
        if occupied_without_scratch(M, N, Kp):
            assert B.arcq_gemm_workspace_size(M, N, Kp) == 0, (M, N, Kp)
            checked += 1
    assert checked > 5000


def test_routes():
    """The kernel, the tile and the number of runs come from one rule: the workspace is what the runs need, the runs are at
    least four stages (NVFP4) or two units (MXFP4) long, and only tiles that exist are named."""
    r = B.Route()
    assert B.lib().arcq_gemm_route(4, 8, 40, ctypes.byref(r)) == B.BAD_SHAPE
    assert B.lib().arcq_gemm_route(4, 8, 64, None) == B.INVALID_ARG
    assert B.lib().arcq_mx_gemm_route(4, 8, 48, 0, ctypes.byref(r)) == B.BAD_SHAPE
    assert B.lib().arcq_mx_gemm_route(4, 8, 64, 0, None) == B.INVALID_ARG
    wide = [(256, 256), (192, 256), (128, 256), (192, 128), (128, 128)]
    narrow = [(64, 32), (64, 64), (96, 64), (128, 64), (64, 128), (96, 128), (128, 128)]
    stream = [(16 * m, 16 * n) for m, n in ((1, 1), (1, 2), (1, 3), (1, 4), (2, 1), (2, 2), (2, 3), (2, 4), (4, 1), (4, 2), (8, 1), (8, 2))]
    seen = set()
    for M, N, Kp in random_sizes(6, 40000, 16):
        kernel, rows, cols, runs, ahead = B.arcq_gemm_route(M, N, Kp)
        seen.add((kernel, rows, cols))
        assert (rows, cols) in {B.ROUTE_STREAM: stream, B.ROUTE_KSPLIT: narrow, B.ROUTE_TILES: wide, B.ROUTE_DIRECT: [(128, 128)]}[kernel]
        assert B.arcq_gemm_workspace_size(M, N, Kp) == (runs * M * N * 4 if runs > 1 else 0)
        assert runs == 1 or (kernel == B.ROUTE_TILES and (rows, cols) == (128, 128) and 2 <= runs <= 8 and 512 * runs <= Kp + 127)
        if kernel == B.ROUTE_STREAM:
            assert M <= rows and (rows == 16 or M > rows // 2)
    assert len(seen) == len(wide) + len(narrow) + len(stream) + 1        # every tile is some shape's
    for M, N, Kp in random_sizes(7, 10000, 32):
        kernel, rows, cols, runs, _ = B.arcq_mx_gemm_route(M, N, Kp, True)
        assert (rows, cols) in {B.ROUTE_STREAM: stream, B.ROUTE_TILES: wide, B.ROUTE_DIRECT: [(128, 128)]}[kernel]
        assert B.arcq_mx_gemm_workspace_size(M, N, Kp) == (runs * M * N * 4 if runs > 1 else 0)
        assert runs == 1 or (kernel == B.ROUTE_TILES and (rows, cols) == (128, 128) and 2 <= runs <= 8)
        assert B.arcq_mx_gemm_route(M, N, Kp)[3] == 1                   # no workspace: never split


# 512-k groups of a row over eight waves: one each, a few waves with one more, all with more; chunks behind the last group do not count
@pytest.mark.parametrize("M,N,Kp,ahead", [
    (16, 14336, 4352, 0), (16, 4096, 4352, 1), (16, 4096, 14592, 0), (32, 28672, 4096, 1), (48, 500, 4352, 1),     # at most eight
    (16, 7168, 4608, 1), (16, 9216, 4608, 0), (16, 28672, 4672, 0), (24, 28672, 5008, 0), (32, 4096, 4608, 1), (32, 5120, 4608, 0),
    (32, 5120, 5120, 1), (32, 9216, 5264, 0), (33, 213, 5008, 0), (38, 282, 10560, 0), (35, 4383, 5072, 0), (64, 500, 5632, 0),
    (16, 28672, 13008, 0), (32, 28672, 8720, 0), (33, 1103, 15616, 0),
    (16, 10240, 8448, 1), (16, 28672, 8448, 1), (32, 28672, 8464, 1), (48, 4096, 8208, 1), (64, 2048, 14592, 1), (32, 16384, 5632, 1),
])
def test_streaming_waves_load_ahead_where_most_of_them_take_another_group(M, N, Kp, ahead):
    route = B.arcq_gemm_route(M, N, Kp)
    assert route[0] == B.ROUTE_STREAM and route[4] == ahead


# Problems at which a path was timed 5 to 40 % faster than the one beside it: short K', where the start of a round counts for more than its
# groups; weight rows that are no multiple of four (each value stored by itself); 96 x 128 tiles that pad more rows than 128 x 128
@pytest.mark.parametrize("M,N,Kp,tile", [
    (46, 9600, 512, (64, 64)), (34, 11392, 704, (64, 64)), (64, 14248, 512, (64, 64)), (48, 14336, 1552, (64, 64)),
    (51, 4288, 22304, None), (36, 4352, 21184, None), (39, 4408, 6144, None), (97, 9024, 1552, (64, 128)),
    (82, 4478, 704, None), (85, 14080, 512, (64, 128)), (741, 2726, 832, (128, 128)), (195, 10832, 12096, (128, 128)), (505, 5376, 6784, (128, 128)),
    (333, 6144, 4240, (96, 128)), (301, 3070, 560, (64, 64)), (64, 28672, 4240, (64, 128)),
])
def test_the_route_is_the_path_that_measured_faster(M, N, Kp, tile):
    kernel, rows, cols, runs, _ = B.arcq_gemm_route(M, N, Kp)
    assert runs == 1 and (kernel == B.ROUTE_STREAM if tile is None else (rows, cols) == tile)


def test_gpu_shape_lists_reach_every_kernel():
    """The lists of test_gpu_ragged.py against the rule as it is: every tile, with the copies of whole rows and with windows; every
    tile of the streaming kernel, loading ahead and not, with several groups per wave and something behind the last."""
    import test_gpu_ragged as R
    for kernel, lists in ((B.ROUTE_TILES, R.STAGED), (B.ROUTE_KSPLIT, R.KSPLIT)):
        for tile, shapes in lists.items():
            assert all(B.arcq_gemm_route(M, N, 16 * nb)[:4] == (kernel, *tile, 1) for M, N, nb in shapes), tile
            assert {nb % 4 == 0 for _, _, nb in shapes} == {True, False}, tile
    for runs, shapes in R.RUNS.items():
        assert all(B.arcq_gemm_route(M, N, 16 * nb)[:4] == (B.ROUTE_TILES, 128, 128, runs) for M, N, nb in shapes), runs
    for (rows, cols, runs), shapes in R.MX.items():
        assert all(B.arcq_mx_gemm_route(M, N, 32 * nb, True)[:4] == (B.ROUTE_TILES, rows, cols, runs) for M, N, nb in shapes)
    routes = {(nb // 32 > 8, nb % 32 > 0) + B.arcq_gemm_route(M, N, 16 * nb)[1:] for M, N, nb in R.STREAM
              if B.arcq_gemm_route(M, N, 16 * nb)[0] == B.ROUTE_STREAM}
    for rows, cols in ((16, 48), (16, 64), (32, 32), (32, 48), (32, 64), (64, 16), (64, 32)):
        assert (True, True, rows, cols, 1, 0) in routes and (True, True, rows, cols, 1, 1) in routes, (rows, cols)
    assert (True, True, 16, 16, 1, 0) in routes and (True, True, 16, 32, 1, 1) in routes and (True, True, 32, 16, 1, 1) in routes


def test_stream_tiles():
    t = ctypes.c_int32(0)
    for fn, head in ((B.lib().arcq_gemm_stream_tiles, ()), (B.lib().arcq_mx_gemm_stream_tiles, (0,))):
        assert fn(4, 8, 40, *head, ctypes.byref(t), ctypes.byref(t)) == B.BAD_SHAPE
        assert fn(4, 8, 64, *head, None, ctypes.byref(t)) == B.INVALID_ARG and fn(4, 8, 64, *head, ctypes.byref(t), None) == B.INVALID_ARG
    for seed, step, route, tiles in ((10, 16, B.arcq_gemm_route, B.arcq_gemm_stream_tiles), (11, 32, B.arcq_mx_gemm_route, B.arcq_mx_gemm_stream_tiles)):
        streaming = 0
        for M, N, Kp in random_sizes(seed, 10000, step):
            kernel, _, cols, _, _ = route(M, N, Kp)
            got = tiles(M, N, Kp)
            if kernel != B.ROUTE_STREAM:
                assert got == (0, 0)
            elif N <= 16384 or M > 32 or N > 57344:
                assert got == (cols // 16, cols // 16)
            else:
                assert got[0] in (4, 5, 6, 7) and cols == 64 and (got[1] == got[0] or got[0] == 4 and got[1] in (2, 3))
            streaming += kernel == B.ROUTE_STREAM
        assert streaming > 200


# a few weight rows behind two whole rounds of four tiles a wave cost MXFP4 less than five tiles a wave in both (timed 2 to 9 % faster)
@pytest.mark.parametrize("M", [1, 16, 32])
@pytest.mark.parametrize("N,Kp,tiles", [(32769, 1056, 4), (32784, 2176, 4), (32785, 2176, 5), (32784, 3584, 4), (32785, 3584, 5), (32769, 4352, 4),
                                        (32800, 4352, 4), (32801, 4352, 5), (32784, 5632, 4), (32800, 4096, 4), (32800, 4064, 5), (33000, 4352, 5)])
def test_mx_weight_rows_behind_two_rounds(M, N, Kp, tiles):
    if B.arcq_mx_gemm_route(M, N, Kp)[0] == B.ROUTE_STREAM:                  # (32 rows: up to K' = 3584 here)
        assert B.arcq_mx_gemm_stream_tiles(M, N, Kp) == (tiles, tiles)
    else:
        assert M == 32 and Kp > 3584


def test_gpu_shape_lists_reach_every_number_of_weight_tiles():
    """The lists of test_gpu_streaming_tiles.py: every kernel of more than four weight tiles a wave, of four and fewer behind them, and of four."""
    import test_gpu_streaming_tiles as T
    rows = lambda M: 1 if M <= 16 else 2
    nvfp4 = {(rows(M), *B.arcq_gemm_stream_tiles(M, N, 16 * nb)) for M, N, nb, *_ in T.NVFP4}
    assert nvfp4 == {(1, 4, 4), (1, 5, 5), (1, 6, 6), (1, 7, 7), (2, 4, 4), (2, 5, 5), (2, 6, 6), (2, 7, 7), (2, 4, 3)}
    mx = {(rows(M), *B.arcq_mx_gemm_stream_tiles(M, N, 32 * nb)) for M, N, nb, *_ in T.MX}
    assert mx == {(1, 4, 4), (1, 5, 5), (1, 6, 6), (1, 7, 7), (2, 5, 5), (2, 4, 2), (2, 4, 3)}
    assert all(B.arcq_gemm_stream_tiles(M, N, 16 * nb) == (t, b) for M, N, nb, t, b in T.NVFP4)
    assert all(B.arcq_mx_gemm_stream_tiles(M, N, 32 * nb) == (t, b) for M, N, nb, t, b in T.MX)


def test_check_perm_argument_errors():
    r = ctypes.c_int(0)
    assert B.lib().arcq_check_perm(None, 16, FAKE, ctypes.byref(r), None) == B.INVALID_ARG
    assert B.lib().arcq_check_perm(FAKE, 0, FAKE, ctypes.byref(r), None) == B.BAD_SHAPE


def test_calibration_argument_errors():
    L = B.lib()
    assert L.arcq_calib_absmax(FAKE, 4, 500, 512, FAKE, None) == B.BAD_SHAPE
    assert L.arcq_calib_absmax(FAKE, -1, 512, 512, FAKE, None) == B.BAD_SHAPE
    assert L.arcq_calib_absmax(FAKE, 4, 512, 496, FAKE, None) == B.BAD_SHAPE
    assert L.arcq_calib_absmax(None, 4, 512, 512, FAKE, None) == B.INVALID_ARG
    assert L.arcq_calib_absmax(FAKE, 4, 512, 512, None, None) == B.INVALID_ARG
    assert L.arcq_calib_absmax(ODD, 4, 512, 512, FAKE, None) == B.BAD_ALIGN
    assert L.arcq_calib_absmax(FAKE, 4, 512, 516, FAKE, None) == B.BAD_ALIGN
    assert L.arcq_calib_absmax(FAKE, 4, 512, 512, ctypes.c_void_p(0x10002), None) == B.BAD_ALIGN
    assert L.arcq_calib_absmax(None, 0, 512, 512, None, None) == B.OK                 # empty batch: nothing to do
    s = ctypes.c_int(0)
    assert L.arcq_calib_select(FAKE, 40, FAKE, FAKE, ctypes.byref(s), None) == B.BAD_SHAPE
    assert L.arcq_calib_select(FAKE, B.MAX_K + 16, FAKE, FAKE, ctypes.byref(s), None) == B.BAD_SHAPE
    assert L.arcq_calib_select(None, 64, FAKE, FAKE, ctypes.byref(s), None) == B.INVALID_ARG
    assert L.arcq_calib_select(FAKE, 64, None, FAKE, ctypes.byref(s), None) == B.INVALID_ARG
    assert L.arcq_calib_select(FAKE, 64, FAKE, None, ctypes.byref(s), None) == B.INVALID_ARG
    assert L.arcq_calib_select(FAKE, 64, ctypes.c_void_p(0x10002), FAKE, ctypes.byref(s), None) == B.BAD_ALIGN


def test_mx_argument_errors():
    L = B.lib()
    for fn in (L.arcq_mx_quantize_act, L.arcq_mx_pack_weight):
        assert fn(FAKE, 4, 528, 528, FAKE, 32, FAKE, FAKE, None) == B.BAD_SHAPE          # K % 32
        assert fn(FAKE, 4, 512, 512, FAKE, 16, FAKE, FAKE, None) == B.BAD_SHAPE          # S % 32
        assert fn(FAKE, 4, 512, 496, FAKE, 32, FAKE, FAKE, None) == B.BAD_SHAPE
        assert fn(None, 4, 512, 512, FAKE, 32, FAKE, FAKE, None) == B.INVALID_ARG
        assert fn(FAKE, 4, 512, 512, FAKE, 32, ctypes.c_void_p(0x10008), FAKE, None) == B.BAD_ALIGN
        assert fn(FAKE, 4, 512, 512, ctypes.c_void_p(0x10004), 32, FAKE, FAKE, None) == B.BAD_ALIGN
        assert fn(None, 0, 512, 512, None, 32, None, None, None) == B.OK
    cb, sb = ctypes.c_size_t(0), ctypes.c_size_t(0)
    assert L.arcq_mx_packed_sizes(10, 512, 64, ctypes.byref(cb), ctypes.byref(sb)) == B.OK
    assert (cb.value, sb.value) == (10 * 576 // 2, 10 * 576 // 32)
    mg = lambda M=4, N=8, Kp=64, ac=FAKE, y=FAKE, dt=0, ldy=8: L.arcq_mx_gemm(ac, FAKE, FAKE, FAKE, M, N, Kp, y, dt, ldy, None)
    assert mg(Kp=48) == B.BAD_SHAPE and mg(Kp=0) == B.BAD_SHAPE and mg(ldy=4) == B.BAD_SHAPE
    assert mg(dt=9) == B.INVALID_ARG and mg(ac=None) == B.INVALID_ARG
    assert mg(ac=ctypes.c_void_p(0x10002)) == B.BAD_ALIGN and mg(y=ctypes.c_void_p(0x10002)) == B.BAD_ALIGN
    assert mg(M=0, ac=None, y=None) == B.OK


def test_variant_entry_points_argument_errors():
    L = B.lib()
    for fn in (L.arcq_quantize_act_ex, L.arcq_pack_weight_ex):
        assert fn(FAKE, 4, 512, 512, FAKE, 32, 1.0, 4, FAKE, FAKE, None) == B.INVALID_ARG      # unknown flag bit
        assert b"flags" in L.arcq_last_error()
        assert fn(FAKE, 4, 512, 512, FAKE, 32, 1.0, 0x80000001, FAKE, FAKE, None) == B.INVALID_ARG
        assert fn(FAKE, 4, 520, 520, FAKE, 32, 1.0, 3, FAKE, FAKE, None) == B.BAD_SHAPE        # the plain rules still hold
        assert fn(None, 4, 512, 512, FAKE, 32, 1.0, 3, FAKE, FAKE, None) == B.INVALID_ARG
        for flags in (0, 1, 2, 3):
            assert fn(None, 0, 512, 512, None, 32, 1.0, flags, None, None, None) == B.OK      # nothing to do
    nq = L.arcq_rmsnorm_quantize_act_ex
    assert nq(FAKE, 4, 512, 512, FAKE, 1e-5, FAKE, 32, 1.0, 8, FAKE, FAKE, None) == B.INVALID_ARG
    # the exact-sum bit belongs to the RMSNorm call alone
    assert nq(None, 0, 512, 512, None, 1e-5, None, 32, 1.0, 4 | 3, None, None, None) == B.OK
    assert L.arcq_quantize_act_ex(None, 0, 512, 512, None, 32, 1.0, 4, None, None, None) == B.INVALID_ARG
    assert B.RMSNORM_EXACT_SUM == 4
    assert nq(FAKE, 4, 512, 512, None, 1e-5, FAKE, 32, 1.0, 1, FAKE, FAKE, None) == B.INVALID_ARG   # gamma
    assert nq(None, 0, 512, 512, None, 1e-5, None, 32, 1.0, 3, None, None, None) == B.OK
    for fn in (L.arcq_mx_quantize_act_ex, L.arcq_mx_pack_weight_ex):
        assert fn(FAKE, 4, 512, 512, FAKE, 32, 4, FAKE, FAKE, None) == B.INVALID_ARG
        assert fn(FAKE, 4, 512, 512, FAKE, 16, 1, FAKE, FAKE, None) == B.BAD_SHAPE
        assert fn(None, 0, 512, 512, None, 32, 3, None, None, None) == B.OK
    assert (B.LAYOUT_INTERLEAVED, B.SCALE_ROUND_UP) == (1, 2)


@pytest.mark.parametrize("name", ["arcq_probe_mfma_f16", "arcq_probe_mfma_fp4"])
def test_probe_argument_errors(name):
    probe = getattr(B.lib(), name)
    fl = ctypes.c_double(0)
    assert probe(0, FAKE, ctypes.byref(fl), None) == B.INVALID_ARG
    assert probe(1 << 21, FAKE, ctypes.byref(fl), None) == B.INVALID_ARG
    assert probe(10, None, ctypes.byref(fl), None) == B.INVALID_ARG
    assert probe(10, FAKE, None, None) == B.INVALID_ARG
    assert probe(10, ctypes.c_void_p(0x10002), ctypes.byref(fl), None) == B.BAD_ALIGN


def test_buffer_copy_argument_errors():
    copy = B.lib().arcq_probe_buffer_copy
    assert copy(FAKE, 64, 0, 2, FAKE, None) == B.INVALID_ARG
    assert copy(FAKE, 64, 68, 4, FAKE, None) == B.INVALID_ARG                # a scalar offset past the buffer
    assert copy(None, 64, 0, 4, FAKE, None) == B.INVALID_ARG and copy(FAKE, 64, 0, 4, None, None) == B.INVALID_ARG
    assert copy(ctypes.c_void_p(0x10004), 64, 0, 4, FAKE, None) == B.BAD_ALIGN
    assert copy(FAKE, 62, 0, 4, FAKE, None) == B.BAD_ALIGN and copy(FAKE, 64, 2, 4, FAKE, None) == B.BAD_ALIGN


def test_ref_gemm_bf16_argument_errors():
    L = B.lib()
    assert L.arcq_ref_gemm_bf16(FAKE, FAKE, 8, 8, 48, FAKE, 8, None) == B.BAD_SHAPE          # K % 32
    assert L.arcq_ref_gemm_bf16(FAKE, FAKE, 8, 8, 64, FAKE, 4, None) == B.BAD_SHAPE          # ldy < N
    assert L.arcq_ref_gemm_bf16(None, FAKE, 8, 8, 64, FAKE, 8, None) == B.INVALID_ARG
    assert L.arcq_ref_gemm_bf16(ctypes.c_void_p(0x10008), FAKE, 8, 8, 64, FAKE, 8, None) == B.BAD_ALIGN
    assert L.arcq_ref_gemm_bf16(FAKE, FAKE, 0, 8, 64, FAKE, 8, None) == B.OK                # empty


def test_mx_gemm_workspace_entry_points():
    L = B.lib()
    n = ctypes.c_size_t(7)
    assert L.arcq_mx_gemm_workspace_size(16, 4096, 4352, ctypes.byref(n)) == B.OK and n.value == 0       # weight-streaming kernel
    assert L.arcq_mx_gemm_workspace_size(2048, 4096, 4352, ctypes.byref(n)) == B.OK and n.value == 0     # enough tiles
    assert L.arcq_mx_gemm_workspace_size(256, 4096, 14592, ctypes.byref(n)) == B.OK
    assert n.value % (256 * 4096 * 4) == 0 and 2 <= n.value // (256 * 4096 * 4) <= 8
    need = n.value
    assert L.arcq_mx_gemm_workspace_size(256, 4096, 48, ctypes.byref(n)) == B.BAD_SHAPE
    assert L.arcq_mx_gemm_workspace_size(256, 4096, 14592, None) == B.INVALID_ARG
    args = (FAKE, FAKE, FAKE, FAKE, 256, 4096, 14592, FAKE, B.DTYPE_F16, 4096)
    assert L.arcq_mx_gemm_ws(*args, None, 0, None) == B.WORKSPACE_TOO_SMALL
    assert L.arcq_mx_gemm_ws(*args, FAKE, need - 1, None) == B.WORKSPACE_TOO_SMALL
    assert L.arcq_mx_gemm_ws(*args, ctypes.c_void_p(0x10010), need, None) == B.BAD_ALIGN
    assert L.arcq_mx_gemm_ws(FAKE, FAKE, FAKE, FAKE, 256, 4096, 14592, FAKE, 7, 4096, FAKE, need, None) == B.INVALID_ARG


def test_second_launches():
    """They take the last columns or the last rows, behind whole tiles of the first launch; neither launch needs a workspace, and the
    second is never taken for K' below 1024."""
    r = B.Rest()
    assert B.lib().arcq_gemm_rest(4, 8, 40, ctypes.byref(r)) == B.BAD_SHAPE
    assert B.lib().arcq_gemm_rest(4, 8, 64, None) == B.INVALID_ARG
    seen = [0] * 4
    for M, N, Kp in random_sizes(8, 40000, 16):
        rest = B.arcq_gemm_rest(M, N, Kp)
        if rest is None:
            continue
        kernel, rows, cols, runs, _ = B.arcq_gemm_route(M, N, Kp)
        assert Kp >= 1024 and runs == 1 and B.arcq_gemm_workspace_size(M, N, Kp) == 0
        if kernel == B.ROUTE_STREAM:
            assert M <= 32 and rest[0] == M and N - rest[1] == 16384 and cols == 64 and rest[2][0] == B.ROUTE_STREAM
        else:
            assert (kernel, rows, cols) in ((B.ROUTE_TILES, 256, 256), (B.ROUTE_TILES, 192, 256), (B.ROUTE_KSPLIT, 128, 128))
        assert (rest[0] == M) != (rest[1] == N) and 0 < rest[0] <= M and 0 < rest[1] <= N
        assert (M - rest[0]) % rows == 0 and (N - rest[1]) % cols == 0
        seen[kernel] += 1
    assert seen[B.ROUTE_STREAM] > 20 and seen[B.ROUTE_KSPLIT] > 50 and seen[B.ROUTE_TILES] > 100
    assert B.arcq_gemm_rest(1777, 10240, 8528)[:2] == (1777, 1024) and B.arcq_gemm_rest(8192, 8192, 29696) is None


def test_tile_order():
    """Every tile once, whatever the numbers of tile rows and columns; an XCD (every eighth workgroup) has a contiguous run of the
    sequence: of a tall problem with few tile columns whole tile rows, but for its first and last."""
    for m, n in ((0, 4), (4, 0), (1 << 11, 1 << 10)):
        assert B.lib().arcq_tile_order(m, n, FAKE, FAKE) == B.BAD_SHAPE
    assert B.lib().arcq_tile_order(4, 4, None, FAKE) == B.INVALID_ARG
    sizes = [(m, n) for m in range(1, 34) for n in range(1, 34)] + [(57, 3), (65, 8), (49, 30), (113, 7), (20, 7), (19, 7), (5, 97), (1, 500), (500, 1)]
    for m, n in sizes:
        order = B.arcq_tile_order(m, n)
        assert sorted(order) == [(r, c) for r in range(m) for c in range(n)], (m, n)
        if n < 8 and m >= 20:
            for xcd in range(8):
                rows = [r for r, _ in order[xcd::8]]
                assert rows == sorted(rows) and len(set(rows)) <= -(-len(rows) // n) + 1, (m, n, xcd)


# sizes whose tiles by rule share K' out to the waves of a workgroup (128 x 256 tiles to pairs, k-split tiles to four) and whose modelled
# times are in favour of tiles that do not
@pytest.mark.parametrize("M,N,Kp,chains", [(3573, 6744, 7472, 2), (2627, 5990, 6128, 2), (541, 25166, 11760, 2), (519, 24363, 9936, 2), (566, 23804, 15120, 2),
                                           (967, 22693, 13920, 2), (2079, 7428, 7552, 2), (2837, 5561, 4560, 2), (521, 6084, 1328, 4),
                                           (2168, 1468, 1392, 4), (249, 12300, 1120, 4)])
def test_no_precision_for_speed(M, N, Kp, chains):
    """Neither launch adds K' up in fewer chains than the tiles of the rule."""
    rest = B.arcq_gemm_rest(M, N, Kp)
    for kernel, rows, cols in [B.arcq_gemm_route(M, N, Kp)[:3]] + ([rest[2]] if rest else []):
        has = {B.ROUTE_STREAM: 4 if rows == 128 else 8, B.ROUTE_KSPLIT: 4, B.ROUTE_TILES: 2 if (rows, cols) == (128, 256) else 1}[kernel]
        assert has >= chains, (kernel, rows, cols)


# 65 to 128 rows, weight rows off the vectors of y: the k-split tiles that weight rows in whole vectors run, no more the streaming kernel
@pytest.mark.parametrize("M,N,Kp", [(121, 24097, 1264), (122, 28115, 1088), (89, 7319, 1520), (112, 23375, 1232), (75, 7103, 1776), (100, 8125, 1152),
                                    (66, 4990, 1040), (80, 24001, 768), (110, 26002, 800)])
def test_stores_of_odd_weight_rows_cost_nothing(M, N, Kp):
    whole = -(-N // 8) * 8
    assert B.arcq_gemm_route(M, N, Kp)[:3] == B.arcq_gemm_route(M, whole, Kp)[:3] and B.arcq_gemm_route(M, N, Kp)[0] == B.ROUTE_KSPLIT
    assert B.arcq_gemm_workspace_size(M, N, Kp) == 0


def test_mx_second_launches():
    r = B.Rest()
    assert B.lib().arcq_mx_gemm_rest(4, 8, 48, 0, ctypes.byref(r)) == B.BAD_SHAPE
    assert B.lib().arcq_mx_gemm_rest(4, 8, 64, 0, None) == B.INVALID_ARG
    # the smallest and largest number of weight rows behind the round, and the shortest K' for one and for two tiles a wave
    for M in (1, 16, 17, 32):
        for N, Kp, two in ((17408, 4096, True), (17407, 4096, False), (17408, 4064, False), (20480, 4096, True), (20481, 4096, False),
                           (24577, 4096, False)):
            rest = B.arcq_mx_gemm_rest(M, N, Kp)
            assert B.arcq_mx_gemm_route(M, N, Kp)[0] == B.ROUTE_STREAM
            assert rest == ((M, N - 16384, (B.ROUTE_STREAM, 16 if M <= 16 else 32, 16)) if two else None), (M, N, Kp)
    for M in (1, 16):
        assert B.arcq_mx_gemm_route(M, 20481, 6112)[0] == B.ROUTE_STREAM and B.arcq_mx_gemm_rest(M, 20481, 6112) is None
        assert B.arcq_mx_gemm_rest(M, 20481, 6144) == (M, 4097, (B.ROUTE_STREAM, 16, 32))
        assert B.arcq_mx_gemm_rest(M, 24576, 6144) == (M, 8192, (B.ROUTE_STREAM, 16, 32))
        assert B.arcq_mx_gemm_rest(M, 24577, 6144) is None
    assert B.arcq_mx_gemm_rest(32, 20481, 12832) == (32, 4097, (B.ROUTE_STREAM, 32, 32))        # without a workspace only
    assert B.arcq_mx_gemm_rest(32, 20481, 12832, True) is None
    # never off the streaming kernel
    assert all(B.arcq_mx_gemm_rest(M, N, Kp, ws) is None or B.arcq_mx_gemm_route(M, N, Kp, ws)[0] == B.ROUTE_STREAM
               for M, N, Kp in random_sizes(9, 20000, 32) for ws in (False, True))


def test_stream_handle_without_torch_private_names(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1234))
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        with monkeypatch.context() as m:
            m.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
            m.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x5678, raising=False)
            assert B._stream() == 0x5678
            m.delattr(torch._C, name)
            assert B._stream() == 0x1234
