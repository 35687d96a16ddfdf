/*
 * arcq_bench.h -- measurement aids of libarcq (no part of the ARCQuant method; see arcq.h for the method's calls):
 * the matrix-rate probes that give the ceiling a GEMM's roofline fraction is read against on a given machine, and
 * the hand-written bf16 GEMM the quantized linear layer is timed against; and what tests ask of the library: routes, tiles,
 * the end of a buffer copy.  Same conventions as arcq.h: device
 * pointers owned by the caller, work enqueued on `stream`, status codes, arcq_last_error().
 */
#ifndef ARCQ_BENCH_H
#define ARCQ_BENCH_H

#include "arcq.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Diagnostic for measurements (no part of the method): enqueues a kernel in which 4096 waves (four per
 * SIMD on 256 CUs) each issue 4 * iters fp16 32x32x16 matrix instructions on register operands, the
 * instruction arcq_gemm is built on, with no memory traffic in the loop.  Timing the launch gives the
 * matrix rate this machine sustains, the ceiling to read arcq_gemm's roofline fraction against.
 * iters   1 .. 2^20
 * sink    device, ARCQ_PROBE_SINK_FLOATS floats, written (keeps the loop alive), 4-byte aligned
 * flop_host  host pointer: receives the floating-point operations of one launch
 */
#define ARCQ_PROBE_SINK_FLOATS 262144
arcq_status arcq_probe_mfma_f16(int iters, float* sink, double* flop_host, void* stream);
/* The same for the instruction arcq_mx_gemm is built on: 4 * iters scaled FP4 32x32x64 matrix instructions
 * per wave (both operands E2M1, unit block scales); same arguments, same sink size. */
arcq_status arcq_probe_mfma_fp4(int iters, float* sink, double* flop_host, void* stream);

/*
 * What a copy into LDS through a buffer descriptor does at the end of its buffer, for a test (arcq_mx_gemm's tiles copy rows past the edge of an
 * operand that way): one wave, each lane `words` words from byte `scalar` + 4 * words * lane of the first `bytes` bytes of src.
 * src    device, readable for scalar + 1024 bytes whatever `bytes` is, 16-byte aligned
 * bytes, scalar  multiples of 4, scalar <= bytes       words  1 or 4
 * out    device, 256 words: what the copy left in LDS, ARCQ_PROBE_UNTOUCHED where it wrote nothing
 */
#define ARCQ_PROBE_UNTOUCHED 0xA5A5A5A5u
arcq_status arcq_probe_buffer_copy(const void* src, uint32_t bytes, uint32_t scalar, int words, uint32_t* out, void* stream);

/*
 * Comparison kernel for measurements (no part of the method): the unquantized linear layer y = x w^T on bf16
 * operands, written on the same tiled skeleton as arcq_mx_gemm (operand rows travel global -> LDS in 128-byte
 * units, v_mfma_f32_32x32x16_bf16, fp32 accumulation), the 16-bit baseline the quantized path is timed against.
 * x  device, bf16 [M, K] row-major, pitch K, 16-byte aligned     w  device, bf16 [N, K] row-major, 16-byte aligned
 * y  device, fp16 [M, N], pitch ldy >= N                         K % 32 == 0, operands below 4 GiB each
 */
arcq_status arcq_ref_gemm_bf16(const void* x, const void* w, int64_t M, int64_t N, int64_t K, void* y, int64_t ldy,
                               void* stream);

/*
 * Which kernel a GEMM problem runs on: a function of its sizes alone (host only, nothing is launched).  Tests ask it, so that
 * a shape written for a tile cannot leave that tile unnoticed when the rule changes; not needed to call the library.
 * ahead: the weight-streaming kernel's waves ask for their next weights while they compute.
 * The streaming kernels' 64 columns stand for more where a wave takes more than four weight tiles (arcq_gemm_stream_tiles below).
 * arcq_gemm_route: operands whose scale bytes lie at odd addresses run another tile where the one named was taken for its modelled time (with
 * 65 to 128 rows the streaming kernel), and they, or K' < 256 off the grid of 64, have no 256 x 256 tiles and may run 192 x 256 or
 * 128 x 256 ones instead.  arcq_mx_gemm_route: such operands (or K' < 512 off the grid of 128) run 256-wide
 * or 128 x 128 tiles instead of 192 x 128 ones; with_workspace: as arcq_mx_gemm_ws (non-zero) or arcq_mx_gemm (0).
 */
#define ARCQ_ROUTE_STREAM 0     /* weight-streaming kernel: tile_cols / 16 weight tiles per wave, or more than four */
#define ARCQ_ROUTE_KSPLIT 1     /* tiles whose waves split every stage along k */
#define ARCQ_ROUTE_TILES 2      /* tiles, K' in `runs` runs across workgroups */
#define ARCQ_ROUTE_DIRECT 3     /* plain kernel (K' < 128 off the streaming kernel, operands of 4 GiB and more) */
typedef struct {
    int32_t kernel, tile_rows, tile_cols, runs, ahead;
} arcq_route;
arcq_status arcq_gemm_route(int64_t M, int64_t N, int64_t Kp, arcq_route* route);
arcq_status arcq_mx_gemm_route(int64_t M, int64_t N, int64_t Kp, int with_workspace, arcq_route* route);
/*
 * Weight tiles of 16 rows that a wave takes in the launch that arcq_gemm_route / arcq_mx_gemm_route names, where that is a streaming kernel (else 0):
 * up to seven where more than 16384 weight rows run in one launch of up to 32 rows.  behind: of the waves behind the first 16384 weight
 * rows, fewer where registers allow no more than four in the first round; otherwise the same.
 */
arcq_status arcq_gemm_stream_tiles(int64_t M, int64_t N, int64_t Kp, int32_t* tiles, int32_t* behind);
arcq_status arcq_mx_gemm_stream_tiles(int64_t M, int64_t N, int64_t Kp, int with_workspace, int32_t* tiles, int32_t* behind);
/*
 * Problems whose last round of tiles would leave much of the chip idle run in two launches: the route above for whole rounds, and
 * this one for the last `rows` x `cols` of the output (0 x 0: there is no second launch; else one of the two is M or N).  Operands
 * whose scale bytes lie at odd addresses run in one launch, except on the streaming kernels, where more than 16384 weight rows may run in two.
 */
typedef struct {
    int64_t rows, cols;
    arcq_route route;
} arcq_rest;
arcq_status arcq_gemm_rest(int64_t M, int64_t N, int64_t Kp, arcq_rest* rest);
arcq_status arcq_mx_gemm_rest(int64_t M, int64_t N, int64_t Kp, int with_workspace, arcq_rest* rest);

/*
 * The order in which the tiled kernels deal tiles to workgroups, as the kernels compute it: workgroup i of a launch over
 * tiles_m x tiles_n tiles (both at least 1, at most 2^20 together) takes tile (rows[i], cols[i]).  Host only, for tests.
 */
arcq_status arcq_tile_order(int64_t tiles_m, int64_t tiles_n, int32_t* rows, int32_t* cols);

#ifdef __cplusplus
}
#endif
#endif /* ARCQ_BENCH_H */
