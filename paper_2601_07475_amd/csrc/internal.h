// Internal declarations shared by the translation units of libarcq (host side only).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <stddef.h>
#include <stdint.h>

#include "../../include/arcq.h"
#include "../../include/arcq_bench.h"

namespace arcq {

// Records a message for arcq_last_error() and returns `code`.
arcq_status fail(arcq_status code, const char* fmt, ...);
void clear_error();

// After a kernel launch: turns a pending HIP launch error into ARCQ_HIP_ERROR.
arcq_status check_launch(const char* what);

// Kernels with more than 48 KB of dynamic LDS need their limit raised once per device.  `done` is a bit mask
// over device indices, one static per kernel instantiation; the limit is raised to the whole 160 KB of a
// compute unit, so one call serves every launch shape of that kernel.
constexpr int kMaxLdsBytes = 160 * 1024;
arcq_status raise_lds_limit(const void* kernel, std::atomic<uint64_t>& done);
// Compute units of the current device (cached per device).
int num_cu();

// mode 0: activations (residual blocks appended); mode 1: weights (outlier blocks duplicated).
// gamma != nullptr (mode 0 only): RMSNorm with that weight and eps in front of the quantizer.
arcq_status launch_quantize(int mode, const void* x, int64_t rows, int64_t K, int64_t ldx,
                            const int32_t* perm, int64_t S, float s_T,
                            uint8_t* codes, uint8_t* scales, const void* gamma, float eps, uint32_t flags,
                            hipStream_t stream);

size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t Kp);
// device address, on the current device, of the library's built-in scratch (ARCQ_NOALLOC_SCRATCH_BYTES)
arcq_status gemm_scratch_pointer(void** out);
arcq_status launch_gemm(const uint8_t* a_codes, const uint8_t* a_scales,
                        const uint8_t* w_codes, const uint8_t* w_scales,
                        int64_t M, int64_t N, int64_t Kp, float alpha,
                        void* y, int y_dtype, int64_t ldy,
                        void* workspace, size_t workspace_bytes, hipStream_t stream);

// Which kernel serves a GEMM problem (a function of its sizes alone): the weight-streaming kernel, the tiles whose waves split
// every stage along k (NVFP4 only), the tiles whose waves do not, or the plain kernel for what those cannot address.
struct GemmPlan {
    int kernel;         // ARCQ_ROUTE_*
    int rows, cols;     // activation and weight rows of a workgroup's tile (ARCQ_ROUTE_STREAM: weight rows of up to four tiles, see `tiles`)
    int runs;           // runs of K' across workgroups (ARCQ_ROUTE_TILES)
    bool ahead;         // ARCQ_ROUTE_STREAM: a wave asks for its next group of chunks while it computes one
    int chunks = 1;     // ARCQ_ROUTE_STREAM: left-over chunks (behind the last group) that a wave takes at a time
    int tiles = 0;      // ARCQ_ROUTE_STREAM: weight tiles of a wave where they are more than four, else 0 (cols / 16 of them)
    int behind = 0;     // ARCQ_ROUTE_STREAM: weight tiles of a wave behind the first round of workgroups, 0: as in it
};
// A problem in one launch, or in two: whole rounds of large tiles over the first `rows` activation rows or the first `cols` weight
// rows, and the others on whatever is fastest for them.
struct GemmParts {
    GemmPlan first, rest;
    int64_t rows, cols;     // of the first launch; all of them: there is no second one
};
GemmParts plan_gemm_parts(int64_t M, int64_t N, int64_t Kp);
inline GemmPlan plan_gemm(int64_t M, int64_t N, int64_t Kp) { return plan_gemm_parts(M, N, Kp).first; }
GemmParts plan_mx_gemm_parts(int64_t M, int64_t N, int64_t Kp, bool workspace);
inline GemmPlan plan_mx_gemm(int64_t M, int64_t N, int64_t Kp, bool workspace) { return plan_mx_gemm_parts(M, N, Kp, workspace).first; }

// Tiled kernel whose waves split every stage along k inside the workgroup (gemm_ksplit.hip): the fastest of its tiles for this
// problem (rows = 0: none serves it), and its launch.
struct KsplitTile {
    int rows, cols;
    double us;          // modelled time
    bool ample;         // some tile occupies more than half of the chip, or the smallest one an eighth of it over a short K'
};
KsplitTile gemm_ksplit_best(int64_t M, int64_t N, int64_t Kp, bool by_value);
arcq_status launch_gemm_ksplit(int rows, int cols, const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                               const uint8_t* w_scales, int64_t M, int64_t N, int64_t Kp, float alpha, void* y, int y_dtype,
                               int64_t ldy, hipStream_t stream);

arcq_status launch_probe_mfma_f16(int iters, float* sink, double* flop_host, hipStream_t stream);
arcq_status launch_probe_mfma_fp4(int iters, float* sink, double* flop_host, hipStream_t stream);
arcq_status launch_probe_buffer_copy(const uint8_t* src, uint32_t bytes, uint32_t scalar, int words, uint32_t* out, hipStream_t stream);
arcq_status launch_ref_gemm_bf16(const void* x, const void* w, int64_t M, int64_t N, int64_t K, _Float16* y, int64_t ldy,
                                 hipStream_t stream);
arcq_status launch_check_perm(const int32_t* perm, int64_t K, uint8_t* flags,
                              int* result_host, hipStream_t stream);

arcq_status launch_calib_absmax(const void* x, int64_t M, int64_t K, int64_t ldx, float* colmax, hipStream_t stream);
arcq_status launch_calib_select(const float* colmax, int64_t K, int32_t* perm, int32_t* info, int* S_host,
                                hipStream_t stream);

// MXFP4 variant (blocks of 32, E8M0 scales, no tensor scale)
arcq_status launch_mx_quantize(int mode, const void* x, int64_t rows, int64_t K, int64_t ldx, const int32_t* perm,
                               int64_t S, uint8_t* codes, uint8_t* scales, uint32_t flags, hipStream_t stream);
// workspace: fp32 partial results of a split reduction dimension, or null (never splits)
arcq_status launch_mx_gemm(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                           const uint8_t* w_scales, int64_t M, int64_t N, int64_t Kp, void* y, int y_dtype, int64_t ldy,
                           void* workspace, hipStream_t stream);
size_t mx_gemm_workspace_bytes(int64_t M, int64_t N, int64_t Kp);
// y = alpha * (partial[0] + partial[1] + ... in index order), partial results fp32 [splits][M][N]
arcq_status launch_splitk_reduce(const float* partial, int splits, int M, int N, float alpha, void* y, int y_dtype,
                                 int64_t ldy, hipStream_t stream);

}  // namespace arcq
