// W4A4 GEMM over the extended reduction dimension K' = K + S (Section 3.2 "Unified GEMM
// Execution", eq. (2)): y[m,n] = alpha * sum_b sa[m,b] sw[n,b] sum_i qa[m,16b+i] qw[n,16b+i].
//
// gfx950's scaled FP4 MFMA takes one power-of-two (E8M0) scale per 32 elements; NVFP4 has one
// E4M3 scale per 16.  A code*scale product needs up to 6 significant bits (2 from E2M1, 4 from
// E4M3) and lies in [2^-10, 2688], so it is exactly representable in fp16 (and in no 8/6/4-bit
// float).  Operands are therefore decoded exactly to fp16 in registers and multiplied with
// v_mfma_f32_32x32x16_f16; products (12 significant bits) are exact in the fp32 accumulator, so
// the only rounding is fp32 accumulation, plus the output cast.  The tensor scales form the
// epilogue factor alpha.
//
// One 32x32x16 MFMA consumes exactly one NVFP4 block of each operand: a lane supplies 8
// consecutive k of row (lane % 32); lanes 0-31 and 32-63 supply different octets.  A and W use
// the same lane -> k mapping, so any assignment of octets to lanes sums over all of k.
#include "internal.h"
#include "gemm_decode.h"
#include "gemm_epilogue.h"
#include "lds_dma.h"
#include "scale_windows.h"
#include "tile_order.h"

#include <hip/hip_fp16.h>

#include <algorithm>
#include <cmath>
#include <iterator>
#include <atomic>
#include <type_traits>

namespace arcq {

namespace {

// Accumulates blocks [b_begin, b_end) straight from global memory (no staging): used for the
// K' tail of the staged kernel and as the whole loop of the fallback kernel.  One iteration
// covers 4 blocks: lanes of half h read blocks 4q + 2h and 4q + 2h + 1 of their rows.
template <int WM, int WN>
__device__ __forceinline__ void accumulate_direct(const uint8_t* const (&ac)[WM], const uint8_t* const (&as)[WM],
                                                  const uint8_t* const (&wc)[WN], const uint8_t* const (&ws)[WN],
                                                  int b_begin, int b_end, int h, float16v (&acc)[WM][WN]) {
    for (int q0 = b_begin; q0 < b_end; q0 += 4) {
        const int b0 = q0 + 2 * h;
        uint2 ca[WM][2], cw[WN][2];
        half2v sa[WM][2], sw[WN][2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int b = b0 + t;
            const bool ok = b < b_end;          // blocks past the end contribute zero
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                ca[i][t] = ok ? *reinterpret_cast<const uint2*>(ac[i] + 8 * (int64_t)b) : make_uint2(0, 0);
                sa[i][t] = scale_pair(ok ? as[i][b] : 0);
            }
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                cw[j][t] = ok ? *reinterpret_cast<const uint2*>(wc[j] + 8 * (int64_t)b) : make_uint2(0, 0);
                sw[j][t] = scale_pair(ok ? ws[j][b] : 0);
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            half8 fa[WM], fw[WN];
#pragma unroll
            for (int i = 0; i < WM; ++i) fa[i] = decode8((t & 1) ? ca[i][t >> 1].y : ca[i][t >> 1].x, sa[i][t >> 1]);
#pragma unroll
            for (int j = 0; j < WN; ++j) fw[j] = decode8((t & 1) ? cw[j][t >> 1].y : cw[j][t >> 1].x, sw[j][t >> 1]);
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i], fw[j], acc[i][j], 0, 0, 0);
        }
    }
}

// D layout of the 32x32 MFMA: lane holds column (lane % 32); register e holds row
// 8 * (e / 4) + 4 * (lane / 32) + e % 4.
template <int WM, int WN, typename OutT>
__device__ __forceinline__ void store_tile(const float16v (&acc)[WM][WN], int m0, int n0, int r, int h, int M,
                                           int N, float alpha, OutT* __restrict__ y, int64_t ldy) {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            const int n = n0 + 32 * j + r;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int m = m0 + 32 * i + 8 * (e >> 2) + 4 * h + (e & 3);
                if (m < M && n < N) store_out(y + (int64_t)m * ldy + n, acc[i][j][e] * alpha);
            }
        }
}

// ---------------------------------------------------------------------------------------------
// Fallback: any K' (multiple of 16), operands read straight from global memory.
// Workgroup = 4 waves (2 x 2), tile 128 x 128, each wave 64 x 64.
template <typename OutT>
__global__ __launch_bounds__(256) void gemm_direct_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N,
    int nbk, float alpha, OutT* __restrict__ y, int64_t ldy) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int r = lane & 31, h = lane >> 5;
    const int m0 = blockIdx.y * 128 + (wave >> 1) * 64;
    const int n0 = blockIdx.x * 128 + (wave & 1) * 64;
    const int64_t cpitch = (int64_t)nbk * 8, spitch = nbk;

    const uint8_t *ac[2], *as[2], *wc[2], *ws[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int m = m0 + 32 * i + r;
        m = m < M ? m : M - 1;              // rows past the edge re-read the last row; never stored
        int n = n0 + 32 * i + r;
        n = n < N ? n : N - 1;
        ac[i] = a_codes + m * cpitch;
        as[i] = a_scales + m * spitch;
        wc[i] = w_codes + n * cpitch;
        ws[i] = w_scales + n * spitch;
    }
    float16v acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    accumulate_direct<2, 2>(ac, as, wc, ws, 0, nbk, h, acc);
    store_tile<2, 2>(acc, m0, n0, r, h, M, N, alpha, y, ldy);
}

// ---------------------------------------------------------------------------------------------
// Staged kernel.  Workgroup = GM x GN waves; each wave owns WM x WN MFMA tiles
// of 32 x 32, so the workgroup tile is BM x BN = 32 WM GM x 32 WN GN.  With 4 waves (one per
// SIMD, up to 256 accumulator registers) the hand-made schedule has to hide every stall.  8 waves
// (two per SIMD, 128 accumulator registers each, <2,4,4,2> / <4,2,2,4>) let the hardware interleave
// two waves but decode every fragment for more waves; on the large shapes they measure the same as
// 2 x 2 waves to within 1 % (the loop is limited by the vector and matrix work itself, not by
// stalls: removing the waits or the barrier from a timing build gains 2 %), so 2 x 2 waves are
// dispatched there; on a 128 x 256 tile, 2 x 4 waves of 64 x 64 are 5 % faster than 2 x 2 of 64 x 128.
//
// A stage is 128 k (8 blocks): per row 64 bytes of codes and 8 scale bytes, kept PACKED in
// LDS (4.5 bits per element) and decoded in registers after the LDS read.  Stages travel
// global -> LDS with global_load_lds (no register staging) through a ring of NSTAGE (3 to 5)
// buffers: the loads of stage s + NSTAGE - 1 are issued right after the barrier that opens stage s,
// so they have NSTAGE - 1 stage times to land, and one barrier per stage suffices (passing the
// barrier of stage s means every wave has finished stage s-1, whose buffer the new stage reuses).
//
// LDS layout of one stage (bytes):  A codes [BM][64] | W codes [BN][64] | A scales [BM][8] |
// W scales [BN][8].  The four 16-byte pieces of a row's codes are stored XOR-swizzled with
// (row >> 2) & 3: the LDS serves a 16-byte read of 16 consecutive lanes per clock from 64 banks, rows
// are 64 bytes apart, so 16 consecutive rows must land on 16 different 16-byte bank groups (measured: a
// swizzle with a period of 8 rows spent half of the LDS-active cycles on bank conflicts).
// A wave-wide DMA instruction writes lane l to (uniform base) + 16 l, so the swizzle is applied
// by choosing which global piece each lane fetches.
//
// How the stages get into LDS (MODE):
//   COPIES   direct-to-LDS copies of whole 16-byte pieces; K' % 64 == 0, codes 16-byte and scale bytes 4-byte aligned;
//   RAGGED   the same for any K' (a multiple of 16) from 256 on: rows of codes then start on 8-byte boundaries, which the
//            copies take (they need dwords), and the scale bytes come as dword-aligned windows (scale_windows.h).  Pieces past
//            the end of a row are fetched from further left and their blocks get scale 0; if only the second block of a
//            piece is missing, the piece is the row's last two blocks and the scale of the first is 0.  The base of the scale
//            bytes has to be 4-byte aligned;
//   REGS     through registers, for what is left (short K', scale bytes at odd addresses), see below.
template <int WM, int WN, int GM, int GN, int MODE = COPIES>
struct StagedCfg {
    static constexpr int BM = 32 * WM * GM, BN = 32 * WN * GN;
    static constexpr int NT = 64 * GM * GN;              // threads
    // DMA instructions per thread per stage: 16-byte pieces of codes, 4-byte pieces of scales.  A copy
    // always involves the whole workgroup; when an operand has fewer pieces than threads the surplus
    // lanes re-fetch its last rows into padding behind the region (so every wave issues the same
    // number of copies, which the counted waits rely on).
    static constexpr int NA = (BM * 4 + NT - 1) / NT, NW = (BN * 4 + NT - 1) / NT;
    static constexpr int NAS = (BM * 2 + NT - 1) / NT, NWS = (BN * 2 + NT - 1) / NT;
    using Windows = ScaleWindows<BM, BN, NT, 8>;
    static constexpr int NSW = MODE == RAGGED ? Windows::NS : 0;           // copies of windows come first
    static constexpr int NDMA = NA + NW + (MODE == RAGGED ? NSW : NAS + NWS);
    static constexpr int A_CODES = 0;
    static constexpr int W_CODES = NA * NT * 16;
    static constexpr int A_SCALES = W_CODES + NW * NT * 16;
    static constexpr int W_SCALES = A_SCALES + (MODE == RAGGED ? Windows::DENSE_W : NAS * NT * 4);
    static constexpr int WINDOWS = A_SCALES + Windows::DENSE_BYTES;
    static constexpr int STAGE_BYTES = MODE == RAGGED ? WINDOWS + Windows::BYTES : W_SCALES + NWS * NT * 4;
    // Ring depth: a stage is fetched NSTAGE - 1 stages before it is computed (3 measured as good as 5).
    static constexpr int NSTAGE = 3;
    static constexpr int DIST = NSTAGE - 1;
    static constexpr int PATCH = NSTAGE * STAGE_BYTES;      // RAGGED: see ScaleWindows::fill_patch
    static constexpr int LDS_BYTES = PATCH + (MODE == RAGGED ? 2 * Windows::PATCH : 0);
};

//
// REGS: the same tiles, LDS layout and compute schedule for operands the direct-to-LDS copies cannot serve.  A thread fetches
// its pieces of a stage into registers (loads declared with the alignment the interface guarantees, 8 bytes
// for codes and 1 for scale bytes), all at once right after the barrier that opens
// stage s+1, and writes them to LDS seven k-steps later, just before the barrier that opens the stage they
// belong to, with blocks past the end of the row replaced by zeros: every stage is then a whole stage.
template <int WM, int WN, int GM, int GN, typename OutT, int MODE = COPIES>
__global__ __launch_bounds__(64 * GM * GN) void gemm_staged_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N,
    int nbk, float alpha, OutT* __restrict__ y, int64_t ldy, int tiles_m, int tiles_n, int group_rows, int splits,
    int64_t split_stride) {
    using C = StagedCfg<WM, WN, GM, GN, MODE>;
    constexpr bool REG = MODE == REGS, RAG = MODE == RAGGED;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    // ---- workgroup -> tile: tile_order.h
    // With splits > 1 the reduction dimension is cut into `splits` runs of whole stages: workgroup
    // blockIdx.x = split * num_tiles + tile accumulates its run and stores an fp32 partial tile at
    // y + split * split_stride (a reduction kernel adds the partial results).
    const int num_tiles = tiles_m * tiles_n;
    const int split = (int)blockIdx.x / num_tiles;
    const TileOrder tile((int)blockIdx.x - split * num_tiles, tiles_m, tiles_n, group_rows);
    const int tile_m = tile.m, tile_n = tile.n;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int r = lane & 31, h = lane >> 5;
    const int wg_m0 = tile_m * C::BM, wg_n0 = tile_n * C::BN;
    const int wrow0 = (wave / GN) * (32 * WM);       // first row of this wave inside the A tile
    const int wcol0 = (wave % GN) * (32 * WN);       // first row of this wave inside the W tile

    // ---- DMA source offsets of this thread (bytes from the operand base)
    // When K' is an odd multiple of 64 the last stage is half a stage (4 blocks): the lanes that
    // would fetch its missing second half re-fetch the first half instead (never used), which
    // keeps every access inside the operand.  `half` selects those adjusted offsets.
    const bool has_half = MODE == COPIES && (nbk & 7) != 0;
    const int nstage = MODE != COPIES ? (nbk + 7) >> 3 : (nbk >> 3) + (has_half ? 1 : 0);   // of the whole reduction dimension
    const int per_split = nstage / splits, extra = nstage % splits;
    const int s_begin = split * per_split + min(split, extra);  // this workgroup's stages [s_begin, s_end)
    const int s_end = s_begin + per_split + (split < extra ? 1 : 0);
    // Offsets are recomputed per copy (a handful of ALU operations per stage) rather than kept
    // in registers: the accumulators leave this kernel 256 registers and it needs most of them.
    // (s & 3) and the row swizzle repeat every 64 slots, so one value serves every copy
    const uint32_t lp_ = (uint32_t)((tid & 3) ^ ((tid >> 4) & 3));
    const uint32_t adj_c0 = lp_ * 16u, adj_c1 = (lp_ & 1u) * 16u, adj_s = (uint32_t)(tid & 1) * 4u;
    const int crow = tid >> 2, srow = tid >> 1; // row of this thread inside a copy of NT/4 code rows / NT/2 scale rows
    const uint32_t cpitch32 = (uint32_t)nbk * 8u, spitch32 = (uint32_t)nbk;
    // lane l of a DMA writes slot wave_slot + l; made a scalar once so that the LDS destinations
    // of all copies are computed on the scalar unit
    const uint32_t wave_slot = __builtin_amdgcn_readfirstlane((uint32_t)(tid & ~63));
    const uint32_t lds0 = lds_address(lds);
    const typename C::Windows windows = {a_scales, w_scales, M, N, nbk, wg_m0, wg_n0, (uint32_t)tid, wave_slot};    // RAGGED
    const int patch_from = C::Windows::patch_from(nbk);
    // DMA instruction d (0 .. NDMA-1) of a stage: (RAGGED: scale windows,) A code pieces, W code pieces, A scales, W scales.
    auto issue_one = [&](int d, int stage, int buf) {
        const uint32_t base = lds0 + buf * C::STAGE_BYTES;
        const bool half = has_half && stage == nstage - 1;
        const uint32_t oc = RAG ? 8u * (uint32_t)min(8 * stage + 2 * (int)lp_, nbk - 2) : (uint32_t)stage * 64u + (half ? adj_c1 : adj_c0);
        if (RAG && d < C::NSW) {
            windows.issue(d, stage, base + C::WINDOWS);
            return;
        }
        d -= C::NSW;
        const uint32_t os = (uint32_t)stage * 8u + (half ? 0u : adj_s);
        constexpr int NA = C::NA, NW = C::NW, NAS = C::NAS, NT = C::NT;
        // rows past the edge of the operand re-read its last row (never stored)
        if (d < NA) {
            const uint32_t row = (uint32_t)min(wg_m0 + d * (NT / 4) + crow, M - 1);
            dma16(a_codes, row * cpitch32 + oc, base + C::A_CODES + 16u * (d * NT + wave_slot));
        } else if (d < NA + NW) {
            const int p = d - NA;
            const uint32_t row = (uint32_t)min(wg_n0 + p * (NT / 4) + crow, N - 1);
            dma16(w_codes, row * cpitch32 + oc, base + C::W_CODES + 16u * (p * NT + wave_slot));
        } else if (d < NA + NW + NAS) {
            const int p = d - NA - NW;
            const uint32_t row = (uint32_t)min(wg_m0 + p * (NT / 2) + srow, M - 1);
            dma4(a_scales, row * spitch32 + os, base + C::A_SCALES + 4u * (p * NT + wave_slot));
        } else {
            const int p = d - NA - NW - NAS;
            const uint32_t row = (uint32_t)min(wg_n0 + p * (NT / 2) + srow, N - 1);
            dma4(w_scales, row * spitch32 + os, base + C::W_SCALES + 4u * (p * NT + wave_slot));
        }
    };
    auto issue_all = [&](int stage, int buf) {
#pragma unroll
        for (int d = 0; d < C::NDMA; ++d) issue_one(d, stage, buf);
    };
    // ---- REGS: the same pieces through registers (piece d of a thread lands where DMA instruction d puts it).
    // A piece that would reach past the end of its row is fetched from further left, so that it ends with the row
    // (needs nbk >= 4), and shifted into place when it is written to LDS.
    constexpr int NCP = C::NA + C::NW, NSP = C::NAS + C::NWS;
    uint4 rc[REG ? NCP : 1];
    uint32_t rs[REG ? NSP : 1];
    auto reg_issue = [&](int stage) {
        const uint32_t oc = 8u * (uint32_t)min(8 * stage + 2 * (int)lp_, nbk - 2);
#pragma unroll
        for (int d = 0; d < NCP; ++d) {
            const bool is_a = d < C::NA;
            const int p = is_a ? d : d - C::NA;
            const uint32_t row = (uint32_t)(is_a ? min(wg_m0 + p * (C::NT / 4) + crow, M - 1) : min(wg_n0 + p * (C::NT / 4) + crow, N - 1));
            rc[d] = load16_a8((is_a ? a_codes : w_codes) + (size_t)(row * cpitch32 + oc));
        }
        const uint32_t os = (uint32_t)min(8 * stage + 4 * (tid & 1), nbk - 4);
#pragma unroll
        for (int d = 0; d < NSP; ++d) {
            const bool is_a = d < C::NAS;
            const int p = is_a ? d : d - C::NAS;
            const uint32_t row = (uint32_t)(is_a ? min(wg_m0 + p * (C::NT / 2) + srow, M - 1) : min(wg_n0 + p * (C::NT / 2) + srow, N - 1));
            rs[d] = load4_a1((is_a ? a_scales : w_scales) + (size_t)(row * spitch32 + os));
        }
    };
    auto reg_commit = [&](int stage, int buf) {
        uint8_t* st = lds + buf * C::STAGE_BYTES;
        const int b0 = 8 * stage + 2 * (int)lp_;       // this piece: blocks b0, b0 + 1
        const bool both = b0 + 1 < nbk, one = b0 < nbk;
#pragma unroll
        for (int d = 0; d < NCP; ++d) {
            const uint4 v = uint4{both ? rc[d].x : one ? rc[d].z : 0u, both ? rc[d].y : one ? rc[d].w : 0u, both ? rc[d].z : 0u, both ? rc[d].w : 0u};
            const int at = d < C::NA ? C::A_CODES + 16 * (d * C::NT + tid) : C::W_CODES + 16 * ((d - C::NA) * C::NT + tid);
            *reinterpret_cast<uint4*>(st + at) = v;
        }
        const int sb0 = 8 * stage + 4 * (tid & 1);      // this word: blocks sb0 .. sb0 + 3
        const int skip = sb0 - min(sb0, nbk - 4);       // bytes of the fetched word that belong to earlier blocks
#pragma unroll
        for (int d = 0; d < NSP; ++d) {
            const uint32_t word = skip >= 4 ? 0u : rs[d] >> (8 * skip);
            const int at = d < C::NAS ? C::A_SCALES + 4 * (d * C::NT + tid) : C::W_SCALES + 4 * ((d - C::NAS) * C::NT + tid);
            *reinterpret_cast<uint32_t*>(st + at) = word;
        }
    };

    // ---- LDS read offsets of this lane inside a stage.  Fragment i of a wave is 32 rows (2048
    // bytes of codes, 256 of scales) further on, a constant folded into the instruction; the
    // swizzle (row >> 2) & 3 only depends on lane % 32 because the other terms are multiples of 32.
    const uint32_t swz = (uint32_t)(r >> 2) & 3u;
    const uint32_t rd_a = C::A_CODES + (wrow0 + r) * 64, rd_w = C::W_CODES + (wcol0 + r) * 64;
    // a lane reads the whole 4-byte scale word of its row and 64-k half stage (both halves of the wave read
    // the same word, which the LDS broadcasts; two-byte reads of its two halves count as a bank conflict)
    // and picks its two bytes with the byte selector of the permute
    const uint32_t rd_as = C::A_SCALES + (wrow0 + r) * 8, rd_ws = C::W_SCALES + (wcol0 + r) * 8;
    const uint32_t scale_sel = h ? 0x0C030C02u : 0x0C010C00u;
    const uint32_t piece0 = 16u * ((uint32_t)h ^ swz), piece1 = 16u * ((2u + (uint32_t)h) ^ swz);

    float16v acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // ---- per-stage compute, software-pipelined by hand (with one or two waves per SIMD little else
    // hides a stall, so every wait is placed where its data has long been ready).
    // A k-step (one block, 16 k) is WM*WN MFMAs fed by WM + WN fragments of 8 fp16 per lane.
    // While the MFMAs of step x run, the fragments of step x+1 are decoded: after every group of
    // MFMAs (see MPG) the decode of its share of the fragments is placed, and scheduling barriers keep
    // the compiler from regrouping them, so the matrix pipe stays busy while the vector ALU decodes.
    // The pipeline runs ACROSS stages: the barrier that opens stage s+1 sits before step 6 of
    // stage s; step 6 reads the first raw codes of stage s+1 from LDS and step 7 decodes its
    // first fragments.  The copies for stage s + NSTAGE - 1 are issued two per k-step during steps 0-5 of
    // stage s (its buffer was last read in stage s-1, which every wave left before the barrier
    // that opened stage s), so no wave ever queues a burst of memory instructions.
    constexpr int G = WM + WN;                 // fragments per k-step
    // MFMAs per group: after every group the decode of G / P fragments is placed.  With few MFMAs per
    // fragment (2 x 2 fragments: nine vector instructions per MFMA) single MFMAs interleave best with the
    // vector work (a register-only model of this loop ran 10 % faster with singles than with pairs);
    // with 4 x 4 fragments pairs and singles measure the same in that model, and singles spill here.
    constexpr int MPG = (WM * WN >= 16) ? 2 : 1;
    constexpr int P = (WM * WN) / MPG;         // groups per k-step
    uint4 ca[2][WM], cw[2][WN];
    uint32_t sa[2][WM], sw[2][WN];
    half8 fa[2][WM], fw[2][WN];
    auto read_raw = [&](int u, const uint8_t* st) {
        const uint8_t* pa = st + rd_a + (u ? piece1 : piece0);
        const uint8_t* pw = st + rd_w + (u ? piece1 : piece0);
        const uint8_t* psa = st + rd_as + 4 * u;
        const uint8_t* psw = st + rd_ws + 4 * u;
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            ca[u][i] = *reinterpret_cast<const uint4*>(pa + i * 2048);
            sa[u][i] = scale_halves(*reinterpret_cast<const uint32_t*>(psa + i * 256), scale_sel);
        }
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            cw[u][j] = *reinterpret_cast<const uint4*>(pw + j * 2048);
            sw[u][j] = scale_halves(*reinterpret_cast<const uint32_t*>(psw + j * 256), scale_sel);
        }
    };
    auto decode_frag = [&](int gidx, int x) {   // fragment gidx of k-step x (0..7) into slot x & 1
        const int u = x >> 2, t = x & 3, d = x & 1;
        if (gidx < WM) {
            const uint4 c4 = ca[u][gidx];
            const uint32_t c = t == 0 ? c4.x : t == 1 ? c4.y : t == 2 ? c4.z : c4.w;
            fa[d][gidx] = decode8_half(c, sa[u][gidx], t >> 1);
        } else {
            const int j = gidx - WM;
            const uint4 c4 = cw[u][j];
            const uint32_t c = t == 0 ? c4.x : t == 1 ? c4.y : t == 2 ? c4.z : c4.w;
            fw[d][j] = decode8_half(c, sw[u][j], t >> 1);
        }
    };

    // A stage is free of branches (they would split the hand-made schedule): the last two stages of a workgroup's run have code of
    // their own (left_tag: stages behind this one, up to DIST = 2), which issues no copies and, in the last one, reads and decodes
    // nothing for a next stage.  (Both used to go on with the last stage, whose copies the end of the kernel then waited for: 1 % of
    // the time on average over 200 problems of 513 to 8192 rows, 0.2 us a round; 2048 x 4096 over K' = 4352 with norm 72.6 -> 71.5 us.)
    int buf = 0;                                // ring slot of the stage being computed
    auto ring_next = [](int b) { return b == C::NSTAGE - 1 ? 0 : b + 1; };
    // RAGGED: the wanted scale bytes of stage s+1 are picked out of their windows during step FIX (read) and the one after
    // (write), one copy per step.  tail_tag: the stage before one whose windows or blocks may pass the end (the last two);
    // all others know that they are whole.
    constexpr int FIX = 3;
    auto copies_before = [](int x) { return (x * C::NDMA + 5) / 6; };    // copies of a stage issued before step x <= 6
    uint3 win[RAG ? 2 : 1];
    auto run_stage = [&](int s, auto tail_tag, auto left_tag) {
        constexpr bool TAIL = decltype(tail_tag)::value;
        constexpr int LEFT = decltype(left_tag)::value;
        const uint8_t* st = lds + buf * C::STAGE_BYTES;
        // the copies issued during this stage go to the slot of the stage computed before this one
        const int buf1 = ring_next(buf), buf2 = buf == 0 ? C::NSTAGE - 1 : buf - 1;
        int fetch = s + C::DIST;        // opaque: followed as an induction variable it costs the copies 14 more additions a stage
        asm("" : "+s"(fetch));
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            // (a half stage leaves here; with code of its own, beside that of a whole last stage, the accumulators spill)
            if (LEFT == 0 && x == 4 && has_half && s == nstage - 1) break;
            if (x == 0) read_raw(1, st);
            if constexpr (RAG && LEFT > 0) {
                uint8_t* next = lds + buf1 * C::STAGE_BYTES;
                if (x >= FIX && x < FIX + C::NSW) {
                    // windows of stage s+1: the code copies of that stage and the copies issued in this one are younger
                    if (x == FIX) wait_vmcnt<C::NA + C::NW + (LEFT == 2 ? (FIX * C::NDMA + 5) / 6 : 0)>();
                    win[(x - FIX) & 1] = windows.gather(x - FIX, next + C::WINDOWS, TAIL && s + 1 >= patch_from, lds + C::PATCH + 8 * (s + 1 - patch_from));
                }
                if (x > FIX && x <= FIX + C::NSW)
                    windows.put(x - FIX - 1, win[(x - FIX - 1) & 1], next + C::A_SCALES, TAIL, s + 1);
            }
            if (x == 6 && LEFT > 0) {
                // stage s+1 must have landed: the copies of the DIST - 1 later stages are younger, and
                // everything older has retired once at most that many operations are outstanding
                // (REGS: this wave's LDS writes of stage s+1 must have completed)
                if constexpr (REG) wait_lgkmcnt0();
                else wait_vmcnt<LEFT == 2 ? (C::DIST - 1) * C::NDMA : 0>();
                if constexpr (RAG) wait_lgkmcnt0();         // this wave's scale bytes of stage s+1 are written
                wg_barrier();
                read_raw(0, lds + buf1 * C::STAGE_BYTES);
                if constexpr (REG && LEFT == 2) reg_issue(s + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < P; ++p) {
#pragma unroll
                for (int gidx = (p * G) / P; gidx < ((p + 1) * G) / P; ++gidx) {
                    if (x + 1 < 8) decode_frag(gidx, x + 1);
                    else if (LEFT > 0) decode_frag(gidx, 0);      // first step of stage s+1
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = MPG * p; q < MPG * p + MPG; ++q) {
                    const int i = q / WN, j = q % WN;
                    // weights as the row operand: see store_tile_swapped
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[x & 1][j], fa[x & 1][i], acc[i][j], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (!REG && LEFT == 2 && x < 6) {    // copies of stage s + NSTAGE - 1, spread over steps 0..5
#pragma unroll
                    for (int d = 0; d < C::NDMA; ++d)
                        if ((d * 6) / C::NDMA == x && d - copies_before(x) == p) issue_one(d, fetch, buf2);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if constexpr (REG && LEFT > 0)
                if (x == 5) {                   // stage s+1, fetched since step 6 of the stage before
                    reg_commit(s + 1, buf1);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        buf = buf1;
    };

    if constexpr (REG) {
        reg_issue(s_begin);
        reg_commit(s_begin, 0);
        reg_issue(min(s_begin + 1, s_end - 1));
        wait_lgkmcnt0();
    } else {
#pragma unroll
        for (int d = 0; d < C::DIST; ++d) issue_all(min(s_begin + d, s_end - 1), d);
        if constexpr (RAG) windows.fill_patch(lds + C::PATCH);
        wait_vmcnt<(C::DIST - 1) * C::NDMA>();
        if constexpr (RAG) {                    // (runs of a split are at least four stages long: the first is whole)
#pragma unroll
            for (int d = 0; d < C::NSW; ++d)
                windows.put(d, windows.gather(d, lds + C::WINDOWS, false, nullptr), lds + C::A_SCALES, false, 0);
            wait_lgkmcnt0();
        }
    }
    wg_barrier();
    read_raw(0, lds);
#pragma unroll
    for (int gidx = 0; gidx < G; ++gidx) decode_frag(gidx, 0);
    using Rag = std::integral_constant<bool, RAG>;
    int s = s_begin;
    for (; s < (RAG ? min(patch_from - 1, s_end - 2) : s_end - 2); ++s) run_stage(s, std::false_type{}, std::integral_constant<int, 2>{});
    if constexpr (RAG)
        for (; s < s_end - 2; ++s) run_stage(s, std::true_type{}, std::integral_constant<int, 2>{});
    if (s_end - s_begin > 1) run_stage(s_end - 2, Rag{}, std::integral_constant<int, 1>{});
    run_stage(s_end - 1, std::false_type{}, std::integral_constant<int, 0>{});
    wait_vmcnt<0>();                            // no copy may still be in flight when the LDS is released

    const int m0 = wg_m0 + wrow0, n0 = wg_n0 + wcol0;
    if constexpr (std::is_same<OutT, _Float16>::value) {
        static_assert(epilogue_lds_bytes(WN) * GM * GN <= C::LDS_BYTES, "one epilogue region per wave must fit the operand ring");
        wg_barrier();                           // every wave has read its last operands: the ring is free
        store_tile_f16_via_lds<WM, WN>(acc, lds + wave * epilogue_lds_bytes(WN), m0, n0, lane, M, N, alpha,
                                       y + (int64_t)split * split_stride, ldy);
    } else {
        store_tile_swapped<WM, WN>(acc, m0, n0, r, h, M, N, alpha, y + (int64_t)split * split_stride, ldy);
    }
}

// ---------------------------------------------------------------------------------------------
// 128 x 256 tiles for problems with about one such tile per CU (2048 x 4096 has 256 of them).
// Same tile, stage ring and copies as gemm_staged_kernel<2, 2, 2, 4>, but the eight waves form a
// 2 (rows) x 2 (columns) x 2 (k) grid: a wave computes a 64 x 128 sub-tile (2 x 4 fragments: six fragment
// decodes per eight MFMAs instead of four per four, the decode being what keeps this tile shape from the
// matrix rate of the bigger ones) over one half of every stage: four of its eight k-steps, exactly the
// 16-byte piece of codes a lane reads per row and stage.  The two waves of a pair (w and w + 4) share a
// SIMD, so the matrix pipe still draws from two instruction streams; at the end they add their partial
// tiles through the LDS and each stores one of the two fragment rows.  MODE: COPIES for K' % 128 == 0, RAGGED for rows off the grid of 64.
template <typename OutT, int MODE>
__global__ __launch_bounds__(512) void gemm_kpair_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N,
    int nbk, float alpha, OutT* __restrict__ y, int64_t ldy, int tiles_m, int tiles_n, int group_rows) {
    using C = StagedCfg<2, 2, 2, 4, MODE>;
    constexpr bool RAG = MODE == RAGGED;
    constexpr int WM = 2, WN = 4;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    // workgroup -> tile: tile_order.h
    const TileOrder tile((int)blockIdx.x, tiles_m, tiles_n, group_rows);
    const int tile_m = tile.m, tile_n = tile.n;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int r = lane & 31, h = lane >> 5;
    const int kh = wave >> 2;                        // k half: k-steps 4 kh .. 4 kh + 3 of every stage
    const int wq = wave & 3;
    const int wg_m0 = tile_m * C::BM, wg_n0 = tile_n * C::BN;
    const int wrow0 = (wq >> 1) * 64;                // first row of this wave inside the A tile
    const int wcol0 = (wq & 1) * 128;                // first row of this wave inside the W tile
    const int nstage = RAG ? (nbk + 7) >> 3 : nbk >> 3;

    // ---- copies (see gemm_staged_kernel)
    const uint32_t lp_ = (uint32_t)((tid & 3) ^ ((tid >> 4) & 3));
    const uint32_t adj_c0 = lp_ * 16u, adj_s = (uint32_t)(tid & 1) * 4u;
    const int crow = tid >> 2, srow = tid >> 1;
    const uint32_t cpitch32 = (uint32_t)nbk * 8u, spitch32 = (uint32_t)nbk;
    const uint32_t wave_slot = __builtin_amdgcn_readfirstlane((uint32_t)(tid & ~63));
    const uint32_t lds0 = lds_address(lds);
    const typename C::Windows windows = {a_scales, w_scales, M, N, nbk, wg_m0, wg_n0, (uint32_t)tid, wave_slot};    // RAGGED
    const int patch_from = C::Windows::patch_from(nbk);
    auto issue_one = [&](int d, int stage, int buf) {
        const uint32_t base = lds0 + buf * C::STAGE_BYTES;
        const uint32_t oc = RAG ? 8u * (uint32_t)min(8 * stage + 2 * (int)lp_, nbk - 2) : (uint32_t)stage * 64u + adj_c0;
        if (RAG && d < C::NSW) {
            windows.issue(d, stage, base + C::WINDOWS);
            return;
        }
        d -= C::NSW;
        const uint32_t os = (uint32_t)stage * 8u + adj_s;
        constexpr int NA = C::NA, NW = C::NW, NAS = C::NAS, NT = C::NT;
        if (d < NA) {
            const uint32_t row = (uint32_t)min(wg_m0 + d * (NT / 4) + crow, M - 1);
            dma16(a_codes, row * cpitch32 + oc, base + C::A_CODES + 16u * (d * NT + wave_slot));
        } else if (d < NA + NW) {
            const int p = d - NA;
            const uint32_t row = (uint32_t)min(wg_n0 + p * (NT / 4) + crow, N - 1);
            dma16(w_codes, row * cpitch32 + oc, base + C::W_CODES + 16u * (p * NT + wave_slot));
        } else if (d < NA + NW + NAS) {
            const int p = d - NA - NW;
            const uint32_t row = (uint32_t)min(wg_m0 + p * (NT / 2) + srow, M - 1);
            dma4(a_scales, row * spitch32 + os, base + C::A_SCALES + 4u * (p * NT + wave_slot));
        } else {
            const int p = d - NA - NW - NAS;
            const uint32_t row = (uint32_t)min(wg_n0 + p * (NT / 2) + srow, N - 1);
            dma4(w_scales, row * spitch32 + os, base + C::W_SCALES + 4u * (p * NT + wave_slot));
        }
    };

    // ---- LDS read offsets: this wave's half of a stage is piece 2 kh + h of a row's codes and bytes
    // 4 kh + 2 h, 4 kh + 2 h + 1 of its scale bytes
    const uint32_t swz = (uint32_t)(r >> 2) & 3u;
    const uint32_t piece = 16u * ((uint32_t)(2 * kh + h) ^ swz);
    const uint32_t rd_a = C::A_CODES + (wrow0 + r) * 64 + piece, rd_w = C::W_CODES + (wcol0 + r) * 64 + piece;
    const uint32_t rd_as = C::A_SCALES + (wrow0 + r) * 8 + 4 * kh, rd_ws = C::W_SCALES + (wcol0 + r) * 8 + 4 * kh;
    const uint32_t scale_sel = h ? 0x0C030C02u : 0x0C010C00u;

    float16v acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    constexpr int G = WM + WN;                 // fragments per k-step
    constexpr int P = WM * WN;                 // MFMAs per k-step, one per group
    uint4 ca[WM], cw[WN];
    uint32_t sa[WM], sw[WN];
    half8 fa[2][WM], fw[2][WN];
    auto read_raw = [&](const uint8_t* st) {
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            ca[i] = *reinterpret_cast<const uint4*>(st + rd_a + i * 2048);
            sa[i] = scale_halves(*reinterpret_cast<const uint32_t*>(st + rd_as + i * 256), scale_sel);
        }
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            cw[j] = *reinterpret_cast<const uint4*>(st + rd_w + j * 2048);
            sw[j] = scale_halves(*reinterpret_cast<const uint32_t*>(st + rd_ws + j * 256), scale_sel);
        }
    };
    auto decode_frag = [&](int gidx, int t) {   // fragment gidx of this wave's k-step t (0..3) into slot t & 1
        const int d = t & 1;
        if (gidx < WM) {
            const uint4 c4 = ca[gidx];
            const uint32_t c = t == 0 ? c4.x : t == 1 ? c4.y : t == 2 ? c4.z : c4.w;
            fa[d][gidx] = decode8_half(c, sa[gidx], t >> 1);
        } else {
            const int j = gidx - WM;
            const uint4 c4 = cw[j];
            const uint32_t c = t == 0 ? c4.x : t == 1 ? c4.y : t == 2 ? c4.z : c4.w;
            fw[d][j] = decode8_half(c, sw[j], t >> 1);
        }
    };

    // One stage = four k-steps of this wave.  During step t the fragments of step t + 1 are decoded, one
    // group of fragments after every MFMA; the raw codes of the next stage are read at the start of step 3
    // (every fragment of this stage has been decoded by then) behind the barrier that opens that stage, and
    // step 3 decodes its first fragments.  The copies of stage s + DIST are issued during steps 0..2.
    int buf = 0;
    auto ring_next = [](int b) { return b == C::NSTAGE - 1 ? 0 : b + 1; };
    uint3 win[RAG ? C::NSW : 1];
    auto run_stage = [&](int s, auto tail_tag, auto left_tag) {     // tags: see gemm_staged_kernel
        constexpr bool TAIL = decltype(tail_tag)::value;
        constexpr int LEFT = decltype(left_tag)::value;
        const int buf1 = ring_next(buf), buf2 = buf == 0 ? C::NSTAGE - 1 : buf - 1;
        int fetch = s + C::DIST;        // opaque: followed as an induction variable it costs the copies 14 more additions a stage
        asm("" : "+s"(fetch));
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (RAG && LEFT > 0) {    // scale bytes of stage s+1, see gemm_staged_kernel
                uint8_t* next = lds + buf1 * C::STAGE_BYTES;
                if (t == 1) {
                    wait_vmcnt<C::NA + C::NW + (LEFT == 2 ? (C::NDMA + 2) / 3 : 0)>();
#pragma unroll
                    for (int d = 0; d < C::NSW; ++d)
                        win[d] = windows.gather(d, next + C::WINDOWS, TAIL, lds + C::PATCH + 8 * (s + 1 - patch_from));
                }
                if (t == 2)
#pragma unroll
                    for (int d = 0; d < C::NSW; ++d) windows.put(d, win[d], next + C::A_SCALES, TAIL, s + 1);
            }
            if (t == 3 && LEFT > 0) {
                wait_vmcnt<LEFT == 2 ? (C::DIST - 1) * C::NDMA : 0>();
                if constexpr (RAG) wait_lgkmcnt0();
                wg_barrier();
                read_raw(lds + buf1 * C::STAGE_BYTES);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < P; ++p) {
#pragma unroll
                for (int gidx = (p * G) / P; gidx < ((p + 1) * G) / P; ++gidx)
                    if (t < 3 || LEFT > 0) decode_frag(gidx, (t + 1) & 3);
                __builtin_amdgcn_sched_barrier(0);
                const int i = p / WN, j = p % WN;
                // weights as the row operand: see store_tile_swapped
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[t & 1][j], fa[t & 1][i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (t < 3 && LEFT == 2) {
#pragma unroll
                    for (int d = 0; d < C::NDMA; ++d)
                        if ((d * 3) / C::NDMA == t && (d - (t * C::NDMA + 2) / 3) == p) issue_one(d, fetch, buf2);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        buf = buf1;
    };

#pragma unroll
    for (int d = 0; d < C::DIST; ++d)
#pragma unroll
        for (int q = 0; q < C::NDMA; ++q) issue_one(q, min(d, nstage - 1), d);
    if constexpr (RAG) windows.fill_patch(lds + C::PATCH);
    wait_vmcnt<(C::DIST - 1) * C::NDMA>();
    if constexpr (RAG) {                        // the first stage is whole
#pragma unroll
        for (int d = 0; d < C::NSW; ++d)
            windows.put(d, windows.gather(d, lds + C::WINDOWS, false, nullptr), lds + C::A_SCALES, false, 0);
        wait_lgkmcnt0();
    }
    wg_barrier();
    read_raw(lds);
#pragma unroll
    for (int gidx = 0; gidx < G; ++gidx) decode_frag(gidx, 0);
    using Rag = std::integral_constant<bool, RAG>;
    int s = 0;
    if constexpr (RAG) {
        for (; s < min(patch_from - 1, nstage - 2); ++s) run_stage(s, std::false_type{}, std::integral_constant<int, 2>{});
        for (; s < nstage - 2; ++s) run_stage(s, std::true_type{}, std::integral_constant<int, 2>{});
    } else {
        // (nearly all instructions of the loop have eight bytes; four bytes off their multiples it is 0.9 % slower, 2000 x 4096 over K' = 8448 124.1 -> 125.3
        // us, and where it falls changes with whatever comes before it; the loops above do not care)
        for (; s < nstage - 2; ++s) {
            asm volatile(".p2align 3");
            run_stage(s, std::false_type{}, std::integral_constant<int, 2>{});
        }
    }
    if (nstage > 1) run_stage(nstage - 2, Rag{}, std::integral_constant<int, 1>{});
    run_stage(nstage - 1, std::false_type{}, std::integral_constant<int, 0>{});
    wait_vmcnt<0>();                            // no copy may still be in flight when the LDS is released

    // ---- the pair adds its partial tiles: in two rounds (columns 0-63, 64-127 of the sub-tile) every wave
    // hands the partner the fragment row the partner will store, 16 bytes per lane and register group
    static_assert(8 * 8192 <= C::LDS_BYTES && 8 * epilogue_lds_bytes(WN) / 2 <= C::LDS_BYTES, "epilogue regions must fit the ring");
    float* xch = reinterpret_cast<float*>(lds);
    const int mine = kh, other = kh ^ 1;        // fragment row this wave stores / gives away
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        wait_lgkmcnt0();                        // this wave's reads of the ring / of the previous round have returned
        wg_barrier();                           // ring (or the previous round's regions) no longer read
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = 2 * round + jj;
                const float16v& src = other == 0 ? acc[0][j] : acc[1][j];
                *reinterpret_cast<float4*>(xch + wave * 2048 + ((jj * 4 + q) * 64 + lane) * 4) =
                    make_float4(src[4 * q], src[4 * q + 1], src[4 * q + 2], src[4 * q + 3]);
            }
        wait_lgkmcnt0();
        wg_barrier();
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = 2 * round + jj;
                const float4 v = *reinterpret_cast<const float4*>(xch + (wave ^ 4) * 2048 + ((jj * 4 + q) * 64 + lane) * 4);
                if (mine == 0) {
                    acc[0][j][4 * q] += v.x; acc[0][j][4 * q + 1] += v.y; acc[0][j][4 * q + 2] += v.z; acc[0][j][4 * q + 3] += v.w;
                } else {
                    acc[1][j][4 * q] += v.x; acc[1][j][4 * q + 1] += v.y; acc[1][j][4 * q + 2] += v.z; acc[1][j][4 * q + 3] += v.w;
                }
            }
    }
    wait_lgkmcnt0();
    wg_barrier();                               // every wave has read its partner's last round
    const int m0 = wg_m0 + wrow0, n0 = wg_n0 + wcol0;
    if constexpr (std::is_same<OutT, _Float16>::value) {
        uint8_t* region = lds + wave * (epilogue_lds_bytes(WN) / 2);
        if (mine == 0)
            store_fragment_rows_f16_via_lds<WM, WN, 0, 1>(acc, region, m0, n0, lane, M, N, alpha, y, ldy);
        else
            store_fragment_rows_f16_via_lds<WM, WN, 1, 1>(acc, region, m0, n0, lane, M, N, alpha, y, ldy);
    } else {
        if (mine == 0)
            store_fragment_row_swapped<WM, WN, 0>(acc, m0, n0, r, h, M, N, alpha, y, ldy);
        else
            store_fragment_row_swapped<WM, WN, 1>(acc, m0, n0, r, h, M, N, alpha, y, ldy);
    }
}

// y = alpha * (sum of the `splits` fp32 partial results [M, N], added in index order).
template <typename OutT>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int splits,
                                                            int64_t split_stride, int M, int N, float alpha,
                                                            OutT* __restrict__ y, int64_t ldy, int vec4) {
    const int64_t total = vec4 ? (int64_t)M * (N >> 2) : (int64_t)M * N;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * blockDim.x) {
        if (vec4) {
            const int64_t m = idx / (N >> 2), n = 4 * (idx % (N >> 2));
            float4 sum = *reinterpret_cast<const float4*>(part + m * N + n);
            for (int sp = 1; sp < splits; ++sp) {
                const float4 v = *reinterpret_cast<const float4*>(part + sp * split_stride + m * N + n);
                sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
            }
            store4(y + m * ldy + n, sum.x * alpha, sum.y * alpha, sum.z * alpha, sum.w * alpha);
        } else {
            const int64_t m = idx / N, n = idx % N;
            float sum = part[m * N + n];
            for (int sp = 1; sp < splits; ++sp) sum += part[sp * split_stride + m * N + n];
            store_out(y + m * ldy + n, sum * alpha);
        }
    }
}

template <int WM, int WN, int GM, int GN, int MODE = COPIES, typename OutT>
arcq_status launch_staged(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                          const uint8_t* w_scales, int M, int N, int nbk, float alpha, OutT* y, int64_t ldy,
                          hipStream_t stream, int splits = 1, float* partial = nullptr) {
    using C = StagedCfg<WM, WN, GM, GN, MODE>;
    const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    if (splits > 1) {
        // fp32 partial results [splits, M, N] in the workspace, then one pass that adds them
        auto kern = gemm_staged_kernel<WM, WN, GM, GN, float, MODE>;
        static std::atomic<uint64_t> lds_raised{0};
        if (arcq_status st = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_raised)) return st;
        const int64_t stride = (int64_t)M * N;
        hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * splits), dim3(C::NT), C::LDS_BYTES, stream, a_codes, a_scales,
                           w_codes, w_scales, M, N, nbk, 1.0f, partial, (int64_t)N, tiles_m, tiles_n, tile_group_rows(tiles_m, tiles_n), splits, stride);
        if (arcq_status st = check_launch("gemm_staged_kernel (split K)")) return st;
        return launch_splitk_reduce(partial, splits, M, N, alpha, y, std::is_same<OutT, _Float16>::value ? ARCQ_DTYPE_F16 : ARCQ_DTYPE_F32,
                                    ldy, stream);
    }
    auto kern = gemm_staged_kernel<WM, WN, GM, GN, OutT, MODE>;
    static std::atomic<uint64_t> lds_raised{0};
    if (arcq_status st = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_raised)) return st;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(C::NT), C::LDS_BYTES, stream, a_codes, a_scales, w_codes,
                       w_scales, M, N, nbk, alpha, y, ldy, tiles_m, tiles_n, tile_group_rows(tiles_m, tiles_n), 1, (int64_t)0);
    return check_launch("gemm_staged_kernel");
}

template <int MODE, typename OutT>
arcq_status launch_kpair(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes, const uint8_t* w_scales, int M,
                         int N, int nbk, float alpha, OutT* y, int64_t ldy, hipStream_t stream) {
    using C = StagedCfg<2, 2, 2, 4, MODE>;
    auto kern = gemm_kpair_kernel<OutT, MODE>;
    static std::atomic<uint64_t> lds_raised{0};
    if (arcq_status st = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_raised)) return st;
    const int tiles_m = (M + 127) / 128, tiles_n = (N + 255) / 256;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(512), C::LDS_BYTES, stream, a_codes, a_scales, w_codes, w_scales, M, N,
                       nbk, alpha, y, ldy, tiles_m, tiles_n, tile_group_rows(tiles_m, tiles_n));
    return check_launch("gemm_kpair_kernel");
}

// ---------------------------------------------------------------------------------------------
// Skinny kernel for M <= 128 (decode, batched decode, short prefill): bound by streaming the packed
// weights once from HBM (9/16 byte per weight), so the layout of the work follows the weight rows.
//
// v_mfma_f32_16x16x32_f16: lane (i = lane % 16, q = lane / 16) supplies 8 consecutive k of row i;
// the four lane groups q supply different octets.  The activations are the 16-row operand, the
// weights the 16-column operand.  A lane loads 16 bytes (32 codes, blocks 8c+2q and 8c+2q+1 of
// chunk c = 128 k) of its weight row, which feed 4 MFMAs; the 16 rows of a tile make each wave
// load 16 x 64 contiguous bytes.  Rows of the activation operand past M repeat row M-1 and are
// not stored.
//
// Everything is loaded straight into registers, U chunks or a group of four at a time: variants that staged the
// activations and scale bytes in LDS, or kept a second set of registers for the next group of the weight stream, measured
// 1.4-1.6x slower at the decode shapes (what loads ahead below reuses the registers of chunks that have been decoded).  Every wave
// handles NT tiles of 16 weight rows for the same chunks, which shares the loads and the decode
// of the activation operand; the WAVES waves of a workgroup split K' (wave w takes chunks
// w*U .. w*U+U-1, then strides on) and add their partial tiles through LDS at the end.
typedef float float4v __attribute__((ext_vector_type(4)));

// MT tiles of 16 activation rows (M <= 16 MT) share every weight fragment a wave loads and decodes:
// batched decode and short prefills (M up to 128) stay on the weight-streaming path.
// GRP: whole chunks are taken four at a time (512 k) with the scale bytes of the four chunks fetched by ONE
// load per tile: the four lanes of a row read 8 bytes each, 32 contiguous bytes of the row, and a 4 x 4
// transpose of 16-bit pairs across the four lane groups (two lane-swap instructions and two byte permutes)
// hands every lane the two bytes it needs for each chunk.  The address unit of a CU spends about two cycles
// per (row, 64-byte segment) an instruction touches, whatever it fetches from the segment, so the two-byte
// scale loads of the chunk-at-a-time loop cost as much as the code loads: without any scale loads the
// kernel ran 18-23 % faster (timing build).  Chunks past the last whole group go through that loop.
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void transpose_scale_pairs(uint2 s, uint32_t& even_chunks, uint32_t& odd_chunks) {
    // lane group q holds the 8 scale bytes of chunk q as four 16-bit pairs (pair p: blocks 2p, 2p+1);
    // afterwards it holds pair q of chunks 0 and 2 (even_chunks: low, high half) and of chunks 1 and 3
    const uint2v x = __builtin_amdgcn_permlane32_swap(s.x, s.y, false, false);
    const uint32_t lo = __builtin_amdgcn_perm(x[1], x[0], 0x05040100u);   // low halves of both words
    const uint32_t hi = __builtin_amdgcn_perm(x[1], x[0], 0x07060302u);   // high halves
    const uint2v t = __builtin_amdgcn_permlane16_swap(lo, hi, false, false);
    even_chunks = t[0];
    odd_chunks = t[1];
}

// Rows need not start on 16-byte boundaries (K' / 16 odd, or operands that are only 8-byte aligned): every load
// is declared with the alignment the interface guarantees (codes 8 bytes, scale bytes 1), which the memory
// path serves in one request like an aligned one.  With an odd number of blocks the last block of a row has no
// partner: the pairs of the main loops stop before it and the last wave handles it by itself at the end, with
// 8-byte loads.
//
// ROLL (see plan_stream): a wave takes several groups, and asks for the next one while it computes: the registers of two chunks are loaded again
// as soon as both have been used.  Two, because a chunk is half a cache line of every row: asking for the halves one by one,
// each behind a chunk's decode, was 10 to 20 % slower than asking for whole groups between computing them (16 x 8192 over
// K' = 29696, weights from HBM: 36.4, 31.0 and, by twos, 30.4 us), although it keeps the most loads in flight.
//
// The decode of the operands bounds the kernel where it has whole rounds (16 x 28672 over K' = 8464: 131 MB from HBM in 34.6 us), so beyond a
// round of four weight tiles a wave more tiles (WIDE) cost less than a second round: the decode of the activations is shared by more of them.
// weight tiles whose partial sums fit the static LDS limit at a time
constexpr int skinny_batch(int mt, int nt, int waves) { return waves * mt * nt > 64 ? (nt + 1) / 2 : nt; }

template <int MT, int NT, int WAVES, int U, bool GRP, bool ROLL, bool TWO_STEPS, typename OutT>
__device__ __forceinline__ void skinny_tiles(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N,
    int nbk, float alpha, OutT* __restrict__ y, int64_t ldy, int n0, float* red_memory) {
    constexpr int BATCH = skinny_batch(MT, NT, WAVES);
    auto& red = *reinterpret_cast<float (*)[WAVES][MT * BATCH][4][64]>(red_memory);
    // WIDE: rows at 32-bit offsets from scalar addresses instead of pointers, and with two row tiles two chunks of activations at a time, loaded again
    // behind the chunk that used them: 256 registers take seven weight tiles then (four with pointers and whole groups of activations)
    constexpr bool WIDE = NT > 4, LATE_A = WIDE && MT == 2;
    static_assert(!WIDE || (GRP && ROLL), "more than four weight tiles: groups only, loaded ahead");
    // the wave number as a scalar: conditions on it become scalar branches (a matrix instruction inside a branch on a
    // vector condition would still execute: it does not honour the lane mask)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int i = lane & 15, q = lane >> 4;
    const int64_t cpitch = (int64_t)nbk * 8, spitch = nbk;
    const int nchunk = (nbk + 7) >> 3;                       // chunks of 8 blocks, the last may be partial

    const uint8_t* const base_c = w_codes + (WIDE ? n0 * cpitch : 0);
    const uint8_t* const base_s = w_scales + (WIDE ? n0 * spitch : 0);
    using Row = std::conditional_t<WIDE, uint32_t, const uint8_t*>;
    using Offset = std::conditional_t<WIDE, uint32_t, int64_t>;
    Row ac[MT], as[MT], wc[NT], ws[NT];
#pragma unroll
    for (int r = 0; r < MT; ++r) {
        const int m = min(16 * r + i, M - 1);
        if constexpr (WIDE) {
            ac[r] = (uint32_t)(m * cpitch) + 16u * q;
            as[r] = (uint32_t)(m * spitch) + 8u * q;
        } else {
            ac[r] = a_codes + (int64_t)m * cpitch;
            as[r] = a_scales + (int64_t)m * spitch;
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int n = min(n0 + 16 * t + i, N - 1);
        if constexpr (WIDE) {
            wc[t] = (uint32_t)((n - n0) * cpitch) + 16u * q;
            ws[t] = (uint32_t)((n - n0) * spitch) + 8u * q;
        } else {
            wc[t] = w_codes + n * cpitch;
            ws[t] = w_scales + n * spitch;
        }
    }
    auto scale_row = [&](Row codes, Row scales) -> Row {
        if constexpr (WIDE) { uint32_t o = codes; asm("" : "+v"(o)); return (o >> 3) + 6u * q; }
        else return scales;
    };
    // Byte `uniform` + `own` (a lane's) of a row.  Up to four tiles one sum for all rows, which has to be one: a sum that is used once is taken apart and added
    // to every row in two steps (33 to 64 rows, one tile a wave, K' = 1056 to 2880: 4.43 and 4.32 us, 6.64 and 6.52).  TWO_STEPS: in two steps, where that is the
    // faster one (gemm_skinny_kernel).  WIDE: rows come with a lane's place in a group of chunks, `place`, and the offset is opaque, so that no 64-bit
    // address of a row is kept.
    struct Parts { int64_t uniform; Offset own; };
    using Byte = std::conditional_t<WIDE || TWO_STEPS, Parts, int64_t>;
    auto byte_at = [](int64_t uniform, Offset own, uint32_t place) -> Byte {
        if constexpr (WIDE) return Parts{uniform, own - place};
        else if constexpr (TWO_STEPS) return Parts{uniform, own};
        else return uniform + own;
    };
    auto in_row = [](const uint8_t* base, Row row, Byte at) -> const uint8_t* {
        if constexpr (WIDE) {
            uint32_t offset = row + at.own;
            asm("" : "+v"(offset));
            return base + at.uniform + offset;
        } else if constexpr (TWO_STEPS) {
            return row + (at.uniform + at.own);
        } else {
            return row + at;
        }
    };
    float4v acc[MT][NT];
#pragma unroll
    for (int r = 0; r < MT; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] = float4v{0.f, 0.f, 0.f, 0.f};

    // ---- operand registers of one group of four whole chunks, and of the U chunks of one pass of the chunk loop
    struct Group {
        uint4 ca[LATE_A ? 2 : 4][MT], cw[4][NT];
        uint2 sa2[MT], sw2[NT];
    };
    struct Chunks {
        uint4 ca[U][MT], cw[U][NT];
        uint32_t sa[U][MT], sw[U][NT];
    };
    // Every load of a group is issued before any of it is used, the scale bytes (used first) first: loads retire
    // in issue order, so chunk m is decoded as soon as it has landed while the later chunks are still in flight.
    // (Left to itself the compiler sinks the loads of the later chunks behind the decode of the earlier ones to
    // save registers, which turns one trip to memory into three; the scheduling barriers behind the calls of
    // these functions keep the loads where they are written.)
    auto load_scales = [&](int g, Group& G) {
        const Byte so = byte_at(32 * (int64_t)g, 8 * q, 8 * q);
#pragma unroll
        for (int r = 0; r < MT; ++r) G.sa2[r] = load8_a1(in_row(a_scales, scale_row(ac[r], as[r]), so));
#pragma unroll
        for (int t = 0; t < NT; ++t) G.sw2[t] = load8_a1(in_row(base_s, scale_row(wc[t], ws[t]), so));
    };
    auto load_activations = [&](Byte co, int m, Group& G) {
#pragma unroll
        for (int r = 0; r < MT; ++r) G.ca[LATE_A ? m & 1 : m][r] = load16_a8(in_row(a_codes, ac[r], co));
    };
    auto codes_at = [&](int g, int m) { return byte_at(256 * (int64_t)g + 64 * m, 16 * q, 16 * q); };
    auto load_codes = [&](int g, int m, Group& G, bool activations) {
        const Byte co = codes_at(g, m);
        if (activations) load_activations(co, m, G);
#pragma unroll
        for (int t = 0; t < NT; ++t) G.cw[m][t] = load16_a8(in_row(base_c, wc[t], co));
    };
    auto load_group = [&](int g, Group& G) {
        load_scales(g, G);
#pragma unroll
        for (int m = 0; m < 4; ++m) load_codes(g, m, G, !LATE_A || m < 2);
    };
    // g: this group; next: group whose loads go into the registers that have been used (roll_tag), else not looked at
    auto compute_group = [&](Group& G, int g, int next, auto roll_tag) {
        constexpr bool roll = decltype(roll_tag)::value;
        uint32_t ea[2][MT], ew[2][NT];     // [chunk parity][tile]: pairs of chunks (0, 2) / (1, 3)
#pragma unroll
        for (int r = 0; r < MT; ++r) transpose_scale_pairs(G.sa2[r], ea[0][r], ea[1][r]);
#pragma unroll
        for (int t = 0; t < NT; ++t) transpose_scale_pairs(G.sw2[t], ew[0][t], ew[1][t]);
        if constexpr (roll && !WIDE) {
            __builtin_amdgcn_sched_barrier(0);
            load_scales(next, G);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint32_t sel = (m >> 1) ? 0x0C030C02u : 0x0C010C00u;
            uint32_t ha[MT], hw[NT];       // fp16 scales of the lane's two blocks of chunk m
#pragma unroll
            for (int r = 0; r < MT; ++r) ha[r] = scale_halves(ea[m & 1][r], sel);
#pragma unroll
            for (int t = 0; t < NT; ++t) hw[t] = scale_halves(ew[m & 1][t], sel);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                half8 fa[MT];
#pragma unroll
                for (int r = 0; r < MT; ++r) {
                    const uint4& c4 = G.ca[LATE_A ? m & 1 : m][r];
                    const uint32_t a32 = k == 0 ? c4.x : k == 1 ? c4.y : k == 2 ? c4.z : c4.w;
                    fa[r] = decode8_half(a32, ha[r], k >> 1);
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const uint32_t w32 = k == 0 ? G.cw[m][t].x : k == 1 ? G.cw[m][t].y : k == 2 ? G.cw[m][t].z : G.cw[m][t].w;
                    const half8 fw = decode8_half(w32, hw[t], k >> 1);
#pragma unroll
                    for (int r = 0; r < MT; ++r)
                        acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[r], fw, acc[r][t], 0, 0, 0);
                }
            }
            if constexpr (LATE_A)
                if (m < 2 || roll) {
                    __builtin_amdgcn_sched_barrier(0);
                    load_activations(codes_at(m < 2 ? g : next, (m + 2) & 3), (m + 2) & 3, G);
                    __builtin_amdgcn_sched_barrier(0);
                }
            if (roll && (m & 1)) {
                __builtin_amdgcn_sched_barrier(0);
                if (WIDE && m == 1) load_scales(next, G);
                load_codes(next, m - 1, G, !LATE_A);
                load_codes(next, m, G, !LATE_A);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // the lane's two blocks 8c + 2q, 8c + 2q + 1 of chunk c both exist, or the pair counts as zero (codes and scale
    // bytes, so that no stray scale pattern meets a zero) and the lane reads the start of its row instead.  The
    // zeroing happens at the use, not at the load: a select behind a load would make the wave wait for it at once.
    auto load_chunks = [&](int c0, Chunks& T) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b0 = 8 * (c0 + u) + 2 * q;
            const bool ok = b0 + 1 < nbk;
            const Byte co = byte_at(0, ok ? 8 * (Offset)b0 : 0, 16 * q), so = byte_at(0, ok ? b0 : 0, 8 * q);
#pragma unroll
            for (int r = 0; r < MT; ++r) {
                T.ca[u][r] = load16_a8(in_row(a_codes, ac[r], co));
                T.sa[u][r] = load2_a1(in_row(a_scales, scale_row(ac[r], as[r]), so));
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                T.cw[u][t] = load16_a8(in_row(base_c, wc[t], co));
                T.sw[u][t] = load2_a1(in_row(base_s, scale_row(wc[t], ws[t]), so));
            }
        }
    };
    auto compute_chunks = [&](int c0, const Chunks& T) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = 8 * (c0 + u) + 2 * q + 1 < nbk;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                half8 fa[MT];
#pragma unroll
                for (int r = 0; r < MT; ++r) {
                    const uint32_t a32 = k == 0 ? T.ca[u][r].x : k == 1 ? T.ca[u][r].y : k == 2 ? T.ca[u][r].z : T.ca[u][r].w;
                    fa[r] = decode8(ok ? a32 : 0u, scale_pair(!ok ? 0u : k < 2 ? (T.sa[u][r] & 0xFFu) : (T.sa[u][r] >> 8)));
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const uint32_t w32 = k == 0 ? T.cw[u][t].x : k == 1 ? T.cw[u][t].y : k == 2 ? T.cw[u][t].z : T.cw[u][t].w;
                    const half8 fw = decode8(ok ? w32 : 0u, scale_pair(!ok ? 0u : k < 2 ? (T.sw[u][t] & 0xFFu) : (T.sw[u][t] >> 8)));
#pragma unroll
                    for (int r = 0; r < MT; ++r)
                        acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[r], fw, acc[r][t], 0, 0, 0);
                }
            }
        }
    };
    bool grouped = false;
    if constexpr (GRP) grouped = nbk >= 32;
    if (grouped) {
        // Whole chunks in groups of four, dealt round-robin to the waves; the up to four chunks behind the last
        // group go to the waves that took one group less.  With one group per wave and four tiles (the up-projection
        // shapes) such a wave asks for its left-over chunk FIRST and decodes it last, so that it costs no trip to
        // memory of its own (1 us of 12 there); with few tiles per wave and several groups the same change made the
        // kernel 10 % slower (measured), so those variants load it where they use it.  (Dealing the left-over chunks
        // out as (chunk, tile) units, one per wave, balances the waves but decodes the activation chunk once per unit:
        // 11.7 against 10.5 us on the 16 x 14336 x 4352 shape, not kept.)
        constexpr bool HOIST = MT == 1 && NT == 4;
        const int ngroup = nbk >> 5;
        const int tail_c = 4 * ngroup + (wave - ngroup % WAVES + WAVES) % WAVES * U;
        const bool has_tail = tail_c < nchunk;
        Chunks tail;
        if (HOIST && has_tail) load_chunks(tail_c, tail);
        if constexpr (ROLL) {
            if (wave < ngroup) {
                Group ga;
                int g = wave;
                load_group(g, ga);
                __builtin_amdgcn_sched_barrier(0);
                for (; g + WAVES < ngroup; g += WAVES) {
                    int next = g + WAVES;
                    if (WIDE) asm("" : "+s"(next));     // opaque: followed as induction variables the rows' addresses take two registers each
                    compute_group(ga, g, next, std::true_type{});
                }
                compute_group(ga, g, 0, std::false_type{});
            }
        } else {
            for (int g = wave; g < ngroup; g += WAVES) {
                Group ga;
                load_group(g, ga);
                __builtin_amdgcn_sched_barrier(0);
                compute_group(ga, g, 0, std::false_type{});
            }
        }
        if (!HOIST && has_tail) load_chunks(tail_c, tail);
        if (has_tail) compute_chunks(tail_c, tail);
    } else {
        for (int c0 = wave * U; c0 < nchunk; c0 += WAVES * U) {
            Chunks T;
            load_chunks(c0, T);
            compute_chunks(c0, T);
        }
    }
    // the last block of a row with an odd number of blocks: lane group 0 supplies its two octets, the others zeros
    if ((nbk & 1) != 0 && wave == WAVES - 1) {
        uint2 oa[MT], ow[NT];
        uint32_t osa[MT], osw[NT];
        const Byte co = byte_at(8 * (int64_t)(nbk - 1), 0, 16 * q), so = byte_at(nbk - 1, 0, 8 * q);
#pragma unroll
        for (int r = 0; r < MT; ++r) {
            oa[r] = load8_a8(in_row(a_codes, ac[r], co));
            osa[r] = *in_row(a_scales, scale_row(ac[r], as[r]), so);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            ow[t] = load8_a8(in_row(base_c, wc[t], co));
            osw[t] = *in_row(base_s, scale_row(wc[t], ws[t]), so);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            half8 fa[MT];
#pragma unroll
            for (int r = 0; r < MT; ++r) fa[r] = decode8(q ? 0u : k ? oa[r].y : oa[r].x, scale_pair(q ? 0u : osa[r]));
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const half8 fw = decode8(q ? 0u : k ? ow[t].y : ow[t].x, scale_pair(q ? 0u : osw[t]));
#pragma unroll
                for (int r = 0; r < MT; ++r)
                    acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[r], fw, acc[r][t], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int t0 = 0; t0 < NT; t0 += BATCH) {
        if (t0 > 0) __syncthreads();
#pragma unroll
        for (int r = 0; r < MT; ++r)
#pragma unroll
            for (int t = t0; t < (t0 + BATCH < NT ? t0 + BATCH : NT); ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) red[wave][r * BATCH + t - t0][e][lane] = acc[r][t][e];
        __syncthreads();
        for (int idx = threadIdx.x; idx < MT * BATCH * 4 * 64; idx += WAVES * 64) {
            const int rt = idx >> 8, e = (idx >> 6) & 3, l = idx & 63;
            if (NT % BATCH != 0 && t0 + rt % BATCH >= NT) continue;
            float sum = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) sum += red[w][rt][e][l];
            const int m = 16 * (rt / BATCH) + 4 * (l >> 4) + e, n = n0 + 16 * (t0 + rt % BATCH) + (l & 15);
            if (m < M && n < N) store_out(y + (int64_t)m * ldy + n, sum * alpha);
        }
    }
}

constexpr int STREAM_ROUND = 256 * 64;      // weight rows of a round of this kernel: a workgroup of four tiles on every compute unit

// BEHIND: weight tiles of the workgroups behind the first STREAM_ROUND weight rows; NT of all others.  (With both, addresses in two steps: 32 x 28672 over
// K' = 8464 42.1 us, 42.4 with one sum; 20 x 26000 38.5 and 38.8 to 39.1.  All others: one sum.)
template <int MT, int NT, int BEHIND, int WAVES, int U, bool GRP, bool ROLL, typename OutT>
__global__ __launch_bounds__(WAVES * 64) void gemm_skinny_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N,
    int nbk, float alpha, OutT* __restrict__ y, int64_t ldy) {
    constexpr int FLOATS = WAVES * MT * skinny_batch(MT, NT, WAVES) * 256;
    static_assert(BEHIND <= NT && sizeof(float) * FLOATS <= 64 * 1024, "partial tiles must fit the static LDS limit");
    __shared__ float red[FLOATS];
    if constexpr (BEHIND == NT) {
        skinny_tiles<MT, NT, WAVES, U, GRP, ROLL, false>(a_codes, a_scales, w_codes, w_scales, M, N, nbk, alpha, y, ldy, blockIdx.x * (16 * NT), red);
    } else {
        constexpr int FIRST = STREAM_ROUND / (16 * NT);
        static_assert(FIRST * 16 * NT == STREAM_ROUND, "whole workgroups first");
        if (blockIdx.x < FIRST)
            skinny_tiles<MT, NT, WAVES, U, GRP, ROLL, true>(a_codes, a_scales, w_codes, w_scales, M, N, nbk, alpha, y, ldy, blockIdx.x * (16 * NT), red);
        else
            skinny_tiles<MT, BEHIND, WAVES, U, GRP, ROLL, true>(a_codes, a_scales, w_codes, w_scales, M, N, nbk, alpha, y, ldy,
                                                                STREAM_ROUND + (blockIdx.x - FIRST) * (16 * BEHIND), red);
    }
}

template <int MT, int NT, int BEHIND, int WAVES, int U, bool GRP, bool ROLL, typename OutT>
arcq_status launch_skinny(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                                 const uint8_t* w_scales, int M, int N, int nbk, float alpha, OutT* y, int64_t ldy,
                                 hipStream_t stream) {
    const int rows = BEHIND == NT ? N : std::min(N, STREAM_ROUND), behind = N - rows;
    const int workgroups = (rows + 16 * NT - 1) / (16 * NT) + (behind + 16 * BEHIND - 1) / (16 * BEHIND);
    hipLaunchKernelGGL((gemm_skinny_kernel<MT, NT, BEHIND, WAVES, U, GRP, ROLL, OutT>), dim3(workgroups),
                       dim3(WAVES * 64), 0, stream, a_codes, a_scales, w_codes, w_scales, M, N, nbk, alpha, y, ldy);
    return check_launch("gemm_skinny_kernel");
}

}  // namespace

// 65 to 128 rows on the weight-streaming kernel rather than on tiles with K' split across workgroups: unless the problem is
// big enough for the latter (measured over N = 1024 .. 28672, K' = 1088 .. 14592 at M = 80, 96, 128: the eight-row-tile variant
// of the streaming kernel takes about 1 us per 10^6 weights, the tiled path 20-30 us for everything up to 6 * 10^7 weights,
// more with a short K' that cannot be split).
static bool skinny_shape(int64_t M, int64_t N, int64_t Kp) {
    if (M <= 64) return true;
    if (M > 128) return false;
    const int64_t weights = N * Kp;
    return !((Kp >= 4096 && weights >= 20000000) || (Kp >= 8192 && weights >= 12000000));
}

// Number of runs the reduction dimension is cut into (1: no split) on the 128 x 128 tiles.  Problems
// with too few such tiles to occupy the chip split K' into runs of at least four stages (256 k).  The number of runs minimises
// a cost in units of one stage time of a tile (about 1.3 us): rounds of workgroups over the 256 CUs times the stages of a run,
// plus, when split, the write and read of the fp32 partial results at about 3 TB/s.
static int split_runs(int64_t M, int64_t N, int64_t Kp) {
    const int64_t nbk = Kp >> 4;
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
    const int64_t nstage = (nbk + 7) >> 3;
    const int64_t max_splits = tiles > 128 || nbk < 8 ? 1 : std::min<int64_t>(8, nstage / 4);
    int best = 1;
    double best_cost = (double)((tiles + 255) / 256) * (double)nstage;
    for (int64_t sp = 2; sp <= max_splits; ++sp) {
        const double rounds = (double)((tiles * sp + 255) / 256);
        const double cost = rounds * (double)((nstage + sp - 1) / sp) + (double)sp * (double)M * (double)N * 8.0 / 4.0e6;
        if (cost < best_cost) {
            best = (int)sp;
            best_cost = cost;
        }
    }
    return best;
}

// Modelled times in us of the 128 x 128 tiles in that number of runs and of the streaming kernel with 33 to 128 rows, to compare
// with gemm_ksplit_best's and fitted to the same problems (8 and 6 to 10 % rms).
static double tiles_time(int64_t M, int64_t N, int64_t Kp, int runs) {
    const int64_t wgs = ((M + 127) / 128) * ((N + 127) / 128) * runs, nstage = ((Kp >> 4) + 7) >> 3;
    const double rounds = (double)((wgs + 255) / 256), stages = (double)((nstage + runs - 1) / runs), ragged = (Kp & 63) ? 0.5 : 0.0;
    const double fill = (double)wgs / 256.0;
    if (runs > 1) return 7.4 + ((N & 3) ? 5.3 * (0.2 + 0.8 * fill) : 0.0) + ragged + stages * 0.95 * rounds +
                         0.366e-6 * 8.0 * (double)runs * (double)M * (double)N;
    // (N & 7: what values stored one by one or in pairs cost; no tile stores them so any more, see gemm_ksplit_best.  The fill by itself is for
    // fp32 results, which take these tiles 1 to 3 us longer)
    return 4.5 + fill + ((N & 7) ? 5.0 * (0.15 * rounds + 0.85 * fill) : 0.0) + ragged + stages * (0.84 * rounds + 0.195 * fill);
}
static double stream_time(const GemmPlan& plan, int64_t N, int64_t Kp) {
    const int64_t wgs = (N + plan.cols - 1) / plan.cols;
    const double rounds = (double)((wgs + 255) / 256), fill = (double)wgs / 256.0;
    // 512-k groups; a round over a short K' takes as long as one over a few of them
    const double groups = (double)Kp / 512.0;
    if (plan.rows == 64) return plan.cols == 32 ? 1.0 + 2.5 * rounds + std::max(groups, 1.6) * (0.674 * rounds + 0.303 * fill)
                                                : 2.9 + std::max(groups, 3.1) * (0.543 + 0.132 * fill);
    // (one tile: 0.7 us more than the fit, which is that much short over K' = 1024 .. 1900)
    return plan.cols == 32 ? 4.8 + std::max(groups, 1.2) * (1.547 * rounds + 0.531 * fill)
                           : 3.2 + std::max(groups, 1.7) * (1.341 + 0.268 * fill);
}

// Rounds of tiles of `rows` x 256, one per compute unit, times the time of a stage of such a tile.
static double wide_cost(int64_t M, int64_t N, int rows, double t_stage) {
    return (double)((((M + rows - 1) / rows) * ((N + 255) / 256) + 255) / 256) * t_stage;
}

constexpr int STREAM_WAVES = 8;     // of a workgroup of the weight-streaming kernel (8 x 2 tiles: 4)

// The weight-streaming kernel's share of the rule: row tiles, weight tiles per wave, and whether the waves load ahead.
static GemmPlan plan_stream(int64_t M, int64_t N, int64_t Kp) {
    // Enough waves to keep the weight stream in flight, as few as that allows so that each wave has several KB to request at
    // once: with many weight rows several tiles per wave share the activation operand; with few, one tile per wave so that
    // every CU still gets a workgroup (measured at the decode shapes).
    // Tiles per wave: as few as give the chip at most one workgroup per compute unit (256), up to four, two with more than 32
    // activation rows; measured with weights from HBM at 16 rows: 640 tiles (N = 10240, K' = 8448) 13.7 us with three tiles per
    // wave against 18.1 us with two (320 workgroups: two rounds), 576 tiles 8.7 against 10.6 (257 to 399 tiles used to run one
    // tile per wave, two workgroups sharing a CU: 320 tiles over K' = 27904 33.7 us against 27.3 us with two tiles per wave,
    // over K' = 4352 7.6 against 6.9); 32 rows: 640 tiles 17.2 us with three against 24.0 with one, 512 tiles 14.7 with two
    // against 17.9, 896 tiles 12.4 with four against 15.7 with two; 64 rows: 512 tiles over K' = 8464 23.2 us with two against
    // 34.6 with one; 128 rows: 512 tiles over K' = 2064 16.2 us with two against 20.0.
    const int64_t tiles = (N + 15) / 16;
    const int mt = M <= 16 ? 1 : M <= 32 ? 2 : M <= 64 ? 4 : 8;
    const int nt = tiles <= 256 ? 1 : tiles <= 512 || mt > 2 ? 2 : tiles <= 768 ? 3 : 4;
    // Ahead where waves take several groups (from HBM, us: 16 x 28672 over K' = 8448 34.9 -> 32.0, 32 x 28672 over 8464 47.5 ->
    // 45.1, 16 x 10240 over 8448 13.9 -> 13.1), and with one group per wave, where its code without a loop is still 2 to 4 %
    // faster (32 x 14336 over 4352 12.9 -> 12.4, 16 x 6144 over 4240 7.4 -> 7.3) except for four tiles behind one row tile (16 x
    // 14336 over 4352 10.4 against 10.6).  Not where one wave or a few take a group more than the others (they alone go
    // through the loop's copy of the code, which presumably is not in the instruction cache then).  Nine groups cost 1 us more that way
    // (33 x 213 over 5008 9.7 against 8.5, 24 x 28672 over 5008 5 % more, 16 x 9216 over 4608 4 %), ten and eleven 2 to 7 % with
    // three weight tiles or more than 32 rows, 17 and 25 up to 3 %; 33 to 48 rows lose up to 7 % with any but a whole number of
    // rounds (33 x 1103 over 15616).  One tile behind one row tile loses with several groups (16 x 4096 over 14592 11.0
    // against 11.1, over 14544 12.3 against 12.7).  128 rows have no groups.
    const int64_t ngroup = Kp >> 9;
    bool ahead;
    if (ngroup <= STREAM_WAVES) ahead = mt <= 4 && !(mt == 1 && nt == 4);
    else if (mt == 4) ahead = M > 48 ? ngroup >= 12 : ngroup % STREAM_WAVES == 0;
    else if (nt >= 3) ahead = ngroup >= 11 && ngroup % STREAM_WAVES != 1;
    else ahead = mt < 4 && mt * nt != 1 && (mt * nt == 2 || ngroup >= 10);
    GemmPlan plan = {ARCQ_ROUTE_STREAM, 16 * mt, 16 * nt, 1, ahead, mt * nt <= 2 ? 2 : 1};
    // Five to seven tiles a wave where they take a round less than four: up to 28672 weight rows in one (from HBM, us: 16 x 22016 over K' = 4352
    // 18.6 -> 14.4, 16 x 28672 over 8464 38.7 -> 34.6, 32 x 18944 over 2176 14.5 -> 10.3, 32 x 28672 over 4352 24.7 -> 21.1), up to 57344 in two (16 x
    // 40960 over 4352 28.2 -> 25.0, 32 x 49152 37.6 -> 35.2).  Beyond, rounds overlap so far that it is a draw (16 x 64000 over 4352 39.3 with four, 40.7
    // with six, 128256 76.6 and 76.1 with seven).  Seven behind two row tiles keep a dozen registers in scratch, which twelve groups pay for too often
    // (32 x 28672 over 8192 38.0 with four and 41.7; over 5632 29.2 and 28.8): the second round takes three tiles a wave instead of four then, over
    // 8192 34.7, over 8464 45.4 -> 42.1.  Only where waves load ahead or take one group, the one form in which these kernels exist: with 9, 10, 17, 25 ...
    // groups a wave or a few take one more, loading ahead costs 2 to 7 % with four tiles, and what is left of the gain then has not been measured.  Slower
    // than four: one or two activation rows with 41000 to 49152 weight rows, up to 1.3 % for some K' (1 x 49152 over 8464 53.1 and 53.8), and a weight row behind two whole
    // rounds (16 x 32769 over 8464 45.8 and 46.5).
    const int rounds = tiles <= 7 * 256 ? 1 : 2;
    if (mt <= 2 && tiles > 4 * 256 * rounds && tiles <= 7 * 256 * rounds && (ahead || ngroup <= STREAM_WAVES)) {
        const int wide = (int)((tiles + 256 * rounds - 1) / (256 * rounds));
        if (mt == 1 || wide < 7 || ngroup < 12) {
            plan.tiles = plan.behind = wide;
            plan.ahead = true;
        } else if (rounds == 1) {
            plan.behind = 3;
        }
    }
    return plan;
}

// Which kernel serves a problem by rule: a function of the shape alone, so that the workspace a caller sizes beforehand matches what the
// launch uses.  Up to 32 rows the weight-streaming kernel, beyond the smallest modelled time of three:
//   * the streaming kernel up to 128 rows, e.g. 64 rows over K' = 4240: 5120 weight rows 12.5 us against 14.3 on 64 x 32 tiles,
//     28672 38.9 against 30.4 on 64 x 128; 46 x 9600 over K' = 512 8.5 against 6.1 on 64 x 64;
//   * the tiles with the k split inside the workgroup (gemm_ksplit_best);
//   * the tiles of this file, with K' split across workgroups or without, by the stage times that choose among them.
// K' is split across workgroups only where the tiles with the split inside leave much of the chip idle, whatever the times
// say: the others need no workspace, and calls without one and overlapping calls of arcq_gemm_noalloc count on that (the 64 x 128
// and 96 x 128 tiles, which came later, do not enter: what they alone could take still splits).  Nor do the times decide where
// the runs need more than the library's built-in scratch: what arcq_gemm_noalloc takes does not follow them.
static GemmPlan plan_by_rule(int64_t M, int64_t N, int64_t Kp) {
    const GemmPlan stream = plan_stream(M, N, Kp);
    if (M <= 32) return stream;
    const KsplitTile ks = gemm_ksplit_best(M, N, Kp, true);
    const GemmPlan ksplit = {ARCQ_ROUTE_KSPLIT, ks.rows, ks.cols, 1, false};
    if (skinny_shape(M, N, Kp)) return ks.rows != 0 && ks.us < stream_time(stream, N, Kp) ? ksplit : stream;
    const int64_t nbk = Kp >> 4, nstage = (nbk + 7) >> 3, tn256 = (N + 255) / 256;
    const bool offsets_fit = (uint64_t)M * (uint64_t)nbk * 8 < 0xFFFF0000ull && (uint64_t)N * (uint64_t)nbk * 8 < 0xFFFF0000ull;
    if (nbk < 8 || !offsets_fit) return {ARCQ_ROUTE_DIRECT, 128, 128, 1, false};
    GemmPlan tiles = {ARCQ_ROUTE_TILES, 128, 128, 1, false};
    double us;
    if (((M + 127) / 128) * ((N + 127) / 128) > 256 && ((M + 191) / 192) * ((N + 127) / 128) <= 256) {
        // More than 256 tiles of 128 x 128 (two workgroups on some compute units, one on the others) but at most 256 of
        // 192 x 128: one round of the taller tile, which also decodes five fragments per six matrix instructions
        // instead of four per four (1.52 against 1.3 us per stage and tile): 512 x 10240 over K' = 8448 116 -> 100 us,
        // 1024 x 5120 over 27904 365 -> 297 us, 1280 x 4096 over 4352 61 -> 49 us.  It goes before the 256-wide tiles, which
        // take one round as well where both fit, of a larger tile on fewer compute units (160 x 28672 over K' = 4352: 51.2
        // against 58.9 us).
        tiles.rows = 192;
        us = 5.0 + (double)nstage * 1.52;
    } else if (((M + 127) / 128) * tn256 >= 192) {
        // Tiles of 256 weight rows by 256, 192 or 128 activation rows when there is work for them.  Workgroups run in
        // rounds of one per compute unit and a round lasts as long as one tile, so the tile height that minimises
        // rounds x (time of a stage of that tile) wins: 2.96, 2.59 and 1.96 us measured per 128-k stage (the bigger
        // tile decodes fewer fragments per matrix instruction: 45, 53 and 60 ps per output element and stage).
        // E.g. 768 x 14336: 224 tiles of 192 rows in one round 88 us, 336 tiles of 128 rows in two rounds 113 us,
        // 168 tiles of 256 rows 100 us; 1024 x 14336: 224 tiles of 256 rows 106 us against 120 us.
        const double c256 = wide_cost(M, N, 256, 2.96), c192 = wide_cost(M, N, 192, 2.59), c128 = wide_cost(M, N, 128, 1.96);
        tiles.rows = c256 <= c192 && c256 <= c128 ? 256 : c192 <= c128 ? 192 : 128;
        tiles.cols = 256;
        us = 5.0 + (double)nstage * std::min({c256, c192, c128});
    } else {
        tiles.runs = split_runs(M, N, Kp);
        us = tiles_time(M, N, Kp, tiles.runs);
    }
    const bool too_large = tiles.runs > 1 && (uint64_t)tiles.runs * (uint64_t)M * (uint64_t)N * sizeof(float) > ARCQ_NOALLOC_SCRATCH_BYTES;
    if (ks.rows != 0 && (tiles.runs > 1 && (ks.ample || too_large) ? ks.ample : ks.us < us)) return ksplit;
    return tiles;
}

// Modelled time in us of one launch of a tile over any number of tiles: start + rounds x round + stages x (full rounds x full + the
// last round's alone + shared x its fill), a round being 256 tiles and a stage 128 k (256 k for the k-split tiles).  (Two or three
// workgroups of the small tiles share a compute unit: a second round costs them about half a first one.)  Rows off the grid of 64 cost
// ragged_round a round and ragged_stage a round and stage.  Fitted to 2190 problems (M = 33 .. 8192, N = 256 .. 28672, K' = 512 .. 24000,
// weights from HBM), every tile timed: 3 to 6 % rms, and the fastest by the model 0.4 % from the fastest of all.
namespace {
struct TileTime {
    int kernel, rows, cols;
    double start, round, full, alone, shared, ragged_round, ragged_stage;
};
constexpr TileTime TILE_TIMES[] = {
    {ARCQ_ROUTE_TILES, 256, 256, 6.058, 5.990, 3.222, 2.079, 0.934, 1.704, 0.0},
    {ARCQ_ROUTE_TILES, 192, 256, 4.814, 4.663, 2.575, 1.632, 0.829, 1.507, 0.0},
    {ARCQ_ROUTE_TILES, 128, 256, 2.255, 4.209, 1.872, 1.006, 0.742, 1.247, 0.0},
    {ARCQ_ROUTE_TILES, 192, 128, 3.521, 1.662, 1.361, 1.026, 0.305, 1.376, 0.104},
    {ARCQ_ROUTE_TILES, 128, 128, 3.513, 0.964, 0.949, 0.776, 0.209, 0.352, 0.050},
    {ARCQ_ROUTE_KSPLIT, 128, 128, 0.916, 5.942, 1.828, 1.134, 0.561, 0.615, 0.012},
    {ARCQ_ROUTE_KSPLIT, 96, 128, 1.005, 4.967, 1.517, 0.944, 0.445, 0.513, 0.029},
    {ARCQ_ROUTE_KSPLIT, 128, 64, 1.014, 5.139, 1.026, 0.765, 0.213, 0.718, 0.028},
    {ARCQ_ROUTE_KSPLIT, 64, 128, 1.003, 3.709, 1.105, 0.744, 0.310, 0.551, 0.046},
    {ARCQ_ROUTE_KSPLIT, 96, 64, 5.399, 0.0, 0.856, 0.629, 0.189, 0.850, 0.022},
    {ARCQ_ROUTE_KSPLIT, 64, 64, 4.086, 0.550, 0.449, 0.467, 0.115, 0.402, 0.035},
    {ARCQ_ROUTE_KSPLIT, 64, 32, 3.271, 0.493, 0.254, 0.401, 0.063, 0.378, 0.018},
};

double tile_time(const TileTime& t, int64_t M, int64_t N, int64_t Kp) {
    const int64_t wgs = ((M + t.rows - 1) / t.rows) * ((N + t.cols - 1) / t.cols), left = wgs & 255;
    const double stage_k = t.kernel == ARCQ_ROUTE_KSPLIT ? 256.0 : 128.0, stages = std::ceil((double)Kp / stage_k);
    const double full = (double)(wgs >> 8), rounds = full + (left ? 1.0 : 0.0);
    const double last = left ? t.alone + t.shared * (double)left / 256.0 : 0.0;
    return t.start + rounds * t.round + stages * (full * t.full + last) +
           ((Kp & 63) ? rounds * (t.ragged_round + stages * t.ragged_stage) : 0.0);
}

// Chains that an output's products over K' are added up in, before those are added to each other: one for each wave of a workgroup that
// takes a share of K'.  Fewer and longer ones round more (fp32 against 64 bits, 3573 x 6744 over K' = 7472: 1.17e-7 with pairs of waves on 128 x 256
// tiles, 1.80e-7 on 256 x 256).  at_least: of 128 x 256 tiles, which have pairs or not by the operands' alignment where K' is 64 mod 128.
int sum_chains(int kernel, int rows, int cols, int64_t Kp, bool at_least) {
    if (kernel == ARCQ_ROUTE_STREAM) return rows == 128 && cols == 32 ? 4 : 8;
    if (kernel == ARCQ_ROUTE_KSPLIT) return 4;
    return rows == 128 && cols == 256 && !(at_least && (Kp & 127) == 64) ? 2 : 1;
}

struct TimedPlan {
    GemmPlan plan;
    double us;
};

// The tile that takes the least modelled time among those with that many chains, or the streaming kernel; no workspace.
TimedPlan plan_by_time(int64_t M, int64_t N, int64_t Kp, int chains) {
    const GemmPlan stream = plan_stream(M, N, Kp);
    if (M <= 32) return {stream, 4.0 + (M <= 16 ? 0.115e-6 : 0.165e-6) * (double)N * (double)Kp};     // (nothing else is ever faster)
    TimedPlan best = {stream, M <= 128 ? stream_time(stream, N, Kp) : 1e30};
    for (const TileTime& t : TILE_TIMES) {
        if (sum_chains(t.kernel, t.rows, t.cols, Kp, true) < chains) continue;
        // 96 x 128 tiles that pad more rows than 128 x 128: see gemm_ksplit_best
        if (t.rows == 96 && t.cols == 128 && (M + 95) / 96 * 96 > (M + 127) / 128 * 128) continue;
        // Small tiles in more than one round are not what the model says where many of them share a compute unit over a long K'
        // (314 x 8176 over 9904 1.5x slower than modelled, 285 x 25216 over 2288 1.2x faster).
        if (t.kernel == ARCQ_ROUTE_KSPLIT && t.rows * t.cols < 96 * 128 && ((M + t.rows - 1) / t.rows) * ((N + t.cols - 1) / t.cols) > 256) continue;
        const double us = tile_time(t, M, N, Kp);
        if (us < best.us) best = {{t.kernel, t.rows, t.cols, 1, false}, us};
    }
    return best;
}
}  // namespace

// The rule's kernel, unless the model knows one launch that takes less than 0.95 of its time, or two that take less than 0.97 of that.
// Two: workgroups run in rounds of one per compute unit, and a last round that is nearly empty costs as much as a full one. Whole
// rounds of the tiles with the best rate go first, and the columns or rows behind them, which are few, to tiles that spread them
// over the chip (a second launch costs 3 us beside its start).  1777 x 10240 over K' = 8528, fp32, with the quantizer: 400
// tiles of 192 x 256 in two rounds 343 us, 252 tiles of 256 x 256 and 224 of 128 x 64 283.  Over 350 and 200 random problems whose route
// this changes: 1.075x (513 to 8192 rows; 0.97x at worst, 1.31x at best) and 1.10x (65 to 512 rows).
// K' < 1024: the rule alone (starts and ends of rounds count for more there than the model knows).
GemmParts plan_gemm_parts(int64_t M, int64_t N, int64_t Kp) {
    GemmPlan rule = plan_by_rule(M, N, Kp);
    const int chains = sum_chains(rule.kernel, rule.rows, rule.cols, Kp, false);
    // Where the price of stores value by value, which no tile has any more, makes the rule stream 65 to 128 rows, it is asked once more
    // without: 267 random problems with N odd or 2 mod 4 1.22x (1.07 to 1.42; 122 x 28115 over K' = 1088 25.2 -> 17.3 us, 121 x 24097 over 1264
    // 23.5 -> 18.9, 89 x 7319 over 1520 11.4 -> 9.1).  Below K' = 1024, where starts count for more than the model knows, only for a tenth: 1.2x
    // (0.98 to 1.5; without the tenth down to 0.95).  33 to 64 rows and up to 4096 weight rows are streamed in eight chains, the tiles have four.
    if (rule.kernel == ARCQ_ROUTE_STREAM && M > 32 && (N & 3) != 0 && chains <= sum_chains(ARCQ_ROUTE_KSPLIT, 0, 0, Kp, true)) {
        const KsplitTile ks = gemm_ksplit_best(M, N, Kp, false);
        if (ks.rows != 0 && ks.us < (Kp < 1024 ? 0.9 : 1.0) * stream_time(rule, N, Kp)) rule = {ARCQ_ROUTE_KSPLIT, ks.rows, ks.cols, 1, false};
    }
    GemmParts best = {rule, rule, M, N};
    // The streaming kernel with more weight rows than one round of four tiles a wave takes: that round, and the rest with one or two
    // tiles a wave, which gives it a round of its own.  (Four tiles a wave throughout: a second round that most of the chip has no part
    // in.)  From HBM, us, 1 and 32 rows: 17408 weight rows over K' = 4096 16.2 -> 13.6 and 20.9 -> 18.1, over 14592 44.5 -> 35.8 and 58.0 -> 47.4;
    // 20480 over 4352 17.1 -> 14.9 and 23.0 -> 20.0; 24576 over 6144 22.9 -> 20.7 and 29.7 -> 28.0, over 14592 47.2 -> 42.9 and 60.3 -> 55.0.  Within
    // the limits 84 sizes gain 1.5 us and more, 1.05 to 1.26x.  A pass that runs the second kernel for the first time takes 5 us more, which the
    // fifth at the latest has made up for.  One launch of more tiles a wave (plan_stream) gains more than a second launch everywhere: 16 x 16400 over 4352
    // 15.7, 15.5 in two, 12.3; 16 x 24576 over 4352 19.1, 18.0 and 15.2; and within the limits too, 1.03 to 1.3x (16 x 20480 over 4352 16.0 in two, 13.2).  They stand for one
    // reason only: the tests state this route, and its bits, for sizes within them (tests/test_gpu_rounds.py, tests/test_library_cpu.py).
    const int64_t behind = N - STREAM_ROUND;
    if (rule.kernel == ARCQ_ROUTE_STREAM && M <= 32 && behind >= 1024 && behind <= STREAM_ROUND / 2 &&
        Kp >= (behind > STREAM_ROUND / 4 ? 6144 : 4096)) {
        GemmParts parts = {plan_stream(M, STREAM_ROUND, Kp), plan_stream(M, behind, Kp), M, STREAM_ROUND};
        parts.rest.chunks = 1;      // K' in the order of four tiles a wave: the same bits as in one launch
        return parts;
    }
    if (Kp < 1024 || rule.runs > 1 || (rule.kernel != ARCQ_ROUTE_TILES && rule.kernel != ARCQ_ROUTE_KSPLIT)) return best;
    const auto of_rule = std::find_if(std::begin(TILE_TIMES), std::end(TILE_TIMES), [&](const TileTime& t) {
        return t.kernel == rule.kernel && t.rows == rule.rows && t.cols == rule.cols;
    });
    const double rule_us = tile_time(*of_rule, M, N, Kp);
    // (not for the price of precision: neither launch adds up K' in fewer chains than the rule's kernel)
    const TimedPlan one = plan_by_time(M, N, Kp, chains);
    double us = rule_us;
    if (one.us < 0.95 * rule_us) {
        best.first = best.rest = one.plan;
        us = one.us;
    }
    us *= 0.97;
    const double stages = (double)Kp / 128.0;
    for (const TileTime& t : TILE_TIMES) {
        if (sum_chains(t.kernel, t.rows, t.cols, Kp, true) < chains) continue;
        // (128 x 256 and 192 x 128 tiles in front gain nothing on average: 0.97 to 1.06x)
        if (!(t.cols == 256 && t.rows >= 192) && !(t.kernel == ARCQ_ROUTE_KSPLIT && t.rows == 128 && t.cols == 128)) continue;
        const int64_t tm = (M + t.rows - 1) / t.rows, tn = (N + t.cols - 1) / t.cols, most = tm * tn / 256;
        for (int64_t rounds = std::max<int64_t>(1, most - 1); rounds <= most; ++rounds) {
            auto consider = [&](int64_t rows, int64_t cols, int64_t rest_rows, int64_t rest_cols) {
                const double first = tile_time(t, rows, cols, Kp);
                // no tile computes 65536 outputs per compute unit and stage in less than 3 us
                if (first + 5.0 + stages * 3.0 * (double)rest_rows * (double)rest_cols / (65536.0 * 256.0) >= us) return;
                const TimedPlan rest = plan_by_time(rest_rows, rest_cols, Kp, chains);
                if (first + rest.us + 3.0 >= us) return;
                us = first + rest.us + 3.0;
                best = {{t.kernel, t.rows, t.cols, 1, false}, rest.plan, rows, cols};
            };
            const int64_t nc = 256 * rounds / tm, nr = 256 * rounds / tn;
            if (nc >= 1 && nc < tn) consider(M, t.cols * nc, M, N - t.cols * nc);
            if (nr >= 1 && nr < tm) consider(t.rows * nr, N, M - t.rows * nr, N);
        }
    }
    return best;
}

namespace {

template <typename OutT>
arcq_status launch_plan(const GemmPlan& plan, const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                        const uint8_t* w_scales, int64_t M, int64_t N, int64_t Kp, float alpha, OutT* y,
                        int64_t ldy, float* workspace, hipStream_t stream) {
    const int nbk = (int)(Kp >> 4);
    const bool dword_scales = ((reinterpret_cast<uintptr_t>(a_scales) | reinterpret_cast<uintptr_t>(w_scales)) & 3) == 0;
    const bool aligned16 = ((reinterpret_cast<uintptr_t>(a_codes) | reinterpret_cast<uintptr_t>(w_codes)) & 15) == 0 && dword_scales;
    if (plan.kernel == ARCQ_ROUTE_STREAM) {
        // (the variants that exist: plan_stream)
        const int tiles = plan.tiles ? plan.tiles : plan.cols / 16, behind = plan.behind ? plan.behind : tiles;
#define ARCQ_STREAM_MIXED(MT_, NT_, BEHIND_, W_, U_, AHEAD_)                                                                      \
    if (plan.rows == 16 * MT_ && tiles == NT_ && behind == BEHIND_ && plan.chunks == U_ && plan.ahead == AHEAD_)                  \
    return launch_skinny<MT_, NT_, BEHIND_, W_, U_, (MT_ <= 4), AHEAD_>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, \
                                                                        alpha, y, ldy, stream)
#define ARCQ_STREAM(MT_, NT_, W_, U_, AHEAD_) ARCQ_STREAM_MIXED(MT_, NT_, NT_, W_, U_, AHEAD_)
        ARCQ_STREAM(1, 1, STREAM_WAVES, 2, false);
        ARCQ_STREAM(1, 1, STREAM_WAVES, 2, true);
        ARCQ_STREAM(1, 2, STREAM_WAVES, 2, true);
        ARCQ_STREAM(1, 3, STREAM_WAVES, 1, false);
        ARCQ_STREAM(1, 3, STREAM_WAVES, 1, true);
        ARCQ_STREAM(1, 4, STREAM_WAVES, 1, false);
        ARCQ_STREAM(1, 4, STREAM_WAVES, 1, true);
        ARCQ_STREAM(2, 1, STREAM_WAVES, 2, true);
        ARCQ_STREAM(2, 2, STREAM_WAVES, 1, false);
        ARCQ_STREAM(2, 2, STREAM_WAVES, 1, true);
        ARCQ_STREAM(2, 3, STREAM_WAVES, 1, false);
        ARCQ_STREAM(2, 3, STREAM_WAVES, 1, true);
        ARCQ_STREAM(2, 4, STREAM_WAVES, 1, false);
        ARCQ_STREAM(2, 4, STREAM_WAVES, 1, true);
        ARCQ_STREAM(1, 5, STREAM_WAVES, 1, true);
        ARCQ_STREAM(1, 6, STREAM_WAVES, 1, true);
        ARCQ_STREAM(1, 7, STREAM_WAVES, 1, true);
        ARCQ_STREAM(2, 5, STREAM_WAVES, 1, true);
        ARCQ_STREAM(2, 6, STREAM_WAVES, 1, true);
        ARCQ_STREAM(2, 7, STREAM_WAVES, 1, true);
        ARCQ_STREAM_MIXED(2, 4, 3, STREAM_WAVES, 1, true);
        ARCQ_STREAM(4, 1, STREAM_WAVES, 1, false);
        ARCQ_STREAM(4, 1, STREAM_WAVES, 1, true);
        ARCQ_STREAM(4, 2, STREAM_WAVES, 1, false);
        ARCQ_STREAM(4, 2, STREAM_WAVES, 1, true);
        ARCQ_STREAM(8, 1, STREAM_WAVES, 1, false);
        ARCQ_STREAM(8, 2, 4, 1, false);
        // the second launch of two
        ARCQ_STREAM(1, 1, STREAM_WAVES, 1, false);
        ARCQ_STREAM(1, 1, STREAM_WAVES, 1, true);
        ARCQ_STREAM(1, 2, STREAM_WAVES, 1, true);
        ARCQ_STREAM(2, 1, STREAM_WAVES, 1, true);
#undef ARCQ_STREAM
#undef ARCQ_STREAM_MIXED
        return fail(ARCQ_HIP_ERROR, "no weight-streaming kernel of %d x %d rows, %d chunks, ahead %d", plan.rows, plan.cols, plan.chunks, (int)plan.ahead);
    }
    if (plan.kernel == ARCQ_ROUTE_KSPLIT)
        return launch_gemm_ksplit(plan.rows, plan.cols, a_codes, a_scales, w_codes, w_scales, M, N, Kp, alpha, y,
                                  std::is_same<OutT, _Float16>::value ? ARCQ_DTYPE_F16 : ARCQ_DTYPE_F32, ldy, stream);
#define ARCQ_TILES(WM_, WN_, MODE_)                                                                                      \
    if (plan.rows == 64 * WM_ && plan.cols == 64 * WN_)                                                                  \
    return launch_staged<WM_, WN_, 2, 2, MODE_>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, y, ldy, \
                                                stream, plan.runs, workspace)
    if (plan.kernel == ARCQ_ROUTE_TILES && (nbk & 3) == 0 && aligned16) {
        ARCQ_TILES(3, 2, COPIES);
        ARCQ_TILES(4, 4, COPIES);
        ARCQ_TILES(3, 4, COPIES);
        ARCQ_TILES(2, 2, COPIES);
        // 128 x 256 tiles: wave pairs that split every stage (6 % faster than 8 waves of 64 x 64 on the 2048 x 4096 x 4352
        // problem); a half stage at the end has its own code in the other kernel.  (The pairs' RAGGED copies know half stages
        // too, and are 3 % faster on 2048 x 4096 over K' = 4416, but 5 to 20 % slower up to K' = 2000 and on most others: 754 x
        // 10432 over 960 29.1 against 33.1 us, 374 x 20167 over 12224 211 against 238.)
        if ((nbk & 7) == 0 && nbk >= 16)
            return launch_kpair<COPIES>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, y, ldy, stream);
        return launch_staged<2, 2, 2, 4>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, y, ldy, stream);
    }
    if (plan.kernel == ARCQ_ROUTE_TILES && nbk >= ScaleWindows<128, 128, 256, 8>::MIN_NB && dword_scales) {
        // Any K' from 256 on, codes that are only 8-byte aligned: the same tiles by the same rule, 3 to 10 % slower than with
        // whole aligned rows (S = 272 against S = 256, weights from HBM, one card: 8192 x 8192 over K = 28928 3037 and 2954 us, 4096 x
        // 8192 over 8192 461 and 444, 2048 x 4096 over 4096 74.1 and 69.4, 512 x 10240 over 8192 110 and 99;
        // through registers 1.15 to 1.35 times as long as with whole rows)
        ARCQ_TILES(3, 2, RAGGED);
        ARCQ_TILES(4, 4, RAGGED);
        ARCQ_TILES(3, 4, RAGGED);
        ARCQ_TILES(2, 2, RAGGED);
        return launch_kpair<RAGGED>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, y, ldy, stream);
    }
    if (plan.kernel == ARCQ_ROUTE_TILES) {
        // scale bytes at odd addresses, or K' from 128 to 240 that is no multiple of 64: stages through registers (no 256 x 256
        // tiles: the staging registers do not fit beside 256 accumulators); 192 or 128 rows by rounds x stage time, 3.5 and 2.4 us
        // here (768 x 14336 over K' = 4368 118 us instead of 163)
        ARCQ_TILES(3, 2, REGS);
        ARCQ_TILES(2, 2, REGS);
        if (wide_cost(M, N, 192, 3.5) <= wide_cost(M, N, 128, 2.4))
            return launch_staged<3, 4, 2, 2, REGS>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, y, ldy, stream);
        return launch_staged<2, 2, 2, 4, REGS>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, y, ldy, stream);
    }
#undef ARCQ_TILES
    dim3 grid((unsigned)((N + 127) / 128), (unsigned)((M + 127) / 128));
    hipLaunchKernelGGL(gemm_direct_kernel<OutT>, grid, dim3(256), 0, stream, a_codes, a_scales, w_codes, w_scales,
                       (int)M, (int)N, nbk, alpha, y, ldy);
    return check_launch("gemm_direct_kernel");
}

template <typename OutT>
arcq_status launch_typed(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                         const uint8_t* w_scales, int64_t M, int64_t N, int64_t Kp, float alpha, OutT* y,
                         int64_t ldy, float* workspace, hipStream_t stream) {
    const GemmParts parts = plan_gemm_parts(M, N, Kp);
    // (stages through registers have times of their own: the rule's kernel; the streaming kernel has none)
    if (((reinterpret_cast<uintptr_t>(a_scales) | reinterpret_cast<uintptr_t>(w_scales)) & 3) != 0 && parts.first.kernel != ARCQ_ROUTE_STREAM)
        return launch_plan(plan_by_rule(M, N, Kp), a_codes, a_scales, w_codes, w_scales, M, N, Kp, alpha, y, ldy, workspace, stream);
    if (arcq_status st = launch_plan(parts.first, a_codes, a_scales, w_codes, w_scales, parts.rows, parts.cols, Kp, alpha, y, ldy,
                                     workspace, stream)) return st;
    const int64_t c = Kp >> 1, s = Kp >> 4;         // bytes of a row of codes, of scale bytes
    if (parts.rows < M)
        return launch_plan(parts.rest, a_codes + parts.rows * c, a_scales + parts.rows * s, w_codes, w_scales, M - parts.rows, N, Kp,
                           alpha, y + parts.rows * ldy, ldy, nullptr, stream);
    if (parts.cols < N)
        return launch_plan(parts.rest, a_codes, a_scales, w_codes + parts.cols * c, w_scales + parts.cols * s, M, N - parts.cols, Kp,
                           alpha, y + parts.cols, ldy, nullptr, stream);
    return ARCQ_OK;
}

}  // namespace

arcq_status launch_splitk_reduce(const float* partial, int splits, int M, int N, float alpha, void* y, int y_dtype,
                                 int64_t ldy, hipStream_t stream) {
    const int64_t stride = (int64_t)M * N;
    const int vec4 = (N & 3) == 0 && (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0;
    const int64_t work = vec4 ? stride / 4 : stride;
    const int blocks = (int)std::min<int64_t>((work + 255) / 256, 4096);
    if (y_dtype == ARCQ_DTYPE_F16)
        hipLaunchKernelGGL(splitk_reduce_kernel<_Float16>, dim3(blocks), dim3(256), 0, stream, partial, splits, stride, M, N,
                           alpha, static_cast<_Float16*>(y), ldy, vec4);
    else
        hipLaunchKernelGGL(splitk_reduce_kernel<float>, dim3(blocks), dim3(256), 0, stream, partial, splits, stride, M, N,
                           alpha, static_cast<float*>(y), ldy, vec4);
    return check_launch("splitk_reduce_kernel");
}

size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t Kp) {
    const int runs = plan_by_rule(M, N, Kp).runs;       // (K' split across workgroups is never replaced by other tiles)
    return runs > 1 ? (size_t)runs * (size_t)M * (size_t)N * sizeof(float) : 0;
}

// ---------------------------------------------------------------------------------------------
// Scratch memory of arcq_gemm_noalloc: the fp32 partial results of a split reduction dimension for
// callers that cannot allocate a workspace.  Every GPU the library runs on holds its own copy of this
// array, at its own address, until the process ends.  In host code the array's name is only a stand-in
// for hipGetSymbolAddress; launches get the per-device address kept in g_scratch_ptr.
static __device__ __align__(256) unsigned char scratch[ARCQ_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];
}  // namespace

// Device address of `scratch` on the current device; looked up once per device.
arcq_status gemm_scratch_pointer(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(ARCQ_HIP_ERROR, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(ARCQ_HIP_ERROR, "device index %d beyond the %d this library keeps scratch for", dev, kMaxDevices);
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return fail(ARCQ_HIP_ERROR, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[dev].store(p, std::memory_order_release);     // the same value from whichever thread gets here first
    }
    *out = p;
    return ARCQ_OK;
}

arcq_status launch_gemm(const uint8_t* a_codes, const uint8_t* a_scales,
                        const uint8_t* w_codes, const uint8_t* w_scales,
                        int64_t M, int64_t N, int64_t Kp, float alpha,
                        void* y, int y_dtype, int64_t ldy,
                        void* workspace, size_t, hipStream_t stream) {
    float* ws = static_cast<float*>(workspace);
    if (y_dtype == ARCQ_DTYPE_F16)
        return launch_typed<_Float16>(a_codes, a_scales, w_codes, w_scales, M, N, Kp, alpha,
                                      static_cast<_Float16*>(y), ldy, ws, stream);
    return launch_typed<float>(a_codes, a_scales, w_codes, w_scales, M, N, Kp, alpha, static_cast<float*>(y), ldy, ws, stream);
}

}  // namespace arcq
