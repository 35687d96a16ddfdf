// GEMM over K' = K + S for MXFP4 operands (Section 3.2 "Unified GEMM Execution", eq. (2), in the MXFP4
// variant of the format): y[m,n] = sum_b 2^(sa[m,b]-127) 2^(sw[n,b]-127) sum_{i<32} qa[m,32b+i] qw[n,32b+i].
//
// This is the format gfx950 multiplies natively: v_mfma_scale_f32_32x32x64_f8f6f4 takes 32 E2M1 values
// per lane and operand (one 16-byte register quad = exactly one MX block of one row) plus one E8M0
// scale byte per lane and operand; a lane holds row (lane % 32) and the k range 32 (lane / 32) .. + 31
// of the 64-k step (checked on the GPU with random codes and scales against this formula).  Products
// of E2M1 values and powers of two are exact; the only rounding is the fp32 accumulation.
// No decode: packed operands go global -> LDS -> registers -> matrix core unchanged.
#include "gemm_epilogue.h"
#include "internal.h"
#include "code_rows.h"
#include "gemm_decode.h"
#include "lds_dma.h"
#include "scale_chunks.h"
#include "tile_order.h"

#include <type_traits>

namespace arcq {

namespace {

typedef int int8v __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float16v mfma_mx(const uint4& a, const uint4& b, const float16v& c, int sa, int sb, int t) {
    const int8v va = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    const int8v vb = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
    // cbsz = blgp = 4: both operands FP4; the scale of a lane is byte 2t of its scale register
    return t == 0 ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va, vb, c, 4, 4, 0, sa, 0, sb)
                  : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va, vb, c, 4, 4, 2, sa, 2, sb);
}

// Staged kernel.  A unit is 256 k: per row 128 bytes of codes (eight 16-byte pieces =
// eight MX blocks) and 8 scale bytes, which come for several units at a time (scale_chunks.h), so that a copy instruction asks for whole 128-byte cache lines
// (8 lanes per row): the texture-address unit of a CU spends about 34 cycles on a copy that touches
// sixteen 64-byte segments and 17.5 on one that touches eight full lines (measured), and with FP4
// MFMAs the copies of a 256 x 256 tile would otherwise take as long as its arithmetic.  Units travel
// global -> LDS with buffer copies (REGS: through registers) through a ring of NUNIT buffers, one barrier per unit.  LDS layout of one unit: A
// codes [BM][128] | W codes [BN][128] (RAGGED and REGS: | A scales [BM][8] | W scales [BN][8]); in front of the units the scale bytes' two chunks or
// windows.  The 256 x 256 tile has two buffers: with whole rows 2 x 64 KB of codes and 2 x 16 KB of scale bytes, all of the 160 KB, with windows 2 x 68
// and 2 x 8 KB.  The eight pieces of a row are stored
// XOR-swizzled with (row >> 1) & 7: the LDS serves a 16-byte read of 16 consecutive lanes per clock from
// 64 banks, rows are 128 bytes apart, so 16 consecutive rows must land on 16 different 16-byte bank groups
// (measured: a swizzle with a period of 8 rows spent 44 % of its LDS cycles on bank conflicts); applied by
// choosing which global piece a lane fetches (a wave-wide copy writes lane l to base + 16 l).
// With the copies of whole rows (COPIES, below) and K' an odd multiple of 128 the last unit is half a unit: its copies re-fetch the first half
// for the missing second half (never used, in bounds).
// BF16: the same skeleton for plain bf16 operands (the comparison kernel arcq_ref_gemm_bf16): a row of a unit is 128
// bytes = 64 bf16 values, there are no scale bytes, and a k-step is one v_mfma_f32_32x32x16_bf16.
// What the loop spends beside the matrix instructions is the copies: a vector multiplication and four to five other vector instructions each, with
// addresses per lane, and the copies of scale bytes, two words a row and unit.  With buffer copies (no vector instruction) and scale bytes for several units
// at once, and without 64-bit divisions in front of the first copy (480 instructions before it, 217 to 284 now): 300 random problems of 65 to 8192 rows 1.09x on
// average (0.995 to 1.40; by tiles 1.06 to 1.16, the same bits; the three were measured together), 8192 x 8192 over K' = 29696 1011 -> 950 us, 4096 x 27648 over 5632
// 383 -> 358, over 5664 458 -> 418 with the quantizer, 1500 x 14336 over 4320 83.2 -> 73.6, 1592 x 2461 over 24000 117 -> 84.
// fp32 results of 256 x 256 tiles: 33 registers in scratch (16 with windows), behind the loop.
// How the units get into LDS (MODE): COPIES for K' % 128 == 0, codes 16-byte and scale bytes 4-byte aligned; RAGGED for any K' (a
// multiple of 32) from 512 on and dword-aligned codes: scale bytes as dword-aligned windows (scale_chunks.h), pieces past the
// end of a row fetched from its last block and their fragments zeroed in the last unit; the base of the scale bytes has
// to be 4-byte aligned.  REGS: what is left, see below.
template <int WM, int WN, int GM, int GN, bool BF16 = false, int MODE = COPIES>
struct MxCfg {
    static constexpr int BM = 32 * WM * GM, BN = 32 * WN * GN;
    static constexpr int NT = 64 * GM * GN;
    static constexpr int NA = (BM * 8 + NT - 1) / NT, NW = (BN * 8 + NT - 1) / NT;       // 16-byte pieces of codes
    static constexpr int NDMA = NA + NW;
    static constexpr int A_CODES = 0;
    static constexpr int W_CODES = NA * NT * 16;
    static constexpr int A_SCALES = W_CODES + NW * NT * 16;             // (COPIES: none in a unit)
    static constexpr int LDS_MOST = 160 * 1024;
    // Scale bytes: chunks or windows of several units (scale_chunks.h); REGS: words of a unit
    static constexpr bool SCALES = !BF16 && MODE != REGS;               // come with copies
    using Wide = ScaleChunkWindows<BM, BN, NT, 3>;
    static constexpr int NAS = BF16 ? 0 : (BM * 2 + NT - 1) / NT, NWS = BF16 ? 0 : (BN * 2 + NT - 1) / NT;     // 4-byte words of scales
    static constexpr int UNIT_BYTES = A_SCALES + (MODE == RAGGED ? Wide::DENSE_BYTES : MODE == REGS ? (NAS + NWS) * NT * 4 : 0);
    static constexpr int NUNIT = 3 * UNIT_BYTES + (!SCALES ? 0 : MODE == COPIES ? 2 * ScaleChunks<BM, BN, NT, 16>::BYTES : 2 * Wide::BYTES + Wide::PATCH) <= LDS_MOST ? 3 : 2;
    // chunks of two units where those of four do not fit beside three ring slots (128 x 256 tiles, 2048 x 4096 over K' = 4352: 31 us on two slots, 24.4 on three)
    using Chunks = ScaleChunks<BM, BN, NT, NUNIT * UNIT_BYTES + 2 * ScaleChunks<BM, BN, NT, 32>::BYTES <= LDS_MOST ? 32 : 16>;
    // windows of one unit where those of three do not fit (256 x 256 tiles)
    using Windows = ScaleChunkWindows<BM, BN, NT, NUNIT * UNIT_BYTES + 2 * Wide::BYTES + Wide::PATCH <= LDS_MOST ? 3 : 1>;
    static constexpr int NG = MODE == COPIES && SCALES ? Chunks::NG : 0;        // copies of scale bytes a unit
    static constexpr int NWG = MODE == RAGGED ? Windows::NG : 0;
    static constexpr int SROW = MODE == COPIES ? 8 * Chunks::Q : 8;     // from a row's scale bytes to the next row's
    static constexpr int W_SCALES = MODE == RAGGED ? Windows::DENSE_W : MODE == REGS ? NAS * NT * 4 : Chunks::W_ROWS * SROW;    // behind those of A
    // chunks or windows, patch (RAGGED: see ScaleChunkWindows::fill_patch), units
    static constexpr int PATCH = !SCALES ? 0 : MODE == COPIES ? 2 * Chunks::BYTES : 2 * Windows::BYTES;
    static constexpr int UNITS = PATCH + (MODE == RAGGED ? Windows::PATCH : 0);
    static constexpr int LDS_BYTES = UNITS + NUNIT * UNIT_BYTES;
    static_assert(LDS_BYTES <= LDS_MOST, "LDS of a compute unit");
    static_assert(NDMA + (MODE == RAGGED ? Windows::NS : NG) < 64, "a counted wait leaves the copies of a unit and of later scale bytes: they have to fit the counter");
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

//
// REGS: the same tiles, LDS layout and schedule for shapes the direct-to-LDS copies do not serve.  A thread fetches its pieces of unit u+2 into registers with ordinary loads
// (declared with the alignment the interface guarantees), all at once right after the barrier that opens unit u+1,
// and writes them to LDS just before the barrier that opens their unit; blocks past the end of a row become zero
// codes (a scale word that would reach past the end is fetched from further left and shifted), so every unit is a
// whole unit.
template <int WM, int WN, int GM, int GN, typename OutT, bool BF16 = false, int MODE = COPIES>
__global__ __launch_bounds__(64 * GM * GN) void mx_gemm_staged_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N, int nb,
    OutT* __restrict__ y, int64_t ldy, int tiles_m, int tiles_n, int group_rows, int splits, int64_t split_stride) {
    using C = MxCfg<WM, WN, GM, GN, BF16, MODE>;
    constexpr bool REG = MODE == REGS, RAG = MODE == RAGGED;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    // The sizes are asked for with the first arguments: left to the compiler, their load comes behind the divisions below and is a trip of
    // its own before the first copy (128 x 128 tiles, 65 to 512 rows: 1 % of the time).
    asm volatile("" ::"s"(M), "s"(N), "s"(nb));
    __builtin_amdgcn_sched_barrier(0);

    // workgroup -> tile: tile_order.h
    // With splits > 1 the units of the reduction dimension are cut into `splits` runs: workgroup
    // blockIdx.x = split * num_tiles + tile accumulates its run and stores an fp32 partial tile at
    // y + split * split_stride (a reduction kernel adds the partial results in index order).
    const int num_tiles = tiles_m * tiles_n;
    const int split = splits > 1 ? (int)blockIdx.x / num_tiles : 0;
    const TileOrder tile((int)blockIdx.x - split * num_tiles, tiles_m, tiles_n, group_rows);
    const int tile_m = tile.m, tile_n = tile.n;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 31, h = lane >> 5;
    const int wg_m0 = tile_m * C::BM, wg_n0 = tile_n * C::BN;
    const int wrow0 = (wave / GN) * (32 * WM), wcol0 = (wave % GN) * (32 * WN);

    const bool has_half = MODE == COPIES && (nb & 7) != 0;            // nb % 8 == 4
    const int nunit = MODE != COPIES ? (nb + 7) >> 3 : (nb >> 3) + (has_half ? 1 : 0);

    // ---- copies: thread -> (row, piece) of a workgroup-wide copy; 8 lanes fetch one row's 128 bytes
    const uint32_t cpitch = (uint32_t)nb * 16u, spitch = (uint32_t)nb;
    const uint32_t lp = (uint32_t)((tid & 7) ^ ((tid >> 4) & 7));               // global piece this lane fetches
    const int crow = tid >> 3, srow = tid >> 1;
    const uint32_t wave_slot = __builtin_amdgcn_readfirstlane((uint32_t)(tid & ~63));
    const uint32_t lds0 = lds_address(lds);
    // this workgroup's run of units [u0, u1); a division is 30 instructions in front of the first copy
    int u0 = 0, u1 = nunit;
    if (splits > 1) {
        u0 = (int)((uint32_t)(split * nunit) / (uint32_t)splits);
        u1 = (int)((uint32_t)((split + 1) * nunit) / (uint32_t)splits);
    }
    const typename C::Chunks chunks(a_scales, w_scales, M, N, nb, wg_m0, wg_n0, (uint32_t)lane, wave_slot >> 6, 8 * u0);      // COPIES
    const typename C::Windows windows(a_scales, w_scales, M, N, nb, wg_m0, wg_n0, (uint32_t)tid, wave_slot, 8 * u0);    // RAGGED
    const int patch_from = C::Windows::patch_from(nb);
    // The offset of this lane's piece of a unit: the same for every copy, whose rows are a scalar apart.
    const CodeRows<C::NT / 8> rows_a(a_codes, M, wg_m0, cpitch), rows_w(w_codes, N, wg_n0, cpitch);
    const uint32_t row_off = (uint32_t)crow * cpitch;
    auto lane_offset = [&](int unit) -> uint32_t {
        if (RAG) return row_off + 16u * (uint32_t)min(8 * unit + (int)lp, nb - 1);
        return row_off + 16u * (has_half && unit == nunit - 1 ? lp & 3u : lp);
    };
    // copy d of a unit: A code pieces, W code pieces
    auto issue_one = [&](int d, int unit, int buf, uint32_t voffset) {
        const uint32_t base = lds0 + C::UNITS + buf * C::UNIT_BYTES + 16u * wave_slot, column = RAG ? 0u : (uint32_t)unit * 128u;
        constexpr int NA = C::NA, NT = C::NT;
        if (d < NA) rows_a.issue(d, voffset, column, base + C::A_CODES + 16 * d * NT);
        else rows_w.issue(d - NA, voffset, column, base + C::W_CODES + 16 * (d - NA) * NT);
    };

    // ---- REGS: the same pieces through registers (piece d of a thread lands where copy d puts it); needs nb >= 4
    constexpr int NCP = C::NA + C::NW, NSP = C::NAS + C::NWS;
    uint4 rc[REG ? NCP : 1];
    uint32_t rs[REG && NSP > 0 ? NSP : 1];
    auto reg_issue = [&](int unit) {
        const uint32_t oc = 16u * (uint32_t)min(8 * unit + (int)lp, nb - 1);
#pragma unroll
        for (int d = 0; d < NCP; ++d) {
            const bool is_a = d < C::NA;
            const int p = is_a ? d : d - C::NA;
            const uint32_t row = (uint32_t)(is_a ? min(wg_m0 + p * (C::NT / 8) + crow, M - 1) : min(wg_n0 + p * (C::NT / 8) + crow, N - 1));
            rc[d] = load16_a4((is_a ? a_codes : w_codes) + (size_t)(row * cpitch + oc));
        }
        const uint32_t os = (uint32_t)min(8 * unit + 4 * (tid & 1), nb - 4);
#pragma unroll
        for (int d = 0; d < NSP; ++d) {
            const bool is_a = d < C::NAS;
            const int p = is_a ? d : d - C::NAS;
            const uint32_t row = (uint32_t)(is_a ? min(wg_m0 + p * (C::NT / 2) + srow, M - 1) : min(wg_n0 + p * (C::NT / 2) + srow, N - 1));
            rs[d] = load4_a1((is_a ? a_scales : w_scales) + (size_t)(row * spitch + os));
        }
    };
    auto reg_commit = [&](int unit, int buf) {
        uint8_t* st = lds + C::UNITS + buf * C::UNIT_BYTES;
        const bool ok = 8 * unit + (int)lp < nb;       // this piece's block exists
#pragma unroll
        for (int d = 0; d < NCP; ++d) {
            const uint4 v = uint4{ok ? rc[d].x : 0u, ok ? rc[d].y : 0u, ok ? rc[d].z : 0u, ok ? rc[d].w : 0u};
            const int at = d < C::NA ? C::A_CODES + 16 * (d * C::NT + tid) : C::W_CODES + 16 * ((d - C::NA) * C::NT + tid);
            *reinterpret_cast<uint4*>(st + at) = v;
        }
        const int sb0 = 8 * unit + 4 * (tid & 1);       // this word: blocks sb0 .. sb0 + 3
        const int skip = sb0 - min(sb0, nb - 4);        // bytes of the fetched word that belong to earlier blocks
#pragma unroll
        for (int d = 0; d < NSP; ++d) {
            const uint32_t word = skip >= 4 ? 0u : rs[d] >> (8 * skip);
            *reinterpret_cast<uint32_t*>(st + C::A_SCALES + 4 * (d * C::NT + tid)) = word;        // (W_SCALES follow at 4 NAS NT)
        }
    };

    // ---- LDS read offsets of this lane: k-step t of a unit takes piece 2t + h of its rows, stored at
    // physical position (2t + h) ^ ((row >> 1) & 7), which only depends on r because the other terms of the
    // row are multiples of 32
    const uint32_t swz = (uint32_t)(r >> 1) & 7u;
    const uint32_t rd_a = C::A_CODES + (wrow0 + r) * 128, rd_w = C::W_CODES + (wcol0 + r) * 128;
    const uint32_t rd_as = MODE == COPIES ? C::Chunks::row_at(wrow0 + r) : (wrow0 + r) * C::SROW;
    const uint32_t rd_ws = C::W_SCALES + (MODE == COPIES ? C::Chunks::row_at(wcol0 + r) : (wcol0 + r) * C::SROW);
    uint32_t pc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) pc[t] = 16u * ((uint32_t)(2 * t + h) ^ swz);

    float16v acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    // EARLY (two ring slots): three sets of fragments, see the pipeline below; otherwise the k-step being computed and the next one
    constexpr bool EARLY = !REG && C::NUNIT == 2;
    constexpr int NSET = EARLY ? 3 : 2;
    uint4 fa[NSET][WM], fw[NSET][WN];
    uint2 sa[WM], sw[WN], sa_n[WM], sw_n[WN];   // scale bytes of the unit (.x: blocks 0-3, .y: 4-7), shifted so
                                                // that bytes 0 and 2 of each word are this lane's
    auto read_codes = [&](int slot, int t, const uint8_t* st) {
#pragma unroll
        for (int i = 0; i < WM; ++i) fa[slot][i] = *reinterpret_cast<const uint4*>(st + rd_a + i * 4096 + pc[t]);
#pragma unroll
        for (int j = 0; j < WN; ++j) fw[slot][j] = *reinterpret_cast<const uint4*>(st + rd_w + j * 4096 + pc[t]);
    };
    // (in the unit's slot, or in the ring of chunks)
    auto read_scales = [&](int unit, int slot, uint2 (&da)[WM], uint2 (&dw)[WN]) {
        if constexpr (!BF16) {
            const uint32_t flip = MODE == COPIES ? C::Chunks::at(unit - u0) : 0u;
            const uint8_t* at = lds + (MODE == COPIES ? C::Chunks::base(unit - u0) : (uint32_t)(C::UNITS + slot * C::UNIT_BYTES + C::A_SCALES));
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                const uint2 v = *reinterpret_cast<const uint2*>(at + (rd_as ^ flip) + i * 32 * C::SROW);
                da[i] = make_uint2(v.x >> (8 * h), v.y >> (8 * h));
            }
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                const uint2 v = *reinterpret_cast<const uint2*>(at + (rd_ws ^ flip) + j * 32 * C::SROW);
                dw[j] = make_uint2(v.x >> (8 * h), v.y >> (8 * h));
            }
        }
    };

    // ---- pipeline, scheduled by hand (one wave per SIMD: nothing else hides a stall).  A unit is
    // NSTEPS WM WN MFMAs.  Three ring slots: the copies of unit u + 2 are issued one at a time between the first
    // MFMAs of unit u (its buffer was last read in unit u-1, which every wave left before the barrier
    // inside unit u-1); the fragments of k-step t+1 are read while k-step t is computed; the barrier
    // that opens unit u+1 and the reads of its first fragments sit before the last half k-step.
    // Two ring slots (EARLY; the 256- and 192-row tiles): the copies of unit u + 2 go to the slot of unit u itself, as soon
    // as every wave has its last fragments of the unit in registers: the fragments of k-steps 1 and 2 are read at the
    // start of the unit, those of k-step 3 at the start of k-step 2 (into the set of k-step 1), and a second barrier at
    // FREE_Q hands the slot over.  The copies then have 64 + 56 - 38 = 82 of the MFMA slots of a 256 x 256 unit to land;
    // issued behind the barrier that opens the next unit they had 36 to 56 (8192 x 8192 over K' = 29696 972 -> 944 us, 1777 x
    // 10240 over 8576 129 -> 118, 4096 x 27648 over 5632 1.00 to 1.02 times as fast: the wait for copies is not all that bounds it).
    constexpr int NM = WM * WN;               // MFMAs per k-step
    int buf = 0;
    // RAGGED: the wanted scale bytes of unit u+1 are picked out of their windows at the start of k-step 1 (read) and in the
    // middle of it (write).  tail_tag: 1: unit u+1 is the last or the one before, whose windows or blocks may pass the end;
    // 2: unit u is the last and may have missing blocks: k-steps past the end are left out, codes past it are zeroed.
    // left_tag: units behind this one, up to 2: the last two units of a workgroup's run have code of their own, which copies
    // nothing and, in the last one, reads nothing for a next unit.  (Both used to copy the last unit once more, and the end of the
    // kernel waited for that: 1.0 % of the time on average over 200 problems of 513 to 8192 rows, 1500 x 14336 over K' = 4320 with the
    // quantizer 85.6 -> 84.2 us.)
    uint3 win[RAG ? C::Windows::G : 1];
    int wchunk = C::Windows::Q == 1 ? 1 : 0, wpart = C::Windows::Q == 1 ? 0 : 1;     // RAGGED: chunk of unit u+1 and its place in it
    auto run_unit = [&](int u, auto tail_tag, auto left_tag) {
        constexpr int NSTEPS = 4;
        constexpr int TAIL = decltype(tail_tag)::value;
        constexpr int LEFT = decltype(left_tag)::value;
        constexpr int LAST_Q = NSTEPS * NM - NM / 2;
        constexpr int COMMIT_Q = LAST_Q - NM / 2;     // REGS: the pieces of unit u+1 go to LDS half a k-step before its barrier
        constexpr int FREE_Q = 2 * NM + (3 * NM) / 8; // EARLY: every fragment of the unit is in registers
        const uint8_t* st = lds + C::UNITS + buf * C::UNIT_BYTES;
        const int buf1 = buf + 1 == C::NUNIT ? 0 : buf + 1, bufd = EARLY ? buf : buf == 0 ? C::NUNIT - 1 : buf - 1;
        int fetch = u + 2;              // opaque: followed as an induction variable it costs the copies 17 more additions a unit
        asm("" : "+s"(fetch));
        const uint32_t voffset = lane_offset(fetch);
#pragma unroll
        for (int t = 0; t < NSTEPS; ++t) {
            if (TAIL == 2 && 8 * u + 2 * t >= nb) break;
            if (LEFT == 0 && t == 2 && has_half && u == nunit - 1) break;       // half a unit
            const int set = !EARLY ? t & 1 : t == 3 ? 1 : t;
            if constexpr (EARLY) {
                if (t == 0) {
                    read_codes(1, 1, st);
                    read_codes(2, 2, st);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (t == 2) {
                    read_codes(1, 3, st);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else if (t + 1 < NSTEPS) {
                read_codes((t + 1) & 1, t + 1, st);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (TAIL == 2 && 8 * u + 2 * t + h >= nb) {
#pragma unroll
                for (int i = 0; i < WM; ++i) fa[set][i] = make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                    const int q = t * NM + i * WN + j;
                    if constexpr (RAG && LEFT > 0) {
                        uint8_t* next = lds + C::UNITS + buf1 * C::UNIT_BYTES;
                        if (q == NM) {
                            // (windows that have landed before the barrier that opened this unit)
#pragma unroll
                            for (int g = 0; g < C::Windows::G; ++g)
                                win[g] = windows.gather(g, wchunk, wpart, lds, TAIL == 1 && u + 1 >= patch_from, lds + C::PATCH);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (q == NM + NM / 2) {
#pragma unroll
                            for (int g = 0; g < C::Windows::G; ++g)
                                windows.put(g, win[g], next + C::A_SCALES, TAIL == 1, u + 1);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    if (REG && LEFT > 0 && q == COMMIT_Q) {
                        reg_commit(u + 1, buf1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (EARLY && LEFT == 2 && q == FREE_Q) {
                        wait_lgkmcnt0();
                        wg_barrier();
                    }
                    if (q == LAST_Q && LEFT > 0) {
                        // unit u+1 must have landed: the copies of the DIST - 1 later units (EARLY: of unit u+2) are younger
                        // (REGS: this wave's LDS writes of unit u+1 must have completed)
                        if constexpr (REG) wait_lgkmcnt0();
                        else wait_vmcnt<LEFT == 2 ? C::NDMA : 0>();
                        if constexpr (RAG) wait_lgkmcnt0();         // this wave's scale bytes of unit u+1 are written
                        wg_barrier();
                        read_codes(0, 0, lds + C::UNITS + buf1 * C::UNIT_BYTES);
                        read_scales(u + 1, buf1, sa_n, sw_n);
                        if constexpr (REG && LEFT == 2) reg_issue(u + 2);
                        if constexpr (RAG) if (++wpart == C::Windows::Q) wpart = 0, ++wchunk;
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    // weights as the row operand: see store_tile_swapped
                    if constexpr (BF16)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fw[set][j]),
                                                                            __builtin_bit_cast(bf16x8, fa[set][i]), acc[i][j], 0, 0, 0);
                    else
                        acc[i][j] = mfma_mx(fw[set][j], fa[set][i], acc[i][j], (int)(t < 2 ? sw[j].x : sw[j].y),
                                            (int)(t < 2 ? sa[i].x : sa[i].y), t & 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (C::NG > 0 && LEFT == 2 && q >= LAST_Q) {        // a group of the scale bytes of later units
#pragma unroll
                        for (int i = 0; i < C::NG; ++i)
                            if (i % (NM - NM / 2) == q - LAST_Q) chunks.issue(i, (u - u0 + 1) % C::Chunks::Q, (u - u0 + 1) / C::Chunks::Q + 1, lds0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (C::NWG > 0 && LEFT == 2 && q == LAST_Q) {
                        windows.issue_group(wpart, wchunk + 1, lds0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (EARLY) {
                        constexpr int E = LAST_Q - FREE_Q;      // the MFMA slots that the copies of unit u + 2 are spread over
                        if (LEFT == 2 && q >= FREE_Q && q < LAST_Q) {
#pragma unroll
                            for (int d = 0; d < C::NDMA; ++d)
                                if (d * E / C::NDMA == q - FREE_Q) issue_one(d, fetch, bufd, voffset);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else if (!REG && LEFT == 2 && q < C::NDMA) {
                        issue_one(q, fetch, bufd, voffset);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
        }
        if constexpr (!BF16 && LEFT > 0) {
#pragma unroll
            for (int i = 0; i < WM; ++i) sa[i] = sa_n[i];
#pragma unroll
            for (int j = 0; j < WN; ++j) sw[j] = sw_n[j];
        }
        buf = buf1;
    };
    static_assert(C::NDMA <= 3 * NM, "copies are issued during the first three k-steps of a unit");

    if constexpr (REG) {
        reg_issue(u0);
        reg_commit(u0, 0);
        reg_issue(min(u0 + 1, nunit - 1));
        wait_lgkmcnt0();
    } else {
        // Scale bytes go out first (1500 x 14336 over K' = 4320 74.7 us, 75.9 behind the first unit's codes), but with three ring slots and whole rows behind
        // those: 128 x 128 tiles over short K' wait for little else (128 x 4096 over 512 4.55 -> 4.45 us together with the shares of issue_first).
        constexpr bool CODES_FIRST = C::SCALES && !RAG && C::NUNIT == 3;
        if constexpr (RAG) {
            windows.issue_chunk(0, lds0);
            if (C::Windows::Q == 1) windows.issue_chunk(1, lds0);       // looked at in the first unit
        }
        if constexpr (C::SCALES && !RAG && !CODES_FIRST) chunks.issue_first((uint32_t)lane, lds0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int d = 0; d < C::NDMA; ++d) issue_one(d, min(u0 + u, nunit - 1), u, lane_offset(min(u0 + u, nunit - 1)));
            if constexpr (CODES_FIRST)
                if (u == 0) chunks.issue_first((uint32_t)lane, lds0);
        }
#pragma unroll
        for (int i = 0; i < C::NG; ++i) chunks.issue(i, 0, 1, lds0);
        if constexpr (C::NWG > 0 && C::Windows::Q > 1) {
            windows.issue_group(0, 1, lds0);
            windows.issue_group(1, 1, lds0);
        }
        // (its loads make the first waves wait for every copy so far: 0.3 us)
        if constexpr (RAG)
            if (C::Windows::needs_patch(M, N, nb, wg_m0, wg_n0)) C::Windows::fill_patch(a_scales, w_scales, M, N, nb, (uint32_t)tid, lds + C::PATCH);
        if (C::NG > 0 && !chunks.active) wait_vmcnt<C::NDMA>();
        else wait_vmcnt<C::NDMA + C::NG + (C::Windows::Q > 1 ? 2 : 0) * C::NWG>();
        if constexpr (RAG) {
            const bool tail = u0 >= patch_from;     // a short run of a split
            if (tail) {                             // uniform: the patch is written by the first waves
                wait_lgkmcnt0();
                wg_barrier();
            }
#pragma unroll
            for (int g = 0; g < C::Windows::G; ++g)
                windows.put(g, windows.gather(g, 0, 0, lds, tail, lds + C::PATCH), lds + C::UNITS + C::A_SCALES, tail, u0);
            wait_lgkmcnt0();
            if (C::Windows::Q == 1) windows.issue_group(0, 2, lds0);    // into the first chunk's place
        }
    }
    wg_barrier();
    read_codes(0, 0, lds + C::UNITS);
    read_scales(u0, 0, sa, sw);
    using Tag0 = std::integral_constant<int, 0>;
    using Tag1 = std::integral_constant<int, 1>;
    using Tag2 = std::integral_constant<int, 2>;
    int u = u0;
    for (; u < (RAG ? min(patch_from - 1, u1 - 2) : u1 - 2); ++u) run_unit(u, Tag0{}, Tag2{});
    if constexpr (RAG) {
        for (; u < u1 - 2; ++u) run_unit(u, Tag1{}, Tag2{});
        if (u1 - u0 > 1) run_unit(u1 - 2, Tag1{}, Tag1{});
        run_unit(u1 - 1, Tag2{}, Tag0{});
    } else {
        if (u1 - u0 > 1) run_unit(u1 - 2, Tag0{}, Tag1{});
        run_unit(u1 - 1, Tag0{}, Tag0{});
    }
    wait_vmcnt<0>();                            // no copy may still be in flight when the LDS is released

    const int m0 = wg_m0 + wrow0, n0 = wg_n0 + wcol0;
    if constexpr (std::is_same<OutT, _Float16>::value) {
        static_assert(epilogue_lds_bytes(WN) * GM * GN <= C::LDS_BYTES, "one epilogue region per wave must fit the operand ring");
        wg_barrier();                           // every wave has read its last operands: the ring is free
        store_tile_f16_via_lds<WM, WN>(acc, lds + wave * epilogue_lds_bytes(WN), m0, n0, lane, M, N, 1.0f, y, ldy);
    } else {
        store_tile_swapped<WM, WN>(acc, m0, n0, r, h, M, N, 1.0f, y + (int64_t)split * split_stride, ldy);
    }
}

// Fallback for any K' (multiple of 32) and any alignment the API admits: operands straight from global
// memory, one 64 x 64 tile per wave.  A k-step is two blocks; when the block count is odd the upper
// half of the lanes contributes zero codes in the last step.
template <typename OutT>
__global__ __launch_bounds__(256) void mx_gemm_direct_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N, int nb,
    OutT* __restrict__ y, int64_t ldy) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // scalar: see gemm.hip
    const int r = lane & 31, h = lane >> 5;
    const int m0 = blockIdx.y * 128 + (wave >> 1) * 64, n0 = blockIdx.x * 128 + (wave & 1) * 64;
    const int64_t cpitch = (int64_t)nb * 16, spitch = nb;
    const uint8_t *ac[2], *as[2], *wc[2], *ws[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = min(m0 + 32 * i + r, M - 1), n = min(n0 + 32 * i + r, N - 1);
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
    for (int b0 = 0; b0 < nb; b0 += 2) {
        const int b = b0 + h;
        const bool ok = b < nb;
        const int bb = ok ? b : 0;
        uint4 fa[2], fw[2];
        int sa[2], sw[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            // 4-byte loads: the API only guarantees 4-byte alignment of the codes on this path
            const uint32_t* pa = reinterpret_cast<const uint32_t*>(ac[i] + 16 * (int64_t)bb);
            const uint32_t* pw = reinterpret_cast<const uint32_t*>(wc[i] + 16 * (int64_t)bb);
            fa[i] = ok ? make_uint4(pa[0], pa[1], pa[2], pa[3]) : make_uint4(0, 0, 0, 0);
            fw[i] = ok ? make_uint4(pw[0], pw[1], pw[2], pw[3]) : make_uint4(0, 0, 0, 0);
            sa[i] = ok ? as[i][bb] : 127;
            sw[i] = ok ? ws[i][bb] : 127;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma_mx(fw[j], fa[i], acc[i][j], sw[j], sa[i], 0);
    }
    store_tile_swapped<2, 2>(acc, m0, n0, r, h, M, N, 1.0f, y, ldy);
}

// Weight-streaming kernel for M <= 64 (decode, batched decode), any K' (a multiple of 32): bound by
// reading the packed weights once (17/32 byte per weight).  v_mfma_scale_f32_16x16x128_f8f6f4: lane
// (i = lane % 16, q = lane / 16) supplies the 32 values of block 4c + q of row i for the 128-k chunk c,
// with that block's scale byte.  A lane loads 16 bytes of codes per row and chunk (a wave: 16 rows x 64
// contiguous bytes) and its block's scale byte.  Blocks past the end of a row (a last chunk of one to three
// blocks) count as zero codes.  Loads are declared with the alignment the interface guarantees (codes 4 bytes,
// scale bytes 1); global memory serves them in one request at any address.  MT tiles of 16 activation rows share every weight fragment; the WAVES
// waves of a workgroup split K' and add their partial tiles through LDS.  Everything is loaded straight
// into registers; latency is hidden by occupancy.
typedef float float4v __attribute__((ext_vector_type(4)));

// GRP: whole chunks are taken four at a time (512 k) with the scale bytes of the four chunks fetched by ONE
// four-byte load per lane: the four lanes of a row read 16 contiguous bytes, and a 4 x 4 byte transpose
// across the four lane groups (two lane-swap instructions and two byte permutes with per-lane selectors)
// leaves every lane with the scale bytes of its block for the four chunks, which the matrix instruction
// picks with its byte selector.  The address unit of a CU spends about two cycles per (row, 64-byte
// segment) an instruction touches, so a four-byte scale load per chunk costs as much as the code load.
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t transpose_scale_bytes(uint32_t s, uint32_t sel_half, uint32_t sel_byte) {
    const uint2v x = __builtin_amdgcn_permlane32_swap(s, s, false, false);     // (q, q ^ 2): own and partner word
    const uint32_t pair = __builtin_amdgcn_perm(x[1], x[0], sel_half);         // bytes {0,1} or {2,3} of chunks (q & 1), (q & 1) + 2
    const uint2v t = __builtin_amdgcn_permlane16_swap(pair, pair, false, false);   // (q, q ^ 1)
    return __builtin_amdgcn_perm(t[1], t[0], sel_byte);                        // byte q of chunks 0, 1, 2, 3
}

// weight tiles whose partial sums fit the static LDS limit at a time
constexpr int mx_skinny_batch(int mt, int nt, int waves) { return waves * mt * nt > 64 ? (nt + 1) / 2 : nt; }

template <int MT, int NT, int WAVES, int U, bool GRP, typename OutT>
__device__ __forceinline__ void mx_skinny_tiles(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N, int nb,
    OutT* __restrict__ y, int64_t ldy, int n0, float* red_memory) {
    constexpr int BATCH = mx_skinny_batch(MT, NT, WAVES);
    auto& red = *reinterpret_cast<float (*)[WAVES][MT * BATCH][4][64]>(red_memory);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // scalar: see gemm.hip
    const int i = lane & 15, q = lane >> 4;
    const int64_t cpitch = (int64_t)nb * 16, spitch = nb;
    const int nchunk = (nb + 3) >> 2;                            // the last chunk may hold fewer than four blocks

    const uint8_t *ac[MT], *as[MT];
#pragma unroll
    for (int r = 0; r < MT; ++r) {
        const int m = min(16 * r + i, M - 1);                    // rows past M repeat row M-1 and are not stored
        ac[r] = a_codes + (int64_t)m * cpitch;
        as[r] = a_scales + (int64_t)m * spitch;
    }
    const uint8_t *wc[NT], *ws[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int n = min(n0 + 16 * t + i, N - 1);
        wc[t] = w_codes + n * cpitch;
        ws[t] = w_scales + n * spitch;
    }
    float4v acc[MT][NT];
#pragma unroll
    for (int r = 0; r < MT; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] = float4v{0.f, 0.f, 0.f, 0.f};

    int cbase = 0, first_wave = 0;              // first chunk and first wave of the chunk-at-a-time loop
    if constexpr (GRP) {
        const int ngroup = nb >> 4;             // groups of four whole chunks
        const uint32_t sel_half = q < 2 ? 0x05040100u : 0x07060302u;
        const uint32_t sel_byte = (q & 1) ? 0x07030501u : 0x06020400u;
        for (int g = wave; g < ngroup; g += WAVES) {
            uint4 ca[4][MT], cw[4][NT];
            uint32_t sa[MT], sw[NT];
            // the scale bytes are needed first (their transpose precedes the first matrix instruction) and loads retire
            // in issue order: asked for first, they do not make the wave wait for the whole group's codes; the
            // scheduling barrier keeps every load of the group ahead of its first use
#pragma unroll
            for (int r = 0; r < MT; ++r) sa[r] = load4_a1(as[r] + 16 * (int64_t)g + 4 * q);
#pragma unroll
            for (int t = 0; t < NT; ++t) sw[t] = load4_a1(ws[t] + 16 * (int64_t)g + 4 * q);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
#pragma unroll
                for (int r = 0; r < MT; ++r) ca[m][r] = load16_a4(ac[r] + 256 * (int64_t)g + 64 * m + 16 * q);
#pragma unroll
                for (int t = 0; t < NT; ++t) cw[m][t] = load16_a4(wc[t] + 256 * (int64_t)g + 64 * m + 16 * q);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < MT; ++r) sa[r] = transpose_scale_bytes(sa[r], sel_half, sel_byte);
#pragma unroll
            for (int t = 0; t < NT; ++t) sw[t] = transpose_scale_bytes(sw[t], sel_half, sel_byte);
            auto step = [&](auto mtag) {
                constexpr int m = decltype(mtag)::value;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int8v vw = {(int)cw[m][t].x, (int)cw[m][t].y, (int)cw[m][t].z, (int)cw[m][t].w, 0, 0, 0, 0};
#pragma unroll
                    for (int r = 0; r < MT; ++r) {
                        const int8v va = {(int)ca[m][r].x, (int)ca[m][r].y, (int)ca[m][r].z, (int)ca[m][r].w, 0, 0, 0, 0};
                        // byte m of the scale registers belongs to chunk m
                        acc[r][t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(va, vw, acc[r][t], 4, 4, m, (int)sa[r], m, (int)sw[t]);
                    }
                }
            };
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
        }
        cbase = 4 * ngroup;
        first_wave = ngroup % WAVES;            // the waves that took one group less come first
    }
    for (int c0 = cbase + ((wave - first_wave + WAVES) % WAVES) * U; c0 < nchunk; c0 += WAVES * U) {
        uint4 ca[U][MT], cw[U][NT];
        uint32_t sa[U][MT], sw[U][NT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // a block past the end of the row: the lane re-reads block 0 and the block counts as zero (codes zeroed where
            // they are used, not here: a select behind a load would make the wave wait for it at once)
            const int64_t b = 4 * (c0 + u) + q < nb ? 4 * (c0 + u) + q : 0;
#pragma unroll
            for (int r = 0; r < MT; ++r) {
                ca[u][r] = load16_a4(ac[r] + 16 * b);
                sa[u][r] = as[r][b];
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                cw[u][t] = load16_a4(wc[t] + 16 * b);
                sw[u][t] = ws[t][b];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool ok = 4 * (c0 + u) + q < nb;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int8v vw = {ok ? (int)cw[u][t].x : 0, ok ? (int)cw[u][t].y : 0, ok ? (int)cw[u][t].z : 0, ok ? (int)cw[u][t].w : 0, 0, 0, 0, 0};
#pragma unroll
                for (int r = 0; r < MT; ++r) {
                    const int8v va = {ok ? (int)ca[u][r].x : 0, ok ? (int)ca[u][r].y : 0, ok ? (int)ca[u][r].z : 0, ok ? (int)ca[u][r].w : 0, 0, 0, 0, 0};
                    // activations as the 16-row operand: lane holds column n = lane % 16, register e row 4 (lane / 16) + e
                    acc[r][t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(va, vw, acc[r][t], 4, 4, 0, (int)sa[u][r], 0, (int)sw[u][t]);
                }
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
            if (m < M && n < N) store_out(y + (int64_t)m * ldy + n, sum);
        }
    }
}

constexpr int MX_STREAM_ROUND = 256 * 64;       // weight rows: a workgroup of eight waves x four tiles on every compute unit

// BEHIND: weight tiles of the workgroups behind the first MX_STREAM_ROUND weight rows; NT of all others
template <int MT, int NT, int BEHIND, int WAVES, int U, bool GRP, typename OutT>
__global__ __launch_bounds__(WAVES * 64) void mx_gemm_skinny_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N, int nb,
    OutT* __restrict__ y, int64_t ldy) {
    constexpr int FLOATS = WAVES * MT * mx_skinny_batch(MT, NT, WAVES) * 256;
    static_assert(BEHIND <= NT && sizeof(float) * FLOATS <= 64 * 1024, "partial tiles must fit the static LDS limit");
    __shared__ float red[FLOATS];
    if constexpr (BEHIND == NT) {
        mx_skinny_tiles<MT, NT, WAVES, U, GRP>(a_codes, a_scales, w_codes, w_scales, M, N, nb, y, ldy, blockIdx.x * (16 * NT), red);
    } else {
        constexpr int FIRST = MX_STREAM_ROUND / (16 * NT);
        static_assert(FIRST * 16 * NT == MX_STREAM_ROUND, "whole workgroups first");
        if (blockIdx.x < FIRST)
            mx_skinny_tiles<MT, NT, WAVES, U, GRP>(a_codes, a_scales, w_codes, w_scales, M, N, nb, y, ldy, blockIdx.x * (16 * NT), red);
        else
            mx_skinny_tiles<MT, BEHIND, WAVES, U, GRP>(a_codes, a_scales, w_codes, w_scales, M, N, nb, y, ldy,
                                                       MX_STREAM_ROUND + (blockIdx.x - FIRST) * (16 * BEHIND), red);
    }
}

template <int MT, int NT, int BEHIND, int WAVES, int U, typename OutT>
arcq_status launch_mx_skinny(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                             const uint8_t* w_scales, int M, int N, int nb, OutT* y, int64_t ldy, hipStream_t stream) {
    const int rows = BEHIND == NT ? N : std::min(N, MX_STREAM_ROUND), behind = N - rows;
    const int workgroups = (rows + 16 * NT - 1) / (16 * NT) + (behind + 16 * BEHIND - 1) / (16 * BEHIND);
    hipLaunchKernelGGL((mx_gemm_skinny_kernel<MT, NT, BEHIND, WAVES, U, (MT <= 4), OutT>), dim3(workgroups),
                       dim3(WAVES * 64), 0, stream, a_codes, a_scales, w_codes, w_scales, M, N, nb, y, ldy);
    return check_launch("mx_gemm_skinny_kernel");
}

template <int WM, int WN, int GM, int GN, int MODE = COPIES, bool BF16 = false, typename OutT>
arcq_status launch_mx_staged(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                             const uint8_t* w_scales, int M, int N, int nb, OutT* y, int64_t ldy, hipStream_t stream,
                             int splits = 1, float* partial = nullptr) {
    using C = MxCfg<WM, WN, GM, GN, BF16, MODE>;
    const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    if (splits > 1) {
        // fp32 partial results [splits, M, N] in the workspace, then one pass that adds them
        auto kern = mx_gemm_staged_kernel<WM, WN, GM, GN, float, BF16, MODE>;
        static std::atomic<uint64_t> lds_raised{0};
        if (arcq_status st = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_raised)) return st;
        hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * splits), dim3(C::NT), C::LDS_BYTES, stream, a_codes, a_scales,
                           w_codes, w_scales, M, N, nb, partial, (int64_t)N, tiles_m, tiles_n, tile_group_rows(tiles_m, tiles_n), splits, (int64_t)M * N);
        if (arcq_status st = check_launch("mx_gemm_staged_kernel (split K)")) return st;
        return launch_splitk_reduce(partial, splits, M, N, 1.0f, y, std::is_same<OutT, _Float16>::value ? ARCQ_DTYPE_F16 : ARCQ_DTYPE_F32,
                                    ldy, stream);
    }
    auto kern = mx_gemm_staged_kernel<WM, WN, GM, GN, OutT, BF16, MODE>;
    static std::atomic<uint64_t> lds_raised{0};
    if (arcq_status st = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_raised)) return st;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(C::NT), C::LDS_BYTES, stream, a_codes, a_scales, w_codes,
                       w_scales, M, N, nb, y, ldy, tiles_m, tiles_n, tile_group_rows(tiles_m, tiles_n), 1, (int64_t)0);
    return check_launch("mx_gemm_staged_kernel");
}

}  // namespace

// Shapes the weight-streaming kernel serves: up to 64 rows while the tiled kernels (with K' split across workgroups
// where tiles are few) are not faster already.  Measured over N = 1024 .. 28672, K' = 4352 .. 28928: up to 16 rows
// below 2 * 10^8 weights (10^8 when K' >= 16384: 5120 x 27904 27.5 us streamed, 19 us tiled); 17 to 32 rows below
// 1.2 * 10^8 (5120 x 27904: 40 us streamed, 19 us tiled); 33 to 64
// rows below 2.2 * 10^7 and fewer than 8192 weight rows (6144 x 4352: 13.2 against 11.2 us).  On the FP4 instruction a 128- or 256-row tile costs no
// more than a 16-row one, so the tiled kernels win as soon as their tiles fill the chip.
static bool mx_streaming_shape(int64_t M, int64_t N, int64_t Kp) {
    const int64_t weights = N * Kp;
    if (M <= 16) return weights < 200000000 && !(Kp >= 16384 && weights >= 100000000);
    return M <= 32 ? weights < 120000000 : M <= 64 && N < 8192 && weights < 22000000;
}

// Number of runs the units of the reduction dimension are cut into when the caller provides a workspace (1: no
// split): a function of the shape alone.  Only the 128 x 128 tiles of few-tile problems split; the cost, in
// microseconds, is rounds of workgroups over the 256 CUs times the units of a run at about 0.65 us a unit, plus,
// when split, the write and read of the fp32 partial results at about 3 TB/s and 5.5 us for the shorter runs'
// pipeline fill and the second launch (fitted to measurements over N = 2048 .. 8192, K' = 4352 .. 29696).
static int mx_split_k(int64_t M, int64_t N, int64_t Kp) {
    const int64_t nb = Kp >> 5;
    const bool streaming = mx_streaming_shape(M, N, Kp);
    if (streaming || nb < 8) return 1;
    if (((M + 255) / 256) * ((N + 255) / 256) >= 256 || ((M + 127) / 128) * ((N + 255) / 256) >= 192) return 1;
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
    if (tiles > 256 && ((M + 191) / 192) * ((N + 127) / 128) <= 256) return 1;      // one round of 192 x 128 tiles
    const int64_t nunit = (nb + 7) >> 3;
    const int64_t max_splits = std::min<int64_t>(8, nunit / 2);
    int best = 1;
    double best_cost = 0.0;
    for (int64_t sp = 1; sp <= max_splits; ++sp) {
        const double rounds = (double)((tiles * sp + 255) / 256);
        double cost = rounds * (double)((nunit + sp - 1) / sp) * 0.65;
        if (sp > 1) cost += (double)sp * (double)M * (double)N * 8.0 / 3.0e6 + 5.5;
        if (sp == 1 || cost < best_cost) {
            best = (int)sp;
            best_cost = cost;
        }
    }
    return best;
}

// Tiles of 256 weight rows by 256, 192 or 128 activation rows when there is work for them (0: there is not): workgroups run in
// rounds of one per compute unit, a round lasts as long as one tile, and a tile's time follows the bytes it copies per
// unit, 136 (rows of A + rows of W): the height that minimises rounds x (height + 256) wins (e.g. 1024 x 10240:
// 240 tiles of 192 rows in one round instead of 320 of 128 rows in two).
static int mx_wide_rows(int64_t M, int64_t N) {
    const int64_t tn256 = (N + 255) / 256;
    if (((M + 127) / 128) * tn256 < 192) return 0;
    auto cost = [&](int64_t bm) { return ((((M + bm - 1) / bm) * tn256 + 255) / 256) * (bm + 256); };
    return cost(256) <= cost(192) && cost(256) <= cost(128) ? 256 : cost(192) <= cost(128) ? 192 : 128;
}

static GemmPlan plan_mx_stream(int64_t M, int64_t N, int64_t Kp) {
    // weight tiles per wave: as few as keep the launch at one workgroup per compute unit, up to four, two with more than 32
    // rows (measured with weights from HBM, 32 rows: 640 tiles 14.8 us with three per wave against 21.7 with one, 896 tiles
    // 10.4 us with four against 13.0 with two, 320 tiles over K' = 8448 11.2 us with two against 15.2 with one)
    const int64_t tiles = (N + 15) / 16;
    const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4;
    const int nt = tiles <= 256 ? 1 : tiles <= 512 || mt > 2 ? 2 : tiles <= 768 ? 3 : 4;
    GemmPlan plan = {ARCQ_ROUTE_STREAM, 16 * mt, 16 * nt, 1, false, mt * nt <= 2 ? 2 : 1};
    // Five to seven tiles a wave where they take a round less than four: up to 28672 weight rows in one (from HBM, us: 1 x 22016 over K' = 4352 14.4 ->
    // 11.4, 16 x 28672 over 5632 20.8 -> 17.5, 32 x 18944 over 2176 11.6 -> 8.7), up to 57344 in two (16 x 40960 over 4352 24.1 -> 21.4, 1 x 57344 over
    // 2176 17.7 -> 16.1).  Two row tiles leave the registers of five; up to 28672 weight rows the second round takes two or three tiles a wave instead
    // of four (32 x 22016 over 4352 18.7 -> 16.2, 32 x 28672 over 2176 12.2 -> 11.7).
    // One tile behind two whole rounds of four, and from K' = 4096 on two, stay on four: the workgroup that has them costs less than a fifth tile in all
    // others (four and five tiles a wave, 1 x 32769 over 4352 16.8 and 18.3, 1 x 32800 18.2 and 18.4, 32 x 32769 over 2176 14.3 and 15.4; 1 x 32785 over 2176
    // 11.5 and 11.3, 1 x 32832 over 4352 20.1 and 18.4).
    const int rounds = tiles <= 7 * 256 ? 1 : 2;
    const int few = rounds == 1 ? 0 : Kp >= 4096 ? 2 : 1;
    if (mt <= 2 && tiles > 4 * 256 * rounds + few && tiles <= 7 * 256 * rounds) {
        const int wide = (int)((tiles + 256 * rounds - 1) / (256 * rounds));
        if (mt == 1 || wide == 5) plan.tiles = plan.behind = wide;
        else if (rounds == 1) plan.behind = wide - 4;
    }
    return plan;
}

static GemmPlan plan_mx_one(int64_t M, int64_t N, int64_t Kp, bool workspace) {
    const int64_t nb = Kp >> 5;
    // up to 64 rows the tiled kernels only win where they can split K' across workgroups, which needs the workspace
    if (mx_streaming_shape(M, N, Kp) || (M <= 64 && !workspace && mx_split_k(M, N, Kp) > 1)) return plan_mx_stream(M, N, Kp);
    const bool offsets_fit = (uint64_t)M * (uint64_t)nb * 16 < 0xFFFF0000ull && (uint64_t)N * (uint64_t)nb * 16 < 0xFFFF0000ull;
    if (!offsets_fit || (nb < 8 && nb != 4)) return {ARCQ_ROUTE_DIRECT, 128, 128, 1, false};
    // more than 256 tiles of 128 x 128 but at most 256 of 192 x 128: one round of the taller tile instead of two
    // workgroups on some compute units (512 x 10240 over K' = 8448: 48 -> 37 us; 1024 x 5120 over 27904: 144 -> 105 us); and
    // before the 256-wide tiles, which put a round of larger tiles on fewer compute units (160 x 28672 over 4352: 28.6 -> 24.2 us)
    if (((M + 127) / 128) * ((N + 127) / 128) > 256 && ((M + 191) / 192) * ((N + 127) / 128) <= 256)
        return {ARCQ_ROUTE_TILES, 192, 128, 1, false};
    if (const int rows = mx_wide_rows(M, N)) return {ARCQ_ROUTE_TILES, rows, 256, 1, false};
    return {ARCQ_ROUTE_TILES, 128, 128, workspace ? mx_split_k(M, N, Kp) : 1, false};
}

GemmParts plan_mx_gemm_parts(int64_t M, int64_t N, int64_t Kp, bool workspace) {
    const GemmPlan one = plan_mx_one(M, N, Kp, workspace);
    // The streaming kernel with more weight rows than one round of four tiles a wave takes: that round, and the rest with one or two tiles a
    // wave in a launch of its own (see plan_gemm_parts in gemm.hip).  From HBM, us, 1 and 16 rows: 17408 weight rows over K' = 4096 13.5 -> 11.7 and
    // 14.9 -> 13.2, 20480 over 4352 14.2 -> 12.6 and 15.8 -> 14.0, over 8448 24.4 -> 20.2 and 27.7 -> 22.9, 24576 over 6144 19.5 -> 17.9 and 22.4 -> 20.3:
    // within NVFP4's limits 52 sizes gain 1.3 us and more, 1.07 to 1.22x.  Elsewhere a second launch loses to one of more tiles a wave (plan_mx_stream: 1 x 16400
    // over 4352 11.0, 12.0 in two, 9.5; 1 x 28672 over 6400 21.6, 22.3 and 19.8; 16 x 24576 over 2176 9.9, 10.4 and 8.0); that it is taken within the limits has NVFP4's
    // one reason, the tests that state this route (plan_gemm_parts).
    const int64_t behind = N - MX_STREAM_ROUND;
    if (one.kernel == ARCQ_ROUTE_STREAM && M <= 32 && behind >= 1024 && behind <= MX_STREAM_ROUND / 2 &&
        Kp >= (behind > MX_STREAM_ROUND / 4 ? 6144 : 4096)) {
        GemmParts parts = {plan_mx_stream(M, MX_STREAM_ROUND, Kp), plan_mx_stream(M, behind, Kp), M, MX_STREAM_ROUND};
        parts.rest.chunks = 1;      // K' in the order of four tiles a wave: the same bits as in one launch
        return parts;
    }
    return {one, one, M, N};
}

namespace {

template <typename OutT>
arcq_status launch_mx_plan(const GemmPlan& plan, const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                           const uint8_t* w_scales, int64_t M, int64_t N, int64_t Kp, OutT* y, int64_t ldy,
                           float* workspace, hipStream_t stream) {
    const int nb = (int)(Kp >> 5);
    const bool dword_scales = ((reinterpret_cast<uintptr_t>(a_scales) | reinterpret_cast<uintptr_t>(w_scales)) & 3) == 0;
    const bool aligned16 = ((reinterpret_cast<uintptr_t>(a_codes) | reinterpret_cast<uintptr_t>(w_codes)) & 15) == 0 && dword_scales;
    if (plan.kernel == ARCQ_ROUTE_STREAM) {
        const int tiles = plan.tiles ? plan.tiles : plan.cols / 16, behind = plan.behind ? plan.behind : tiles;
#define ARCQ_MX_STREAM_MIXED(MT_, NT_, BEHIND_, U_)                                                 \
    if (plan.rows == 16 * MT_ && tiles == NT_ && behind == BEHIND_ && plan.chunks == U_)             \
    return launch_mx_skinny<MT_, NT_, BEHIND_, 8, U_>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nb, y, ldy, stream)
#define ARCQ_MX_STREAM(MT_, NT_, U_) ARCQ_MX_STREAM_MIXED(MT_, NT_, NT_, U_)
        ARCQ_MX_STREAM(1, 1, 2);
        ARCQ_MX_STREAM(1, 2, 2);
        ARCQ_MX_STREAM(1, 3, 1);
        ARCQ_MX_STREAM(1, 4, 1);
        ARCQ_MX_STREAM(2, 1, 2);
        ARCQ_MX_STREAM(2, 2, 1);
        ARCQ_MX_STREAM(2, 3, 1);
        ARCQ_MX_STREAM(2, 4, 1);
        ARCQ_MX_STREAM(1, 5, 1);
        ARCQ_MX_STREAM(1, 6, 1);
        ARCQ_MX_STREAM(1, 7, 1);
        ARCQ_MX_STREAM(2, 5, 1);
        ARCQ_MX_STREAM_MIXED(2, 4, 2, 1);
        ARCQ_MX_STREAM_MIXED(2, 4, 3, 1);
        ARCQ_MX_STREAM(4, 1, 1);
        ARCQ_MX_STREAM(4, 2, 1);
        // the second launch of two
        ARCQ_MX_STREAM(1, 1, 1);
        ARCQ_MX_STREAM(1, 2, 1);
        ARCQ_MX_STREAM(2, 1, 1);
#undef ARCQ_MX_STREAM
#undef ARCQ_MX_STREAM_MIXED
        return fail(ARCQ_HIP_ERROR, "no weight-streaming kernel of %d x %d rows, %d chunks", plan.rows, plan.cols, plan.chunks);
    }
    // How the units get into LDS: whole aligned pieces; any K' (a multiple of 32) from 512 on, codes at their minimum alignment;
    // through registers, for scale bytes at odd addresses and short K' (no 192 x 128 tiles there)
    const int mode = (nb & 3) == 0 && aligned16 ? COPIES
                     : nb >= ScaleChunkWindows<128, 128, 256, 3>::MIN_NB && dword_scales ? RAGGED : REGS;
    auto tiled = [&](auto mode_tag) {
        constexpr int MODE = decltype(mode_tag)::value;
        const bool tall = plan.rows == 192 && plan.cols == 128;
        const int wide = plan.cols == 256 ? plan.rows : MODE == REGS && tall ? mx_wide_rows(M, N) : 0;
        if constexpr (MODE != REGS)
            if (tall)
                return launch_mx_staged<3, 2, 2, 2, MODE>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nb, y, ldy, stream);
        if (wide == 256)
            return launch_mx_staged<4, 4, 2, 2, MODE>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nb, y, ldy, stream);
        if (wide == 192)
            return launch_mx_staged<3, 4, 2, 2, MODE>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nb, y, ldy, stream);
        if (wide == 128)
            return launch_mx_staged<2, 4, 2, 2, MODE>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nb, y, ldy, stream);
        return launch_mx_staged<2, 2, 2, 2, MODE>(a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nb, y, ldy, stream,
                                                  plan.runs, workspace);
    };
    if (plan.kernel == ARCQ_ROUTE_TILES && (mode != REGS || nb >= 8))
        return mode == COPIES   ? tiled(std::integral_constant<int, COPIES>{})
               : mode == RAGGED ? tiled(std::integral_constant<int, RAGGED>{})
                                : tiled(std::integral_constant<int, REGS>{});
    dim3 grid((unsigned)((N + 127) / 128), (unsigned)((M + 127) / 128));
    hipLaunchKernelGGL(mx_gemm_direct_kernel<OutT>, grid, dim3(256), 0, stream, a_codes, a_scales, w_codes, w_scales,
                       (int)M, (int)N, nb, y, ldy);
    return check_launch("mx_gemm_direct_kernel");
}

template <typename OutT>
arcq_status launch_mx_typed(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                            const uint8_t* w_scales, int64_t M, int64_t N, int64_t Kp, OutT* y, int64_t ldy,
                            float* workspace, hipStream_t stream) {
    const GemmParts parts = plan_mx_gemm_parts(M, N, Kp, workspace != nullptr);
    if (arcq_status st = launch_mx_plan(parts.first, a_codes, a_scales, w_codes, w_scales, M, parts.cols, Kp, y, ldy, workspace, stream)) return st;
    if (parts.cols == N) return ARCQ_OK;
    return launch_mx_plan(parts.rest, a_codes, a_scales, w_codes + parts.cols * (Kp >> 1), w_scales + parts.cols * (Kp >> 5), M,
                          N - parts.cols, Kp, y + parts.cols, ldy, nullptr, stream);
}

}  // namespace

// Comparison kernel: y = x w^T for plain bf16 operands (x [M, K], w [N, K], row-major, 16-byte aligned, K % 32 == 0)
// on the tiled skeleton above, fp32 accumulation, fp16 output.  nb counts 16-byte pieces of a row.
arcq_status launch_ref_gemm_bf16(const void* x, const void* w, int64_t M, int64_t N, int64_t K, _Float16* y, int64_t ldy,
                                 hipStream_t stream) {
    const uint8_t* a = static_cast<const uint8_t*>(x);
    const uint8_t* b = static_cast<const uint8_t*>(w);
    const int nb = (int)(K >> 3);
    const int64_t t256 = ((M + 255) / 256) * ((N + 255) / 256);
    if (t256 >= 256) return launch_mx_staged<4, 4, 2, 2, COPIES, true>(a, nullptr, b, nullptr, (int)M, (int)N, nb, y, ldy, stream);
    const int64_t t128x256 = ((M + 127) / 128) * ((N + 255) / 256);
    if (t128x256 >= 192) return launch_mx_staged<2, 4, 2, 2, COPIES, true>(a, nullptr, b, nullptr, (int)M, (int)N, nb, y, ldy, stream);
    return launch_mx_staged<2, 2, 2, 2, COPIES, true>(a, nullptr, b, nullptr, (int)M, (int)N, nb, y, ldy, stream);
}

size_t mx_gemm_workspace_bytes(int64_t M, int64_t N, int64_t Kp) {
    const int splits = mx_split_k(M, N, Kp);
    return splits > 1 ? (size_t)splits * (size_t)M * (size_t)N * sizeof(float) : 0;
}

arcq_status launch_mx_gemm(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                           const uint8_t* w_scales, int64_t M, int64_t N, int64_t Kp, void* y, int y_dtype, int64_t ldy,
                           void* workspace, hipStream_t stream) {
    float* ws = static_cast<float*>(workspace);
    if (y_dtype == ARCQ_DTYPE_F16)
        return launch_mx_typed<_Float16>(a_codes, a_scales, w_codes, w_scales, M, N, Kp, static_cast<_Float16*>(y), ldy, ws, stream);
    return launch_mx_typed<float>(a_codes, a_scales, w_codes, w_scales, M, N, Kp, static_cast<float*>(y), ldy, ws, stream);
}

}  // namespace arcq
