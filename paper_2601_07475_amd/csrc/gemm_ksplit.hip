// Tiled W4A4 GEMM for problems with few output tiles (a few hundred activation rows; Section 3.2 eq. (2)): the waves
// of a workgroup split every stage along k INSIDE the compute unit, so a small output tile still keeps all four
// SIMDs busy and the chip gets one tile per compute unit without a round trip of fp32 partial results through
// HBM and a second launch (which is what splitting K' across workgroups costs).
//
// Workgroup tile BM x BN = 32 WM GM x 32 WN GN, computed by GM x GN x KS waves: wave (wq, kh) accumulates the
// WM x WN fragments of sub-tile wq over the k-quarter kh of every stage.  A stage is 64 KS k (256 for KS = 4): per
// row 32 KS code bytes (2 KS pieces of 16 bytes) and 4 KS scale bytes, kept packed in LDS and decoded in registers
// (gemm_decode.h); wave kh reads pieces 2 kh and 2 kh + 1 of a row (lanes 0-31 the first, lanes 32-63 the second:
// four k-steps, as in the wave-pair kernel of gemm.hip, whose schedule this kernel shares) and the scale word at
// byte 4 kh.  Stages travel global -> LDS with global_load_lds through a ring of three buffers.  The 16-byte
// pieces of a row are XOR-swizzled so that 16 consecutive rows fall on 16 different bank groups (rows are 128
// bytes apart for KS = 4: swizzle (row >> 1) & 7; 64 bytes for KS = 2: (row >> 2) & 3).
// At the end the KS partial tiles are added through the LDS in KS - 1 rounds; fragment f of a sub-tile is owned
// (finished and stored) by wave kh = f % KS (with six fragments and four waves two waves own two, two own one).
#include "internal.h"
#include "gemm_decode.h"
#include "gemm_epilogue.h"
#include "lds_dma.h"
#include "scale_windows.h"
#include "tile_order.h"

#include <type_traits>

namespace arcq {

namespace {

// How the stages get into LDS, as in gemm.hip: COPIES for K' % 64 == 0, RAGGED for any K' (dword-aligned scale bytes), REGS for
// scale bytes at odd addresses (see below).
template <int WM, int WN, int GM, int GN, int KS, int MODE = COPIES>
struct KsplitCfg {
    static_assert(KS == 2 || KS == 4, "k halves or quarters");
    static constexpr int BM = 32 * WM * GM, BN = 32 * WN * GN;
    static constexpr int NWAVE = GM * GN * KS, NT = 64 * NWAVE;
    static constexpr int ROWB = 32 * KS;            // code bytes of a row per stage
    static constexpr int PPR = 2 * KS;              // 16-byte pieces of a row per stage
    static constexpr int SROWB = 4 * KS;            // scale bytes of a row per stage
    // copy instructions per thread and stage (a copy always involves the whole workgroup; surplus lanes re-fetch
    // the operand's last rows into padding behind its region, so that every wave issues the same number)
    static constexpr int NA = (BM * PPR + NT - 1) / NT, NW = (BN * PPR + NT - 1) / NT;
    static constexpr int NAS = (BM * KS + NT - 1) / NT, NWS = (BN * KS + NT - 1) / NT;
    using Windows = ScaleWindows<BM, BN, NT, 4 * KS>;
    static constexpr int NSW = MODE == RAGGED ? Windows::NS : 0;           // copies of windows come first
    static constexpr int NDMA = NA + NW + (MODE == RAGGED ? NSW : NAS + NWS);
    static constexpr int A_CODES = 0;
    static constexpr int W_CODES = NA * NT * 16;
    static constexpr int A_SCALES = W_CODES + NW * NT * 16;
    static constexpr int W_SCALES = A_SCALES + (MODE == RAGGED ? Windows::DENSE_W : NAS * NT * 4);
    static constexpr int WINDOWS = A_SCALES + Windows::DENSE_BYTES;
    static constexpr int STAGE_BYTES = MODE == RAGGED ? WINDOWS + Windows::BYTES : W_SCALES + NWS * NT * 4;
    static constexpr int NSTAGE = 3, DIST = 2;
    static constexpr int OWN = (WM * WN + KS - 1) / KS;  // fragments a wave finishes and stores (at most)
    static constexpr int PATCH = NSTAGE * STAGE_BYTES;      // RAGGED: see ScaleWindows::fill_patch
    static constexpr int LDS_BYTES = PATCH + (MODE == RAGGED ? 2 * Windows::PATCH : 0);
    static_assert(NWAVE * OWN * 4096 <= LDS_BYTES, "the exchange regions must fit the operand ring");
    static_assert((NT / PPR) % 16 == 0 && (NT / KS) % 1 == 0, "row swizzle must not depend on the copy index");
    static_assert((DIST - 1) * NDMA < 64, "the vector-memory counter has 6 bits");
};

// One 32 x 32 fragment computed with the weights as the row operand: lane holds output row m0 + lane % 32, register
// e holds column n0 + 8 (e / 4) + 4 (lane / 32) + e % 4.
template <typename OutT>
__device__ __forceinline__ void store_fragment(const float16v& a, int m0, int n0, int r, int h, int M, int N, float alpha,
                                               OutT* __restrict__ y, int64_t ldy) {
    const int m = m0 + r;
    if (m >= M) return;
    OutT* yrow = y + (int64_t)m * ldy;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int n = n0 + 8 * g + 4 * h;
        const float v0 = a[4 * g] * alpha, v1 = a[4 * g + 1] * alpha, v2 = a[4 * g + 2] * alpha, v3 = a[4 * g + 3] * alpha;
        if (n + 3 < N) {
            store4(yrow + n, v0, v1, v2, v3);
        } else {
            if (n < N) store_out(yrow + n, v0);
            if (n + 1 < N) store_out(yrow + n + 1, v1);
            if (n + 2 < N) store_out(yrow + n + 2, v2);
            if (n + 3 < N) store_out(yrow + n + 3, v3);
        }
    }
}

// REGS: any K' (a multiple of 16) and operands that are only 8-byte aligned: a thread fetches its pieces of stage s + 2
// into registers with ordinary loads (declared with the alignment the interface guarantees), right after the barrier
// that opens stage s + 1, and writes them to LDS before the barrier that opens their stage; blocks past the end of a row
// become zero codes and zero scale bytes (a piece that would reach past the row's end is fetched from further left and
// shifted), so the last stage needs no special case.
template <int WM, int WN, int GM, int GN, int KS, typename OutT, int MODE = COPIES>
__global__ __launch_bounds__(64 * GM * GN * KS) void gemm_ksplit_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales,
    const uint8_t* __restrict__ w_codes, const uint8_t* __restrict__ w_scales, int M, int N,
    int nbk, float alpha, OutT* __restrict__ y, int64_t ldy, int tiles_m, int tiles_n, int group_rows) {
    using C = KsplitCfg<WM, WN, GM, GN, KS, MODE>;
    constexpr bool REG = MODE == REGS, RAG = MODE == RAGGED;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];

    // workgroup -> tile: tile_order.h
    const TileOrder tile((int)blockIdx.x, tiles_m, tiles_n, group_rows);
    const int tile_m = tile.m, tile_n = tile.n;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int r = lane & 31, h = lane >> 5;
    const int kh = wave / (GM * GN);                 // k share: k-steps 4 kh .. 4 kh + 3 of every stage
    const int wq = wave % (GM * GN);
    const int wg_m0 = tile_m * C::BM, wg_n0 = tile_n * C::BN;
    const int wrow0 = (wq / GN) * (32 * WM);         // first row of this wave inside the A tile
    const int wcol0 = (wq % GN) * (32 * WN);         // first row of this wave inside the W tile
    // stages of 4 KS blocks; the last one may hold only `part` k shares (K' is a multiple of 64, not of 64 KS): the
    // copies of its missing shares re-fetch the first share (in bounds, never used) and the waves of those shares read
    // their scale bytes as zero, so that their fragments decode to zeros
    const int nstage = (nbk + 4 * KS - 1) / (4 * KS);
    const int part = MODE != COPIES ? 0 : (nbk % (4 * KS)) / 4; // 0: the last stage is whole (RAGGED, REGS: made whole with zeros)

    // ---- copies
    auto swz = [](int row) -> uint32_t { return KS == 4 ? (uint32_t)(row >> 1) & 7u : (uint32_t)(row >> 2) & 3u; };
    const int crow = tid / C::PPR, srow = tid / KS;  // row of this thread inside a copy of NT / PPR code rows / NT / KS scale rows
    const uint32_t adj_c = 16u * ((uint32_t)(tid % C::PPR) ^ swz(crow));
    const uint32_t adj_s = 4u * (uint32_t)(tid % KS);
    const uint32_t cpitch32 = (uint32_t)nbk * 8u, spitch32 = (uint32_t)nbk;
    const uint32_t wave_slot = __builtin_amdgcn_readfirstlane((uint32_t)(tid & ~63));
    const uint32_t lds0 = lds_address(lds);
    const uint32_t piece_g = (uint32_t)(tid % C::PPR) ^ swz(crow);      // global piece this lane fetches
    const bool piece_missing = part != 0 && (int)(piece_g >> 1) >= part, scale_missing = part != 0 && tid % KS >= part;
    const uint32_t adj_c_last = piece_missing ? 16u * (piece_g & 1u) : adj_c, adj_s_last = scale_missing ? 0u : adj_s;
    const typename C::Windows windows = {a_scales, w_scales, M, N, nbk, wg_m0, wg_n0, (uint32_t)tid, wave_slot};    // RAGGED
    const int patch_from = C::Windows::patch_from(nbk);
    auto issue_one = [&](int d, int stage, int buf) {
        const uint32_t base = lds0 + buf * C::STAGE_BYTES;
        const bool last = stage == nstage - 1;
        const uint32_t oc = RAG ? 8u * (uint32_t)min(4 * KS * stage + 2 * (int)piece_g, nbk - 2)
                                : (uint32_t)stage * C::ROWB + (last ? adj_c_last : adj_c);
        if (RAG && d < C::NSW) {
            windows.issue(d, stage, base + C::WINDOWS);
            return;
        }
        d -= C::NSW;
        const uint32_t os = (uint32_t)stage * C::SROWB + (last ? adj_s_last : adj_s);
        constexpr int NA = C::NA, NW = C::NW, NAS = C::NAS, NT = C::NT;
        // rows past the edge of the operand re-read its last row (never stored)
        if (d < NA) {
            const uint32_t row = (uint32_t)min(wg_m0 + d * (NT / C::PPR) + crow, M - 1);
            dma16(a_codes, row * cpitch32 + oc, base + C::A_CODES + 16u * (d * NT + wave_slot));
        } else if (d < NA + NW) {
            const int p = d - NA;
            const uint32_t row = (uint32_t)min(wg_n0 + p * (NT / C::PPR) + crow, N - 1);
            dma16(w_codes, row * cpitch32 + oc, base + C::W_CODES + 16u * (p * NT + wave_slot));
        } else if (d < NA + NW + NAS) {
            const int p = d - NA - NW;
            const uint32_t row = (uint32_t)min(wg_m0 + p * (NT / KS) + srow, M - 1);
            dma4(a_scales, row * spitch32 + os, base + C::A_SCALES + 4u * (p * NT + wave_slot));
        } else {
            const int p = d - NA - NW - NAS;
            const uint32_t row = (uint32_t)min(wg_n0 + p * (NT / KS) + srow, N - 1);
            dma4(w_scales, row * spitch32 + os, base + C::W_SCALES + 4u * (p * NT + wave_slot));
        }
    };

    // ---- REGS: the same pieces through registers (piece d of a thread lands where copy d puts it); needs nbk >= 4
    constexpr int NCP = C::NA + C::NW, NSP = C::NAS + C::NWS;
    uint4 rc[REG ? NCP : 1];
    uint32_t rs[REG ? NSP : 1];
    auto reg_issue = [&](int stage) {
        const uint32_t oc = 8u * (uint32_t)min(4 * KS * stage + 2 * (int)piece_g, nbk - 2);
#pragma unroll
        for (int d = 0; d < NCP; ++d) {
            const bool is_a = d < C::NA;
            const int p = is_a ? d : d - C::NA;
            const uint32_t row = (uint32_t)(is_a ? min(wg_m0 + p * (C::NT / C::PPR) + crow, M - 1) : min(wg_n0 + p * (C::NT / C::PPR) + crow, N - 1));
            rc[d] = load16_a8((is_a ? a_codes : w_codes) + (size_t)(row * cpitch32 + oc));
        }
        const uint32_t os = (uint32_t)min(4 * KS * stage + 4 * (tid % KS), nbk - 4);
#pragma unroll
        for (int d = 0; d < NSP; ++d) {
            const bool is_a = d < C::NAS;
            const int p = is_a ? d : d - C::NAS;
            const uint32_t row = (uint32_t)(is_a ? min(wg_m0 + p * (C::NT / KS) + srow, M - 1) : min(wg_n0 + p * (C::NT / KS) + srow, N - 1));
            rs[d] = load4_a1((is_a ? a_scales : w_scales) + (size_t)(row * spitch32 + os));
        }
    };
    auto reg_commit = [&](int stage, int buf) {
        uint8_t* st = lds + buf * C::STAGE_BYTES;
        const int b0 = 4 * KS * stage + 2 * (int)piece_g;      // this piece: blocks b0, b0 + 1
        const bool both = b0 + 1 < nbk, one = b0 < nbk;
#pragma unroll
        for (int d = 0; d < NCP; ++d) {
            const uint4 v = uint4{both ? rc[d].x : one ? rc[d].z : 0u, both ? rc[d].y : one ? rc[d].w : 0u, both ? rc[d].z : 0u, both ? rc[d].w : 0u};
            const int at = d < C::NA ? C::A_CODES + 16 * (d * C::NT + tid) : C::W_CODES + 16 * ((d - C::NA) * C::NT + tid);
            *reinterpret_cast<uint4*>(st + at) = v;
        }
        const int sb0 = 4 * KS * stage + 4 * (tid % KS);       // this word: blocks sb0 .. sb0 + 3
        const int skip = sb0 - min(sb0, nbk - 4);               // bytes of the fetched word that belong to earlier blocks
#pragma unroll
        for (int d = 0; d < NSP; ++d) {
            const uint32_t word = skip >= 4 ? 0u : rs[d] >> (8 * skip);
            const int at = d < C::NAS ? C::A_SCALES + 4 * (d * C::NT + tid) : C::W_SCALES + 4 * ((d - C::NAS) * C::NT + tid);
            *reinterpret_cast<uint32_t*>(st + at) = word;
        }
    };

    // ---- LDS read offsets: this wave's share of a stage is piece 2 kh + h of a row's codes and the scale word at
    // byte 4 kh; fragment i of a wave is 32 rows further on (the swizzle only depends on lane % 32 because the other
    // terms are multiples of 32)
    const uint32_t piece = 16u * ((uint32_t)(2 * kh + h) ^ swz(r));
    const uint32_t rd_a = C::A_CODES + (wrow0 + r) * C::ROWB + piece, rd_w = C::W_CODES + (wcol0 + r) * C::ROWB + piece;
    const uint32_t rd_as = C::A_SCALES + (wrow0 + r) * C::SROWB + 4 * kh, rd_ws = C::W_SCALES + (wcol0 + r) * C::SROWB + 4 * kh;
    const uint32_t scale_sel = h ? 0x0C030C02u : 0x0C010C00u;

    float16v acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    constexpr int G = WM + WN;                 // fragments per k-step
    constexpr int MPG = (WM * WN >= 16) ? 2 : 1;   // MFMAs per group (singles spill with 4 x 4 fragments)
    constexpr int P = WM * WN / MPG;           // groups per k-step: after every group the decode of G / P fragments
    uint4 ca[WM], cw[WN];
    uint32_t sa[WM], sw[WN];
    half8 fa[2][WM], fw[2][WN];
    const bool share_missing = part != 0 && kh >= part;     // this wave has nothing in the last stage
    auto read_raw = [&](const uint8_t* st, bool zero) {
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            ca[i] = *reinterpret_cast<const uint4*>(st + rd_a + i * (32 * C::ROWB));
            const uint32_t word = *reinterpret_cast<const uint32_t*>(st + rd_as + i * (32 * C::SROWB));
            sa[i] = scale_halves(zero ? 0u : word, scale_sel);
        }
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            cw[j] = *reinterpret_cast<const uint4*>(st + rd_w + j * (32 * C::ROWB));
            const uint32_t word = *reinterpret_cast<const uint32_t*>(st + rd_ws + j * (32 * C::SROWB));
            sw[j] = scale_halves(zero ? 0u : word, scale_sel);
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

    // One stage = four k-steps of this wave.  During step t the fragments of step t + 1 are decoded, one group of
    // fragments after every MFMA; the raw codes of the next stage are read at the start of step 3 (every fragment of
    // this stage has been decoded by then) behind the barrier that opens that stage, and step 3 decodes its first
    // fragments.  The copies of stage s + DIST are issued during steps 0..2, into the buffer of stage s - 1, which
    // every wave left before the barrier that opened stage s.
    int buf = 0;
    auto ring_next = [](int b) { return b == C::NSTAGE - 1 ? 0 : b + 1; };
    // RAGGED: the scale bytes of stage s+1 are picked out of their windows during step 1 (read) and 2 (write); tail_tag: the stage
    // before one whose windows or blocks may pass the end (the last two), all others know that they are whole.
    // left_tag: stages behind this one, up to DIST = 2: the last two stages issue no copies and the last one reads and decodes nothing for a
    // next one.  (Both used to go on with the last stage, whose copies the end of the kernel then waited for: 2.8 % of the time on average
    // over 140 problems, 5 % where K' <= 4500, 20 for each tile.  With the last stages taken care of, a ring of four stages is still 1 % slower and
    // one of five 1.5 %; the barrier and the reads of the next stage a k-step earlier 1.7 %.)
    uint3 win[RAG ? C::NSW : 1];
    auto run_stage = [&](int s, auto tail_tag, auto left_tag) {
        constexpr bool TAIL = decltype(tail_tag)::value;
        constexpr int LEFT = decltype(left_tag)::value;
        const int buf1 = ring_next(buf), buf2 = buf == 0 ? C::NSTAGE - 1 : buf - 1;
        int fetch = s + C::DIST;        // opaque: see gemm_staged_kernel
        asm("" : "+s"(fetch));
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (RAG && LEFT > 0) {
                uint8_t* next = lds + buf1 * C::STAGE_BYTES;
                if (t == 1) {
                    wait_vmcnt<C::NA + C::NW + (LEFT == 2 ? (C::NDMA + 2) / 3 : 0)>();
#pragma unroll
                    for (int d = 0; d < C::NSW; ++d)
                        win[d] = windows.gather(d, next + C::WINDOWS, TAIL, lds + C::PATCH + 4 * KS * (s + 1 - patch_from));
                }
                if (t == 2)
#pragma unroll
                    for (int d = 0; d < C::NSW; ++d) windows.put(d, win[d], next + C::A_SCALES, TAIL, s + 1);
            }
            if (t == 3 && LEFT > 0) {
                if constexpr (REG) {
                    reg_commit(s + 1, buf1);       // fetched since step 3 of the stage before
                    wait_lgkmcnt0();
                } else {
                    wait_vmcnt<LEFT == 2 ? (C::DIST - 1) * C::NDMA : 0>();
                    if constexpr (RAG) wait_lgkmcnt0();
                }
                wg_barrier();
                read_raw(lds + buf1 * C::STAGE_BYTES, share_missing && LEFT == 1);
                if constexpr (REG && LEFT == 2) reg_issue(s + 2);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int p = 0; p < P; ++p) {
#pragma unroll
                for (int gidx = (p * G) / P; gidx < ((p + 1) * G) / P; ++gidx)
                    if (t < 3 || LEFT > 0) decode_frag(gidx, (t + 1) & 3);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = MPG * p; q < MPG * p + MPG; ++q) {
                    const int i = q / WN, j = q % WN;
                    // weights as the row operand: see store_fragment
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[t & 1][j], fa[t & 1][i], acc[i][j], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (!REG && t < 3 && LEFT == 2) {
#pragma unroll
                    for (int d = 0; d < C::NDMA; ++d)
                        if ((d * 3) / C::NDMA == t && (d - (t * C::NDMA + 2) / 3) == p) issue_one(d, fetch, buf2);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        buf = buf1;
    };
    static_assert((C::NDMA + 2) / 3 <= P, "the copies of a stage are spread over the MFMAs of three k-steps");

    if constexpr (REG) {
        reg_issue(0);
        reg_commit(0, 0);
        reg_issue(min(1, nstage - 1));
        wait_lgkmcnt0();
    } else {
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
    }
    wg_barrier();
    read_raw(lds, share_missing && nstage == 1);
#pragma unroll
    for (int gidx = 0; gidx < G; ++gidx) decode_frag(gidx, 0);
    using Rag = std::integral_constant<bool, RAG>;
    int s = 0;
    for (; s < (RAG ? min(patch_from - 1, nstage - 2) : nstage - 2); ++s) run_stage(s, std::false_type{}, std::integral_constant<int, 2>{});
    if constexpr (RAG)
        for (; s < nstage - 2; ++s) run_stage(s, std::true_type{}, std::integral_constant<int, 2>{});
    if (nstage > 1) run_stage(nstage - 2, Rag{}, std::integral_constant<int, 1>{});
    run_stage(nstage - 1, std::false_type{}, std::integral_constant<int, 0>{});
    wait_vmcnt<0>();                            // no copy may still be in flight when the LDS is released

    // ---- the KS partial tiles of a sub-tile are added through the LDS: in round rho every wave hands the fragments
    // owned by wave kh + rho (same sub-tile) over and adds what wave kh - rho left for it
    float* xch = reinterpret_cast<float*>(lds);
    auto region = [&](int k_share) { return xch + ((k_share * (GM * GN) + wq) * C::OWN) * 1024; };
#pragma unroll
    for (int rho = 1; rho < KS; ++rho) {
        const int dst = (kh + rho) % KS, src = (kh + KS - rho) % KS;
        wait_lgkmcnt0();                        // this wave's reads of the ring / of the previous round have returned
        wg_barrier();                           // ring (or the previous round's regions) no longer read by anyone
#pragma unroll
        for (int f = 0; f < WM * WN; ++f)
            if (f % KS == dst) {                // uniform over the wave
                float* slot = region(kh) + (f / KS) * 1024;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4*>(slot + (q * 64 + lane) * 4) =
                        make_float4(acc[f / WN][f % WN][4 * q], acc[f / WN][f % WN][4 * q + 1], acc[f / WN][f % WN][4 * q + 2],
                                    acc[f / WN][f % WN][4 * q + 3]);
            }
        wait_lgkmcnt0();
        wg_barrier();
#pragma unroll
        for (int f = 0; f < WM * WN; ++f)
            if (f % KS == kh) {
                const float* slot = region(src) + (f / KS) * 1024;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 v = *reinterpret_cast<const float4*>(slot + (q * 64 + lane) * 4);
                    acc[f / WN][f % WN][4 * q] += v.x;
                    acc[f / WN][f % WN][4 * q + 1] += v.y;
                    acc[f / WN][f % WN][4 * q + 2] += v.z;
                    acc[f / WN][f % WN][4 * q + 3] += v.w;
                }
            }
    }
    const int m0 = wg_m0 + wrow0, n0 = wg_n0 + wcol0;
#pragma unroll
    for (int f = 0; f < WM * WN; ++f)
        if (f % KS == kh) store_fragment(acc[f / WN][f % WN], m0 + 32 * (f / WN), n0 + 32 * (f % WN), r, h, M, N, alpha, y, ldy);
}

template <int WM, int WN, int GM, int GN, int KS, int MODE, typename OutT>
arcq_status launch_ksplit(const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes, const uint8_t* w_scales,
                          int M, int N, int nbk, float alpha, OutT* y, int64_t ldy, hipStream_t stream) {
    using C = KsplitCfg<WM, WN, GM, GN, KS, MODE>;
    auto kern = gemm_ksplit_kernel<WM, WN, GM, GN, KS, OutT, MODE>;
    static std::atomic<uint64_t> lds_raised{0};
    if (arcq_status st = raise_lds_limit(reinterpret_cast<const void*>(kern), lds_raised)) return st;
    const int tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(C::NT), C::LDS_BYTES, stream, a_codes, a_scales, w_codes, w_scales,
                       M, N, nbk, alpha, y, ldy, tiles_m, tiles_n, tile_group_rows(tiles_m, tiles_n));
    return check_launch("gemm_ksplit_kernel");
}

template <int MODE, typename OutT>
arcq_status launch_ksplit_typed(int rows, int cols, const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                                const uint8_t* w_scales, int M, int N, int nbk, float alpha, OutT* y, int64_t ldy,
                                hipStream_t stream) {
#define ARCQ_KSPLIT(WM_, WN_, GN_)                  \
    if (rows == 32 * WM_ && cols == 32 * WN_ * GN_) \
    return launch_ksplit<WM_, WN_, 1, GN_, 4, MODE>(a_codes, a_scales, w_codes, w_scales, M, N, nbk, alpha, y, ldy, stream)
    ARCQ_KSPLIT(2, 1, 1);
    ARCQ_KSPLIT(2, 2, 1);
    ARCQ_KSPLIT(3, 2, 1);
    ARCQ_KSPLIT(4, 2, 1);
    ARCQ_KSPLIT(2, 2, 2);
    ARCQ_KSPLIT(3, 2, 2);
#undef ARCQ_KSPLIT
    return launch_ksplit<2, 4, 2, 1, 4, MODE>(a_codes, a_scales, w_codes, w_scales, M, N, nbk, alpha, y, ldy, stream);     // 128 x 128
}

}  // namespace

// The tile that takes the least time, and that time in us; rows = 0 and a time beyond any other's where none serves the problem.
// Only tiles that cover it with at most one workgroup per compute unit (256) are looked at: with more, a second round costs
// as much as the first; and with 32 at least, below which K' is better split across workgroups.  The time of a tile over K' is
// start + stages (alone + shared x workgroups / 256): a workgroup takes longer the more of the chip is busy (clock, and the
// weights' way from HBM); rows off the grid of 64 have their windows of scale bytes, 0.5 us.  Fitted to 6700 problems (M = 33 .. 8000, N = 16 ..
// 30000, K' = 512 .. 30000, weights from HBM), each path of each timed: 4 to 8 % rms.  The choice among these, the streaming kernel and
// the tiles of gemm.hip by the modelled times is 2 % from the best of all on average, where fixed limits of 144 to 256 workgroups on five
// tile shapes were 5 %; eleven of the 6700 are more than 4 % slower than with those limits, 1000 more than 4 % faster.
// by_value: with what it cost then (single, on a full chip) that values were stored one by one where weight rows are no multiple of four.
// They are stored by fours at any address now.  The rule keeps the price because it decides about splitting K' across workgroups, and with it
// about workspaces; plan_gemm_parts asks without it where it matters otherwise: for what is streamed, and from K' = 1024 on by the times.
// 96 x 128 tiles are left out where they pad more rows than 128 x 128: what is multiplied in vain costs clock that the model does
// not know of (195 x 10832 over K' = 12096: 90.6 us against 81.8).
KsplitTile gemm_ksplit_best(int64_t M, int64_t N, int64_t Kp, bool by_value) {
    struct Tile {
        int rows, cols;
        double start, alone, shared, single;
    };
    static constexpr Tile tiles[] = {{64, 32, 4.1, 0.421, 0.089, 1.1}, {64, 64, 4.95, 0.484, 0.200, 1.95}, {96, 64, 6.1, 0.641, 0.250, 2.65},
                                     {64, 128, 5.4, 0.759, 0.461, 3.7}, {128, 64, 7.0, 0.818, 0.209, 3.4}, {96, 128, 6.9, 0.966, 0.533, 5.1},
                                     {128, 128, 7.9, 1.206, 0.598, 6.8}};
    KsplitTile best = {0, 0, 1e30, false};
    const int64_t nbk = Kp >> 4;
    if (nbk < 32) return best;                            // at least two stages
    if ((uint64_t)M * (uint64_t)nbk * 8 >= 0xFFFF0000ull || (uint64_t)N * (uint64_t)nbk * 8 >= 0xFFFF0000ull) return best;
    for (const Tile& t : tiles) {
        const int64_t tiles_m = (M + t.rows - 1) / t.rows, wgs = tiles_m * ((N + t.cols - 1) / t.cols);
        if (wgs > 256 || wgs < 32) continue;
        const bool added = t.cols == 128 && t.rows < 128;   // 64 x 128 and 96 x 128: see plan_gemm
        if (!added && (wgs >= 144 || (t.cols == 32 && M > 64 && nbk <= 544))) best.ample = true;
        if (t.rows == 96 && t.cols == 128 && tiles_m * 96 > (M + 127) / 128 * 128) continue;
        const double fill = (double)wgs / 256.0;
        const double c = t.start + (by_value && (N & 3) ? t.single * (0.2 + 0.8 * fill) : 0.0) + ((Kp & 63) ? 0.5 : 0.0) +
                         (double)((nbk + 15) / 16) * (t.alone + t.shared * fill);
        if (c < best.us) {
            best.rows = t.rows;
            best.cols = t.cols;
            best.us = c;
        }
    }
    return best;
}

arcq_status launch_gemm_ksplit(int rows, int cols, const uint8_t* a_codes, const uint8_t* a_scales, const uint8_t* w_codes,
                               const uint8_t* w_scales, int64_t M, int64_t N, int64_t Kp, float alpha, void* y, int y_dtype,
                               int64_t ldy, hipStream_t stream) {
    const int nbk = (int)(Kp >> 4);
    // whole pieces need rows that start on 16-byte boundaries (K' a multiple of 64 covers the scale bytes too); scale windows need
    // the base of the scale bytes on a dword (256 x 4096 over K' = 4352 / 4368: 14.6 / 16.3 us; through registers 18.5)
    const bool copies = (nbk & 3) == 0 &&
                        ((reinterpret_cast<uintptr_t>(a_codes) | reinterpret_cast<uintptr_t>(w_codes)) & 15) == 0 &&
                        ((reinterpret_cast<uintptr_t>(a_scales) | reinterpret_cast<uintptr_t>(w_scales)) & 3) == 0;
    const bool windows = ((reinterpret_cast<uintptr_t>(a_scales) | reinterpret_cast<uintptr_t>(w_scales)) & 3) == 0;
    auto launch = [&](auto* out) {
        return copies    ? launch_ksplit_typed<COPIES>(rows, cols, a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, out, ldy, stream)
               : windows ? launch_ksplit_typed<RAGGED>(rows, cols, a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, out, ldy, stream)
                         : launch_ksplit_typed<REGS>(rows, cols, a_codes, a_scales, w_codes, w_scales, (int)M, (int)N, nbk, alpha, out, ldy, stream);
    };
    return y_dtype == ARCQ_DTYPE_F16 ? launch(static_cast<_Float16*>(y)) : launch(static_cast<float*>(y));
}

}  // namespace arcq
