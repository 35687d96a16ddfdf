// Scale bytes of the MXFP4 tiles (eight per row and unit of 256 k), through direct-to-LDS copies that fetch those of several units at a time.
//
// Two words a row and unit, as a copy of their own, cost as many instructions as a quarter of the codes and the address unit of the CU as much as all of them
// (71 cycles an instruction of 32 rows, against 17 to 20 for eight lines of 128 bytes).  32 bytes a row cost 79 cycles for 32 rows in pieces of 16 bytes a
// lane, and 8 cycles for eight rows in words: pieces, a quarter of the instructions, in the loops, and words before them, where a wave waits
// for the first chunk.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lds_dma.h"

namespace arcq {

// Units are counted from the first one of the workgroup's run here; `first_byte` is where that one's scale bytes are in a row.
// Copies of rows past the edge of an operand, and of chunks past the end of its last row, start at its end at the latest: a scalar offset beyond it would
// leave the range check of a buffer nothing to compare with (lds_dma.h).

// As few copies a wave and group as let `waves` waves with rows of one operand each have all rows.
constexpr int copies_of_group(int copies_a, int copies_w, int groups, int waves) {
    int ng = 1;
    while ((copies_a + groups * ng - 1) / (groups * ng) + (copies_w + groups * ng - 1) / (groups * ng) > waves) ++ng;
    return ng;
}

// Rows of scale bytes that start on dwords (blocks per row a multiple of four): CHUNK bytes of every row (16 or 32), those of Q units, are
// one chunk, and the readers take the bytes of their unit straight out of a ring of two chunks.
// A chunk is copied in Q groups, one a unit, behind the barrier that opens the next unit: unit u brings group (u + 1) % Q of chunk
// (u + 1) / Q + 1.  The chunk that was in its place was last read before that barrier, and the copies of unit u have landed when the code copies
// of unit u + 3 are all that is younger: a unit before the chunk is read.
// Every wave has rows of one operand, the first ones those of A, so that a copy takes no decisions; left-over waves have none.
template <int BM, int BN, int NT, int CHUNK>
struct ScaleChunks {
    static constexpr int Q = CHUNK / 8, LANES = CHUNK / 16, R = 64 / LANES;         // units of a chunk, lanes of a row, rows of a copy
    static constexpr int TA = (BM + R - 1) / R, TW = (BN + R - 1) / R, WAVES = NT / 64;
    static constexpr int NG = copies_of_group(TA, TW, Q, WAVES);    // copies of a wave in each group
    static constexpr int WA = (TA + Q * NG - 1) / (Q * NG), WW = (TW + Q * NG - 1) / (Q * NG);      // waves with rows of A, of W
    static constexpr int NA = (TA + WA - 1) / WA, NW = (TW + WW - 1) / WW;          // copies of such a wave
    static constexpr int SHARE = WAVES >= 2 * (WA + WW) && NA == NW ? 2 : 1;        // waves that share the first chunk's copies of a wave
    static constexpr int W_ROWS = WA * NA * R;                      // row that the W tile's rows start at
    static constexpr int BYTES = (W_ROWS + WW * NW * R) * CHUNK;

    buffer_t rows;              // scale bytes of this wave's operand from the wave's first row on
    uint32_t voffset;           // of this lane
    uint32_t step, first_byte;
    uint32_t to, copies;        // this wave's place in a chunk, and its copies
    bool active;                // whether it has any
    uint32_t share;             // of the first chunk

    // Words of a row are exchanged by the row's number, so that the eight bytes of 32 rows, which an instruction reads, are on more different banks
    // (8192 x 8192 over K' = 29696, all rows alike 1068 us, every other eight rows exchanged 1012).
    __device__ __forceinline__ static uint32_t exchanged(uint32_t row) { return LANES == 2 ? row >> 3 & 1u : 0u; }
    // a unit's bytes of a row: at row_at(row) ^ at(unit) behind base(unit), rows of the W tile from W_ROWS on
    __device__ __forceinline__ static uint32_t row_at(uint32_t row) { return CHUNK * row + 16u * exchanged(row); }
    __device__ __forceinline__ static uint32_t at(int unit) { return (uint32_t)(unit % Q * 8); }
    __device__ __forceinline__ static uint32_t base(int unit) { return (uint32_t)(unit / Q & 1) * BYTES; }

    __device__ __forceinline__ ScaleChunks(const uint8_t* a, const uint8_t* w, int M, int N, int nb, int m0, int n0, uint32_t lane, uint32_t wave,
                                           int first_byte_) : step((uint32_t)(R * nb)), first_byte((uint32_t)first_byte_) {
        active = WA + WW == WAVES || wave < (uint32_t)(WA + WW);
        share = SHARE > 1 && !active ? 1u : 0u;
        if (SHARE > 1) wave %= (uint32_t)(WA + WW);
        const bool of_a = wave < (uint32_t)WA;
        copies = of_a ? NA : NW;
        const uint32_t in_tile = of_a ? wave * (NA * R) : (wave - WA) * (NW * R);
        to = (in_tile + (of_a ? 0u : (uint32_t)W_ROWS)) * CHUNK;
        const uint32_t bytes = (uint32_t)(of_a ? M : N) * (uint32_t)nb, start = ((uint32_t)(of_a ? m0 : n0) + in_tile) * (uint32_t)nb;
        // (a wave whose rows are all past the edge has none)
        rows = buffer_of((of_a ? a : w) + min(start, bytes), bytes - min(start, bytes));
        voffset = lane / LANES * (uint32_t)nb + 16u * (lane % LANES ^ exchanged(lane / LANES));
    }
    // The first chunk, in words, of which waves without rows take a share (128 x 128 tiles: eight copies a wave instead of sixteen for half of the waves,
    // each behind four to seven scalar instructions).
    __device__ __forceinline__ void issue_first(uint32_t lane, uint32_t ring) const {
        if (SHARE == 1 && !active) return;
        constexpr int WORDS = CHUNK / 4, RW = 64 / WORDS;           // lanes of a row, rows of a copy: 8 and 8, 4 and 16
        constexpr int MOST = (NA > NW ? NA : NW) * R / RW / SHARE;
        static_assert(MOST % 2 == 0, "a share begins with an even copy");
        const uint32_t row = lane / WORDS, word = lane % WORDS;
        const uint32_t even = row * (step / R) + 4u * word, odd = row * (step / R) + 4u * (word ^ (LANES == 2 ? 4u : 0u));
        const uint32_t all = copies * (R / RW);                     // (a wave with fewer than the others repeats its last two, which are unlike each other)
#pragma unroll
        for (int k = 0; k < MOST; ++k) {
            const uint32_t i = NA == NW ? MOST * share + k : min((uint32_t)k, all - 2u + (k & 1));
            copy4(rows, k & 1 ? odd : even, min(first_byte + i * (RW * (step / R)), rows[2]), ring + to + i * (RW * CHUNK));
        }
    }
    // copy i of a group of a chunk (a wave with fewer copies than the groups have repeats its last one)
    __device__ __forceinline__ void issue(int i, int group, int chunk, uint32_t ring) const {
        if (!active) return;
        const uint32_t k = min((uint32_t)(group * NG + i), copies - 1u);
        copy16(rows, voffset, min(first_byte + (uint32_t)(CHUNK * chunk) + k * step, rows[2]), ring + (uint32_t)(chunk & 1) * BYTES + to + k * (R * CHUNK));
    }
};

// Rows of scale bytes that start at any address (K' a multiple of the block only).
//
// A copy needs dword-aligned addresses, and the scale bytes of chunk c, units Q c to Q c + Q - 1, of row m start at byte m * nb + first_byte + 8 Q c of the
// operand (nb blocks per row).  Every row fetches a window of 32 bytes (three units; 16 for one) that
// starts at that address rounded down to a dword: the wanted bytes lie phase = m * nb % 4 bytes into the window, the same for
// every chunk, and rows a multiple of four apart have the same phase.  Once a window has landed, lanes of the wave that fetched it read the bytes
// of one unit, shift them and write them to their place in the unit (`gather` and `put`, a few instructions per thread and
// unit), so that the GEMM loop finds the layout it knows.
// There are two buffers.  A chunk is copied in Q groups, one a unit, behind the barrier that opens the next unit: unit u brings group (u + 2) % Q of chunk
// (u + 2) / Q + 1, once the wave has picked out the bytes of unit u + 1.  (Ahead of the unit's code copies, one group later: up to 6 % slower where
// there are three ring slots, whose copies then have less time to land.)
//
// The operand's last one to three bytes, where they are no word, are read one by one at the start into `patch`, a word per operand.
template <int BM, int BN, int NT, int UNITS>
struct ScaleChunkWindows {
    static_assert(UNITS == 1 || UNITS == 3, "16 or 32 bytes a row");
    static constexpr int Q = UNITS, LANES = Q == 3 ? 2 : 1, WINDOW = 16 * LANES, R = 64 / LANES;
    static constexpr int ROWS = NT / LANES;                         // rows of a copy of the whole workgroup
    static constexpr int NSA = (BM + ROWS - 1) / ROWS, NS = NSA + (BN + ROWS - 1) / ROWS;       // copies per thread and chunk
    static constexpr int NG = (NS + Q - 1) / Q;                     // and group
    static constexpr int G = (NS + LANES - 1) / LANES;              // gathers per thread and unit: a row a lane
    static constexpr int BYTES = NS * ROWS * WINDOW;                // of a chunk
    static constexpr int DENSE_BYTES = NS * ROWS * 8;               // of the wanted bytes: 8 per row of A, then of W
    static constexpr int DENSE_W = NSA * ROWS * 8;
    static constexpr int PATCH = 16;
    static constexpr int MIN_NB = 16;                               // shortest rows served

    buffer_t a, w;              // scale bytes of the operands from the tiles' first rows on, whole words
    uint32_t voffset;           // of this lane
    uint32_t nb, first_byte, tid, wave_slot;

    __device__ __forceinline__ ScaleChunkWindows(const uint8_t* a_scales, const uint8_t* w_scales, int M, int N, int nb_, int m0, int n0, uint32_t tid_,
                                                 uint32_t wave_slot_, int first_byte_)
        : a(buffer_of(a_scales + (uint32_t)m0 * (uint32_t)nb_, ((uint32_t)M * (uint32_t)nb_ & ~3u) - (uint32_t)m0 * (uint32_t)nb_)),
          w(buffer_of(w_scales + (uint32_t)n0 * (uint32_t)nb_, ((uint32_t)N * (uint32_t)nb_ & ~3u) - (uint32_t)n0 * (uint32_t)nb_)),
          voffset((tid_ / LANES * (uint32_t)nb_ & ~3u) + 16u * (tid_ % LANES)), nb((uint32_t)nb_), first_byte((uint32_t)first_byte_), tid(tid_),
          wave_slot(wave_slot_) {}

    // whether the tile has rows that touch a word which is not whole
    __device__ __forceinline__ static bool needs_patch(int M, int N, int nb, int m0, int n0) {
        return (m0 + BM >= M && (M * nb & 3) != 0) || (n0 + BN >= N && (N * nb & 3) != 0);
    }
    // first unit of a row (not of the run) that may touch the operand's last word; not the row's first, and at most one follows
    __device__ __forceinline__ static int patch_from(int nb) { return (nb - 6) / 8; }

    __device__ __forceinline__ void issue(int d, int chunk, uint32_t windows) const {
        const buffer_t& rows = d < NSA ? a : w;
        copy16(rows, voffset, min(first_byte + (uint32_t)(8 * Q * chunk) + (uint32_t)((d < NSA ? d : d - NSA) * ROWS) * nb, rows[2]),
               windows + (uint32_t)(chunk & 1) * BYTES + 16u * ((uint32_t)(d * NT) + wave_slot));
    }
    __device__ __forceinline__ void issue_chunk(int chunk, uint32_t windows) const {
#pragma unroll
        for (int d = 0; d < NS; ++d) issue(d, chunk, windows);
    }
    __device__ __forceinline__ void issue_group(int group, int chunk, uint32_t windows) const {     // (the last group may repeat the last copy)
#pragma unroll
        for (int i = 0; i < NG; ++i) issue(min(group * NG + i, NS - 1), chunk, windows);
    }

    __device__ __forceinline__ static void fill_patch(const uint8_t* a_scales, const uint8_t* w_scales, int M, int N, int nb, uint32_t tid, uint8_t* area) {
        if (tid < 8) {
            const uint32_t total = (uint32_t)(tid < 4 ? M : N) * (uint32_t)nb, at = (total & ~3u) + (tid & 3u);
            area[tid] = at < total ? (tid < 4 ? a_scales : w_scales)[at] : (uint8_t)0;
        }
    }

    // ---- a lane's share of gather g: a row's eight bytes, of the rows that its wave copied
    __device__ __forceinline__ uint32_t copy_of(int g) const {      // (lanes of the last gather without a copy of their own repeat the last one)
        const uint32_t i = LANES == 2 ? 2u * g + (tid >> 5 & 1u) : (uint32_t)g;
        return NS % LANES ? min(i, (uint32_t)NS - 1u) : i;
    }
    __device__ __forceinline__ uint32_t row_of(int g) const { return copy_of(g) * (uint32_t)ROWS + wave_slot / LANES + tid % R; }       // rows of A, then of W

    // The three words that hold them, of unit Q chunk + j.  tail: the unit is the row's patch_from() or later.
    __device__ __forceinline__ uint3 gather(int g, int chunk, int j, const uint8_t* windows, bool tail, const uint8_t* patch) const {
        const uint32_t row = row_of(g);
        const uint8_t* src = windows + (chunk & 1) * BYTES + WINDOW * row + 8 * j;
        const uint2 lo = *reinterpret_cast<const uint2*>(src);
        uint3 v = make_uint3(lo.x, lo.y, *reinterpret_cast<const uint32_t*>(src + 8));
        if (tail) {
            const bool of_a = copy_of(g) < (uint32_t)NSA;
            const uint32_t from = ((row - (of_a ? 0u : (uint32_t)(NSA * ROWS))) * nb & ~3u) + first_byte + (uint32_t)(8 * (Q * chunk + j));
            const uint32_t end = of_a ? a[2] : w[2];
            const uint32_t last = *reinterpret_cast<const uint32_t*>(patch + (of_a ? 0 : 4));
            if (from >= end) v.x = last;
            if (from + 4 >= end) v.y = last;
            if (from + 8 >= end) v.z = last;
        }
        return v;
    }

    // Their shift and write.  unit: of the row.  Bytes past the end of the row become 0 (tail).
    __device__ __forceinline__ void put(int g, const uint3& v, uint8_t* dense, bool tail, int unit) const {
        const uint32_t phase = tid % R * nb & 3u;
        uint2 out = make_uint2(__builtin_amdgcn_alignbyte(v.y, v.x, phase), __builtin_amdgcn_alignbyte(v.z, v.y, phase));
        if (tail) {
            const int left = (int)nb - 8 * unit;        // blocks of the row from the first of the eight on
            if (left < 8) {
                uint64_t all = (uint64_t)out.y << 32 | out.x;
                all = left <= 0 ? 0 : all & (~0ull >> (64 - 8 * left));
                out = make_uint2((uint32_t)all, (uint32_t)(all >> 32));
            }
        }
        *reinterpret_cast<uint2*>(dense + row_of(g) * 8) = out;
    }
};

}  // namespace arcq
