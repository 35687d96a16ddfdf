// Scale bytes of operands whose rows of scale bytes start at any address (K' a multiple of the block only), through
// direct-to-LDS copies.
//
// A copy needs dword-aligned addresses, and row m's scale bytes of stage s start at byte m * nb + STEP * s of the operand
// (nb blocks per row, STEP scale bytes per row and stage, 8 or 16).  Every row therefore fetches a window of 16 or 32 bytes that
// starts at that address rounded down to a dword: the wanted bytes lie phase = (m * nb) % 4 bytes into the window, the same for
// every stage, and rows a multiple of four apart have the same phase.  Once a window has landed, the lane that fetched it reads
// it, shifts it and writes the wanted bytes to their place in the stage (`gather` and `put`, a few instructions per thread and
// stage, placed where the window landed long ago), so that the GEMM loops find the layout they know.
// (Leaving the shift to the readers costs more, 256 x 4096 over K' = 4352 forced onto this path: 17.7 us with word pairs and a
// permute, 15.0 with words at any address while they happen to be aligned and 21.5 when they are not; 14.4 without windows.)
//
// The windows of the operand's last row pass its end in the last two stages at most.  Copies are clamped to the operand; that
// row's bytes come from `patch` instead, read one by one at the start.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lds_dma.h"

namespace arcq {

template <int BM, int BN, int NT, int STEP>
struct ScaleWindows {
    static_assert(STEP == 8 || STEP == 16, "scale bytes per row and stage");
    static constexpr int LPR = STEP / 8;                            // slots per row: 16 bytes of the window, 8 wanted bytes
    static constexpr int PITCH = 16 * LPR;                          // bytes of a window
    static constexpr int A_SLOTS = (BM * LPR + 63) / 64 * 64;       // whole waves, so that a wave copies from one operand
    static constexpr int NS = (A_SLOTS + BN * LPR + NT - 1) / NT;   // copies per thread and stage
    static constexpr int BYTES = NS * NT * 16;                      // of the windows of a stage
    static constexpr int DENSE_BYTES = NS * NT * 8;                 // of the wanted bytes: STEP per row of A, then of W
    static constexpr int DENSE_W = A_SLOTS * 8;
    static constexpr int PATCH = 32 * LPR;                          // bytes kept per operand: two windows, STEP apart
    static constexpr int MIN_NB = PITCH;                            // shortest rows served

    const uint8_t *a, *w;       // scale bytes of the operands, dword-aligned
    int M, N, nb, m0, n0;       // rows, blocks per row, first rows of the tile (multiples of four)
    uint32_t tid, wave_slot;    // thread, and the first thread of its wave as a scalar

    // first stage in which the last row's window may pass the end of the operand; it is not the first stage of the row, and
    // at most one stage follows
    __device__ __forceinline__ static int patch_from(int nb) { return (nb - PITCH) / STEP + 1; }

    __device__ __forceinline__ bool is_a(int d) const { return (uint32_t)(d * NT) + wave_slot < (uint32_t)A_SLOTS; }
    __device__ __forceinline__ uint32_t slot(int d) const {         // within the operand's slots
        return (uint32_t)(d * NT) + tid - (is_a(d) ? 0u : (uint32_t)A_SLOTS);
    }

    __device__ __forceinline__ void issue(int d, int stage, uint32_t lds_base) const {
        const uint32_t at = slot(d);
        const int rows = is_a(d) ? M : N;
        const uint32_t row = (uint32_t)min((is_a(d) ? m0 : n0) + (int)(at / LPR), rows - 1);
        const uint32_t off = row * (uint32_t)nb + (uint32_t)(STEP * stage) + 16u * (at % LPR);
        const uint32_t limit = (uint32_t)rows * (uint32_t)nb - 16u;
        dma16(is_a(d) ? a : w, min(off, limit) & ~3u, lds_base + 16u * ((uint32_t)(d * NT) + wave_slot));
    }

    // The bytes from the last row's first window that may pass the end on, zeros past the end.  area: 2 * PATCH bytes of LDS.
    __device__ __forceinline__ void fill_patch(uint8_t* area) const {
        if (tid < 2 * PATCH) {
            const bool of_a = tid < PATCH;
            const uint32_t total = (uint32_t)(of_a ? M : N) * (uint32_t)nb;
            const uint32_t at = ((total - (uint32_t)nb + (uint32_t)(STEP * patch_from(nb))) & ~3u) + (tid & (PATCH - 1));
            area[tid] = at < total ? (of_a ? a : w)[at] : (uint8_t)0;
        }
    }

    // The three words that hold this thread's eight wanted bytes of copy d of a landed stage.  tail: the stage is
    // patch_from() + 0 or 1, patch its window in the patch area.
    __device__ __forceinline__ uint3 gather(int d, const uint8_t* windows, bool tail, const uint8_t* patch) const {
        const uint8_t* src = windows + 16 * (d * NT + (int)tid);
        if constexpr (LPR == 2) src -= 8 * (slot(d) & 1u);          // the second slot's bytes start in the middle of the window
        if (tail && (is_a(d) ? m0 : n0) + (int)(slot(d) / LPR) == (is_a(d) ? M : N) - 1)
            src = patch + (is_a(d) ? 0 : PATCH) + 8 * (slot(d) % LPR);
        const uint2 lo = *reinterpret_cast<const uint2*>(src);
        return make_uint3(lo.x, lo.y, *reinterpret_cast<const uint32_t*>(src + 8));
    }

    // Their shift and write.  left: blocks of the row from the first of the eight on, where fewer than eight may be left (tail).
    // Bytes past the end become 0.  Blocks are copied two to a 16-byte piece: the last block of an odd row was
    // copied as the second one of its piece, so its byte moves up by one.
    __device__ __forceinline__ void put(int d, const uint3& v, uint8_t* dense, bool tail, int stage) const {
        const uint32_t phase = ((tid / LPR) * (uint32_t)nb) & 3u;
        uint2 out = make_uint2(__builtin_amdgcn_alignbyte(v.y, v.x, phase), __builtin_amdgcn_alignbyte(v.z, v.y, phase));
        if (tail) {
            const int left = nb - STEP * stage - 8 * (int)(slot(d) % LPR);
            if (left < 8) {
                uint64_t all = (uint64_t)out.y << 32 | out.x;
                all = left <= 0 ? 0 : all & (~0ull >> (64 - 8 * left));
                if (left > 0 && (left & 1)) {
                    const uint64_t below = (1ull << (8 * (left - 1))) - 1;
                    all = (all & below) | (all & ~below) << 8;
                }
                out = make_uint2((uint32_t)all, (uint32_t)(all >> 32));
            }
        }
        *reinterpret_cast<uint2*>(dense + 8 * (d * NT + (int)tid)) = out;
    }
};

}  // namespace arcq
