// The rows of codes that a tile of the MXFP4 and bf16 kernels has of one operand, copied straight into LDS through a buffer descriptor (lds_dma.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lds_dma.h"

namespace arcq {

// A copy of the whole workgroup takes ROWS rows, copy d those from ROWS d of the tile on; rows past the edge of the operand arrive as zeros (never
// stored).  A copy that has no row left starts at the last one, so that its scalar offset stays within the operand; all but that row's lanes are past it.
// (Loop-invariant, as the row offsets themselves: the loops of the tiles have the instructions that they had without it.)
template <int ROWS>
struct CodeRows {
    buffer_t rows;
    uint32_t pitch, last;       // bytes of a row; last row, counted from the tile's first

    __device__ __forceinline__ CodeRows(const uint8_t* codes, int all, int first, uint32_t pitch_)
        : rows(buffer_of(codes + (int64_t)first * pitch_, (uint32_t)(all - first) * pitch_)), pitch(pitch_), last((uint32_t)(all - first) - 1u) {}

    // voffset: row of the copy times pitch, and the bytes into the row that are the lane's own; column < pitch: those of every lane
    __device__ __forceinline__ void issue(int d, uint32_t voffset, uint32_t column, uint32_t lds_wave_base) const {
        copy16(rows, voffset, column, min((uint32_t)(d * ROWS), last) * pitch, lds_wave_base);
    }
};

}  // namespace arcq
