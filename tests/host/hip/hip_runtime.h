// What the device headers under test need of the HIP runtime, for a host compiler.
#pragma once
#include <stdint.h>

#define __host__
#define __device__
#define __forceinline__ inline

struct uint2 { uint32_t x, y; };
struct uint3 { uint32_t x, y, z; };
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
inline uint3 make_uint3(uint32_t x, uint32_t y, uint32_t z) { return {x, y, z}; }
template <typename T> inline T min(T a, T b) { return b < a ? b : a; }
// bytes `shift` to `shift` + 3 of the eight of high : low
inline uint32_t __builtin_amdgcn_alignbyte(uint32_t high, uint32_t low, uint32_t shift) {
    return (uint32_t)(((uint64_t)high << 32 | low) >> (8 * (shift & 3)));
}
