// Offline calibration (Section 3.2 "Adaptive Outlier Identification"): per-channel absolute maximum
// over calibration activations, then the channel order and the outlier count S.
//
// Statistics are fp32 values >= 0 held as their bit patterns, which order like unsigned integers:
// the running maximum is an integer atomic maximum and the sort key is the pattern itself.
#include "internal.h"

#include <hip/hip_fp16.h>

#include <cstring>

namespace arcq {

namespace {

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// |a|, |b| as fp16 bit patterns, element-wise maximum (patterns of non-negative halves order like integers)
__device__ __forceinline__ uint32_t absmax2(uint32_t acc, uint32_t v) {
    const u16x2 a = __builtin_bit_cast(u16x2, acc), b = __builtin_bit_cast(u16x2, v & 0x7FFF7FFFu);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(a, b));
}

// Four waves per workgroup: lane l of every wave owns the 8 channels 8 (64 blockIdx.x + l) .. + 7; wave w
// scans rows w, w + 4, ... of strip blockIdx.y with 16-byte loads (a wave instruction reads 1 KB of one
// row), eight rows in flight; the four waves combine through LDS and merge the maxima into the running statistic with
// integer atomic maxima (atomics on one address serialise in the L2, so there are few strips and one atomic per
// channel and strip).  A lane merges neighbouring channels with its neighbours, so that an atomic instruction covers two
// cache lines instead of sixteen, and leaves out the channels whose statistic, read when the workgroup
// started, is no smaller already: from the second batch on that is nearly all of them.
// HBM-bound: 2 bytes per element read once.
constexpr int ABSMAX_UNROLL = 8;
__global__ __launch_bounds__(256) void absmax_kernel(const uint16_t* __restrict__ x, int64_t ldx, int M, int K,
                                                     int rows_per_strip, uint32_t* __restrict__ colmax) {
    __shared__ uint4 part[4][64];
    const int tid = threadIdx.y * 64 + threadIdx.x, ch = blockIdx.x * 512 + 2 * tid;    // this thread merges channels ch, ch + 1
    const uint2 seen = ch < K ? make_uint2(colmax[ch], colmax[ch + 1]) : make_uint2(0, 0);
    const int c8 = min((int)(blockIdx.x * 64 + threadIdx.x), (K >> 3) - 1);     // surplus lanes repeat the last group
    const int m0 = blockIdx.y * rows_per_strip + threadIdx.y, m1 = min(M, (int)(blockIdx.y + 1) * rows_per_strip);
    const uint4* src = reinterpret_cast<const uint4*>(x + 8 * (int64_t)c8);
    const int64_t pitch16 = ldx >> 3;                       // row pitch in 16-byte units
    uint4 mx[ABSMAX_UNROLL];
#pragma unroll
    for (int u = 0; u < ABSMAX_UNROLL; ++u) mx[u] = make_uint4(0, 0, 0, 0);
    int m = m0;
    for (; m + 4 * (ABSMAX_UNROLL - 1) < m1; m += 4 * ABSMAX_UNROLL) {
        uint4 v[ABSMAX_UNROLL];
#pragma unroll
        for (int u = 0; u < ABSMAX_UNROLL; ++u) v[u] = src[(int64_t)(m + 4 * u) * pitch16];
#pragma unroll
        for (int u = 0; u < ABSMAX_UNROLL; ++u) {
            mx[u].x = absmax2(mx[u].x, v[u].x);
            mx[u].y = absmax2(mx[u].y, v[u].y);
            mx[u].z = absmax2(mx[u].z, v[u].z);
            mx[u].w = absmax2(mx[u].w, v[u].w);
        }
    }
    for (; m < m1; m += 4) {
        const uint4 v = src[(int64_t)m * pitch16];
        mx[0].x = absmax2(mx[0].x, v.x);
        mx[0].y = absmax2(mx[0].y, v.y);
        mx[0].z = absmax2(mx[0].z, v.z);
        mx[0].w = absmax2(mx[0].w, v.w);
    }
#pragma unroll
    for (int u = 1; u < ABSMAX_UNROLL; ++u) {
        mx[0].x = absmax2(mx[0].x, mx[u].x);
        mx[0].y = absmax2(mx[0].y, mx[u].y);
        mx[0].z = absmax2(mx[0].z, mx[u].z);
        mx[0].w = absmax2(mx[0].w, mx[u].w);
    }
    part[threadIdx.y][threadIdx.x] = mx[0];
    __syncthreads();
    const uint32_t* halves = reinterpret_cast<const uint32_t*>(part);   // [wave][pair of channels]
    uint32_t m2 = halves[tid];
#pragma unroll
    for (int w = 1; w < 4; ++w) m2 = absmax2(m2, halves[256 * w + tid]);
    const uint32_t lo = __float_as_uint(__half2float(__ushort_as_half((unsigned short)(m2 & 0xFFFFu))));
    const uint32_t hi = __float_as_uint(__half2float(__ushort_as_half((unsigned short)(m2 >> 16))));
    if (ch < K) {                                               // K is even
        if (lo > seen.x) atomicMax(colmax + ch, lo);
        if (hi > seen.y) atomicMax(colmax + ch + 1, hi);
    }
}

// Layer maximum, tau = 2^-3 max (exact), number of channels above tau, S rounded up to a block of 16, by one workgroup of
// 1024 threads.  info = {S, S_raw, bits(max), bits(tau)}.
// s_host (or null): S once more, for the host.
__device__ __forceinline__ void calib_stats(const uint32_t* __restrict__ colmax, int K, int32_t* __restrict__ info, int* part,
                                            int32_t* s_host) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t mx = 0;
    for (int k = tid; k < K; k += 1024) mx = max(mx, colmax[k]);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, m, 64));
    if (lane == 0) part[wave] = (int)mx;
    __syncthreads();
    uint32_t total = 0;
    for (int w = 0; w < 16; ++w) total = max(total, (uint32_t)part[w]);
    const float tau = __uint_as_float(total) * 0.125f;
    int cnt = 0;
    for (int k = tid; k < K; k += 1024) cnt += __uint_as_float(colmax[k]) > tau ? 1 : 0;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) cnt += __shfl_xor(cnt, m, 64);
    __syncthreads();
    if (lane == 0) part[wave] = cnt;
    __syncthreads();
    if (tid == 0) {
        int s_raw = 0;
        for (int w = 0; w < 16; ++w) s_raw += part[w];
        const int s = min(K, (s_raw + 15) / 16 * 16);
        info[0] = s;
        info[1] = s_raw;
        info[2] = (int32_t)total;
        info[3] = (int32_t)__float_as_uint(tau);
        if (s_host) __hip_atomic_store(s_host, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Stable ascending order by counting: the position of channel k is the number of channels that come
// before it (smaller statistic, or equal statistic and smaller index).  Every position is hit exactly
// once whatever the values, so the output is always a permutation.  K^2 comparisons, bound by the vector
// instructions (a compare and an add with carry each).  The first workgroup finds the layer's statistics instead, which took a
// launch of their own (5 us).
// HALVES: a workgroup ranks 32 channels, and its 16 waves take a sixteenth of the keys each, of which either half of a wave compares its
// own half with the 32 channels: 256 workgroups for K = 8192.  Keys of lower index come before an equal one, keys of higher index do
// not: patterns order like integers, so the former are compared with the channel's key + 1.
// Otherwise it ranks 64 channels, one per lane, against keys that are the same for all lanes and come through the scalar unit:
// 1.6 times fewer cycles a comparison, but 128 workgroups for K = 8192.  Both, us (HALVES first): K = 4096 6.3 and 9.2, 8192 10.8 and 14.5,
// 9216 18.4 and 15.6, 12288 23.9 and 19.4, 14336 27 and 22, 28672 101 and 63, 65536 449 and 250: beyond 8192 HALVES' workgroups are more than one a
// compute unit.
constexpr int HALVES_UP_TO = 8192;      // channels
template <bool HALVES>
__global__ __launch_bounds__(1024) void calib_select_kernel(const uint32_t* __restrict__ colmax, int K, int32_t* __restrict__ perm,
                                                            int32_t* __restrict__ info, int32_t* __restrict__ s_host) {
    __shared__ int part[16][64];
    if (blockIdx.x == 0) {
        calib_stats(colmax, K, info, &part[0][0], s_host);
        return;
    }
    constexpr int RANKED = HALVES ? 32 : 64;
    const int lane = threadIdx.x & 63, wave = HALVES ? (int)(threadIdx.x >> 6) : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int k0 = (blockIdx.x - 1) * RANKED, k = k0 + (lane & (RANKED - 1));
    const uint32_t mine = colmax[min(k, K - 1)];
    int before = 0;
    if constexpr (HALVES) {
        // slices of a multiple of 32 keys, so that a workgroup's channels lie in one; every bound is a multiple of 16
        const int slice = (K + 1023) / 1024 * 32;
        const int j0 = min((2 * wave + (lane >> 5)) * slice, K), j1 = min(j0 + slice, K);
        for (int j = j0; j < j1; j += 16) {
            // (the channels' own 32 keys, which need their indices as well, are left to the first wave)
            const uint32_t bound = j + 16 <= k0 ? mine + 1 : j >= k0 + RANKED ? mine : 0u;
            u32x4_a4 key[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) key[e] = *reinterpret_cast<const u32x4_a4*>(colmax + j + 4 * e);
#pragma unroll
            for (int e = 0; e < 16; ++e) before += key[e >> 2][e & 3] < bound ? 1 : 0;
        }
        if (wave == 0) {
            const int first = k0 + 16 * (lane >> 5);                // 16 keys for either half
            if (first < K)
#pragma unroll
                for (int e = 0; e < 16; ++e) before += colmax[first + e] < (first + e < k ? mine + 1 : mine) ? 1 : 0;
        }
        // (no pattern is greater than the greatest: every key of lower index comes before it)
        if (mine + 1 == 0) before += max(min(j1, k0) - j0, 0) + (wave == 0 ? min(max(k - k0 - 16 * (lane >> 5), 0), 16) : 0);
    } else {
        const int slice = (K + 1023) / 1024 * 64;               // a multiple of 64: a workgroup's channels lie in one slice
        const int j0 = min(wave * slice, K), j1 = min(j0 + slice, K);
        int j = j0;
        for (const int to = min(j1, max(j0, k0)); j < to; j += 16)      // (every bound is a multiple of 16)
#pragma unroll
            for (int e = 0; e < 16; ++e) before += colmax[j + e] <= mine ? 1 : 0;
        for (const int to = min(j1, max(j0, k0 + 64)); j < to; ++j) before += colmax[j] < mine || (colmax[j] == mine && j < k) ? 1 : 0;
        for (; j < j1; j += 16)
#pragma unroll
            for (int e = 0; e < 16; ++e) before += colmax[j + e] < mine ? 1 : 0;
    }
    part[wave][lane] = before;
    __syncthreads();
    if (threadIdx.x < RANKED && k < K) {
        int position = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) position += part[w][lane] + (HALVES ? part[w][lane + 32] : 0);
        perm[position] = k;
    }
}

}  // namespace

arcq_status launch_calib_absmax(const void* x, int64_t M, int64_t K, int64_t ldx, float* colmax, hipStream_t stream) {
    const int colblocks = (int)((K / 8 + 63) / 64);
    // about 1024 workgroups (4 per CU, 128 KB in flight per CU), strips of at least 32 rows
    int64_t rows_per_strip = (M * colblocks + 1023) / 1024;
    if (rows_per_strip < 32) rows_per_strip = 32;
    const int64_t strips = (M + rows_per_strip - 1) / rows_per_strip;
    hipLaunchKernelGGL(absmax_kernel, dim3(colblocks, (unsigned)strips), dim3(64, 4), 0, stream,
                       static_cast<const uint16_t*>(x), ldx, (int)M, (int)K, (int)rows_per_strip,
                       reinterpret_cast<uint32_t*>(colmax));
    return check_launch("absmax_kernel");
}

arcq_status launch_calib_select(const float* colmax, int64_t K, int32_t* perm, int32_t* info, int* S_host,
                                hipStream_t stream) {
    const uint32_t* keys = reinterpret_cast<const uint32_t*>(colmax);
    // Page-locked memory takes S from the kernel itself, at a multiple of four bytes; any other needs a copy, which the host waits for 10 us
    // longer (K = 8192: 31 against 22 us a call).
    int32_t* direct = nullptr;
    if (S_host && (reinterpret_cast<uintptr_t>(S_host) & 3) == 0) {
        hipPointerAttribute_t at;
        if (hipPointerGetAttributes(&at, S_host) != hipSuccess) (void)hipGetLastError();    // memory the runtime does not know is no error of this call
        else if (at.type == hipMemoryTypeHost) direct = static_cast<int32_t*>(at.devicePointer);
    }
    const bool halves = K <= HALVES_UP_TO;
    const unsigned workgroups = (unsigned)(halves ? (K + 31) / 32 : (K + 63) / 64) + 1;
    hipLaunchKernelGGL(halves ? calib_select_kernel<true> : calib_select_kernel<false>, dim3(workgroups), dim3(1024), 0, stream, keys,
                       (int)K, perm, info, direct);
    if (arcq_status st = check_launch("calib_select_kernel")) return st;
    if (S_host) {
        int32_t s = 0;
        hipError_t e = direct ? hipSuccess : hipMemcpyAsync(&s, info, sizeof(s), hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return fail(ARCQ_HIP_ERROR, "arcq_calib_select: %s", hipGetErrorString(e));
        if (!direct) std::memcpy(S_host, &s, sizeof(s));        // at any address
    }
    return ARCQ_OK;
}

}  // namespace arcq
