// Counting the magnitudes of 16-bit rows, shared by the translation units that do it (rank ladder, Round-to-Nearest).
#pragma once
#include "mlmc_device.h"

namespace mlmc {

constexpr int C16_KEYS = 1 << 15;       // magnitudes of a 16-bit entry: its bits without the sign
constexpr int C16_THREADS = 1024;
constexpr int C16_BLOCK = 128;          // magnitudes of one exponent
constexpr int C16_LDS = C16_KEYS + 64;  // words: a counter per magnitude; zeros are counted per lane behind them

typedef uint32_t u32x4_b16 __attribute__((ext_vector_type(4), aligned(2)));

// Counts of the magnitudes of entries [i0, i1) of a 16-bit row, in LDS (s_h[C16_LDS]), by a workgroup of C16_THREADS threads; at the
// return every counter is final (s_h[0] among them).  One LDS atomic per entry.  Zeros, which a gradient may mostly consist of, go to a
// counter per lane: on one word the lanes of a wave take turns.  16-byte loads (8 entries) at any alignment, past the cache, four of a wave's in
// flight while four are counted: bound by the read, 4 rows of 1.24e8 entries in 166 us (6.0 TB/s; with plain 8-byte loads 188).
// MARK: (10 us more of the 166) for every 512 entries of a whole piece a 64-bit word at marks[(entry - i0) / 512], bit l: one of the eight entries from 8 l on is in win.
// Returns how many of them the wave has marked.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 both16(int32_t x) { const u16x2 r = {(uint16_t)x, (uint16_t)x}; return r; }
struct C16Window { uint32_t lo, span, base; };   // magnitudes lo .. lo + span - 1, and those from base on
template <bool MARK>
__device__ __forceinline__ uint32_t count16_slice(const uint16_t* row, int64_t i0, int64_t i1, uint32_t* s_h, const C16Window& win, uint64_t* marks) {
    const int tid = threadIdx.x;
    for (int i = tid; i < C16_LDS / 4; i += C16_THREADS) ((uint4*)s_h)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    const uint32_t lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int NW = C16_THREADS / 64, PIECE = 2048;
    char* h = (char*)s_h;
    const uint32_t zero_at = (uint32_t)(C16_KEYS * 4) + lane * 4u;
    auto count1 = [&](uint32_t at) { atomicAdd((uint32_t*)(h + (at ? at : zero_at)), 1u); };
    auto count2 = [&](uint32_t w) {
        count1((w << 2) & 0x1FFFCu);
        count1((w >> 14) & 0x1FFFCu);
    };
    auto fetch = [&](int64_t p, u32x4_b16 (&b)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = __builtin_nontemporal_load((const u32x4_b16*)(row + i0 + p * PIECE + q * 512 + lane * 8));
    };
    const u16x2 wlo = both16((int32_t)win.lo);
    uint32_t marked = 0;
    auto use = [&](const u32x4_b16 (&b)[4], int64_t p) {
        uint32_t words = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (MARK) {
                u16x2 lowest = {0xFFFFu, 0xFFFFu}, highest = {0, 0};   // of the distances from lo, of the magnitudes
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const u16x2 k = __builtin_bit_cast(u16x2, b[q][i] & 0x7FFF7FFFu);
                    lowest = __builtin_elementwise_min(lowest, (u16x2)(k - wlo));
                    highest = __builtin_elementwise_max(highest, k);
                }
                const uint32_t l0 = lowest.x, l1 = lowest.y, h0 = highest.x, h1 = highest.y;
                const uint64_t m = __ballot((l0 < l1 ? l0 : l1) < win.span || (h0 > h1 ? h0 : h1) >= win.base);
                marked += (uint32_t)__popcll(m);
                words = write_lane((uint32_t)m, 2 * q, words);
                words = write_lane((uint32_t)(m >> 32), 2 * q + 1, words);
            }
            count2(b[q].x); count2(b[q].y); count2(b[q].z); count2(b[q].w);
        }
        if (MARK && lane < 8) ((uint32_t*)marks)[p * 8 + lane] = words;
    };
    const int64_t n = i1 > i0 ? (i1 - i0) / PIECE : 0;   // whole pieces; wave w takes w, w + NW, ...
    u32x4_b16 b0[4], b1[4];
    int64_t p = wave;
    if (p < n) {
        fetch(p, b0);
        while (true) {   // uniform
            const bool more1 = p + NW < n;
            if (more1) fetch(p + NW, b1);
            use(b0, p);
            if (!more1) break;
            p += NW;
            const bool more0 = p + NW < n;
            if (more0) fetch(p + NW, b0);
            use(b1, p);
            if (!more0) break;
            p += NW;
        }
    }
    for (int64_t j = i0 + n * PIECE + tid; j < i1; j += C16_THREADS) count1(((uint32_t)row[j] << 2) & 0x1FFFCu);
    __syncthreads();
    if (wave == 0) {
        const uint32_t z = wave_sum(s_h[C16_KEYS + lane]);
        if (lane == 0) s_h[0] = z;
    }
    __syncthreads();
    return marked;
}

}  // namespace mlmc
