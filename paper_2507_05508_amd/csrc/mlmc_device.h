// Device-side helpers: wave64 primitives, row loaders, key arithmetic, Philox4x32-10.
#pragma once
#include "mlmc_internal.h"

namespace mlmc {

__device__ __forceinline__ uint32_t lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// number of set bits of m below this lane
__device__ __forceinline__ uint32_t mbcnt(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// old with lane l (uniform) replaced by v (uniform); clang has the intrinsic but no builtin of this name
__device__ int llvm_amdgcn_writelane(int v, int l, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ uint32_t write_lane(uint32_t v, int l, uint32_t old) { return (uint32_t)llvm_amdgcn_writelane((int)v, l, (int)old); }

// Orders LDS traffic between the lanes of one wave (no instruction beyond the waits the fences need).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        uint32_t u = __shfl_xor(v, o, 64);
        v = u > v ? u : v;
    }
    return v;
}

// Exclusive prefix over the lanes of a small count c (0..7), and the wave total.
__device__ __forceinline__ uint32_t wave_excl_small(uint32_t c, uint32_t& total) {
    uint64_t b0 = __ballot(c & 1u), b1 = __ballot(c & 2u), b2 = __ballot(c & 4u);
    total = __popcll(b0) + 2u * __popcll(b1) + 4u * __popcll(b2);
    return mbcnt(b0) + 2u * mbcnt(b1) + 4u * mbcnt(b2);
}

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
    return v;
}

// Exclusive scan over a workgroup of NT threads (NT multiple of 64, <= 1024). `lds` holds NT/64 + 1 words.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds, uint32_t& total) {
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t u = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += u;
    }
    __syncthreads();
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int w = 0; w < NT / 64; ++w) {
            uint32_t t = lds[w];
            lds[w] = run;
            run += t;
        }
        lds[NT / 64] = run;
    }
    __syncthreads();
    total = lds[NT / 64];
    return lds[wave] + inc - v;
}

// Strided loop over [i0, i1) for a group of NT threads (this thread starts at i0 + t): U loads are issued back to
// back before the first is consumed.  A loop whose every load sits behind its own bounds check is compiled to one
// load, one wait per iteration; here whole batches take a branch-free path and the ragged rest is one more batch
// whose out-of-range loads are redirected to the last element and discarded.
template <int U, int NT, class Load, class Proc>
__device__ __forceinline__ void batched_loop(uint32_t i0, uint32_t i1, uint32_t t, Load load, Proc proc) {
    if (i1 <= i0) return;
    uint32_t i = i0 + t;
    if (i1 >= (uint32_t)((U - 1) * NT)) {
        const uint32_t lim = i1 - (uint32_t)((U - 1) * NT);   // i + (U-1)*NT < i1  <=>  i < lim
        for (; i < lim; i += (uint32_t)(U * NT)) {
            decltype(load(0u)) v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = load(i + (uint32_t)(u * NT));
#pragma unroll
            for (int u = 0; u < U; ++u) proc(i + (uint32_t)(u * NT), v[u]);
        }
    }
    if (i < i1) {   // fewer than U strides are left for this thread
        decltype(load(0u)) v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t k = i + (uint32_t)(u * NT);
            v[u] = load(k < i1 ? k : i1 - 1u);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t k = i + (uint32_t)(u * NT);
            if (k < i1) proc(k, v[u]);
        }
    }
}

// ---- keys ----------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t key_of_bits(uint32_t fp32_bits) { return fp32_bits & 0x7FFFFFFFu; }

// square of the 24-bit significand (no hidden bit when the exponent field is 0): < 2^48
__device__ __forceinline__ uint64_t sig_square(uint32_t key) {
    uint32_t frac = key & 0x7FFFFFu;
    uint32_t sig = (key >> 23) ? (frac | 0x800000u) : frac;
    return (uint64_t)sig * (uint64_t)sig;
}

// ---- row loaders: four consecutive elements starting at j (j % 4 == 0), as fp32 bit patterns -------
// DT = MLMC_F32 / MLMC_BF16.  VEC: one 16-byte (8-byte for bf16) load for the four; it needs the alignment of an element
// only (the memory system takes unaligned wide loads: the maximum of 8 rows of 11,689,513 fp32 elements takes 62 us, as that of
// aligned rows does, and took 68 us with single-element loads).
typedef uint32_t u32x4_f32 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_bf16 __attribute__((ext_vector_type(2), aligned(2)));
template <int DT, bool VEC>
struct RowLoader {
    const void* row;
    int64_t d;
    __device__ __forceinline__ RowLoader(const void* g, int64_t ld, int64_t d_, int r) : d(d_) {
        if (DT == MLMC_F32)
            row = (const void*)((const float*)g + (int64_t)r * ld);
        else
            row = (const void*)((const uint16_t*)g + (int64_t)r * ld);
    }
    // returns the number of valid elements (0..4); invalid ones read as +0
    __device__ __forceinline__ int load4(int64_t j, uint32_t (&b)[4]) const {
        int64_t left = d - j;
        int nv = left >= 4 ? 4 : (left > 0 ? (int)left : 0);
        if (DT == MLMC_F32) {
            const uint32_t* p = (const uint32_t*)row + j;
            if (VEC && nv == 4) {
                const u32x4_f32 v = *(const u32x4_f32*)p;
                b[0] = v.x; b[1] = v.y; b[2] = v.z; b[3] = v.w;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) b[c] = c < nv ? p[c] : 0u;
            }
        } else {
            const uint16_t* p = (const uint16_t*)row + j;
            if (VEC && nv == 4) {
                const u32x2_bf16 v = *(const u32x2_bf16*)p;
                b[0] = v.x << 16; b[1] = v.x & 0xFFFF0000u; b[2] = v.y << 16; b[3] = v.y & 0xFFFF0000u;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) b[c] = c < nv ? ((uint32_t)p[c] << 16) : 0u;
            }
        }
        return nv;
    }
    // four consecutive elements that are all inside the row (j + 4 <= d): no branch, so that several of these
    // loads can be in flight before the first result is needed
    __device__ __forceinline__ void load4_full(int64_t j, uint32_t (&b)[4]) const {
        if (DT == MLMC_F32) {
            const uint32_t* p = (const uint32_t*)row + j;
            if (VEC) {
                const u32x4_f32 v = *(const u32x4_f32*)p;
                b[0] = v.x; b[1] = v.y; b[2] = v.z; b[3] = v.w;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) b[c] = p[c];
            }
        } else {
            const uint16_t* p = (const uint16_t*)row + j;
            if (VEC) {
                const u32x2_bf16 v = *(const u32x2_bf16*)p;
                b[0] = v.x << 16; b[1] = v.x & 0xFFFF0000u; b[2] = v.y << 16; b[3] = v.y & 0xFFFF0000u;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) b[c] = (uint32_t)p[c] << 16;
            }
        }
    }
    // load4_full for a row that is streamed through once: a non-temporal load, so that the row does not push
    // what the kernel writes and reads back soon after (its staged lists) out of the L2.  It is also the faster read of more than the
    // last cache holds: 384 MB at 6.4 TB/s against 5.5, 1 GB 6.7 / 5.9 (up to 256 MB both reach 6.2).
    // (But what it reads is not kept for the next reader: the Round-to-Nearest norms keep plain loads, the extraction behind them gains from it, 95 us against 105.)
    __device__ __forceinline__ void load4_stream(int64_t j, uint32_t (&b)[4]) const {
        if (DT == MLMC_F32 && VEC) {
            const u32x4_f32 v = __builtin_nontemporal_load((const u32x4_f32*)((const uint32_t*)row + j));
            b[0] = v.x; b[1] = v.y; b[2] = v.z; b[3] = v.w;
        } else if (DT != MLMC_F32 && VEC) {
            const u32x2_bf16 v = __builtin_nontemporal_load((const u32x2_bf16*)((const uint16_t*)row + j));
            b[0] = v.x << 16; b[1] = v.x & 0xFFFF0000u; b[2] = v.y << 16; b[3] = v.y & 0xFFFF0000u;
        } else {
            load4_full(j, b);
        }
    }
    __device__ __forceinline__ uint32_t load1_stream(int64_t j) const {
        if (DT == MLMC_F32) return __builtin_nontemporal_load((const uint32_t*)row + j);
        return (uint32_t)__builtin_nontemporal_load((const uint16_t*)row + j) << 16;
    }
    __device__ __forceinline__ uint32_t load1(int64_t j) const {
        if (DT == MLMC_F32) return ((const uint32_t*)row)[j];
        return (uint32_t)((const uint16_t*)row)[j] << 16;
    }
};

// [i0, i1) of a row by the NW waves of a workgroup, 1024 elements at a time with the next 1024 in flight; i0 is a multiple of
// 1024.  f(keys of four times four consecutive elements of every lane, how many of each four are there).  f gets all sixteen
// at once so that it waits for its loads before it stores anything: the waits count loads and stores alike but can only
// rely on the loads, so a store between them would cut the loads in flight short.  STREAM: the row is read past the cache (load4_stream).
template <int DT, int NW, bool STREAM, class F>
__device__ __forceinline__ void stream_slice(const RowLoader<DT, true>& ld, int64_t i0, int64_t i1, uint32_t wave, uint32_t lane, F f) {
    const int n = (int)((i1 - i0) >> 10);
    uint32_t b0[4][4], b1[4][4];
    auto fetch = [&](int p, uint32_t (&b)[4][4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t j = i0 + (int64_t)p * 1024 + q * 256 + lane * 4;
            if (STREAM) ld.load4_stream(j, b[q]);
            else ld.load4_full(j, b[q]);
        }
    };
    auto use = [&](uint32_t (&b)[4][4]) {
        const int nv[4] = {4, 4, 4, 4};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) b[q][c] = key_of_bits(b[q][c]);
        f(b, nv);
    };
    int p = (int)wave;
    if (p < n) {
        fetch(p, b0);
        while (true) {   // uniform
            const bool more1 = p + NW < n;
            if (more1) fetch(p + NW, b1);
            use(b0);
            if (!more1) break;
            p += NW;
            const bool more0 = p + NW < n;
            if (more0) fetch(p + NW, b0);
            use(b1);
            if (!more0) break;
            p += NW;
        }
    }
    if ((int)wave == n % NW && i0 + (int64_t)n * 1024 < i1) {   // the ragged rest
        int nv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t j = i0 + (int64_t)n * 1024 + q * 256 + lane * 4;
            nv[q] = j < i1 ? ld.load4(j, b0[q]) : 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) b0[q][c] = c < nv[q] ? key_of_bits(b0[q][c]) : 0u;
        }
        f(b0, nv);
    }
}

// ---- Philox4x32-10 (Salmon et al., SC'11), from the published round function ----------------------
__device__ __forceinline__ uint32_t philox_word0(uint64_t seed, uint64_t step, uint32_t worker) {
    uint32_t c0 = (uint32_t)step, c1 = (uint32_t)(step >> 32), c2 = worker, c3 = 0u;
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        uint64_t pa = (uint64_t)0xD2511F53u * c0;
        uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
        uint32_t n0 = (uint32_t)(pb >> 32) ^ c1 ^ k0;
        uint32_t n2 = (uint32_t)(pa >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
    }
    return c0;
}

// Level draw shared by the Top-k and bit-wise paths: integer inverse CDF of one 32-bit uniform.
// p: L probabilities (local array).  Returns the level in 1..L.
__device__ __forceinline__ int draw_from_p(const double* p, int L, uint32_t x) {
    double c = 0.0;
    int level = L;
    bool found = false;
    for (int l = 0; l < L; ++l) {
        c = __dadd_rn(c, p[l]);
        double t = floor(__dmul_rn(c, 4294967296.0));
        uint64_t T;
        if (!(t > 0.0)) T = 0;
        else if (t >= 4294967296.0) T = 4294967296ull;
        else T = (uint64_t)t;
        if (l == L - 1) T = 4294967296ull;
        if (!found && (uint64_t)x < T) {
            level = l + 1;
            found = true;
        }
    }
    return level;
}

// ---- exact sums of squares: a 640-bit integer count of 2^-298 units -> correctly rounded fp64 ----------
struct BigAcc {
    uint32_t* w;  // 20 words, least significant first
    // value * 2^-298 rounded to nearest-even fp64
    __device__ double to_double() const {
        int top = -1;
        for (int i = 19; i >= 0; --i) if (w[i]) { top = i; break; }
        if (top < 0) return 0.0;
        const int P = top * 32 + 31 - __clz(w[top]);  // index of the most significant set bit
        auto word = [&](int i) -> uint64_t { return (i < 0 || i >= 20) ? 0ull : (uint64_t)w[i]; };
        if (P <= 52) {  // fits the significand exactly
            uint64_t v = word(0) | (word(1) << 32);
            return ldexp((double)v, -298);
        }
        // bits P .. P-52 as the significand, bit P-53 as guard, anything below as sticky
        const int g = P - 53;                       // guard bit index (>= 0)
        const int wi = g >> 5, bs = g & 31;         // window starting at the guard bit: 54 bits needed
        uint64_t win = (word(wi) >> bs) | (word(wi + 1) << (32 - bs));
        if (bs > 0) win |= word(wi + 2) << (64 - bs);
        const uint32_t guard = (uint32_t)(win & 1ull);
        uint64_t mant = (win >> 1) & ((1ull << 53) - 1ull);
        bool sticky = bs ? (w[wi] & ((1u << bs) - 1u)) != 0 : false;
        for (int i = wi - 1; i >= 0 && !sticky; --i) sticky = w[i] != 0;
        if (guard && (sticky || (mant & 1ull))) ++mant;
        return ldexp((double)mant, P - 52 - 298);
    }
};

// The same integer as LDS counters of 32-bit words (64 bits each, carries not yet propagated): v << shift is split into three words that are
// added with LDS atomics in any order; fewer than 2^32 addends cannot overflow a counter.
__device__ __forceinline__ void wide_add(unsigned long long* wide, uint64_t v, int shift) {
    if (!v) return;
    const int wi = shift >> 5, bs = shift & 31;
    uint32_t parts[3];
    parts[0] = (uint32_t)(v << bs);
    parts[1] = (uint32_t)(bs ? v >> (32 - bs) : v >> 32);
    parts[2] = bs ? (uint32_t)(v >> (64 - bs)) : 0u;
#pragma unroll
    for (int i = 0; i < 3; ++i)
        if (parts[i] && wi + i < 20) atomicAdd(&wide[wi + i], (unsigned long long)parts[i]);
}
// One thread: the carries propagated into `words` (20 of them), the value as a correctly rounded double.
__device__ __forceinline__ double wide_to_double(const unsigned long long* wide, uint32_t* words) {
    uint64_t w[20];
#pragma unroll
    for (int i = 0; i < 20; ++i) w[i] = wide[i];
    uint64_t carry = 0;
#pragma unroll
    for (int i = 0; i < 20; ++i) {
        const uint64_t t = w[i] + carry;
        words[i] = (uint32_t)t;
        carry = t >> 32;
    }
    BigAcc acc;
    acc.w = words;
    return acc.to_double();
}

// ---------------------------------------------------------------------------------------------------
// Level draw of one row (Alg. 2 / Alg. 3 "Sample l ~ p") by one wave, a lane per level: the sums, whose order fixes their roundings, go through the
// lanes one by one, the divisions and the integer thresholds are made side by side (one thread took 6 us for twelve levels).
__device__ __forceinline__ double lane_f64(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}
// p: the lane's probability (lane l: level l + 1, l < L <= 64).  Returns the level in 1..L, to every lane.
__device__ __forceinline__ int wave_draw_from_p(double p, int L, uint32_t x) {
    const int lane = (int)lane_id();
    double c = 0.0, mine = 0.0;
    for (int l = 0; l < L; ++l) {
        c = __dadd_rn(c, lane_f64(p, l));
        mine = lane == l ? c : mine;
    }
    const double t = floor(__dmul_rn(mine, 4294967296.0));
    uint64_t T = !(t > 0.0) ? 0ull : t >= 4294967296.0 ? 4294967296ull : (uint64_t)t;
    if (lane == L - 1) T = 4294967296ull;
    const uint64_t below = __ballot(lane < L && (uint64_t)x < T);   // the last level's lane is always among them
    return (int)__builtin_ctzll(below) + 1;
}
// Probability of level l + 1 (l < L, a lane's own; a whole wave); norm: the level's, where this call computes them.
__device__ __forceinline__ double level_p(const TopkArgs& a, int row, double norm, int l) {
    const int L = a.L;
    if (a.draw_mode == 0) return a.p_fixed[l];
    if (a.draw_mode == 1) return a.p_dev[(size_t)row * L + l];
    const double n = a.draw_mode == 2 ? a.p_dev[(size_t)row * L + l] : norm;
    double tot = 0.0;
    for (int i = 0; i < L; ++i) tot = __dadd_rn(tot, lane_f64(n, i));
    return tot == 0.0 ? __ddiv_rn(1.0, (double)L) : __ddiv_rn(n, tot);
}
__device__ inline int draw_row(const TopkArgs& a, int row, const double* norms_row) {   // returns the level
    const int L = a.L, lane = (int)lane_id(), l = lane < L ? lane : L - 1;
    const double p = level_p(a, row, a.draw_mode == 3 ? norms_row[l] : 0.0, l);
    const uint32_t x = philox_word0(a.seed, a.step, (uint32_t)row);
    const int level = wave_draw_from_p(p, L, x);
    const double pl = lane_f64(p, level - 1);
    if (lane == 0) {
        RowInfo* ri = a.rinfo + row;
        ri->level = level;
        ri->weight = pl == 0.0 ? 0.0f : (float)__ddiv_rn(1.0, pl);
        ri->draw_x = x;
        a.level[row] = level;
    }
    return level;
}

}  // namespace mlmc
