// Top-k MLMC of 16-bit rows on gfx950.  A 16-bit row has at most 2^15 magnitudes: one read that counts them gives every rank threshold,
// every band's exact sum of squares and, slice by slice, where the message of a slice begins, so that a second read writes it.
//
//   k_c16_sample, k_c16_forecast   large plans: which magnitudes the message will need, from a sample
//   k_c16_hist    first read: counts of a slice of a row in LDS, one workgroup per slice                      [mlmc_count16.h]
//   k_c16_reduce  per magnitude: the row's total and, short slices, the entries in the slices before each slice
//   k_c16_scan    per row: threshold keys and how many of their equals are inside, norms (Lemma 3.4), level draw
//   k_c16_write   short slices: the second read writes the message, a slice per workgroup
//   k_c16_mark, k_c16_offsets, k_c16_expand   long slices: the second read leaves the tiles' entries in lists, which become the message
//
// Against the way of the 32-bit rows (sampled histogram, selection read with candidate lists, ranking, message from staged lists), which these
// rows took before, adaptive, compress + aggregate: 4 rows of 1.24e8 entries 817 -> 534 us, 32 of 1e6 271 -> 93.
#include "mlmc_count16.h"

namespace mlmc {

// ---------------------------------------------------------------------------------------------------
// The forecast of a row's message, so that the one read that every entry takes part in can mark what the message will need (a bit per eight entries: the
// rows' scales differ from stretch to stretch, and most lines of a row have nothing of the drawn band) and the second read leaves out the rest.
// k_c16_sample counts one block of 1024 entries in 32 by the upper 13 bits of the magnitudes, in up to 64 parts a row;
// k_c16_forecast, a workgroup per row, takes thresholds and norms from the sample, draws the level as the row will (adaptive: all levels within one per cent
// of the whole of where the drawn word falls) and leaves a window of magnitudes that holds its band and its base band, sampling errors allowed for.
// What it misses costs a read (k_c16_mark), nothing else; where it would mark too much, nothing is marked.  4 rows of 1.24e8 entries, 16 levels, adaptive: 10 + 19 us and 166 -> 176 for the first read,
// the second 182 -> 56 (28 to 92 by the levels drawn, 8 of 48 rows with bands of a thirtieth or more); whole pass 575 -> 484.
constexpr int C16_CB = 8192, C16_CSHIFT = 2;   // a sampled counter: four magnitudes
constexpr int C16_SAMPLE = 5;
constexpr int C16_PARTS = 64;                  // at most: one workgroup adds them up
__global__ __launch_bounds__(512) void k_c16_sample(TopkArgs a) {
    __shared__ __align__(16) uint32_t s_h[C16_CB];
    __shared__ uint32_t s_occ[8];
    const int row = blockIdx.y, tid = threadIdx.x;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < C16_CB / 4; i += 512) ((uint4*)s_h)[i] = make_uint4(0, 0, 0, 0);
    if (tid < 8) s_occ[tid] = 0u;
    __syncthreads();
    const uint16_t* g = (const uint16_t*)a.g + (int64_t)row * a.ld;
    const int64_t nblk = a.d >> 10, first = ((int64_t)1 << C16_SAMPLE) >> 1, ns = nblk > first ? ((nblk - first - 1) >> C16_SAMPLE) + 1 : 0;   // whole blocks
    auto count = [&](uint32_t w) {
        atomicAdd(&s_h[(w >> C16_CSHIFT) & (uint32_t)(C16_CB - 1)], 1u);
        atomicAdd(&s_h[(w >> (16 + C16_CSHIFT)) & (uint32_t)(C16_CB - 1)], 1u);
    };
    constexpr int U = 4;   // blocks in flight
    for (int64_t i = (int64_t)blockIdx.x * 8 + wave; i < ns; i += (int64_t)gridDim.x * 8 * U) {   // uniform
        u32x4_b16 v[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t b = i + (int64_t)gridDim.x * 8 * u;
            const uint16_t* p = g + ((((b < ns ? b : i) << C16_SAMPLE) + first) << 10) + lane * 8;
#pragma unroll
            for (int h = 0; h < 2; ++h) v[u][h] = *(const u32x4_b16*)(p + 512 * h);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + (int64_t)gridDim.x * 8 * u >= ns) break;   // uniform
            uint32_t other = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q) other |= (v[u][h][q] ^ v[u][0][0]) | (v[u][h][q] ^ (v[u][0][0] << 16 | v[u][0][0] >> 16));
            if ((other & 0x7FFF7FFFu) == 0u) {   // sixteen times one magnitude: rows that are mostly zero
                atomicAdd(&s_h[(v[u][0][0] >> C16_CSHIFT) & (uint32_t)(C16_CB - 1)], 16u);
                continue;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) { count(v[u][h].x); count(v[u][h].y); count(v[u][h].z); count(v[u][h].w); }
        }
    }
    __syncthreads();
    // exponents that occur: 32 counters, eight lanes
    uint4* part = (uint4*)(a.c16_part + ((size_t)row * (a.c16_wgs + 1) + blockIdx.x) * C16_KEYS);
#pragma unroll
    for (int it = 0; it < C16_CB / 4 / 512; ++it) {
        const int i = it * 512 + tid;
        const uint4 v = ((const uint4*)s_h)[i];
        const uint64_t m = __ballot((v.x | v.y | v.z | v.w) != 0u);
        const bool on = ((m >> (lane & 56u)) & 0xFFull) != 0u;
        if (on) part[i] = v;
        if (on && (lane & 7u) == 0u) atomicOr(&s_occ[i >> 8], 1u << ((i >> 3) & 31));
    }
    __syncthreads();
    if (tid < 8) a.c16_occ[((size_t)row * a.c16_wgs + blockIdx.x) * 8 + tid] = s_occ[tid];
}

__global__ __launch_bounds__(1024) void k_c16_forecast(TopkArgs a) {
    __shared__ __align__(16) uint32_t s_bin[C16_CB];
    __shared__ uint32_t s_occ[C16_PARTS * 8], s_any[8];
    __shared__ uint8_t s_exp[256];                           // the exponents that occur
    __shared__ uint32_t s_scan[17];
    __shared__ double s_w[16], s_above[1024];                // squares of the sampled entries above a thread's
    __shared__ uint4 s_r[TMAX];                              // sampled ranks of the boundaries; ranks that are surely above and below them
    __shared__ uint32_t s_hi[TMAX], s_lo[TMAX];              // magnitudes there
    __shared__ double s_e[TMAX];                             // squares of the sampled entries above a boundary
    const int row = blockIdx.x, tid = threadIdx.x, L = a.L, W = a.c16_wgs < C16_PARTS ? a.c16_wgs : C16_PARTS;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 8) s_any[tid] = 0u;
    for (int i = tid; i < C16_CB / 4; i += 1024) ((uint4*)s_bin)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    for (int i = tid; i < W * 8; i += 1024) {
        const uint32_t o = a.c16_occ[(size_t)row * a.c16_wgs * 8 + i];
        s_occ[i] = o;
        if (o) atomicOr(&s_any[i & 7], o);
    }
    __syncthreads();
    uint32_t nexp = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t o = s_any[i];
        if (tid < 32 && ((o >> tid) & 1u)) s_exp[nexp + __popc(o & ((1u << tid) - 1u))] = (uint8_t)(32 * i + tid);
        nexp += __popc(o);
    }
    __syncthreads();
    // eight lanes an exponent of a part, eight exponents a wave, eight of these in flight
    const uint32_t nch = (nexp + 7u) / 8u, items = nch * (uint32_t)W;
    for (uint32_t i0 = wave; i0 < items; i0 += 16 * 8) {   // uniform
        uint4 v[8];
        uint32_t at[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t i = i0 + 16u * u < items ? i0 + 16u * u : 0u, s = i / nch, j = (i - s * nch) * 8u + (lane >> 3), e = s_exp[j < nexp ? j : 0];
            at[u] = e * 32 + (lane & 7u) * 4;
            v[u] = make_uint4(0, 0, 0, 0);
            if (i0 + 16u * u < items && j < nexp && ((s_occ[s * 8 + (e >> 5)] >> (e & 31)) & 1u))   // (the others are not written)
                v[u] = *(const uint4*)(a.c16_part + ((size_t)row * (a.c16_wgs + 1) + s) * C16_KEYS + at[u]);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (v[u].x) atomicAdd(&s_bin[at[u]], v[u].x);
            if (v[u].y) atomicAdd(&s_bin[at[u] + 1], v[u].y);
            if (v[u].z) atomicAdd(&s_bin[at[u] + 2], v[u].z);
            if (v[u].w) atomicAdd(&s_bin[at[u] + 3], v[u].w);
        }
    }
    __syncthreads();
    const int bin0 = C16_CB - 8 * (tid + 1);   // this thread's eight counters, descending with the thread
    uint32_t n[8], sum = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint4 v = ((const uint4*)(s_bin + bin0))[h];
        n[4 * h] = v.x; n[4 * h + 1] = v.y; n[4 * h + 2] = v.z; n[4 * h + 3] = v.w;
    }
    auto square = [](uint32_t bin) -> double {
        const double v = (double)__uint_as_float((bin << C16_CSHIFT | 2u) << 16);
        return v * v;
    };
    double en = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (n[i]) en += square((uint32_t)(bin0 + i)) * (double)n[i];
        sum += n[i];
    }
    uint32_t total;
    const uint32_t before = block_excl_scan<1024>(sum, s_scan, total);
    double inc = en;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double u = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += u;
    }
    if (lane == 63) s_w[wave] = inc;
    {   // s_bin[p]: entries of the counters 0 .. p in descending order
        uint32_t upto = before;
#pragma unroll
        for (int i = 7; i >= 0; --i) { upto += n[i]; s_bin[8 * tid + 7 - i] = upto; }   // (block_excl_scan's barriers lie behind the reads)
    }
    if (tid <= L) {
        const double f = (double)total / (double)a.d;
        const uint32_t r = (uint32_t)((double)a.k[tid] * f);
        const float m = 5.0f * sqrtf((float)r) + 8.0f;
        s_r[tid] = make_uint4(r, (float)r > m ? r - (uint32_t)m : 0u, r + (uint32_t)m, 0u);
        s_hi[tid] = (uint32_t)C16_KEYS - 1u;
        s_lo[tid] = 0u;
    }
    __syncthreads();
    double e0 = 0.0, all = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        if (w == (int)wave) e0 = all;
        all += s_w[w];
    }
    s_above[tid] = e0 + inc - en;
    __syncthreads();
    if (tid < 3 * (L + 1)) {   // a rank each: its counter by bisection
        const int t = tid % (L + 1), what = tid / (L + 1);
        const uint32_t r = what == 0 ? s_r[t].x : what == 1 ? s_r[t].y : s_r[t].z;
        if (r >= total) {
            if (what == 0) s_e[t] = all;
        } else {
            int lo = 0, hi = C16_CB - 1;   // the first with more than r entries up to it
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (s_bin[mid] > r) hi = mid;
                else lo = mid + 1;
            }
            const uint32_t bin = (uint32_t)(C16_CB - 1 - lo);
            if (what == 0) {
                double e = s_above[lo >> 3];
                uint32_t at = (lo >> 3) ? s_bin[(lo & ~7) - 1] : 0u;
                for (int p = lo & ~7; p < lo; ++p) {
                    if (s_bin[p] != at) e += square((uint32_t)(C16_CB - 1 - p)) * (double)(s_bin[p] - at);
                    at = s_bin[p];
                }
                s_e[t] = r > at ? e + square(bin) * (double)(r - at) : e;
            } else if (what == 1) {
                if (r) s_hi[t] = bin << C16_CSHIFT | ((1u << C16_CSHIFT) - 1u);
            } else {
                s_lo[t] = bin << C16_CSHIFT;
            }
        }
    }
    __syncthreads();
    if (wave == 0) {
        const int l = (int)lane < L ? (int)lane : L - 1;
        const double d2 = s_e[l + 1] - s_e[l];
        const double p = level_p(a, row, d2 > 0.0 ? sqrt(d2) : 0.0, l);
        const uint32_t x = philox_word0(a.seed, a.step, (uint32_t)row), eps = a.draw_mode == 3 ? 42949673u : 0u;
        const int l0 = wave_draw_from_p(p, L, x > eps ? x - eps : 0u), l1 = wave_draw_from_p(p, L, x < ~eps ? x + eps : ~0u);
        if (lane == 0) {
            RowInfo* ri = a.rinfo + row;
            ri->mark_lo = s_lo[l1];
            ri->mark_hi = s_hi[l0 - 1];
            ri->mark_base = a.k[0] > 0 ? s_lo[0] : (uint32_t)C16_KEYS;
            // What the first read would mark: sampled entries of the window and from the base band's key on (s_bin: descending).  Entries and not ranks, because
            // many may be equal to a boundary's key: of rows of one value, or bands that end among zeros, all (4 rows of 6e7, pass 1512 -> 1926 and 855 -> 1253 us when they
            // were marked by their ranks), of a base band of three tenths every eight (703 -> 752).  The limit lets bands of an eighth with their margins pass; wider ones have a mark in most
            // lines of any row.
            auto upto = [&](uint32_t key) -> uint32_t { return key < (uint32_t)C16_KEYS ? s_bin[C16_CB - 1 - (int)(key >> C16_CSHIFT)] : 0u; };
            auto above = [&](uint32_t key) -> uint32_t { return upto(key + (1u << C16_CSHIFT)); };
            const uint32_t base = upto(ri->mark_base), over = above(ri->mark_hi), band = upto(ri->mark_lo);
            const uint32_t marked = base + (band > base ? band - (over > base ? over : base) : 0u);
            ri->mark_on = marked <= total / 32u * 5u ? 1 : 0;
            ri->marked = 0;
        }
    }
}

// One workgroup per (slice, row), one per CU: the counters fill its LDS.  Bound by the read.
// FORECAST: rows with a forecast are marked.
template <bool FORECAST>
__global__ __launch_bounds__(C16_THREADS) void k_c16_hist(TopkArgs a) {
    __shared__ __align__(16) uint32_t s_h[C16_LDS];
    const int row = blockIdx.y;
    if (row == 0 && blockIdx.x == 0 && threadIdx.x == 0) *a.dev_status = 0;   // nothing of this launch reports through it
    const int64_t i0 = (int64_t)blockIdx.x * a.c16_slice, i1 = i0 + a.c16_slice < a.d ? i0 + a.c16_slice : a.d;
    const uint16_t* g = (const uint16_t*)a.g + (int64_t)row * a.ld;
    RowInfo* ri = a.rinfo + row;
    __shared__ uint32_t s_marked;
    const bool marking = FORECAST && ri->mark_on;   // uniform
    uint32_t marked = 0;
    if (FORECAST && threadIdx.x == 0) s_marked = 0;
    if (marking)
        marked = count16_slice<true>(g, i0, i1, s_h, C16Window{ri->mark_lo, ri->mark_hi - ri->mark_lo + 1u, ri->mark_base}, a.c16_mark + ((size_t)row * a.ntiles * TILE + i0) / 512);
    else
        count16_slice<false>(g, i0, i1, s_h, C16Window{}, nullptr);
    // Blocks of C16_BLOCK magnitudes that occur, and which those are: the values of a row have some twenty of the 256 exponents.
    __shared__ uint32_t s_occ[C16_KEYS / C16_BLOCK / 32];
    if (threadIdx.x < C16_KEYS / C16_BLOCK / 32) s_occ[threadIdx.x] = 0u;
    if (marking && lane_id() == 0) atomicAdd(&s_marked, marked);
    __syncthreads();
    if (marking && threadIdx.x == 0) atomicAdd(&ri->marked, s_marked);
    uint4* part = (uint4*)(a.c16_part + ((size_t)row * (a.c16_wgs + 1) + blockIdx.x) * C16_KEYS);
    static_assert(C16_BLOCK == 128 && C16_THREADS == 1024, "half a wave per block, 32 blocks in a turn of the workgroup");
#pragma unroll
    for (int it = 0; it < C16_KEYS / 4 / C16_THREADS; ++it) {
        const int i = it * C16_THREADS + (int)threadIdx.x;
        const uint4 v = ((const uint4*)s_h)[i];
        const uint64_t m = __ballot((v.x | v.y | v.z | v.w) != 0u);
        const uint32_t lo = (uint32_t)m ? 1u : 0u, hi = (uint32_t)(m >> 32) ? 2u : 0u;
        if (lane_id() < 32u ? lo : hi) part[i] = v;
        if (lane_id() == 0 && (lo | hi)) atomicOr(&s_occ[it], (lo | hi) << (2 * (threadIdx.x >> 6)));
    }
    __syncthreads();
    if (threadIdx.x < C16_KEYS / C16_BLOCK / 32) a.c16_occ[((size_t)row * a.c16_wgs + blockIdx.x) * (C16_KEYS / C16_BLOCK / 32) + threadIdx.x] = s_occ[threadIdx.x];
}

// Slice c16_wgs of c16_part: the totals; BEFORE: the counts of slice s become those of the slices before it (in blocks that occur in the row; the
// others are not written).  A workgroup per block of magnitudes, done at once where it does not occur; G groups of consecutive slices side by side, at
// most PER slices each, so that a thread's loads are all in flight at once.
// 32 rows of 1e6 entries 7.7 us, 4 of 1.24e8 4.8 (every block written and read: 15.7 and 13.3).
template <int G, int PER, bool BEFORE>
__global__ __launch_bounds__(C16_BLOCK * G) void k_c16_reduce(TopkArgs a) {
    __shared__ uint32_t s_sum[G][C16_BLOCK];
    const int W = a.c16_wgs, tid = threadIdx.x, grp = tid / C16_BLOCK, key = tid % C16_BLOCK, row = blockIdx.y, blk = blockIdx.x;
    const int s0 = grp * PER, n = s0 >= W ? 0 : (s0 + PER < W ? PER : W - s0);
    constexpr int WORDS = C16_KEYS / C16_BLOCK / 32;
    const uint32_t* occ = a.c16_occ + (size_t)row * W * WORDS + blk / 32;
    uint32_t* p = a.c16_part + (size_t)row * (W + 1) * C16_KEYS + (size_t)blk * C16_BLOCK + key;
    static_assert(PER <= 32 && G * PER <= 256 && G * PER <= 2 * C16_BLOCK, "a thread per slice");
    const bool mine = tid < W && ((occ[(size_t)(tid < W ? tid : 0) * WORDS] >> (blk % 32)) & 1u);
    if (!__syncthreads_or(mine ? 1 : 0)) {
        if (grp == 0) p[(size_t)W * C16_KEYS] = 0u;
        return;
    }
    uint32_t v[PER], sum = 0, has = 0;   // has: in which of the group's slices the block occurs (elsewhere it is not written)
    {
        const int l = (int)lane_id();
        has = (uint32_t)__ballot(l < n && ((occ[(size_t)(l < n ? s0 + l : 0) * WORDS] >> (blk % 32)) & 1u));
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = (has >> i) & 1u ? p[(size_t)(s0 + i) * C16_KEYS] : 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) sum += v[i];
    s_sum[grp][key] = sum;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t t = s_sum[g][key];
        run += g < grp ? t : 0u;
        total += t;
    }
    if (BEFORE) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (i < n) p[(size_t)(s0 + i) * C16_KEYS] = run;
            run += v[i];
        }
    }
    if (grp == 0) p[(size_t)W * C16_KEYS] = total;
}

// One workgroup per row, bound by its chain of LDS reads, barriers and the draw: 12 levels 14.4 us, 16 levels 15.3 (17.4 and 19.5 with the boundaries read one
// after the other where they are compared).  thr_tau[t]: the magnitude at rank k_t - 1 (C16_KEYS: k_t == 0); thr_jx[t]: how many entries equal to it, in index
// order, are within the top k_t.
__global__ __launch_bounds__(1024) void k_c16_scan(TopkArgs a) {
    __shared__ uint32_t s_scan[17];
    __shared__ uint32_t s_k[TMAX + 1];   // the ladder: ranks are below 2^31
    __shared__ uint32_t s_big[TMAX][20];
    __shared__ unsigned long long s_wide[TMAX][20];
    __shared__ double s_norm[LMAX];
    __shared__ uint32_t s_top;
    const int row = blockIdx.x, tid = threadIdx.x, L = a.L;
    RowInfo* ri = a.rinfo + row;
    const int lo_key = C16_KEYS - 32 * (tid + 1);   // this thread's 32 magnitudes: lo_key .. lo_key + 31, descending with the thread
    uint32_t n[32];
    {
        const uint4* src = (const uint4*)(a.c16_part + ((size_t)row * (a.c16_wgs + 1) + a.c16_wgs) * C16_KEYS + lo_key);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint4 q = src[i];
            n[4 * i] = q.x; n[4 * i + 1] = q.y; n[4 * i + 2] = q.z; n[4 * i + 3] = q.w;
        }
    }
    if (tid <= TMAX) s_k[tid] = tid <= L ? (uint32_t)a.k[tid] : 0xFFFFFFFFu;   // behind the last boundary: one that nothing reaches
    for (int i = tid; i < TMAX * 20; i += 1024) (&s_wide[0][0])[i] = 0ull;
    if (tid == 0) s_top = 0u;
    uint32_t sum = 0;
    int top = -1;
#pragma unroll
    for (int i = 0; i < 32; ++i) { sum += n[i]; if (n[i]) top = i; }
    uint32_t total;
    const uint32_t before = block_excl_scan<1024>(sum, s_scan, total);
    {   // which blocks occur: four threads hold one
        const uint64_t m = __ballot(sum != 0u);
        if (lane_id() == 0) {
            uint32_t w16 = 0;   // this wave's sixteen blocks, the highest in bit 15 (a wave's magnitudes descend)
#pragma unroll
            for (int b = 0; b < 16; ++b) w16 |= ((m >> (4 * b)) & 15ull) ? 1u << (15 - b) : 0u;
            ((uint16_t*)ri->occ)[15 - (tid >> 6)] = (uint16_t)w16;
        }
    }
    if (sum && before == 0u) s_top = (uint32_t)(lo_key + top);   // the row's largest magnitude: one thread
    if (tid == 0 && (int64_t)total != a.d) atomicOr(a.dev_status, MLMC_DEV_INTERNAL);
    if (tid <= L && s_k[tid] == 0) { ri->thr_tau[tid] = (uint32_t)C16_KEYS; ri->thr_jx[tid] = 0u; }
    if (sum) {
        const uint32_t r0 = before;  // rank of this thread's first entry
        int t = 0;                     // the first band boundary behind rank r0: rank r0 lies in band t
#pragma unroll 4
        for (int u = 0; u <= L; ++u) t += s_k[u] <= r0 ? 1 : 0;
        uint32_t next = s_k[t];
        const int E = lo_key >> 7, e1 = E ? E : 1;   // one exponent for all 32
        const int sh = 2 * (e1 - 1) + 32;
        uint64_t acc = 0;
        if (next > r0 + sum) {   // all of them in one band
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const uint32_t sig = (uint32_t)((lo_key + i) & 127) | (E ? 128u : 0u);
                acc += (uint64_t)n[i] * (sig * sig);   // the square of the significand in units of 2^32
            }
        } else {
            uint32_t r = r0;
#pragma unroll
            for (int i = 31; i >= 0; --i) {
                const uint32_t sig = (uint32_t)((lo_key + i) & 127) | (E ? 128u : 0u);
                const uint64_t sq = sig * sig;
                uint32_t left = n[i];
                while (next <= r + left) {   // boundary t lies among these entries or right behind them
                    const uint32_t take = next - r;
                    ri->thr_tau[t] = (uint32_t)(lo_key + i);
                    ri->thr_jx[t] = n[i] - (left - take);
                    acc += (uint64_t)take * sq;
                    if (a.all_thresholds && t >= 1) wide_add(s_wide[t], acc, sh);
                    acc = 0;
                    left -= take;
                    r += take;
                    next = s_k[++t];
                }
                acc += (uint64_t)left * sq;
                r += left;
            }
        }
        if (a.all_thresholds && t >= 1 && t <= L) wide_add(s_wide[t], acc, sh);
    }
    __syncthreads();
    if (a.all_thresholds && tid >= 1 && tid <= L) {
        const double nrm = __dsqrt_rn(wide_to_double(s_wide[tid], s_big[tid]));
        s_norm[tid - 1] = nrm;
        a.norms[(size_t)row * L + (tid - 1)] = nrm;
        if (a.norms_user) a.norms_user[(size_t)row * L + (tid - 1)] = nrm;
    }
    __syncthreads();
    if (tid == 0) {
        ri->topkey = s_top;
        if (s_top >= 0x7F80u) atomicOr(a.dev_status, MLMC_DEV_NONFINITE);
    }
    if (tid < 64 && a.draw_mode >= 0) draw_row(a, row, s_norm);
}

// ---------------------------------------------------------------------------------------------------
// A step of the message kernels: C16_STEP entries, a wave takes 1024 consecutive ones in two loads, a lane 8 of either half.
constexpr int C16_STEP = 16 * C16_THREADS;
constexpr int C16_WAVES = C16_THREADS / 64;
// Per half, in its top bit (the other bits hold anything): key < bound, keys below 2^15, bounds up to it.
__device__ __forceinline__ uint32_t below16(u16x2 key, u16x2 bound) { return __builtin_bit_cast(uint32_t, (u16x2)(key - bound)); }
__device__ __forceinline__ uint32_t in_range16(u16x2 key, u16x2 lo, u16x2 hi) { return below16(key, hi) & ~below16(key, lo); }   // lo <= key < hi
// bit e of the result: entry e of a lane's 16 satisfies f (top bits per pair of keys).  The top bits are pushed in from above, two entries
// per instruction: six or seven instructions a pair (as 0 or 1 per half they were twelve, the compiler taking a halfword's minimum with 1 for a comparison).
template <class F>
__device__ __forceinline__ uint32_t mask16(const uint32_t (&b)[8], F f) {
    uint32_t acc = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = (acc >> 2) | (f(__builtin_bit_cast(u16x2, b[i] & 0x7FFF7FFFu)) & 0x80008000u);
    return ((acc >> 16) & 0xAAAAu) | ((acc >> 1) & 0x5555u);
}
// A lane's entries of the step that starts at entry j of the row (j: the lane's own first entry), [j, i1) of it there.
__device__ __forceinline__ void fetch_step(const uint16_t* g, int64_t j, u32x4_b16 (&v)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) v[h] = __builtin_nontemporal_load((const u32x4_b16*)(g + j + 512 * h));
}
__device__ __forceinline__ uint32_t fetch_part(const uint16_t* g, int64_t j, int64_t i1, u32x4_b16 (&v)[2]) {   // a step that ends early: which entries are there
    uint32_t valid = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t jh = j + 512 * h, left = i1 - jh;
        v[h] = (u32x4_b16){0u, 0u, 0u, 0u};
        if (left >= 8) {
            v[h] = __builtin_nontemporal_load((const u32x4_b16*)(g + jh));
            valid |= 0xFFu << (8 * h);
        } else if (left > 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e < left) {
                    v[h][e >> 1] |= (uint32_t)g[jh + e] << (16 * (e & 1));
                    valid |= 1u << (8 * h + e);
                }
        }
    }
    return valid;
}
__device__ __forceinline__ void words_of(const u32x4_b16 (&v)[2], uint32_t (&b)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = v[i >> 2][i & 3];
}

// The three thresholds of a row's message (0, l-1, l) as a stretch of the row sees them: an entry is inside the i-th when its key is at least
// lo[i]; where `cut` has bit i, `left[i]` of the entries equal to tau[i] = lo[i] - 1, in index order, are inside too (fewer than there are).
struct C16Cuts {
    int32_t lo[3], tau[3];
    uint32_t left[3];
    uint32_t cut;
};
// `before` entries equal to tau lie in front of the stretch, `here` in it, q in all are inside.
__device__ __forceinline__ void set_cut(C16Cuts& c, int i, int32_t tau, uint32_t before, uint32_t here, uint32_t q) {
    c.tau[i] = tau;
    c.left[i] = 0;
    c.lo[i] = tau + 1 < C16_KEYS ? tau + 1 : C16_KEYS;
    if (before < q) {
        if (before + here <= q) c.lo[i] = tau;
        else { c.cut |= 1u << i; c.left[i] = q - before; }
    }
}
// Slice s of the row: its thresholds, the message entries of the row in front of it and its own.  A whole workgroup of NT threads.
template <int NT>
__device__ __forceinline__ void slice_state(const TopkArgs& a, int row, int s, C16Cuts& c, uint32_t& base, uint32_t& members, uint32_t* s_red) {
    const RowInfo* ri = a.rinfo + row;
    const uint32_t* p0 = a.c16_part + ((size_t)row * (a.c16_wgs + 1) + s) * C16_KEYS;
    const uint32_t* p1 = p0 + C16_KEYS;
    const int lev = ri->level, top = (int)ri->topkey, tid = threadIdx.x;
    uint32_t in0 = 0, in1 = 0;   // entries equal to a threshold that are inside it: in front of the slice, to its end
    c.cut = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int t = i == 0 ? 0 : lev - 2 + i;
        const int32_t tau = (int32_t)ri->thr_tau[t];
        const uint32_t q = ri->thr_jx[t];
        const uint32_t b = tau < C16_KEYS ? p0[tau] : 0u, e = tau < C16_KEYS ? p1[tau] : 0u;
        set_cut(c, i, tau, b, e - b, q);
        const uint32_t sign = i == 1 ? ~0u : 1u;
        in0 += sign * (b < q ? b : q);
        in1 += sign * (e < q ? e : q);
    }
    uint32_t m0 = 0, m1 = 0;
    auto add = [&](int k) {   // blocks that do not occur are not written
        if ((ri->occ[k / C16_BLOCK / 32] >> (k / C16_BLOCK % 32)) & 1u) { m0 += p0[k]; m1 += p1[k]; }
    };
    for (int k = c.tau[0] + 1 + tid; k <= top; k += NT) add(k);
    const int t1 = c.tau[1] < top ? c.tau[1] : top;
    for (int k = c.tau[2] + 1 + tid; k <= t1; k += NT) add(k);
    m0 = wave_sum(m0);
    m1 = wave_sum(m1);
    const int wave = tid >> 6;
    if (lane_id() == 0) { s_red[wave] = m0; s_red[NT / 64 + wave] = m1; }
    __syncthreads();
    for (int i = 0; i < NT / 64; ++i) { in0 += s_red[i]; in1 += s_red[NT / 64 + i]; }
    __syncthreads();
    base = in0;
    members = in1 - in0;
}

// ---------------------------------------------------------------------------------------------------
// Long rows: the message by way of tile lists.  k_c16_mark leaves, tile by tile, the entries that may be in the message (its members and, where
// a threshold splits them, all entries equal to it) in index order, k_c16_offsets turns the counts of the tiles into places, k_c16_expand
// writes the message.  Waves are on their own throughout, so a row of stretches with different scales, some of which hold a hundred times as
// many members as others, keeps no workgroup waiting: 4 rows of 1.24e8 entries in 148 stretches took 480 us with a slice per workgroup (k_c16_write),
// and 317 with the fuller slices cut into parts after a count of 190; this way 182 + 13 + 43, the first of them 56 where the first read has marked what is needed.
struct C16Message {       // a row's thresholds 0, l-1, l
    uint32_t lo[3];       // keys from here on are inside whatever their position
    uint32_t tau[3];      // the key whose entries are split (C16_KEYS: none are)
    uint32_t q[3];        // of them, in index order, the first q are inside
};
__device__ __forceinline__ C16Message message_of(const RowInfo* ri, const uint32_t* total) {
    C16Message m;
    const int lev = ri->level;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int t = i == 0 ? 0 : lev - 2 + i;
        const uint32_t tau = ri->thr_tau[t], q = ri->thr_jx[t];
        const bool split = tau < (uint32_t)C16_KEYS && q < total[tau];
        m.lo[i] = tau + (split ? 1u : 0u);
        m.tau[i] = split ? tau : (uint32_t)C16_KEYS;
        m.q[i] = q;
    }
    return m;
}
constexpr int MK_THREADS = 256, MK_WAVES = MK_THREADS / 64;
__global__ __launch_bounds__(MK_THREADS, 6) void k_c16_mark(TopkArgs a) {
    __shared__ __align__(16) uint32_t s_ent[MK_WAVES][1024];
    const int row = blockIdx.y;
    const uint32_t lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t* total = a.c16_part + ((size_t)row * (a.c16_wgs + 1) + a.c16_wgs) * C16_KEYS;
    C16Message ms = message_of(a.rinfo + row, total);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        ms.lo[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)ms.lo[i]);
        ms.tau[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)ms.tau[i]);
    }
    // candidates: keys in [f2, e2k) or [f0, ...)
    const int32_t lo0 = (int32_t)(ms.tau[0] < (uint32_t)C16_KEYS ? ms.tau[0] : ms.lo[0]), lo2 = (int32_t)(ms.tau[2] < (uint32_t)C16_KEYS ? ms.tau[2] : ms.lo[2]);
    const u16x2 f2 = both16(lo2), e2k = both16((int32_t)ms.lo[1]), f0 = both16(lo0);
    const bool based = lo0 < C16_KEYS;   // uniform: a base band
    const uint16_t* g = (const uint16_t*)a.g + (int64_t)row * a.ld;
    uint32_t* ent = s_ent[wave];
    const int64_t stride = (int64_t)gridDim.x * MK_WAVES, nfull = a.d / TILE;
    const uint32_t t0 = ms.tau[0] << 16, t1 = ms.tau[1] << 16, t2 = ms.tau[2] << 16;
    uint32_t* list = nullptr;
    uint32_t head = 0, e0 = 0, e1 = 0, e2 = 0;   // uniform: candidates of the tile so far, those equal to a split key
    // 1024 entries of a tile, block `blk` of it
    auto block = [&](const u32x4_b16& va, const u32x4_b16& vb, uint32_t blk, uint32_t valid) {
        const uint32_t b[8] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
        uint32_t m;
        if (based) m = mask16(b, [&](u16x2 k) { return in_range16(k, f2, e2k) | ~below16(k, f0); }) & valid;
        else m = mask16(b, [&](u16x2 k) { return in_range16(k, f2, e2k); }) & valid;
        if (__ballot(m != 0u) == 0ull) return;   // uniform
        const uint32_t c0 = __popc(m & 0xFFu), c1 = __popc(m >> 8);
        const uint32_t inc = wave_incl_scan(c0 | (c1 << 16));
        const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63), tot0 = tot & 0xFFFFu, n = tot0 + (tot >> 16);
        const uint32_t at0 = (inc & 0xFFFFu) - c0, at1 = tot0 + (inc >> 16) - c1;
        const uint32_t off = blk * 1024u + lane * 8u;
        wave_lds_sync();
        if (n > 192u) {   // uniform: entry by entry
            uint32_t at = at0;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                if (k == 8) at = at1;
                if ((m >> k) & 1u) { ent[at] = (k & 1 ? b[k >> 1] & 0xFFFF0000u : b[k >> 1] << 16) | (off + (uint32_t)k + (k >= 8 ? 504u : 0u)); ++at; }
            }
        } else {
            uint32_t rank = 0;
            while (m) {
                const uint32_t k = (uint32_t)__builtin_ctz(m), q = k >> 1;
                const uint32_t x0 = q & 1u ? b[1] : b[0], x1 = q & 1u ? b[3] : b[2], x2 = q & 1u ? b[5] : b[4], x3 = q & 1u ? b[7] : b[6];
                const uint32_t y0 = q & 2u ? x1 : x0, y1 = q & 2u ? x3 : x2, z = q & 4u ? y1 : y0;
                ent[k < 8u ? at0 + rank : at1 + rank - c0] = (k & 1u ? z & 0xFFFF0000u : z << 16) | (off + k + (k >= 8u ? 504u : 0u));
                ++rank;
                m &= m - 1u;
            }
        }
        wave_lds_sync();
        for (uint32_t i = 0; i < n; i += 64) {
            const bool on = i + lane < n;
            const uint32_t e = on ? ent[i + lane] : 0x80000000u, key = on ? e & 0x7FFF0000u : ~0u;
            if (on) list[head + i + lane] = e;
            e0 += (uint32_t)__popcll(__ballot(key == t0));
            e1 += (uint32_t)__popcll(__ballot(key == t1));
            e2 += (uint32_t)__popcll(__ballot(key == t2));
        }
        head += n;
    };
    uint4* cnt = a.c16_cnt + (size_t)row * a.ntiles;
    auto begin = [&](int64_t tile) {
        list = a.c16_list + ((size_t)row * a.ntiles + tile) * TILE;
        head = e0 = e1 = e2 = 0;
    };
    auto end = [&](int64_t tile) { if (lane == 0) cnt[tile] = make_uint4(head, e0, e1, e2); };
    auto fetch = [&](int64_t tile, int half, u32x4_b16 (&v)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = __builtin_nontemporal_load((const u32x4_b16*)(g + tile * TILE + half * 2048 + q * 512 + lane * 8));
    };
    int64_t tile = (int64_t)blockIdx.x * MK_WAVES + wave;
    const RowInfo* ri = a.rinfo + row;
    if (a.c16_mark && ri->mark_on && (int64_t)ri->marked <= a.d / 16 && lo2 >= (int32_t)ri->mark_lo && ms.lo[1] <= ri->mark_hi + 1u &&
        (uint32_t)lo0 >= ri->mark_base) {   // uniform
        // The first read has marked all the candidates of the row: eight entries per mark, a lane each, in index order.  At most half of the eights: taking their
        // candidates one by one then costs less than the lines that are left out save (4 rows of 1.2e8: 40 % of the eights marked 232 us against 240 for the plain read, 61 %
        // 268 against 248; a test per tile instead of one per row took registers and a scan per tile, 55 -> 74 with few marks).
        const uint64_t* marks = a.c16_mark + (size_t)row * a.ntiles * (TILE / 512);
        uint16_t* place = (uint16_t*)ent;   // [2][512] the marked eights of a tile, of the next one
        // the marks of a tile, word 2 i + h of them in lane 2 i + h
        auto marks_at = [&](int64_t t) -> uint32_t { return ((const uint32_t*)(marks + t * 8))[lane & 15u]; };
        // marked eights of a tile; their places, and the first 64 of them on their way
        auto open = [&](int64_t t, uint32_t w, uint32_t par, u32x4_b16& v) -> uint32_t {
            uint32_t c = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)w, 2 * i + 1) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)w, 2 * i);
                if (m == 0ull) continue;   // uniform
                if ((m >> lane) & 1ull) place[par * 512u + c + mbcnt(m)] = (uint16_t)(i * 64 + (int)lane);
                c += (uint32_t)__popcll(m);
            }
            wave_lds_sync();
            v = __builtin_nontemporal_load((const u32x4_b16*)(g + t * TILE + (uint32_t)place[par * 512u + (lane < c ? lane : c - 1u)] * 8u));
            return c;
        };
        for (; tile < nfull; tile += 64 * stride) {
            // 64 of the wave's tiles at a time: a lane looks whether its tile has a mark, and settles those that have none
            const int64_t mine = tile + (int64_t)lane * stride;
            bool any = false;
            if (mine < nfull) {
                const uint4* w = (const uint4*)(marks + mine * 8);
                uint32_t o = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) { const uint4 x = w[i]; o |= x.x | x.y | x.z | x.w; }
                any = o != 0u;
                if (!any) cnt[mine] = make_uint4(0, 0, 0, 0);
            }
            uint64_t todo = __ballot(any);
            if (todo == 0ull) continue;   // uniform
            auto take = [&]() -> int64_t {
                const int64_t t = tile + (int64_t)__builtin_ctzll(todo) * stride;
                todo &= todo - 1;
                return t;
            };
            u32x4_b16 v, vn = (u32x4_b16){0u, 0u, 0u, 0u};
            int64_t t = take(), tn = t;
            uint32_t par = 0, c = open(t, marks_at(t), 0u, v), cn = 0, wn = 0;
            if (todo) { tn = take(); wn = marks_at(tn); }
            while (true) {   // uniform
                const bool more = tn != t;
                if (more) cn = open(tn, wn, par ^ 1u, vn);
                const int64_t ta = todo ? take() : tn;
                if (ta != tn) wn = marks_at(ta);
                begin(t);
                uint32_t eq01 = 0, eq2 = 0;
                for (uint32_t j0 = 0;; j0 += 64) {   // uniform
                    const uint32_t b[4] = {v.x, v.y, v.z, v.w}, mine8 = place[par * 512u + (j0 + lane < c ? j0 + lane : c - 1u)];
                    uint32_t acc = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const u16x2 key = __builtin_bit_cast(u16x2, b[i] & 0x7FFF7FFFu);
                        acc = (acc >> 2) | ((in_range16(key, f2, e2k) | ~below16(key, f0)) & 0x80008000u);
                    }
                    // entry e of the lane's eight: even ones from the lower halves, odd ones from the upper ones
                    uint32_t m = j0 + lane < c ? ((acc >> 9) & 0x55u) | ((acc >> 24) & 0xAAu) : 0u;
                    const uint32_t inc = wave_incl_scan((uint32_t)__popc(m));
                    uint32_t at = head + inc - (uint32_t)__popc(m);
                    while (m) {
                        const uint32_t q = (uint32_t)__builtin_ctz(m);
                        const uint32_t x0 = q & 2u ? b[1] : b[0], x1 = q & 2u ? b[3] : b[2], x = q & 4u ? x1 : x0;
                        const uint32_t e = q & 1u ? x & 0xFFFF0000u : x << 16, key = e & 0x7FFF0000u;
                        list[at] = e | (mine8 * 8u + q);
                        eq01 += (key == t0 ? 1u : 0u) | (key == t1 ? 0x10000u : 0u);
                        eq2 += key == t2 ? 1u : 0u;
                        ++at;
                        m &= m - 1u;
                    }
                    head += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
                    if (j0 + 64u >= c) break;
                    v = __builtin_nontemporal_load((const u32x4_b16*)(g + t * TILE + (uint32_t)place[par * 512u + (j0 + 64u + lane < c ? j0 + 64u + lane : c - 1u)] * 8u));
                }
                eq01 = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(eq01), 63);   // (at most 4096 each)
                eq2 = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(eq2), 63);
                e0 = eq01 & 0xFFFFu;
                e1 = eq01 >> 16;
                e2 = eq2;
                end(t);
                if (!more) break;
                t = tn;
                tn = ta;
                c = cn;
                v = vn;
                par ^= 1u;
                wave_lds_sync();
            }
        }
        tile = nfull % stride == (int64_t)blockIdx.x * MK_WAVES + wave ? nfull : a.ntiles;
    } else if (tile < nfull) {
        u32x4_b16 va[4], vb[4];
        fetch(tile, 0, va);
        while (true) {   // uniform
            fetch(tile, 1, vb);
            begin(tile);
            block(va[0], va[1], 0, 0xFFFFu);
            block(va[2], va[3], 1, 0xFFFFu);
            const bool more = tile + stride < nfull;
            if (more) fetch(tile + stride, 0, va);
            block(vb[0], vb[1], 2, 0xFFFFu);
            block(vb[2], vb[3], 3, 0xFFFFu);
            end(tile);
            if (!more) break;
            tile += stride;
        }
        tile += stride;
    }
    if (tile == nfull && tile < a.ntiles) {   // the row's last tile, when it is not whole
        begin(tile);
        for (uint32_t blk = 0; blk < 4; ++blk) {
            u32x4_b16 v[2];
            const uint32_t valid = fetch_part(g, tile * TILE + blk * 1024 + lane * 8, a.d, v);
            block(v[0], v[1], blk, valid);
        }
        end(tile);
    }
}

// Of the e entries equal to key v that follow E others, how many are in the message: inside threshold 0, or inside l and not inside l-1.
__device__ __forceinline__ uint32_t equals_inside(const C16Message& m, uint32_t v, uint32_t E, uint32_t e) {
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        uint32_t f = 0;
        if (v >= m.lo[i]) f = e;
        else if (v == m.tau[i] && m.q[i] > E) f = m.q[i] - E < e ? m.q[i] - E : e;
        n += i == 1 ? 0u - f : f;
    }
    return n;
}
// The tiles' places in the message, and how many of the split entries lie before every tile.  A workgroup takes `span` tiles of a row, 1024 at a time, after
// adding up those in front of them (with one workgroup per row, its threads on a run of tiles each, 72 us at 30381 tiles; this way
// 13, of which a launch takes 5).
__global__ __launch_bounds__(1024) void k_c16_offsets(TopkArgs a, int64_t span) {
    __shared__ uint32_t s_scan[17];
    __shared__ int64_t s_k[TMAX];
    __shared__ unsigned long long s_rows;
    __shared__ uint32_t s_sum[4];
    const int row = blockIdx.y, tid = threadIdx.x;
    if (tid < TMAX) s_k[tid] = tid <= a.L ? a.k[tid] : 0;
    if (tid == 0) s_rows = 0ull;
    if (tid < 4) s_sum[tid] = 0u;
    const uint4* cnt = a.c16_cnt + (size_t)row * a.ntiles;
    const int64_t t0 = (int64_t)blockIdx.x * span, t1 = t0 + span < a.ntiles ? t0 + span : a.ntiles;
    uint4 sum = make_uint4(0, 0, 0, 0);
    batched_loop<8, 1024>(0u, (uint32_t)t0, (uint32_t)tid, [&](uint32_t t) { return cnt[t]; }, [&](uint32_t, uint4 c) {
        sum.x += c.x; sum.y += c.y; sum.z += c.z; sum.w += c.w;
    });
    __syncthreads();
    if (t0 > 0) {   // uniform
        sum.x = wave_sum(sum.x); sum.y = wave_sum(sum.y); sum.z = wave_sum(sum.z); sum.w = wave_sum(sum.w);
        if (lane_id() == 0) { atomicAdd(&s_sum[0], sum.x); atomicAdd(&s_sum[1], sum.y); atomicAdd(&s_sum[2], sum.z); atomicAdd(&s_sum[3], sum.w); }
    }
    const bool last = t1 == a.ntiles;
    const int lev = a.rinfo[row].level;
    if (last && tid < row) {
        const int li = a.level[tid];
        atomicAdd(&s_rows, (unsigned long long)(s_k[0] + s_k[li] - s_k[li - 1]));
    }
    static_assert(MLMC_MAX_WORKERS <= 1024, "a thread per row");
    const C16Message m = message_of(a.rinfo + row, a.c16_part + ((size_t)row * (a.c16_wgs + 1) + a.c16_wgs) * C16_KEYS);
    // each split key once
    const bool s0 = m.tau[0] < (uint32_t)C16_KEYS, s1 = m.tau[1] < (uint32_t)C16_KEYS && !(s0 && m.tau[1] == m.tau[0]),
               s2 = m.tau[2] < (uint32_t)C16_KEYS && !(s0 && m.tau[2] == m.tau[0]) && !(s1 && m.tau[2] == m.tau[1]);
    // the message entries of a stretch of tiles
    auto inside = [&](const uint4& at, const uint4& c) -> uint32_t {
        uint32_t n = c.x;
        if (s0) n += equals_inside(m, m.tau[0], at.y, c.y) - c.y;
        if (s1) n += equals_inside(m, m.tau[1], at.z, c.z) - c.z;
        if (s2) n += equals_inside(m, m.tau[2], at.w, c.w) - c.w;
        return n;
    };
    __syncthreads();
    uint4 run = make_uint4(0, s_sum[1], s_sum[2], s_sum[3]);
    run.x = inside(make_uint4(0, 0, 0, 0), make_uint4(s_sum[0], s_sum[1], s_sum[2], s_sum[3]));
    uint4* pre = a.c16_pre + (size_t)row * a.ntiles;
    uint32_t* tile_off = a.tile_off + (size_t)row * (a.ntiles + 1);
    for (int64_t tb = t0; tb < t1; tb += 1024) {   // uniform
        const int64_t t = tb + tid;
        const uint4 c = t < t1 ? cnt[t] : make_uint4(0, 0, 0, 0);
        uint4 at = run, all;
        at.y += block_excl_scan<1024>(c.y, s_scan, all.y);
        at.z += block_excl_scan<1024>(c.z, s_scan, all.z);
        at.w += block_excl_scan<1024>(c.w, s_scan, all.w);
        at.x += block_excl_scan<1024>(inside(at, c), s_scan, all.x);
        if (t < t1) {
            tile_off[t] = at.x;
            pre[t] = make_uint4(c.x, at.y, at.z, at.w);
        }
        run.x += all.x; run.y += all.y; run.z += all.z; run.w += all.w;
    }
    if (last && tid == 0) {
        const int64_t rowstart = (int64_t)s_rows, nnz = s_k[0] + s_k[lev] - s_k[lev - 1];
        tile_off[a.ntiles] = (uint32_t)nnz;
        a.rinfo[row].msg.rowstart = rowstart;
        if ((int64_t)run.x != nnz) atomicOr(a.dev_status, MLMC_DEV_INTERNAL);
        a.row_off[row] = rowstart;
        if (row == a.M - 1) {
            a.row_off[a.M] = rowstart + nnz;
            if (rowstart + nnz > a.capacity) atomicOr(a.dev_status, MLMC_DEV_CAPACITY);
        }
    }
}
// A wave per tile, 64 entries of its list at a time.
__global__ __launch_bounds__(256) void k_c16_expand(TopkArgs a) {
    const int row = blockIdx.y;
    const uint32_t lane = lane_id();
    const RowInfo* ri = a.rinfo + row;
    const C16Message m = message_of(ri, a.c16_part + ((size_t)row * (a.c16_wgs + 1) + a.c16_wgs) * C16_KEYS);
    const float w = ri->weight;
    const int64_t rowstart = ri->msg.rowstart, room = a.capacity - rowstart;
    const bool any_split = m.tau[0] < (uint32_t)C16_KEYS || m.tau[1] < (uint32_t)C16_KEYS || m.tau[2] < (uint32_t)C16_KEYS;
    uint32_t* idx = a.idx + rowstart;
    float* val = a.val + rowstart;
    for (int64_t tile = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); tile < a.ntiles; tile += (int64_t)gridDim.x * 4) {
        const uint4 c = a.c16_pre[(size_t)row * a.ntiles + tile];
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.x);
        if (n == 0) continue;   // uniform
        uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.tile_off[(size_t)row * (a.ntiles + 1) + tile]);
        uint32_t E[3] = {c.y, c.z, c.w};
        const uint32_t* list = a.c16_list + ((size_t)row * a.ntiles + tile) * TILE;
        constexpr int U = 4;
        uint32_t e[U], next[U];
        auto fetch = [&](uint32_t i0, uint32_t (&v)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) { const uint32_t i = i0 + 64u * u + lane; v[u] = list[i < n ? i : n - 1u]; }
        };
        fetch(0, next);
        for (uint32_t i0 = 0; i0 < n; i0 += 64 * U) {
#pragma unroll
            for (int u = 0; u < U; ++u) e[u] = next[u];
            if (i0 + 64 * U < n) fetch(i0 + 64 * U, next);   // uniform; full tiles are many rounds, one after the other
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool on = i0 + 64u * u + lane < n;
                const uint32_t key = (e[u] >> 16) & 0x7FFFu;
                bool in[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    in[i] = key >= m.lo[i];
                    if (any_split) {   // uniform
                        const uint64_t eq = __ballot(on && key == m.tau[i]);
                        in[i] = in[i] || (key == m.tau[i] && E[i] + mbcnt(eq) < m.q[i]);
                        E[i] += (uint32_t)__popcll(eq);
                    }
                }
                const bool member = on && (in[0] || (in[2] && !in[1]));
                const uint64_t mm = __ballot(member);
                const uint32_t pos = at + mbcnt(mm);
                if (member && (int64_t)pos < room) {
                    const float v = __uint_as_float(e[u] & 0xFFFF0000u);
                    idx[pos] = (uint32_t)(tile * TILE) + (e[u] & 0xFFFu);
                    val[pos] = in[0] ? v : __fmul_rn(v, w);
                }
                at += (uint32_t)__popcll(mm);
            }
        }
    }
}

// Short slices: the message (Eq. (6)) of a slice by one workgroup.  A step's members are found as one 16-bit mask per lane, ranked by a scan
// over the lanes and one record per wave in LDS, and gathered in LDS ({entry's bits, offset in the step}); the next step writes them out densely, four
// to a store.  One barrier per step, the loads of the next step in flight (of two or three: slower), those of the first one issued before the slice's state.
// Of a threshold's equals the first few are inside.  Only in the one slice in which they run out is that a matter of position: there a wave's
// record holds its equals too, from which every wave tells by itself which waves' are inside, and the one wave that holds the last of them ranks them.
// One slice per threshold and row is such a one, and the launch ends with them: counted by lane shuffles and a second barrier, all three thresholds whether
// split or not, 32 rows of 1e6 entries took 46 us, now 34; 8 of 5e6 52 and 37, 4 of 2.5e6 20 and 15, 8 of 65537 14 and 9.
__global__ __launch_bounds__(C16_THREADS) void k_c16_write(TopkArgs a) {
    __shared__ __align__(16) uint32_t s_ent[2][C16_STEP];   // members of a step in index order: bits << 16 | base band by position << 15 | offset
    __shared__ uint2 s_pub[2][C16_WAVES];          // a wave's members by key and the equals of the split thresholds, 16 bits each
    __shared__ uint32_t s_red[2 * C16_WAVES];
    __shared__ int64_t s_k[TMAX];
    __shared__ unsigned long long s_rows;
    const int tid = threadIdx.x;
    const uint32_t lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = blockIdx.y, slice = blockIdx.x;
    const RowInfo* ri = a.rinfo + row;
    const int64_t i0 = (int64_t)slice * a.c16_slice, i1 = i0 + a.c16_slice < a.d ? i0 + a.c16_slice : a.d;
    const bool last = i1 == a.d;
    const uint16_t* g = (const uint16_t*)a.g + (int64_t)row * a.ld;
    const uint32_t lane_off = (uint32_t)wave * 1024u + lane * 8u;   // this lane's first entry of a step; the other half is 512 further on
    const int nfull = (int)((i1 - i0) / C16_STEP), nsteps = (int)((i1 - i0 + C16_STEP - 1) / C16_STEP);
    const int64_t mine = i0 + lane_off;
    u32x4_b16 buf[2], ahead[2];
    if (nfull > 0) fetch_step(g, mine, buf);   // in flight while the slice's state is put together
    if (tid < TMAX) s_k[tid] = tid <= a.L ? a.k[tid] : 0;
    if (tid == 0) s_rows = 0ull;
    __syncthreads();
    const int lev = ri->level;
    const float w = ri->weight;
    if (tid < row) {   // at most C16_THREADS rows
        const int li = a.level[tid];
        atomicAdd(&s_rows, (unsigned long long)(s_k[0] + s_k[li] - s_k[li - 1]));
    }
    static_assert(MLMC_MAX_WORKERS <= C16_THREADS, "a thread per row");
    C16Cuts cuts;
    uint32_t base, left_in_row = 0;
    slice_state<C16_THREADS>(a, row, slice, cuts, base, left_in_row, s_red);
    __syncthreads();
    const int64_t rowstart = (int64_t)s_rows;
    const int64_t nnz = s_k[0] + s_k[lev] - s_k[lev - 1];
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        cuts.lo[i] = __builtin_amdgcn_readfirstlane(cuts.lo[i]);
        cuts.tau[i] = __builtin_amdgcn_readfirstlane(cuts.tau[i]);
        cuts.left[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)cuts.left[i]);
    }
    cuts.cut = (uint32_t)__builtin_amdgcn_readfirstlane((int)cuts.cut);
    uint32_t* tile_off = a.tile_off + (size_t)row * (a.ntiles + 1);
    if (last && tid == 0) {
        a.row_off[row] = rowstart;
        tile_off[a.ntiles] = (uint32_t)nnz;
        if (row == a.M - 1) {
            a.row_off[a.M] = rowstart + nnz;
            if (rowstart + nnz > a.capacity) atomicOr(a.dev_status, MLMC_DEV_CAPACITY);
        }
    }
    uint32_t* idx = a.idx + rowstart;
    float* val = a.val + rowstart;
    const int64_t room = a.capacity - rowstart;   // entries past the capacity are not written

    uint32_t run = base;
    uint32_t par = 0, prev_first = 0, prev_count = 0, prev_sb = 0;
    const uint32_t lo0 = (uint32_t)cuts.lo[0] << 16;   // a key's place in an entry
    typedef uint32_t u32x4_out __attribute__((ext_vector_type(4), aligned(4)));
    typedef float f32x4_out __attribute__((ext_vector_type(4), aligned(4)));
    auto value = [&](uint32_t e) -> float {
        const float v = __uint_as_float(e & 0xFFFF0000u);
        return (e & 0x7FFF0000u) >= lo0 || (e & 0x8000u) ? v : __fmul_rn(v, w);
    };
    auto write_out = [&](uint32_t p, uint32_t first, uint32_t count, uint32_t sb) {
        if ((int64_t)first + count <= room) {   // uniform
            const uint32_t quads = count / 4;
            for (uint32_t i = tid; i < quads; i += C16_THREADS) {
                const uint4 e = *(const uint4*)&s_ent[p][4 * i];
                u32x4_out j;
                f32x4_out v;
                j.x = sb + (e.x & 0x3FFFu); j.y = sb + (e.y & 0x3FFFu); j.z = sb + (e.z & 0x3FFFu); j.w = sb + (e.w & 0x3FFFu);
                v.x = value(e.x); v.y = value(e.y); v.z = value(e.z); v.w = value(e.w);
                *(u32x4_out*)(idx + first + 4 * i) = j;
                *(f32x4_out*)(val + first + 4 * i) = v;
            }
            const uint32_t i = quads * 4 + tid;
            if (i < count) {
                const uint32_t e = s_ent[p][i];
                idx[first + i] = sb + (e & 0x3FFFu);
                val[first + i] = value(e);
            }
        } else {
            for (uint32_t i = tid; i < count && (int64_t)first + i < room; i += C16_THREADS) {
                const uint32_t e = s_ent[p][i];
                idx[first + i] = sb + (e & 0x3FFFu);
                val[first + i] = value(e);
            }
        }
    };
    auto step = [&](int s, const u32x4_b16 (&v)[2], uint32_t valid) {
        uint32_t b[8];
        words_of(v, b);
        const int64_t sb = i0 + (int64_t)s * C16_STEP;
        // members by their key alone
        const u16x2 from = both16(cuts.lo[2]), to = both16(cuts.lo[1]);
        uint32_t m;
        if (cuts.lo[0] < C16_KEYS) {   // uniform: a base band
            const u16x2 f0 = both16(cuts.lo[0]);
            m = mask16(b, [&](u16x2 k) { return in_range16(k, from, to) | ~below16(k, f0); }) & valid;
        } else {
            m = mask16(b, [&](u16x2 k) { return in_range16(k, from, to); }) & valid;
        }
        auto total_of = [](uint32_t c) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(c), 63); };
        // and the equals of the thresholds that are split in this slice
        uint32_t e[3] = {0, 0, 0}, pub_x = __popc(m), pub_y = 0;
        const uint32_t cut = cuts.cut;   // uniform
        if (cut) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if ((cut >> i) & 1u) e[i] = mask16(b, [&](u16x2 k) { return in_range16(k, both16(cuts.tau[i]), both16(cuts.tau[i] + 1)); }) & valid;
            pub_x |= __popc(e[0]) << 16;
            pub_y = total_of(__popc(e[1]) | __popc(e[2]) << 16);
        }
        pub_x = total_of(pub_x);
        if (lane == 0) s_pub[par][wave] = make_uint2(pub_x, pub_y);
        __syncthreads();
        if (prev_count) write_out(par ^ 1u, prev_first, prev_count, prev_sb);   // every wave is past its gathering of that step
        const uint2 pub = s_pub[par][lane & (C16_WAVES - 1)];   // lane u: wave u's
        uint32_t tot = pub.x & 0xFFFFu, by_position = 0;          // by_position: base band members that their keys do not tell
        if (cut) {
            // of every wave's equals those that are inside: `left` of them in the order of the waves
            const uint32_t eq[3] = {pub.x >> 16, pub.y & 0xFFFFu, pub.y >> 16};
            uint32_t keep[3] = {0, 0, 0};
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (!((cut >> i) & 1u)) continue;
                const uint32_t upto = wave_incl_scan(eq[i]), before = upto - eq[i], left = cuts.left[i];
                const uint32_t here = before >= left ? 0u : eq[i] < left - before ? eq[i] : left - before;
                tot += i == 1 ? 0u - here : here;
                const uint32_t own = (uint32_t)__builtin_amdgcn_readlane((int)here, wave), all = (uint32_t)__builtin_amdgcn_readlane((int)upto, C16_WAVES - 1);
                if (own == (uint32_t)__builtin_amdgcn_readlane((int)eq[i], wave)) {
                    keep[i] = e[i];
                } else if (own) {   // uniform over the wave: they run out among its own
                    const uint32_t c0 = __popc(e[i] & 0xFFu), c1 = __popc(e[i] >> 8);
                    const uint32_t inc = wave_incl_scan(c0 | (c1 << 16));
                    const uint32_t tot0 = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63) & 0xFFFFu;
                    uint32_t r = (inc & 0xFFFFu) - c0;
#pragma unroll 1
                    for (int k = 0; k < 16; ++k) {
                        if (k == 8) r = tot0 + (inc >> 16) - c1;
                        if ((e[i] >> k) & 1u) { if (r < own) keep[i] |= 1u << k; ++r; }
                    }
                }
                if (all > left) cuts.cut &= ~(1u << i);   // none behind this step
                else cuts.left[i] = left - all;
            }
            by_position = keep[0];
            m = keep[0] | ((m | keep[2]) & ~keep[1]);
        }
        const uint32_t c0 = __popc(m & 0xFFu), c1 = __popc(m >> 8);
        const uint32_t inc = wave_incl_scan(c0 | (c1 << 16));
        const uint32_t tot0 = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63) & 0xFFFFu;
        const uint32_t upto = wave_incl_scan(tot);   // lane u: waves 0 .. u
        const uint32_t wtot = (uint32_t)__builtin_amdgcn_readlane((int)tot, wave), total = (uint32_t)__builtin_amdgcn_readlane((int)upto, C16_WAVES - 1);
        const uint32_t pre = (uint32_t)__builtin_amdgcn_readlane((int)upto, wave) - wtot;
        if ((wave & 3) == 0 && lane == 0 && sb + wave * 1024 < i1) tile_off[sb / TILE + wave / 4] = run + pre;
        if (wtot) {   // uniform
            uint32_t* out = s_ent[par];
            const uint32_t at0 = pre + (inc & 0xFFFFu) - c0, at1 = pre + tot0 + (inc >> 16) - c1;   // first member of either half
            auto put = [&](uint32_t at, uint32_t bits, uint32_t k) {   // bits: the entry in the upper half
                out[at] = bits | (((by_position >> k) & 1u) << 15) | (lane_off + k + (k >= 8u ? 504u : 0u));
            };
            if (wtot > 192u) {   // uniform: entry by entry
                uint32_t at = at0;
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    if (k == 8) at = at1;
                    if ((m >> k) & 1u) { put(at, k & 1 ? b[k >> 1] & 0xFFFF0000u : b[k >> 1] << 16, (uint32_t)k); ++at; }
                }
            } else {
                uint32_t rank = 0;
                while (m) {
                    const uint32_t k = (uint32_t)__builtin_ctz(m), q = k >> 1;
                    const uint32_t x0 = q & 1u ? b[1] : b[0], x1 = q & 1u ? b[3] : b[2], x2 = q & 1u ? b[5] : b[4], x3 = q & 1u ? b[7] : b[6];
                    const uint32_t y0 = q & 2u ? x1 : x0, y1 = q & 2u ? x3 : x2, z = q & 4u ? y1 : y0;
                    put(k < 8u ? at0 + rank : at1 + rank - c0, k & 1u ? z & 0xFFFF0000u : z << 16, k);
                    ++rank;
                    m &= m - 1u;
                }
            }
        }
        prev_first = run;
        prev_count = total;
        prev_sb = (uint32_t)sb;
        run += total;
        par ^= 1u;
    };
    static_assert(TILE == 4 * 1024 && C16_STEP <= 0x4000, "a tile is four waves' entries; offsets have 14 bits");
    int s = 0;
#pragma unroll 1
    for (; s < nfull; ++s) {
        fetch_step(g, mine + (int64_t)(s + 1 < nfull ? s + 1 : s) * C16_STEP, ahead);   // the last one again: a load without a condition, which the waits can count
        step(s, buf, 0xFFFFu);
        buf[0] = ahead[0];
        buf[1] = ahead[1];
    }
    if (s < nsteps) {
        const uint32_t valid = fetch_part(g, mine + (int64_t)s * C16_STEP, i1, buf);
        step(s, buf, valid);
    }
    __syncthreads();
    if (prev_count) write_out(par ^ 1u, prev_first, prev_count, prev_sb);
    if (last && tid == 0 && (int64_t)run != nnz) atomicOr(a.dev_status, MLMC_DEV_INTERNAL);
}

// message == false: norms only.
mlmc_status topk16_run(const mlmc_plan_t* pl, const TopkArgs& args, bool message, hipStream_t st) {
    TopkArgs a = args;
    if (!message) a.c16_mark = nullptr;
    const dim3 grid(pl->c16_wgs, pl->M);
    if (a.c16_mark) {
        MLMC_LAUNCH(K_HIST, st, k_c16_sample<<<dim3(pl->c16_wgs < C16_PARTS ? pl->c16_wgs : C16_PARTS, pl->M), 512, 0, st>>>(a));
        MLMC_LAUNCH(K_SCAN, st, k_c16_forecast<<<pl->M, 1024, 0, st>>>(a));
    }
    if (a.c16_mark) MLMC_LAUNCH(K_C16_HIST, st, k_c16_hist<true><<<grid, C16_THREADS, 0, st>>>(a));
    else MLMC_LAUNCH(K_C16_HIST, st, k_c16_hist<false><<<grid, C16_THREADS, 0, st>>>(a));
    const dim3 rgrid(C16_KEYS / C16_BLOCK, pl->M);
#define MLMC_C16_REDUCE(G, PER)                                                                                          \
    do {                                                                                                                \
        if (message && !a.c16_list) MLMC_LAUNCH(K_C16_REDUCE, st, k_c16_reduce<G, PER, true><<<rgrid, C16_BLOCK * G, 0, st>>>(a)); \
        else MLMC_LAUNCH(K_C16_REDUCE, st, k_c16_reduce<G, PER, false><<<rgrid, C16_BLOCK * G, 0, st>>>(a));              \
    } while (0)
    if (pl->c16_wgs > 64) MLMC_C16_REDUCE(8, 32);
    else if (pl->c16_wgs > 8) MLMC_C16_REDUCE(2, 32);
    else if (pl->c16_wgs > 1) MLMC_C16_REDUCE(2, 4);
    else MLMC_C16_REDUCE(1, 1);
#undef MLMC_C16_REDUCE
    MLMC_LAUNCH(K_C16_SCAN, st, k_c16_scan<<<pl->M, 1024, 0, st>>>(a));
    if (!message) return MLMC_OK;
    if (a.c16_list) {
        int64_t mw = (pl->ntiles + MK_WAVES - 1) / MK_WAVES;
        const int64_t cap = 2048 / pl->M > 0 ? 2048 / pl->M : 1;
        // with a forecast some rows have little to do: their workgroups make room for those of the others (4 rows of 1.24e8 entries 70 -> 56 us on average)
        const int64_t mcap = a.c16_mark ? 4 * cap : cap;
        const dim3 mgrid((unsigned)(mw < mcap ? mw : mcap), pl->M), egrid((unsigned)(mw < 4 * cap ? mw : 4 * cap), pl->M);
        MLMC_LAUNCH(K_C16_MARK, st, k_c16_mark<<<mgrid, MK_THREADS, 0, st>>>(a));
        const int64_t span = (pl->ntiles + 65535) / 65536 * 1024;   // at most 64 workgroups a row: what they add up in front of their tiles stays small
        MLMC_LAUNCH(K_C16_OFFSETS, st, k_c16_offsets<<<dim3((unsigned)((pl->ntiles + span - 1) / span), pl->M), 1024, 0, st>>>(a, span));
        MLMC_LAUNCH(K_C16_WRITE, st, k_c16_expand<<<egrid, 256, 0, st>>>(a));
    } else {
        MLMC_LAUNCH(K_C16_WRITE, st, k_c16_write<<<grid, C16_THREADS, 0, st>>>(a));
    }
    return MLMC_OK;
}

}  // namespace mlmc
