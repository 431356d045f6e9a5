// Top-k MLMC of short 32-bit rows on gfx950: a row fits the registers of one workgroup, which finds everything about it in one launch.
//
//   k_row_select  per row: exact rank thresholds by three digits (14 + 9 + 8 bits) counted in LDS, all of them side by side; band sums
//                 (Lemma 3.4), norms, level draw
//   k_row_write   per row: the message in index order
//
// Such rows are bound by launches and latency: nine to twelve launches of 5 to 15 us in the way of the longer rows (sampled histogram, selection
// read, ranking, message, each over several workgroups a row and with its own tables in memory to clear), two here.  The selection of a row of
// 65536 takes 22 us with fixed p (load 4, first digit 5, table 1, candidates listed 6, the other digits 2, places 4) and 39 with adaptive p (sums of squares 8,
// norms and draw 4 more); the message 6.  compress, us, the longer rows' way / this one: 4 rows of 65536, fixed p 54 / 28, adaptive 76 / 45; 1 of 16384 53 / 20, 73 / 31;
// 64 of 32768 74 / 26, 130 / 40.  What rows of few or close values cost is LDS atomics of many lanes on one word, so zeros are in no list and in no
// atomic, and where a row's candidates do not fit the list its counts are kept in copies.  4 rows of 65536, fixed p and adaptive, us, the longer rows' way / this
// one before / now: three in ten zero 61 / 57 / 27, 83 / 146 / 46; nine in ten 120 / 61 / 27, 550 / 130 / 44; quarters of a normal 77 / 62 / 58, 113 / 135 / 108; all
// within 4e-4 of one 96 / 107 / 66, 128 / 241 / 105; 30 % of one value 220 / 109 / 82, 290 / 160 / 109.
#include <type_traits>

#include "mlmc_device.h"

namespace mlmc {

constexpr int RW_THREADS = 1024;
constexpr int RW_WAVES = RW_THREADS / 64;
constexpr int RW_PIECES = 16;                  // pieces of 256 entries of a wave
static_assert(ROW_MAX == RW_WAVES * RW_PIECES * 256, "a row in the registers of a workgroup");

// A wave's consecutive pieces of the row; a lane holds four consecutive entries of each.
struct RowPieces {
    uint32_t b[RW_PIECES][4];
    int first, n;                              // uniform: the wave's first piece, how many it has
    int d;
    __device__ __forceinline__ void load(const TopkArgs& a, int row, int wave, uint32_t lane) {
        d = (int)a.d;
        const int all = (d + 255) / 256, per = (all + RW_WAVES - 1) / RW_WAVES;
        first = wave * per;
        n = all - first < per ? all - first : per;
        const RowLoader<MLMC_F32, true> ld(a.g, a.ld, a.d, row);
#pragma unroll
        for (int q = 0; q < RW_PIECES; ++q) {
            if (q >= n) continue;   // uniform
            if ((first + q + 1) * 256 <= d) ld.load4_full((int64_t)(first + q) * 256 + lane * 4, b[q]);
            else (void)ld.load4((int64_t)(first + q) * 256 + lane * 4, b[q]);
        }
    }
    // how many of the lane's four entries of piece q there are
    __device__ __forceinline__ int valid(int q, uint32_t lane) const {
        const int left = d - (first + q) * 256 - (int)lane * 4;
        return left >= 4 ? 4 : left > 0 ? left : 0;
    }
};

// One more in h[b] for the lanes that want it, lanes that share the first one's word, and then the next one's (ROUNDS in all), at once.
template <int ROUNDS>
__device__ __forceinline__ void count_peeled(uint32_t* h, uint32_t b, bool want) {
#pragma unroll
    for (int i = 0; i < ROUNDS; ++i) {
        const uint64_t w = __ballot(want);
        if (w == 0) return;
        const int first = __builtin_ctzll(w);
        const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)b, first);
        const uint64_t same = __ballot(want && b == b0);
        if ((int)lane_id() == first) atomicAdd(&h[b0], (uint32_t)__popcll(same));
        want = want && b != b0;
    }
    if (want) atomicAdd(&h[b], 1u);
}

// Descending search in a histogram held by one wave: lane l owns bins [BPL l, BPL l + BPL).  The bin that holds 1-based rank r, the rank inside it, its count.
template <int BPL>
__device__ __forceinline__ void row_rank_search(const uint32_t* h, uint32_t r, uint32_t& bin, uint32_t& rin, uint32_t& cnt) {
    const uint32_t lane = lane_id();
    uint32_t v[BPL], sum = 0;
#pragma unroll
    for (int i = 0; i < BPL; ++i) { v[i] = h[BPL * lane + i]; sum += v[i]; }
    const uint32_t inc = wave_incl_scan(sum);
    uint32_t above = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63) - inc;   // in the bins of higher lanes
    uint32_t fb = 0, fr = 0, fc = 0;
#pragma unroll
    for (int i = BPL - 1; i >= 0; --i) {
        if (above < r && r <= above + v[i]) { fb = BPL * lane + (uint32_t)i; fr = r - above; fc = v[i]; }
        above += v[i];
    }
    const uint64_t m = __ballot(fc != 0u);
    const int src = m ? (int)__builtin_ctzll(m) : 0;
    bin = (uint32_t)__builtin_amdgcn_readlane((int)fb, src);
    rin = (uint32_t)__builtin_amdgcn_readlane((int)fr, src);
    cnt = (uint32_t)__builtin_amdgcn_readlane((int)fc, src);
}

constexpr int RW_QUARTERS = 4;                 // stretches of a wave's pieces: what a wave of the message launch takes
constexpr int RW_D2 = 512, RW_D3 = 256;        // bins of the second and third digit
static_assert(TMAX * RW_D2 >= NB1 && TMAX * 20 * 8 <= TMAX * RW_D3 * 4, "shared arrays");

// Copies of a digit's counts where the whole row is counted: tables of BINS words, as many copies of all of them as the place of TMAX tables holds, at most 16
// (log2 of it).  A copy begins a word behind the end of the one before and a table's words change places by its number: rows of few values are in the
// same few bins of every table, which would be few banks.
__device__ __forceinline__ int copies_log2(int tables) { return tables > 16 ? 0 : tables > 8 ? 1 : tables > 4 ? 2 : tables > 2 ? 3 : 4; }
__device__ __forceinline__ uint32_t copy_at(int words, int log2_copies) { return (lane_id() & ((1u << log2_copies) - 1u)) * (uint32_t)(words + 1); }
template <int BINS>
__device__ __forceinline__ uint32_t place_in_copy(uint32_t table, uint32_t bin) { return table * BINS + (bin ^ ((table & 15u) << 2)); }
// The counts in the first copy, every word in its own place, by a whole workgroup; `zeros` more in word `zero_at` (< 0: nowhere).
template <int BINS>
__device__ __forceinline__ void add_copies(uint32_t* h, int words, int log2_copies, int zero_at, uint32_t zeros) {
    static_assert(BINS % 64 == 0, "a wave's words change places among themselves");
    for (int i = threadIdx.x; i < words; i += RW_THREADS) {
        const uint32_t at = place_in_copy<BINS>(i / BINS, i % BINS);
        uint32_t v = i == zero_at ? zeros : 0u;
        for (int c = 0; c < (1 << log2_copies); ++c) v += h[c * (words + 1) + at];
        wave_lds_sync();
        h[i] = v;
    }
}
static_assert(32 * RW_D3 + 16 <= TMAX * RW_D3 && 32 * RW_D2 + 16 <= TMAX * RW_D2, "tables times copies is at most 32");

// thr_tau[t]: the key at rank k_t - 1 (0xFFFFFFFF: k_t == 0); thr_jx[t]: how many entries equal to it, in index order, are within the top k_t;
// thr_zone[t]: 1 where that is not all of them.
template <bool SUMS>
__global__ __launch_bounds__(RW_THREADS) void k_row_select(TopkArgs a) {
    __shared__ __align__(16) uint32_t s_a[TMAX * RW_D2];   // first digit's counts [NB1]; second digit's, per slot; then where a prefix is a threshold's: its sub-slot, bit 31 set
    __shared__ __align__(16) uint32_t s_b[TMAX * RW_D3];   // third digit's counts, per sub-slot; then the sums of the bands
    __shared__ __align__(16) uint8_t s_tab[NB1];           // of a first digit: 0x80 | slot where it holds a threshold, else the band of its entries
    __shared__ __align__(16) unsigned long long s_sum[SUMS ? GMAX * REP_SUM : 1];
    __shared__ uint32_t s_scan[RW_WAVES + 1];
    __shared__ uint32_t s_need[TMAX];
    __shared__ int32_t s_t[TMAX], s_slot[TMAX], s_first[TMAX + 1];   // thresholds that are needed; their slots; a slot's first one
    __shared__ int32_t s_sub1st[TMAX + 1], s_nsub;   // a sub-slot's first one
    __shared__ uint32_t s_bkt[TMAX], s_rank[TMAX], s_bin[TMAX], s_tau[TMAX], s_q[TMAX], s_eq[TMAX];
    __shared__ uint16_t s_gexp[GMAX], s_gband[GMAX];
    __shared__ double s_norm[LMAX];
    __shared__ int32_t s_na, s_ns, s_lev;
    __shared__ uint32_t s_ncand, s_zeros;
    __shared__ uint4 s_part[RW_WAVES * RW_QUARTERS];
    __shared__ uint32_t s_status;
    const int row = blockIdx.x, tid = threadIdx.x, L = a.L;
    const uint32_t lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    RowInfo* ri = a.rinfo + row;
    RowPieces r;
    r.load(a, row, wave, lane);
    for (int i = tid; i < NB1 / 4; i += RW_THREADS) ((uint4*)s_a)[i] = make_uint4(0, 0, 0, 0);
    if (SUMS) for (int i = tid; i < GMAX * REP_SUM; i += RW_THREADS) s_sum[i] = 0ull;
    if (tid == 0) { s_status = 0u; s_ncand = 0u; }
    __syncthreads();
    if (wave == 0) {   // which thresholds are needed: all of them, or 0, l - 1 and l once the level is drawn
        if (!a.all_thresholds) {
            const int lev = draw_row(a, row, a.norms + (size_t)row * L);
            if (tid == 0) s_lev = lev;
            const int n = lev == 1 ? 2 : 3;
            if (tid < n) {
                const int t = tid == 0 ? 0 : lev - n + 1 + tid;
                s_t[tid] = t;
                s_need[tid] = (uint32_t)a.k[t];
            }
            if (tid == 0) s_na = n;
        } else {
            if (tid <= L) { s_t[tid] = tid; s_need[tid] = (uint32_t)a.k[tid]; }
            if (tid == 0) s_na = L + 1;
        }
    }
    // LDS atomics of many lanes on one word take a turn each.  Zeros, which a gradient may to a good part consist of, are what is missing in the counts and
    // are in no list; and rows of few values are seen in the first entries.
    bool crowded = false;   // uniform
    if (r.n > 0) {
        const uint32_t k0 = key_of_bits(r.b[0][0]);
        const uint64_t there = __ballot(k0 != 0u);
        if (there) {
            const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)(k0 >> B1_SHIFT), (int)__builtin_ctzll(there));
            crowded = __popcll(__ballot(k0 >> B1_SHIFT == b0) & there) >= 24;
        }
    }
    auto every = [&](auto f) {   // f(key), all lanes; zero past the row's end
#pragma unroll
        for (int q = 0; q < RW_PIECES; ++q) {
            if (q >= r.n) continue;
#pragma unroll
            for (int c = 0; c < 4; ++c) f(key_of_bits(r.b[q][c]));
        }
    };
    static_assert(TMAX * RW_D2 >= NB1 + 64, "a word per lane that nobody reads");
    if (__builtin_expect(crowded, 0)) every([&](uint32_t key) { count_peeled<3>(s_a, key >> B1_SHIFT, key != 0u); });
    else every([&](uint32_t key) { atomicAdd(&s_a[key ? key >> B1_SHIFT : (uint32_t)NB1 + lane], 1u); });
    __syncthreads();
    const int na = s_na;
    // ---- first digit: thread t holds 16 buckets, descending with the thread ----
    const int b_lo = NB1 - 16 * (tid + 1);
    {
        uint32_t hv[16], sum = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 v = ((const uint4*)(s_a + b_lo))[i];
            hv[4 * i] = v.x; hv[4 * i + 1] = v.y; hv[4 * i + 2] = v.z; hv[4 * i + 3] = v.w;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += hv[i];
        uint32_t total;
        const uint32_t before = block_excl_scan<RW_THREADS>(sum, s_scan, total);
        if (tid == RW_THREADS - 1) {   // the lowest buckets, and nothing behind them
            if (total > (uint32_t)a.d) atomicOr(&s_status, (uint32_t)MLMC_DEV_INTERNAL);
            hv[0] += (uint32_t)a.d - total;
            sum += (uint32_t)a.d - total;
            s_zeros = (uint32_t)a.d - total;
        }
        static_assert((0x7F800000u >> B1_SHIFT) % 16 == 0, "the buckets of Inf and NaN are whole threads'");
        if (b_lo >= (int)(0x7F800000u >> B1_SHIFT) && sum) atomicOr(&s_status, (uint32_t)MLMC_DEV_NONFINITE);
        for (int u = 0; u < na; ++u) {
            const uint32_t k = s_need[u];
            if (k - before - 1u >= sum) continue;   // before < k <= before + sum
            uint32_t run = before;
#pragma unroll
            for (int i = 15; i >= 0; --i) {
                if (k - run - 1u < hv[i]) { s_bkt[u] = (uint32_t)(b_lo + i); s_rank[u] = k - run; }
                run += hv[i];
            }
        }
        if (tid < na && s_need[tid] == 0u) s_bkt[tid] = NB1;   // nothing is inside
    }
    __syncthreads();
    auto slots = [&](bool valid, uint32_t what, int32_t& slot, bool& fresh) -> int {   // wave 0: equal neighbours among the thresholds share a slot
        const uint32_t prev = (uint32_t)__shfl_up((int)what, 1, 64);
        const uint64_t vm = __ballot(valid);
        fresh = valid && (lane == 0 || !((vm >> (lane - 1u)) & 1ull) || prev != what);
        const uint64_t fm = __ballot(fresh);
        slot = (int32_t)(mbcnt(fm) + (fresh ? 1u : 0u)) - 1;
        return (int)__popcll(fm);
    };
    if (wave == 0) {
        const bool valid = (int)lane < na && s_bkt[(int)lane < na ? lane : 0u] < (uint32_t)NB1;
        int32_t slot;
        bool fresh;
        const int ns = slots(valid, (int)lane < na ? s_bkt[lane] : 0u, slot, fresh);
        if ((int)lane < na) s_slot[lane] = valid ? slot : -1;
        if (fresh) s_first[slot] = (int32_t)lane;
        if (lane == 0) { s_ns = ns; s_first[ns] = na; }
    }
    __syncthreads();
    const int ns = s_ns, zero_slot = s_bkt[na - 1] == 0u ? ns - 1 : -1;   // of the threshold in the zeros' bucket, the lowest
    // the table, and the sum groups' exponents and bands: (255 - exponent) + band grows by one step at least whenever either changes
    auto group = [&](uint32_t bucket, uint32_t band) {
        const uint32_t E = bucket >> 6, g = 255u - E + band;
        s_gexp[g] = (uint16_t)(E ? E : 1u);
        s_gband[g] = (uint16_t)band;
    };
    {   // a bucket's band: the thresholds in higher buckets; a thread's 16 bytes side by side
        uint32_t above = 0, w[4] = {0, 0, 0, 0};
        for (int u = 0; u < na; ++u) {
            const int at = (int)s_bkt[u] - b_lo;
            above += at > 15 ? 1u : 0u;
            if (at > 0 && at <= 15) {   // one of this thread's: the buckets below it
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int n = at - 4 * k;   // so many of these four
                    w[k] += n >= 4 ? 0x01010101u : n > 0 ? 0x01010101u >> (8 * (4 - n)) : 0u;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] += above * 0x01010101u;
        *(uint4*)(s_tab + b_lo) = make_uint4(w[0], w[1], w[2], w[3]);
        if (SUMS) group((uint32_t)b_lo, above);
    }
    __syncthreads();
    if (tid < na && s_slot[tid] >= 0) {
        s_tab[s_bkt[tid]] = (uint8_t)(0x80u | (uint32_t)s_slot[tid]);
        if (SUMS) { group(s_bkt[tid], (uint32_t)tid); group(s_bkt[tid], (uint32_t)tid + 1u); }
    }
    for (int i = tid; i < ns * RW_D2; i += RW_THREADS) s_a[i] = 0;   // (every thread has read its counts)
    for (int i = tid; i < TMAX * RW_D3; i += RW_THREADS) s_b[i] = 0;
    __syncthreads();
    // ---- second digit, of the entries that share a threshold's first one: a few per cent of the row, listed for what follows as long as there is room ----
    uint32_t* list = s_a + ns * RW_D2;
    const uint32_t room = (uint32_t)(TMAX * RW_D2 - ns * RW_D2);
    auto fours = [&](auto with_zeros, auto f) {   // f(codes, keys, with_zeros: whether it is another than zero, which piece), all lanes; zero past the row's end
#pragma unroll
        for (int q = 0; q < RW_PIECES; ++q) {
            if (q >= r.n) continue;
            uint32_t code[4], key[4];
            bool on[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                key[c] = key_of_bits(r.b[q][c]);
                code[c] = s_tab[key[c] >> B1_SHIFT];
                on[c] = !decltype(with_zeros)::value || key[c] != 0u;
            }
            f(code, key, on, q);
        }
    };
    using yes = std::true_type;
    using no = std::false_type;
    {
        uint64_t mine = 0;   // which of the lane's entries
        auto mark = [&](const uint32_t (&code)[4], const uint32_t (&)[4], const bool (&on)[4], int q) {
#pragma unroll
            for (int c = 0; c < 4; ++c) mine |= (uint64_t)(on[c] && (code[c] & 0x80u)) << (4 * q + c);
        };
        if (__builtin_expect(zero_slot >= 0, 0)) fours(yes{}, mark);   // uniform
        else fours(no{}, mark);
        const uint32_t c = (uint32_t)__popcll(mine), inc = wave_incl_scan(c);
        uint32_t at = 0;
        if (lane == 63) at = atomicAdd(&s_ncand, inc);
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + inc - c;
#pragma unroll
        for (int q = 0; q < RW_PIECES; ++q) {
            if (q >= r.n) continue;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if ((mine >> (4 * q + k)) & 1u) {
                    if (at < room) list[at] = key_of_bits(r.b[q][k]);
                    ++at;
                }
        }
    }
    __syncthreads();
    const uint32_t ncand = s_ncand;
    const bool listed = ncand <= room, clumped = crowded || ncand > room / 2;   // clumped: many of them may be of one value
    auto candidates = [&](auto f) {   // the listed ones: f(slot, key, whether there is one), all lanes of a wave
        for (uint32_t i = (uint32_t)wave * 64u; i < ncand; i += RW_THREADS) {   // uniform
            const bool on = i + lane < ncand;
            const uint32_t key = list[on ? i + lane : i];
            f(s_tab[key >> B1_SHIFT] & 0x7Fu, key, on);
        }
    };
    auto prefixes = [&](const uint32_t (&code)[4], const uint32_t (&key)[4], uint32_t (&w)[4]) {   // what stands at the first two digits; code: a candidate's, or anything
#pragma unroll
        for (int c = 0; c < 4; ++c) w[c] = s_a[code[c] & 0x80u ? (code[c] & 0x7Fu) * RW_D2 + ((key[c] >> 8) & (RW_D2 - 1u)) : 0u];
    };
    // Where they do not fit (many equal keys, or close ones) the row is gone through again, and the list's place holds copies of the counts
    if (__builtin_expect(listed, 1)) {
        candidates([&](uint32_t slot, uint32_t key, bool on) {
            const uint32_t at = on ? slot * RW_D2 + ((key >> 8) & (RW_D2 - 1u)) : 0u;
            if (__builtin_expect(clumped, 0)) count_peeled<1>(s_a, at, on);
            else if (on) atomicAdd(&s_a[at], 1u);
        });
        if (tid == 0 && zero_slot >= 0) atomicAdd(&s_a[zero_slot * RW_D2], s_zeros);
    } else {
        const int words = ns * RW_D2, lc = copies_log2(ns);
        for (int i = tid; i < ((words + 1) << lc) - 1; i += RW_THREADS) s_a[i] = 0;
        __syncthreads();
        uint32_t* h = s_a + copy_at(words, lc);
        fours(yes{}, [&](const uint32_t (&code)[4], const uint32_t (&key)[4], const bool (&on)[4], int) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (on[c] && (code[c] & 0x80u)) atomicAdd(&h[place_in_copy<RW_D2>(code[c] & 0x7Fu, (key[c] >> 8) & (RW_D2 - 1u))], 1u);
        });
        __syncthreads();
        add_copies<RW_D2>(s_a, words, lc, zero_slot * RW_D2, s_zeros);
    }
    __syncthreads();
    for (int u = wave; u < na; u += RW_WAVES) {
        if (s_slot[u] < 0) continue;   // uniform
        uint32_t bin, rin, cnt;
        row_rank_search<RW_D2 / 64>(s_a + s_slot[u] * RW_D2, s_rank[u], bin, rin, cnt);
        if (lane == 0) { s_bin[u] = bin; s_q[u] = rin; }
    }
    __syncthreads();
    if (wave == 0) {
        const bool valid = (int)lane < na && s_slot[(int)lane < na ? lane : 0u] >= 0;
        const uint32_t pfx = valid ? (uint32_t)s_slot[lane] * RW_D2 + s_bin[lane] : 0u;
        int32_t sub;
        bool fresh;
        const int nsub = slots(valid, pfx, sub, fresh);
        if (fresh) { s_a[pfx] = 0x80000000u | (uint32_t)sub; s_sub1st[sub] = (int32_t)lane; }
        if (valid) s_eq[lane] = (uint32_t)sub;
        if (lane == 0) { s_nsub = nsub; s_sub1st[nsub] = na; }
    }
    __syncthreads();
    // ---- third digit ----
    const uint32_t zero_sub = zero_slot >= 0 ? s_a[zero_slot * RW_D2] : 0u;
    const int zero_at = zero_sub >> 31 ? (int)(zero_sub & 63u) * RW_D3 : -1;
    if (__builtin_expect(listed, 1)) {
        if (tid == 0 && zero_at >= 0) atomicAdd(&s_b[zero_at], s_zeros);
        candidates([&](uint32_t slot, uint32_t key, bool on) {
            const uint32_t w = s_a[on ? slot * RW_D2 + ((key >> 8) & (RW_D2 - 1u)) : 0u];
            const bool want = on && (w >> 31);
            const uint32_t at = (w & 63u) * RW_D3 + (key & (RW_D3 - 1u));
            if (__builtin_expect(clumped, 0)) count_peeled<1>(s_b, at, want);
            else if (want) atomicAdd(&s_b[at], 1u);
        });
    } else {
        const int words = s_nsub * RW_D3, lc = copies_log2(s_nsub);
        uint32_t* h = s_b + copy_at(words, lc);
        fours(yes{}, [&](const uint32_t (&code)[4], const uint32_t (&key)[4], const bool (&on)[4], int) {
            uint32_t w[4];
            prefixes(code, key, w);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (on[c] && (code[c] & 0x80u) && (w[c] >> 31)) atomicAdd(&h[place_in_copy<RW_D3>(w[c] & 63u, key[c] & (RW_D3 - 1u))], 1u);
        });
        __syncthreads();
        add_copies<RW_D3>(s_b, words, lc, zero_at, s_zeros);
    }
    __syncthreads();
    for (int u = wave; u < na; u += RW_WAVES) {
        uint32_t tau = 0xFFFFFFFFu, rin = 0, cnt = 0;
        if (s_slot[u] >= 0) {   // uniform
            uint32_t low;
            row_rank_search<RW_D3 / 64>(s_b + s_eq[u] * RW_D3, s_q[u], low, rin, cnt);
            tau = s_bkt[u] << B1_SHIFT | s_bin[u] << 8 | low;
        }
        if (lane == 0) {
            ri->thr_tau[s_t[u]] = tau;
            ri->thr_jx[s_t[u]] = rin;
            ri->thr_zone[s_t[u]] = rin < cnt ? 1 : 0;
            s_tau[u] = tau;
            s_rank[u] = rin;
            s_bin[u] = cnt;   // equals of the threshold
            if (s_slot[u] >= 0 && (rin < 1u || rin > cnt)) atomicOr(&s_status, (uint32_t)MLMC_DEV_INTERNAL);
        }
    }
    __syncthreads();
    if (tid == 0) ri->status = s_status;
    // ---- where the message of every stretch of four pieces begins: members by key, entries equal to a threshold that splits its equals ----
    auto places = [&](int lev) {
        uint32_t lo[3], tau[3], inside[3], nnz = 0;
        bool split[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int t = i == 0 ? 0 : lev - 2 + i;
            const int u = a.all_thresholds ? t : i == 0 ? 0 : lev == 1 ? i - 1 : i;   // where threshold t stands among those needed
            nnz += i == 1 ? 0u - s_need[u] : s_need[u];
            tau[i] = s_tau[u];
            inside[i] = s_rank[u];
            split[i] = s_rank[u] < s_bin[u];
            lo[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(split[i] ? tau[i] + 1u : tau[i]));
        }
        const uint32_t width = lo[1] - lo[2];
        constexpr int PQ = RW_PIECES / RW_QUARTERS;
        auto count = [&](auto with_base, auto with_split) {   // uniform
            constexpr bool BASED = decltype(with_base)::value, SPLIT = decltype(with_split)::value;
#pragma unroll
            for (int h = 0; h < RW_QUARTERS; ++h) {
                uint32_t n[4] = {0, 0, 0, 0};
#pragma unroll
                for (int q = h * PQ; q < (h + 1) * PQ; ++q) {
                    if (q >= r.n) continue;
                    auto piece = [&](int nv) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const uint32_t key = key_of_bits(r.b[q][c]);
                            bool m = key - lo[2] < width;
                            if (BASED) m = m || key >= lo[0];
                            n[0] += m && c < nv ? 1u : 0u;
                            if (SPLIT)
#pragma unroll
                                for (int i = 0; i < 3; ++i) n[1 + i] += split[i] && key == tau[i] && c < nv ? 1u : 0u;
                        }
                    };
                    if ((r.first + q + 1) * 256 <= r.d) piece(4);   // uniform
                    else piece(r.valid(q, lane));
                }
                n[0] = wave_incl_scan(n[0]);
                if (SPLIT)
#pragma unroll
                    for (int i = 1; i < 4; ++i) n[i] = wave_incl_scan(n[i]);
                if (lane == 63) s_part[wave * RW_QUARTERS + h] = make_uint4(n[0], n[1], n[2], n[3]);
            }
        };
        if (split[0] || split[1] || split[2]) count(yes{}, yes{});
        else if (lo[0] != 0xFFFFFFFFu) count(yes{}, no{});
        else count(no{}, no{});
        __syncthreads();
        if (wave == 0) {
            static_assert(RW_WAVES * RW_QUARTERS == 64, "a lane per stretch");
            const uint4 c = s_part[lane];
            uint4 at;
            at.x = wave_incl_scan(c.x) - c.x;
            at.y = wave_incl_scan(c.y) - c.y;
            at.z = wave_incl_scan(c.z) - c.z;
            at.w = wave_incl_scan(c.w) - c.w;
            const uint32_t e[3] = {at.y, at.z, at.w}, here[3] = {c.y, c.z, c.w};
            uint32_t end = at.x + c.x;
#pragma unroll
            for (int i = 0; i < 3; ++i) {   // |in0| + |in2| - |in1|: the sets are nested
                const uint32_t f = !split[i] ? 0u : e[i] < inside[i] ? e[i] : inside[i], g = e[i] + here[i], h = !split[i] ? 0u : g < inside[i] ? g : inside[i];
                at.x += i == 1 ? 0u - f : f;
                end += i == 1 ? 0u - h : h;
            }
            if (lane == 63 && end != nnz) ri->status = s_status | (uint32_t)MLMC_DEV_INTERNAL;   // an entry too few or too many was counted
            a.row_part[(size_t)row * 64 + lane] = at;
        }
    };
    if (!SUMS) {
        places(s_lev);
        return;
    }

    // ---- exact sums of squares: per (exponent, band) in LDS; the entries equal to a threshold are counted already ----
    unsigned long long (*s_wide)[20] = (unsigned long long(*)[20])s_b;
    for (int i = tid; i < TMAX * 20; i += RW_THREADS) (&s_wide[0][0])[i] = 0ull;
    auto add_square = [&](uint32_t band, uint32_t key) {
        atomicAdd(&s_sum[(255u - (key >> 23) + band) * REP_SUM + (lane & (REP_SUM - 1u))], (unsigned long long)sig_square(key));
    };
    if (__builtin_expect(listed, 1)) {
        auto others = [&](const uint32_t (&code)[4], const uint32_t (&key)[4], const bool (&on)[4], int) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (on[c] && !(code[c] & 0x80u)) add_square(code[c], key[c]);
        };
        if (__builtin_expect(s_zeros != 0u, 0)) fours(yes{}, others);   // uniform
        else fours(no{}, others);                                       // (what is past the end adds nothing)
        candidates([&](uint32_t slot, uint32_t key, bool on) {
            int u = s_first[on ? slot : 0u];
            const int u1 = s_first[on ? slot + 1u : 0u];
            for (; u < u1; ++u) {   // thresholds descend: the first one not above the key ends its search
                const uint32_t tau = s_tau[u];
                if (key < tau) continue;
                on = on && key != tau;
                break;
            }
            if (on) add_square((uint32_t)u, key);
        });
    } else {
        for (int i = tid; i < ns * RW_D2; i += RW_THREADS) {   // of a prefix: its first threshold and the one behind its last, or the band of its entries
            const uint32_t w = s_a[i];
            int u;
            if (w >> 31) {
                u = (int)(0x80000000u | (uint32_t)s_sub1st[(w & 63u) + 1u] << 8 | (uint32_t)s_sub1st[w & 63u]);
            } else {
                u = s_first[i / RW_D2];
                const int u1 = s_first[i / RW_D2 + 1];
                while (u < u1 && (uint32_t)(i % RW_D2) < ((s_tau[u] >> 8) & (RW_D2 - 1u))) ++u;
            }
            s_a[i] = (uint32_t)u;
        }
        __syncthreads();
        fours(yes{}, [&](const uint32_t (&code)[4], const uint32_t (&key)[4], const bool (&on)[4], int) {
            uint32_t w[4], tau[4], band[4];
            prefixes(code, key, w);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                band[c] = code[c] & 0x80u ? w[c] : code[c];
                tau[c] = s_tau[band[c] >> 31 ? band[c] & 63u : 0u];
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                bool add = on[c];
                if (band[c] >> 31) {
                    uint32_t u = band[c] & 63u;
                    const uint32_t u1 = (band[c] >> 8) & 63u;
                    uint32_t t = tau[c];
                    while (key[c] < t) {
                        if (++u == u1) break;
                        t = s_tau[u];
                    }
                    add = add && (u == u1 || key[c] != t);
                    band[c] = u;
                }
                if (add) add_square(band[c], key[c]);
            }
        });
    }
    static_assert(ROW_MAX <= 1 << 16, "squares below 2^48 in a 64-bit counter");
    __syncthreads();
    for (int g = tid; g < GMAX; g += RW_THREADS) {
        unsigned long long lo = 0, hi = 0;
#pragma unroll
        for (int i = 0; i < REP_SUM; ++i) {
            const unsigned long long v = s_sum[g * REP_SUM + ((i + tid) & (REP_SUM - 1))];
            lo += v & 0xFFFFFFFFull;
            hi += v >> 32;
        }
        if (lo | hi) {
            const int band = s_gband[g], sh = 2 * ((int)s_gexp[g] - 1);
            if (band >= 1 && band <= L) { wide_add(s_wide[band], lo, sh); wide_add(s_wide[band], hi, sh + 32); }
        }
    }
    if (tid < na && s_slot[tid] >= 0) {   // the entries equal to threshold u's key: those that are inside it but not inside u - 1; behind the last of them the rest
        const int u = tid;
        const uint32_t tau = s_tau[u], E = tau >> 23;
        const uint64_t sq = sig_square(tau);
        const int sh = 2 * ((int)(E ? E : 1u) - 1);
        auto add = [&](int band, uint32_t n) {
            if (band < 1 || band > L || n == 0u) return;
            wide_add(s_wide[band], (sq & 0xFFFFFFFFull) * n, sh);
            wide_add(s_wide[band], (sq >> 32) * n, sh + 32);
        };
        add(u, s_rank[u] - (u > 0 && s_tau[u - 1] == tau ? s_rank[u - 1] : 0u));
        if (u == na - 1 || s_tau[u + 1] != tau) add(u + 1, s_bin[u] - s_rank[u]);
    }
    __syncthreads();
    if (tid >= 1 && tid <= L) {
        const double nrm = __dsqrt_rn(wide_to_double(s_wide[tid], s_a + tid * 20));
        s_norm[tid - 1] = nrm;
        a.norms[(size_t)row * L + (tid - 1)] = nrm;
        if (a.norms_user) a.norms_user[(size_t)row * L + (tid - 1)] = nrm;
    }
    __syncthreads();
    if (a.draw_mode != 3) return;   // uniform: norms only
    if (wave == 0) {
        const int lev = draw_row(a, row, s_norm);
        if (tid == 0) s_lev = lev;
    }
    __syncthreads();
    places(s_lev);
}

// What the rows report, and whether the message fits: by one workgroup, the only one that writes the status word.
template <int NT>
__device__ __forceinline__ void row_status(const TopkArgs& a, int tid, uint32_t bits) {
    for (int i = tid; i < a.M; i += NT) bits |= a.rinfo[i].status;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) bits |= (uint32_t)__shfl_xor((int)bits, o, 64);
    __shared__ uint32_t s_bits;
    if (tid == 0) s_bits = 0u;
    __syncthreads();
    if ((tid & 63) == 0) atomicOr(&s_bits, bits);
    __syncthreads();
    if (tid == 0) *a.dev_status = (int32_t)s_bits;
}
__global__ __launch_bounds__(RW_THREADS) void k_row_status(TopkArgs a) { row_status<RW_THREADS>(a, threadIdx.x, 0u); }

// A wave takes a stretch of up to four pieces, whose place in the message is known: nothing waits for another wave.
constexpr int RWW_THREADS = 256;
__global__ __launch_bounds__(RWW_THREADS) void k_row_write(TopkArgs a) {
    __shared__ int64_t s_k[TMAX], s_rows[RWW_THREADS / 64];
    const int row = blockIdx.y, tid = threadIdx.x;
    const uint32_t lane = lane_id();
    const int u = (int)blockIdx.x * (RWW_THREADS / 64) + __builtin_amdgcn_readfirstlane(tid >> 6);   // stretch: quarter u % 4 of wave u / 4 of the selection
    constexpr int PQ = RW_PIECES / RW_QUARTERS;
    const int d = (int)a.d, all = (d + 255) / 256, per = (all + RW_WAVES - 1) / RW_WAVES;
    const int p0 = (u / RW_QUARTERS) * per + (u % RW_QUARTERS) * PQ;
    int p1 = (u / RW_QUARTERS + 1) * per;
    p1 = p1 < all ? p1 : all;
    const int n = p1 - p0 < PQ ? p1 - p0 : PQ;   // <= 0: nothing here
    const RowLoader<MLMC_F32, true> ld(a.g, a.ld, a.d, row);
    uint32_t b[PQ][4];
    int nv[PQ];
#pragma unroll
    for (int q = 0; q < PQ; ++q) nv[q] = q < n ? ld.load4((int64_t)(p0 + q) * 256 + lane * 4, b[q]) : 0;
    const uint4 part = a.row_part[(size_t)row * 64 + u];
    if (tid <= a.L) s_k[tid] = a.k[tid];
    const RowInfo* ri = a.rinfo + row;
    const int lev = ri->level;
    const float w = ri->weight;
    uint32_t lo[3], tau[3], inside[3];   // keys from lo on are inside; of those equal to tau, where they are split, the first `inside`
    bool split[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int t = i == 0 ? 0 : lev - 2 + i;
        tau[i] = ri->thr_tau[t];
        inside[i] = ri->thr_jx[t];
        split[i] = ri->thr_zone[t] != 0;
        lo[i] = split[i] ? tau[i] + 1u : tau[i];
    }
    __syncthreads();
    int64_t rowstart = 0;   // the messages of the rows before this one
    for (int i = tid; i < row; i += RWW_THREADS) {
        const int li = a.level[i];
        rowstart += s_k[0] + s_k[li] - s_k[li - 1];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) rowstart += (int64_t)__shfl_xor((long long)rowstart, o, 64);
    if (lane == 0) s_rows[tid >> 6] = rowstart;
    __syncthreads();
    rowstart = s_rows[0] + s_rows[1] + s_rows[2] + s_rows[3];
    const int64_t nnz = s_k[0] + s_k[lev] - s_k[lev - 1], room = a.capacity - rowstart;
    uint32_t* idx = a.idx + rowstart;
    float* val = a.val + rowstart;
    uint32_t* tile_off = a.tile_off + (size_t)row * (a.ntiles + 1);
    uint32_t run = part.x, eq[3] = {part.y, part.z, part.w};
#pragma unroll
    for (int q = 0; q < PQ; ++q) {
        if (q >= n) continue;   // uniform
        if (((p0 + q) & (TILE / 256 - 1)) == 0 && lane == 0) tile_off[(p0 + q) / (TILE / 256)] = run;
        uint32_t in[3] = {0, 0, 0};
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 3; ++i) in[i] |= (c < nv[q] && key_of_bits(b[q][c]) >= lo[i] ? 1u : 0u) << c;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (!split[i]) continue;   // uniform
            uint32_t rank = eq[i];
            uint64_t m[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                m[c] = __ballot(c < nv[q] && key_of_bits(b[q][c]) == tau[i]);
                rank += mbcnt(m[c]);
                eq[i] += (uint32_t)__popcll(m[c]);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t e = (uint32_t)(m[c] >> lane) & 1u;
                in[i] |= (rank < inside[i] ? e : 0u) << c;
                rank += e;
            }
        }
        const uint32_t m4 = in[0] | (in[2] & ~in[1]);
        uint32_t at = run;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint64_t m = __ballot((m4 >> c) & 1u);
            at += mbcnt(m);
            run += (uint32_t)__popcll(m);
        }
        const uint32_t j = (uint32_t)(p0 + q) * 256u + lane * 4u;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if ((m4 >> c) & 1u) {
                const float v = __uint_as_float(b[q][c]);
                if ((int64_t)at < room) { idx[at] = j + (uint32_t)c; val[at] = (in[0] >> c) & 1u ? v : __fmul_rn(v, w); }
                ++at;
            }
    }
    if (blockIdx.x != 0) return;   // uniform
    if (tid == 0) {
        tile_off[a.ntiles] = (uint32_t)nnz;
        a.row_off[row] = rowstart;
        if (row == a.M - 1) a.row_off[a.M] = rowstart + nnz;
    }
    if (row == a.M - 1) row_status<RWW_THREADS>(a, tid, rowstart + nnz > a.capacity ? (uint32_t)MLMC_DEV_CAPACITY : 0u);   // uniform; it knows where the message ends
}

// message == false: norms only.
mlmc_status row_topk_run(const mlmc_plan_t* pl, const TopkArgs& a, bool message, hipStream_t st) {
    if (a.all_thresholds) MLMC_LAUNCH(K_ROW_SELECT, st, k_row_select<true><<<pl->M, RW_THREADS, 0, st>>>(a));
    else MLMC_LAUNCH(K_ROW_SELECT, st, k_row_select<false><<<pl->M, RW_THREADS, 0, st>>>(a));
    if (message) MLMC_LAUNCH(K_ROW_WRITE, st, k_row_write<<<dim3(64 / (RWW_THREADS / 64), pl->M), RWW_THREADS, 0, st>>>(a));
    else MLMC_LAUNCH(K_ROW_WRITE, st, k_row_status<<<1, RW_THREADS, 0, st>>>(a));
    return MLMC_OK;
}

}  // namespace mlmc
