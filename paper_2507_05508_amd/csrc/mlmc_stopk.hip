// s-segmented Top-k MLMC on gfx950 (Sec. 2.2 "s-Top-k", Sec. 3.2, Lemma 3.4, App. D): the ladder k_l = min(s l, d),
// l = 0..L = ceil(d / s), g^0 = 0, adaptive level probabilities over all L bands.  The residual of level l is the
// l-th segment of the row sorted by magnitude.  Ladders of up to SE_LMAX levels are handled without a sort (second half of this
// file); longer ones, whose segments are a few entries, short rows and few short rows of 16 bits sort the whole row once:
//
//   k_rs_hist / k_rs_scan / k_rs_scatter   stable least-significant-digit radix sort of {inverted |g| key, index} pairs,
//                 8 bits per pass (4 passes for fp32, 2 for bf16 inputs whose keys have 16 significant bits); the
//                 first pass reads the gradients themselves.  Stable + initial index order = ties by lower index.
//   k_sb_norms    Delta_l for every band: exact integer sum of the squares of a segment (640-bit accumulate in LDS),
//                 rounded once to fp64, sqrt (Lemma 3.4, App. D)
//   k_sb_draw     p_l = Delta_l / sum Delta in level order, integer inverse CDF of the Philox word, weight (Alg. 3)
//   k_sb_mark / k_sb_offsets / k_sb_write   the drawn segment as an index-ordered message: its entries are marked in
//                 a bitmap over the row, tiles are counted and scanned, entries written in index order with their
//                 fp32 weight applied (Eq. (6))
#include "mlmc_device.h"

namespace mlmc {

constexpr int RS_TILE = 4096;     // elements of one sort block
constexpr int RS_THREADS = 256;   // four waves; wave w owns a quarter of the block, in order
constexpr int RS_PER_WAVE = RS_TILE / (RS_THREADS / 64);
constexpr int RS_GROUPS = RS_PER_WAVE / 64;   // 64-element groups of a wave

__device__ __forceinline__ uint32_t inv_key(uint32_t bits) { return 0x7FFFFFFFu - key_of_bits(bits); }   // ascending = magnitude descending

// One element of a sort pass.  FIRST: the pairs are formed from the gradients (index = position).
template <int DT, bool FIRST>
__device__ __forceinline__ uint2 rs_load(const StopkArgs& a, const RowLoader<DT, false>& ld, const uint2* src, int row, int64_t i) {
    if (FIRST) return make_uint2(inv_key(ld.load1(i)), (uint32_t)i);
    return src[(size_t)row * a.d + i];
}

// Digit counts of every block: counts[row][bin][blk].
template <int DT, bool FIRST>
__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(StopkArgs a, const uint2* src, int shift) {
    __shared__ uint32_t s_h[256];
    const int row = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x;
    s_h[tid] = 0;
    __syncthreads();
    RowLoader<DT, false> ld(a.g, a.ld, a.d, row);
    const int64_t i0 = (int64_t)blk * RS_TILE;
    const int64_t i1 = i0 + RS_TILE < a.d ? i0 + RS_TILE : a.d;
    bool nonfinite = false;
    // the block's loads issued sixteen at a time per thread (a loop of single loads waits for each in turn)
    batched_loop<RS_TILE / RS_THREADS, RS_THREADS>(0u, (uint32_t)(i1 - i0), (uint32_t)tid,
        [&](uint32_t i) { return rs_load<DT, FIRST>(a, ld, src, row, i0 + i).x; },
        [&](uint32_t, uint32_t key) {
            atomicAdd(&s_h[(key >> shift) & 255u], 1u);
            if (FIRST) nonfinite |= key <= 0x7FFFFFFFu - 0x7F800000u;   // Inf / NaN keys (ordered by their bit pattern)
        });
    if (FIRST && __ballot(nonfinite) && lane_id() == 0) atomicOr(a.dev_status, MLMC_DEV_NONFINITE);
    __syncthreads();
    a.counts[((size_t)row * 256 + tid) * a.nblk + blk] = s_h[tid];
}

// Exclusive prefix of counts[row][bin][.] over the blocks, one workgroup per (bin, row), and the bin's total; the
// scatter adds the totals of the lower bins.
__global__ __launch_bounds__(1024) void k_rs_scan(StopkArgs a) {
    __shared__ uint32_t s_scan[1024 / 64 + 1];
    const int bin = blockIdx.x, row = blockIdx.y, tid = threadIdx.x;
    uint32_t* c = a.counts + ((size_t)row * 256 + bin) * a.nblk;
    uint32_t carry = 0;
    for (int j0 = 0; j0 < a.nblk; j0 += 1024) {
        const int j = j0 + tid;
        const uint32_t v = j < a.nblk ? c[j] : 0u;
        uint32_t total;
        const uint32_t ex = block_excl_scan<1024>(v, s_scan, total);
        if (j < a.nblk) c[j] = carry + ex;
        carry += total;
    }
    if (tid == 0) a.bin_total[row * 256 + bin] = carry;
}

// Stable scatter of one pass.  Order is kept at every step: a wave walks its elements in order, lanes of a group
// rank themselves among the lanes with the same digit below them, waves and blocks start where the prefixes say.
// The block's pairs are first put in digit order in LDS, then written out: pairs of one digit go to consecutive
// addresses, so the writes come in runs instead of single 8-byte stores.
template <int DT, bool FIRST>
__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(StopkArgs a, const uint2* src, uint2* dst, int shift) {
    __shared__ uint32_t s_hist[RS_THREADS / 64][256];   // per wave and digit: the count, then (in place) the slot in the block's digit-ordered staging area
    uint32_t (*s_base)[256] = s_hist;
    __shared__ uint32_t s_gstart[256];                  // global position of the block's first pair of a digit minus its slot
    __shared__ uint32_t s_scan[RS_THREADS / 64 + 1];
    __shared__ uint2 s_stage[RS_TILE];
    const int row = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < (RS_THREADS / 64) * 256; i += RS_THREADS) (&s_hist[0][0])[i] = 0;
    __syncthreads();
    RowLoader<DT, false> ld(a.g, a.ld, a.d, row);
    const int64_t b0 = (int64_t)blk * RS_TILE;
    const int64_t w0 = b0 + (int64_t)wave * RS_PER_WAVE;
    uint2 e[RS_GROUPS];
    if (b0 + RS_TILE <= a.d) {   // a whole block (uniform): no bounds check between the loads, they are issued together
#pragma unroll
        for (int q = 0; q < RS_GROUPS; ++q) e[q] = rs_load<DT, FIRST>(a, ld, src, row, w0 + q * 64 + lane);
    } else {
#pragma unroll
        for (int q = 0; q < RS_GROUPS; ++q) {
            const int64_t i = w0 + q * 64 + lane;
            e[q] = i < a.d ? rs_load<DT, FIRST>(a, ld, src, row, i) : make_uint2(0u, 0u);
        }
    }
#pragma unroll
    for (int q = 0; q < RS_GROUPS; ++q)
        if (w0 + q * 64 + lane < a.d) atomicAdd(&s_hist[wave][(e[q].x >> shift) & 255u], 1u);
    __syncthreads();
    {
        // digit `tid`: its pairs of this block start at (lower bins of the row) + (earlier blocks of the bin) in the
        // output, and at (lower digits of this block) in the staging area
        uint32_t row_total, blk_total, mine = 0;
#pragma unroll
        for (int w = 0; w < RS_THREADS / 64; ++w) mine += s_hist[w][tid];
        const uint32_t lower = block_excl_scan<RS_THREADS>(a.bin_total[row * 256 + tid], s_scan, row_total);
        if (tid == 0 && (int64_t)row_total != a.d) atomicOr(a.dev_status, MLMC_DEV_INTERNAL);
        const uint32_t slot0 = block_excl_scan<RS_THREADS>(mine, s_scan, blk_total);
        s_gstart[tid] = lower + a.counts[((size_t)row * 256 + tid) * a.nblk + blk] - slot0;
        uint32_t run = slot0;
#pragma unroll
        for (int w = 0; w < RS_THREADS / 64; ++w) {
            const uint32_t c = s_hist[w][tid];
            s_base[w][tid] = run;
            run += c;
        }
    }
    __syncthreads();
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int q = 0; q < RS_GROUPS; ++q) {
        const bool valid = w0 + q * 64 + lane < a.d;
        const uint32_t digit = (e[q].x >> shift) & 255u;
        uint64_t peers = __ballot(valid);   // lanes with this lane's digit
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t m = __ballot(valid && ((digit >> b) & 1u));
            peers &= ((digit >> b) & 1u) ? m : ~m;
        }
        const uint32_t rank = (uint32_t)__popcll(peers & below);
        const uint32_t base = s_base[wave][digit];
        wave_lds_sync();   // every lane has read its base before a leader moves it on
        if (valid && rank == 0) s_base[wave][digit] = base + (uint32_t)__popcll(peers);
        wave_lds_sync();
        if (valid) s_stage[base + rank] = e[q];
    }
    __syncthreads();
    uint2* out = dst + (size_t)row * a.d;
    const int nvalid = (int)(a.d - b0 < RS_TILE ? a.d - b0 : RS_TILE);
    for (int i = tid; i < nvalid; i += RS_THREADS) {
        const uint2 p = s_stage[i];
        out[s_gstart[(p.x >> shift) & 255u] + (uint32_t)i] = p;
    }
}

// Delta_l of every band of every row from the sorted pairs: a wave takes bands in turn.  The squares of a segment are
// added exactly: sig^2 * 2^(2 (E' - 1)) in units of 2^-298, split into 32-bit words that go to 64-bit counters of their
// word positions (LDS atomics, any order), one carry pass, one rounding to fp64, sqrt.
constexpr int SN_WAVES = 4;
__global__ __launch_bounds__(SN_WAVES * 64) void k_sb_norms(StopkArgs a, const uint2* sorted) {
    __shared__ unsigned long long s_wide[SN_WAVES][20];
    __shared__ uint32_t s_big[SN_WAVES][20];
    const int row = blockIdx.y;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint2* sp = sorted + (size_t)row * a.d;
    for (int64_t band = (int64_t)blockIdx.x * SN_WAVES + wave; band < a.L; band += (int64_t)gridDim.x * SN_WAVES) {
        if (lane < 20) s_wide[wave][lane] = 0ull;
        wave_lds_sync();
        const int64_t lo = band * a.s, hi = lo + a.s < a.d ? lo + a.s : a.d;
        // A lane meets its keys in descending order, so their exponents come in runs: the squares of a run are summed in
        // registers (low and high halves apart, no overflow for any segment length) and reach LDS once per run.
        auto flush = [&](uint32_t E, uint64_t slo, uint64_t shi) {
            const int shift = 2 * ((int)(E ? E : 1u) - 1);
            auto add = [&](uint64_t v, int sh) {
                if (!v) return;
                const int wi = sh >> 5, bs = sh & 31;
                const uint32_t p0 = (uint32_t)(v << bs);
                const uint32_t p1 = (uint32_t)(bs ? v >> (32 - bs) : v >> 32);
                const uint32_t p2 = bs ? (uint32_t)(v >> (64 - bs)) : 0u;
                if (p0 && wi < 20) atomicAdd(&s_wide[wave][wi], (unsigned long long)p0);
                if (p1 && wi + 1 < 20) atomicAdd(&s_wide[wave][wi + 1], (unsigned long long)p1);
                if (p2 && wi + 2 < 20) atomicAdd(&s_wide[wave][wi + 2], (unsigned long long)p2);
            };
            add(slo, shift);
            add(shi, shift + 32);
        };
        uint32_t curE = 0xFFFFFFFFu;
        uint64_t slo = 0, shi = 0;
        // eight loads of a lane in flight (past the segment's end: its last entry, ignored), consumed in order
        for (int64_t i = lo + lane; i < hi; i += 64 * 8) {
            uint32_t kx[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t j = i + 64 * u;
                kx[u] = sp[j < hi ? j : hi - 1].x;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (i + 64 * u < hi) {
                    const uint32_t key = 0x7FFFFFFFu - kx[u];
                    const uint32_t E = key >> 23;
                    if (E != curE) {
                        if (curE != 0xFFFFFFFFu) flush(curE, slo, shi);
                        curE = E;
                        slo = 0;
                        shi = 0;
                    }
                    const uint64_t sq = sig_square(key);
                    slo += sq & 0xFFFFFFFFull;
                    shi += sq >> 32;
                }
            }
        }
        if (curE != 0xFFFFFFFFu) flush(curE, slo, shi);
        wave_lds_sync();
        if (lane == 0) {
            unsigned long long carry = 0;
            for (int i = 0; i < 20; ++i) {
                const unsigned long long t = s_wide[wave][i] + carry;
                s_big[wave][i] = (uint32_t)t;
                carry = t >> 32;
            }
            BigAcc acc;
            acc.w = s_big[wave];
            const double nrm = __dsqrt_rn(acc.to_double());
            a.norms[(size_t)row * a.L + band] = nrm;
            if (a.norms_user) a.norms_user[(size_t)row * a.L + band] = nrm;
        }
        wave_lds_sync();
    }
}

// Level draw of every row (Alg. 3): p_l = Delta_l / (Delta_1 + ... + Delta_L).  The sum and the running CDF are taken in
// level order by one thread (the order fixes the roundings) - but only the additions: the quotients before them and the
// integer thresholds and comparisons after them are independent per level and spread over the workgroup.  The norms
// pass through LDS in chunks.  Bound by the chain of additions, which the second time ends where the draw is settled: 1000 levels 25.7 -> 12.8 us
// against reads that are waited for and a CDF to its end; 8 rows of 1.17e7, compress + aggregate, 419 -> 408.
constexpr int SD_CHUNK = 8192;
static_assert(SD_CHUNK % 16 == 0, "entries are taken by sixteen");
// next(i, v): takes s_n[i .. i + 16), i = 0, 16, ... below n (a multiple of 16), in order; true: enough.  Returns the first entry it was not given.  Sixteen
// reads are in flight while the sixteen before them are added: waited for in turn, they took as long as the additions.
template <class F>
__device__ __forceinline__ int sd_sixteens(const double* s_n, int n, F next) {
    auto fetch = [&](int i, double (&v)[16]) {
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = s_n[i + u];
        __builtin_amdgcn_sched_barrier(0);   // issued before the additions that follow
    };
    double va[16], vb[16];
    fetch(0, va);
    for (int i = 0;; i += 32) {
        fetch(i + 16 < n ? i + 16 : 0, vb);   // past the end: not used
        if (next(i, va) || i + 16 >= n) return i + 16;
        fetch(i + 32 < n ? i + 32 : 0, va);
        if (next(i + 16, vb) || i + 32 >= n) return i + 32;
    }
}
__global__ __launch_bounds__(1024) void k_sb_draw(StopkArgs a) {
    __shared__ double s_n[SD_CHUNK];     // norms, then probabilities, of the chunk
    __shared__ double s_cdf[SD_CHUNK];   // running sums of the probabilities up to every level of the chunk
    __shared__ double s_tot;
    __shared__ int32_t s_done;           // levels of the chunk that have their running sum
    __shared__ int32_t s_found;          // lowest level met so far whose threshold lies above the drawn word
    const int row = blockIdx.x, tid = threadIdx.x;
    const double* nr = a.norms + (size_t)row * a.L;
    const int L = a.L;
    double tot = 0.0;
    for (int c0 = 0; c0 < L; c0 += SD_CHUNK) {
        const int n = L - c0 < SD_CHUNK ? L - c0 : SD_CHUNK, n16 = (n + 15) & ~15;
        __syncthreads();
        for (int i = tid; i < n16; i += 1024) s_n[i] = i < n ? nr[c0 + i] : 0.0;   // (a zero more changes no sum)
        __syncthreads();
        if (tid == 0)
            (void)sd_sixteens(s_n, n16, [&](int, const double (&v)[16]) {
#pragma unroll
                for (int u = 0; u < 16; ++u) tot = __dadd_rn(tot, v[u]);
                return false;
            });
    }
    if (tid == 0) { s_tot = tot; s_found = 0x7FFFFFFF; }
    __syncthreads();
    tot = s_tot;
    const uint32_t x = philox_word0(a.seed, a.step, (uint32_t)row);
    const double uni = __ddiv_rn(1.0, (double)L);
    const double stop = __dmul_rn((double)x + 1.0, 0x1p-32);   // (exact) a running sum from here on has its threshold above the drawn word: no later level is needed
    double c = 0.0, pl = 0.0;
    int level = L;
    for (int c0 = 0; c0 < L; c0 += SD_CHUNK) {
        const int n = L - c0 < SD_CHUNK ? L - c0 : SD_CHUNK, n16 = (n + 15) & ~15;
        __syncthreads();
        for (int i = tid; i < n16; i += 1024) s_n[i] = i >= n ? 0.0 : tot == 0.0 ? uni : __ddiv_rn(nr[c0 + i], tot);
        __syncthreads();
        if (tid == 0)
            s_done = sd_sixteens(s_n, n16, [&](int at, const double (&v)[16]) {
                double run[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) { c = __dadd_rn(c, v[u]); run[u] = c; }
#pragma unroll
                for (int u = 0; u < 16; ++u) s_cdf[at + u] = run[u];
                return c >= stop;
            });
        __syncthreads();
        const int done = s_done < n ? s_done : n;
        for (int i = tid; i < done; i += 1024) {
            const double t = floor(__dmul_rn(s_cdf[i], 4294967296.0));
            uint64_t T;
            if (!(t > 0.0)) T = 0;
            else if (t >= 4294967296.0) T = 4294967296ull;
            else T = (uint64_t)t;
            if (c0 + i == L - 1) T = 4294967296ull;
            if ((uint64_t)x < T) atomicMin(&s_found, c0 + i + 1);
        }
        __syncthreads();
        if (s_found != 0x7FFFFFFF) {   // uniform: the chunk holds the level, and s_n its probability
            level = s_found;
            pl = s_n[level - 1 - c0];
            break;
        }
    }
    if (tid == 0) {
        SRow* sr = a.srow + row;
        sr->level = level;
        sr->weight = pl == 0.0 ? 0.0f : (float)__ddiv_rn(1.0, pl);
        const int64_t lo = (int64_t)(level - 1) * a.s;
        sr->lo = lo;
        sr->count = lo + a.s < a.d ? a.s : a.d - lo;
        if (a.se_thr) {   // ladders that are not sorted
            const uint2* thr = a.se_thr + (size_t)row * (a.L + 1) + level;
            const uint2 h = thr[-1], o = thr[0], got = a.se_marks ? a.se_got[row] : make_uint2(~0u, 0u);
            a.sseg[row] = SSeg{h, o, o.x >= got.x && h.x <= got.y ? 1 : 0, level, sr->weight, 0.0f};
        }
        a.level[row] = level;
    }
}

__global__ __launch_bounds__(256) void k_sb_clear(uint4* p, size_t n16, int32_t* dev_status) {
    const uint4 z = make_uint4(0, 0, 0, 0);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) p[i] = z;
    if (dev_status && blockIdx.x == 0 && threadIdx.x == 0) *dev_status = 0;
}

// The entries of the drawn segment, marked in the row's bitmap (bit j of the row: entry j is in the message) and counted
// per tile of 4096 indices.
__global__ __launch_bounds__(256) void k_sb_mark(StopkArgs a, const uint2* sorted) {
    const int row = blockIdx.y;
    const SRow sr = a.srow[row];
    uint32_t* bm = a.bitmap + (size_t)row * a.bm_words;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < sr.count; i += (int64_t)gridDim.x * 256) {
        const uint32_t j = sorted[(size_t)row * a.d + sr.lo + i].y;
        atomicOr(&bm[j >> 5], 1u << (j & 31u));
        atomicAdd(&a.tile_cnt[(size_t)row * a.ntiles + (j >> 12)], 1u);   // indices are distinct: an entry counts once
    }
}

// Per row: entries before every tile of 4096 indices, and where the row's message starts.
__global__ __launch_bounds__(1024) void k_sb_offsets(StopkArgs a) {
    __shared__ uint32_t s_scan[1024 / 64 + 1];
    const int row = blockIdx.x, tid = threadIdx.x;
    uint32_t* to = a.tile_off + (size_t)row * (a.ntiles + 1);
    const uint32_t* tc = a.tile_cnt + (size_t)row * a.ntiles;
    uint32_t carry = 0;
    for (int64_t j0 = 0; j0 < a.ntiles; j0 += 1024) {
        const int64_t t = j0 + tid;
        const uint32_t c = t < a.ntiles ? tc[t] : 0u;
        uint32_t round_total;
        const uint32_t ex = block_excl_scan<1024>(c, s_scan, round_total);
        if (t < a.ntiles) to[t] = carry + ex;
        carry += round_total;
    }
    const uint32_t total = carry;
    if (tid == 0) {
        to[a.ntiles] = total;
        if ((int64_t)total != a.srow[row].count) atomicOr(a.dev_status, MLMC_DEV_INTERNAL);
        int64_t start = 0;
        for (int r = 0; r < row; ++r) start += a.srow[r].count;
        a.row_off[row] = start;
        if (row == a.M - 1) {
            a.row_off[a.M] = start + total;
            if (start + (int64_t)total > a.capacity) atomicOr(a.dev_status, MLMC_DEV_CAPACITY);
        }
    }
}

// The message of a row in index order: a wave takes a tile, a lane two words of its bitmap.
template <int DT>
__global__ __launch_bounds__(256) void k_sb_write(StopkArgs a) {
    const int row = blockIdx.y;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = (int64_t)blockIdx.x * 4 + wave;
    if (tile >= a.ntiles) return;
    const uint32_t* bm = a.bitmap + (size_t)row * a.bm_words;
    const uint32_t* to = a.tile_off + (size_t)row * (a.ntiles + 1);
    if (to[tile + 1] == to[tile]) return;   // nothing of the segment in this tile
    RowLoader<DT, false> ld(a.g, a.ld, a.d, row);
    const float w = a.srow[row].weight;
    const int64_t w0 = tile * (TILE / 32) + lane * 2;
    uint32_t b0 = w0 < a.bm_words ? bm[w0] : 0u, b1 = w0 + 1 < a.bm_words ? bm[w0 + 1] : 0u;
    const uint32_t mine = (uint32_t)__popc(b0) + (uint32_t)__popc(b1);
    uint32_t inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += u;
    }
    int64_t at = a.row_off[row] + to[tile] + (inc - mine);
    auto emit = [&](uint32_t bits, int64_t jbase) {
        while (bits) {
            const int b = __builtin_ctz(bits);
            bits &= bits - 1u;
            const int64_t j = jbase + b;
            if (at < a.capacity) {
                a.idx[at] = (uint32_t)j;
                a.val[at] = __fmul_rn(__uint_as_float(ld.load1(j)), w);
            }
            ++at;
        }
    };
    emit(b0, w0 * 32);
    emit(b1, (w0 + 1) * 32);
}

// ---------------------------------------------------------------------------------------------------
template <int DT>
static mlmc_status launch_stopk(const mlmc_plan_t* pl, const StopkArgs& a, bool message, hipStream_t st) {
    const dim3 sgrid(a.nblk, pl->M);
    // bitmaps, tile counts and device status start at zero
    {
        const size_t n16 = a.clear_bytes / 16;   // the bitmaps and, right behind them, the tile counts
        int blocks = (int)((n16 + 255) / 256);
        if (blocks > 2048) blocks = 2048;
        MLMC_LAUNCH(K_ZERO, st, k_sb_clear<<<blocks, 256, 0, st>>>((uint4*)a.bitmap, n16, a.dev_status));
    }
    // sort: pass 0 reads the gradients; bf16 keys have their low 16 bits clear, so their two low digits are constant
    const int first_shift = pl->dtype == MLMC_BF16 ? 16 : 0;
    uint2* bufs[2] = {a.pa, a.pb};
    int cur = 0;   // the pass writes bufs[cur]
    for (int shift = first_shift; shift < 32; shift += 8) {
        const uint2* src = shift == first_shift ? nullptr : bufs[cur ^ 1];
        if (shift == first_shift) {
            MLMC_LAUNCH(K_RS_HIST, st, k_rs_hist<DT, true><<<sgrid, RS_THREADS, 0, st>>>(a, src, shift));
            MLMC_LAUNCH(K_RS_SCAN, st, k_rs_scan<<<dim3(256, pl->M), 1024, 0, st>>>(a));
            MLMC_LAUNCH(K_RS_SCATTER, st, k_rs_scatter<DT, true><<<sgrid, RS_THREADS, 0, st>>>(a, src, bufs[cur], shift));
        } else {
            MLMC_LAUNCH(K_RS_HIST, st, k_rs_hist<DT, false><<<sgrid, RS_THREADS, 0, st>>>(a, src, shift));
            MLMC_LAUNCH(K_RS_SCAN, st, k_rs_scan<<<dim3(256, pl->M), 1024, 0, st>>>(a));
            MLMC_LAUNCH(K_RS_SCATTER, st, k_rs_scatter<DT, false><<<sgrid, RS_THREADS, 0, st>>>(a, src, bufs[cur], shift));
        }
        cur ^= 1;
    }
    const uint2* sorted = bufs[cur ^ 1];
    {
        int64_t gx = (a.L + SN_WAVES - 1) / SN_WAVES;
        const int64_t cap = 8192 / pl->M > 0 ? 8192 / pl->M : 1;
        if (gx > cap) gx = cap;
        MLMC_LAUNCH(K_SB_NORMS, st, k_sb_norms<<<dim3((unsigned)gx, pl->M), SN_WAVES * 64, 0, st>>>(a, sorted));
    }
    if (!message) return MLMC_OK;
    MLMC_LAUNCH(K_SB_DRAW, st, k_sb_draw<<<pl->M, 1024, 0, st>>>(a));
    {
        int64_t gx = (a.s + 255) / 256;
        if (gx > 1024) gx = 1024;
        MLMC_LAUNCH(K_SB_MARK, st, k_sb_mark<<<dim3((unsigned)gx, pl->M), 256, 0, st>>>(a, sorted));
    }
    MLMC_LAUNCH(K_SB_OFFSETS, st, k_sb_offsets<<<pl->M, 1024, 0, st>>>(a));
    MLMC_LAUNCH(K_SB_WRITE, st, k_sb_write<DT><<<dim3((unsigned)((a.ntiles + 3) / 4), pl->M), 256, 0, st>>>(a));
    return MLMC_OK;
}

// ---------------------------------------------------------------------------------------------------
// The way without a sort, for ladders of up to SE_LMAX levels.  What the norms need is, per band, the exact sum of its
// squares, and what the message needs is two thresholds; neither needs an order among the entries of a band.  So:
//   k_se_coarse / k_se_map   a histogram of sampled blocks (13 bits of the key) gives a monotone map key -> one of at most
//                 SE_BINS bins of about equal occupancy, every bin inside one exponent, zero in a bin of its own
//   k_se_count / k_se_reduce exact counts of the bins (first read of the rows), per workgroup, then summed over the workgroups
//   k_se_scan     ranks of the bins: a bin whose ranks lie inside one band is a REGION of that band, one that holds band
//                 boundaries a ZONE (for L = 1000 and the occupancies met here about 5 % of the entries), unless all its
//                 entries have one key, in which case the boundaries' parts follow from the counts
//   k_se_split    second read: squares of region entries are added per (band, exponent) in LDS, keys of zone entries go to
//                 their zones' lists, whose places are exact (the counts are)
//   k_se_zone     per zone of few entries: keys in order, thresholds of its boundaries (key, how many of the equal keys are
//                 inside), sums of its parts
//   k_se_wide     the same for zones of many entries (repeated keys; rows that the sample misjudged), by counts of their keys
//   k_se_norms / k_sb_draw   Delta_l, level
//   k_se_mark / k_se_offsets / k_se_write   bitmap of the drawn segment and its message; entries equal to a
//                 threshold whose equal keys are split are told apart by their rank in index order: a third read of the rows.  In large plans
//                 (se_marks) the exact counts of the bins give the norms to about 1e-4, and with them, before the second read, a key window that holds
//                 the drawn segment nearly always: that read leaves a bit per four entries and only those are looked at (73 -> 13 us, the second one
//                 121 -> 119 with what the forecast and the marks cost it, 11)
// Two reads of the rows, three in smaller plans, and about 10 bytes per entry of other traffic against 4 x 24 bytes and more for the sort of pairs:
// 8 rows of 1.17e7 fp32 entries at 1000 levels, compress + aggregate: 2788 -> 430 us; with the forecast, one addition per entry in the second read
// and zones of one boundary ranked in one bucket 401 -> 325.  The line at SE_LMAX levels is where the
// class of a bin and the list cursors of a zone per boundary still fit LDS beside the map and the sums.
constexpr int SE_CB = 8192;             // coarse buckets: key >> SE_CSHIFT
constexpr int SE_CSHIFT = 18;
constexpr int SE_THREADS = 1024;
constexpr int SE_WAVES = SE_THREADS / 64;
constexpr int SE_ZCAP = 2048;           // keys that a zone's workgroup puts in order in LDS
// Zones of more entries: first counts of 2^SE_ZBITS sub-bins, then of the (at most 16) keys of every sub-bin that holds boundaries.
// Up to SE_ZBIG entries one workgroup does both in LDS; more are taken in slices of SE_ZSLICE by many, the counts in the
// zone's place of the second list: 2^SE_ZBITS + 16 SE_LMAX words and one for the ticket.
constexpr int SE_ZBITS = 14;
constexpr uint32_t SE_ZSUB = 1u << SE_ZBITS, SE_ZSLICE = 65536;   // a slice's squares (below 2^48 each) fit a 64-bit sum
static_assert(SE_CSHIFT - SE_ZBITS <= 4 && SE_ZBIG == (1 << SE_ZBITS) + 16 * SE_LMAX, "place of a zone's counts");
// Slots of k_se_split: the sums of the L + 256 groups in 2^se_rep lane-interleaved copies, behind them the cursors of the zones (fewer than L).
constexpr int SE_SLOTS = 2 * SE_LMAX + 256;
static_assert(SE_SLOTS < 0x10000, "class of a bin: its slot");

// entry: of the key's coarse bucket, shift | base << 16 (a shift takes the low five bits of its count as they are)
__device__ __forceinline__ uint32_t se_bin(uint32_t entry, uint32_t key) {
    return (entry >> 16) + ((key & ((1u << SE_CSHIFT) - 1u)) >> (entry & 31u)) + (key < 1u ? key : 1u);
}

// One more in h[b] for the active lanes that want it.  LDS atomics of many lanes on one word take a turn each (about three
// clocks): where many share the first one's word, and then the next one's, they are added at once.
__device__ __forceinline__ void se_count_peeled(uint32_t* h, uint32_t b, bool want) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint64_t w = __ballot(want);
        if (w == 0) return;
        const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)b, __builtin_ctzll(w));
        const uint64_t same = __ballot(want && b == b0);
        if (__popcll(same) < 8) break;   // uniform
        if (lane_id() == (uint32_t)__builtin_ctzll(w)) atomicAdd(&h[b0], (uint32_t)__popcll(same));
        want = want && b != b0;
    }
    if (want) atomicAdd(&h[b], 1u);
}

// Coarse histogram of the sampled blocks of 1024 entries (block b is sampled when b % 2^shift == 2^shift / 2).
template <int DT>
__global__ __launch_bounds__(512) void k_se_coarse(StopkArgs a) {
    __shared__ uint32_t s_h[SE_CB];
    const int row = blockIdx.y, tid = threadIdx.x;
    const int64_t nblk = (a.d + 1023) >> 10, first = ((int64_t)1 << a.se_shift) >> 1;
    for (int i = tid; i < SE_CB; i += 512) s_h[i] = 0;
    __syncthreads();
    RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    for (int64_t i = (int64_t)blockIdx.x * 8 + wave; (i << a.se_shift) + first < nblk; i += (int64_t)gridDim.x * 8) {
        const int64_t base = ((i << a.se_shift) + first) * 1024;
        uint32_t b[4][4];
        int nv[4] = {4, 4, 4, 4};
        if (base + 1024 <= a.d) {   // uniform
#pragma unroll
            for (int q = 0; q < 4; ++q) ld.load4_full(base + q * 256 + lane * 4, b[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) nv[q] = ld.load4(base + q * 256 + lane * 4, b[q]);
        }
        uint32_t other = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                b[q][c] = c < nv[q] ? key_of_bits(b[q][c]) >> SE_CSHIFT : SE_CB;
                other |= b[q][c] ^ b[0][0];
            }
        if (other == 0 && nv[0] == 4) {   // (all four are whole: a missing entry is unlike any other)
            atomicAdd(&s_h[b[0][0]], 16u);   // LDS atomics of many lanes on one word take turns: rows of one value
            continue;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (b[q][c] < (uint32_t)SE_CB) atomicAdd(&s_h[b[q][c]], 1u);
    }
    __syncthreads();
    uint32_t* h = a.se_coarse + (size_t)row * SE_CB;
    for (int i = tid; i < SE_CB; i += 512)
        if (s_h[i]) atomicAdd(&h[i], s_h[i]);
}

// Per row: the map.  A sampled bucket gets a power of two of bins in proportion to its count, any other one; the share is
// the largest of five that fit.  16-bit inputs: a bucket has four keys, it gets a bin for each.
template <int DT>
__global__ __launch_bounds__(1024) void k_se_map(StopkArgs a) {
    __shared__ uint32_t s_scan[1024 / 64 + 1], s_need[5];
    constexpr int PER = SE_CB / 1024;
    constexpr uint32_t ROOM = SE_BINS - 1;          // zero has a bin of its own
    constexpr uint32_t SHARE = ROOM - SE_CB;
    const int row = blockIdx.x, tid = threadIdx.x;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) { c[i] = a.se_coarse[(size_t)row * SE_CB + tid * PER + i]; sum += c[i]; }
    uint32_t ns;
    if (tid < 5) s_need[tid] = 0;
    block_excl_scan<1024>(sum, s_scan, ns);
    // log2 of the bins of bucket i at share m / 4 (16-bit inputs: m = 8 stands for a bin per key, 4 for one per bucket)
    const unsigned long long unit = ((unsigned long long)SHARE << 30) / ns;   // bins per sampled entry at share 1, times 2^30
    auto bits = [&](int i, uint32_t m) -> uint32_t {
        if (!c[i]) return 0u;
        if (DT == MLMC_BF16) return m == 8u ? 2u : 0u;
        const uint32_t v = (uint32_t)((c[i] * unit * m) >> 32);   // rounded down; c unit <= SHARE 2^30
        const uint32_t k = v ? 31u - (uint32_t)__clz((int)v) : 0u;
        return k < (uint32_t)SE_CSHIFT ? k : (uint32_t)SE_CSHIFT;
    };
#pragma unroll
    for (uint32_t m = 4; m <= 8; ++m) {
        uint32_t need = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) need += 1u << bits(i, m);
        need = wave_sum(need);
        if (lane_id() == 0) atomicAdd(&s_need[m - 4u], need);
    }
    __syncthreads();
    uint32_t m = 8;
    while (m > 4u && s_need[m - 4u] > ROOM) --m;   // m = 4 always fits
    uint32_t kb[PER], need = 0, nbins;
#pragma unroll
    for (int i = 0; i < PER; ++i) { kb[i] = bits(i, m); need += 1u << kb[i]; }
    const uint32_t before = block_excl_scan<1024>(need, s_scan, nbins);
    uint32_t* map = a.se_map + (size_t)row * SE_CB;
    uint32_t base = before;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t e = base << 16 | ((uint32_t)SE_CSHIFT - kb[i]);
        map[tid * PER + i] = e;
        base += 1u << kb[i];
    }
    if (tid == 0) {
        a.se_info[(size_t)row * SE_BINS] = make_uint2(0u, 0u);
        a.se_nbins[row] = nbins + 1;
    }
}

// Exact counts of a workgroup's slice of a row.
template <int DT, bool STREAM>
__global__ __launch_bounds__(SE_THREADS) void k_se_count(StopkArgs a) {
    __shared__ __align__(16) uint32_t s_map[SE_CB];
    __shared__ __align__(16) uint32_t s_cnt[SE_BINS];
    const int row = blockIdx.y, tid = threadIdx.x;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < SE_CB / 4; i += SE_THREADS) ((uint4*)s_map)[i] = ((const uint4*)(a.se_map + (size_t)row * SE_CB))[i];
    for (int i = tid; i < SE_BINS / 4; i += SE_THREADS) ((uint4*)s_cnt)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    // The bins' records, {lowest key, shift}, for the launches behind this one: a share of the buckets for every workgroup of the row (the one
    // workgroup that makes the map took 16 us with them, 8 rows of 1.17e7 entries, 7.8 without).  A wave takes 16 buckets: small ones a lane each, large ones together.
    uint2* info = a.se_info + (size_t)row * SE_BINS;
    for (uint32_t b0 = (wave * gridDim.x + blockIdx.x) * 16u; b0 < (uint32_t)SE_CB; b0 += gridDim.x * (uint32_t)(SE_WAVES * 16)) {
        const uint32_t e = s_map[b0 + (lane & 15u)], sh = e & 31u, n = lane < 16u ? 1u << (SE_CSHIFT - sh) : 0u;
        if (n <= 8u)
            for (uint32_t i = 0; i < n; ++i) {
                const uint32_t key = ((b0 + lane) << SE_CSHIFT) + (i << sh);
                info[1 + (e >> 16) + i] = make_uint2(key ? key : 1u, sh);   // zeros are in bin 0: a threshold at this bin leaves them out
            }
        uint64_t big = __ballot(n > 8u);
        while (big) {   // uniform
            const int l = __builtin_ctzll(big);
            big &= big - 1;
            const uint32_t eb = (uint32_t)__builtin_amdgcn_readlane((int)e, l), shb = eb & 31u, nb = 1u << (SE_CSHIFT - shb);
            for (uint32_t i = lane; i < nb; i += 64) {
                const uint32_t key = ((b0 + (uint32_t)l) << SE_CSHIFT) + (i << shb);
                info[1 + (eb >> 16) + i] = make_uint2(key ? key : 1u, shb);
            }
        }
    }
    RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    const int64_t i0 = (int64_t)blockIdx.x * a.se_slice, i1 = i0 + a.se_slice < a.d ? i0 + a.se_slice : a.d;
    uint32_t maxkey = 0;
    stream_slice<DT, SE_WAVES, STREAM>(ld, i0, i1, wave, lane, [&](const uint32_t (&k)[4][4], const int (&nv)[4]) {
        uint32_t e[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) e[q][c] = s_map[k[q][c] >> SE_CSHIFT];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c < nv[q]) {
                    atomicAdd(&s_cnt[se_bin(e[q][c], k[q][c])], 1u);
                    maxkey = k[q][c] > maxkey ? k[q][c] : maxkey;
                }
    });
    if (__ballot(maxkey >= 0x7F800000u) && lane == 0) atomicOr(a.dev_status, MLMC_DEV_NONFINITE);
    __syncthreads();
    uint4* part = (uint4*)(a.se_part + ((size_t)row * gridDim.x + blockIdx.x) * SE_BINS);
    const int n4 = ((int)a.se_nbins[row] + 3) / 4;
    for (int i = tid; i < n4; i += SE_THREADS) part[i] = ((const uint4*)s_cnt)[i];
}

// Per bin: exclusive prefix over the workgroups, in place, and the total; the total of every 256 bins.
constexpr int SE_BLOCKS = (SE_BINS + 255) / 256;
__global__ __launch_bounds__(256) void k_se_reduce(StopkArgs a) {
    __shared__ uint32_t s_scan[256 / 64 + 1];
    const int row = blockIdx.y;
    const uint32_t bin = blockIdx.x * 256 + threadIdx.x;
    const uint32_t nbins = a.se_nbins[row];
    if (blockIdx.x * 256 >= nbins) return;
    uint32_t* p = a.se_part + (size_t)row * a.se_wgs * SE_BINS + bin;
    uint32_t run = 0;
    int g = bin < nbins ? 0 : a.se_wgs;
    for (; g + 8 <= a.se_wgs; g += 8) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(size_t)(g + u) * SE_BINS];
#pragma unroll
        for (int u = 0; u < 8; ++u) { p[(size_t)(g + u) * SE_BINS] = run; run += v[u]; }
    }
    for (; g < a.se_wgs; ++g) {
        const uint32_t v = p[(size_t)g * SE_BINS];
        p[(size_t)g * SE_BINS] = run;
        run += v;
    }
    if (bin < nbins) a.se_total[(size_t)row * SE_BINS + bin] = run;
    uint32_t all;
    block_excl_scan<256>(run, s_scan, all);
    if (threadIdx.x == 0) a.se_bsum[row * SE_BLOCKS + blockIdx.x] = all;
}

// value * 2^shift (in units of 2^-298) into the 64-bit word counters of a band
__device__ __forceinline__ void se_add(unsigned long long* wide, uint64_t v, int shift) {
    if (!v) return;
    const int wi = shift >> 5, bs = shift & 31;
    const uint32_t p0 = (uint32_t)(v << bs);
    const uint32_t p1 = (uint32_t)(bs ? v >> (32 - bs) : v >> 32);
    const uint32_t p2 = bs ? (uint32_t)(v >> (64 - bs)) : 0u;
    if (p0 && wi < SE_WORDS) atomicAdd(&wide[wi], (unsigned long long)p0);
    if (p1 && wi + 1 < SE_WORDS) atomicAdd(&wide[wi + 1], (unsigned long long)p1);
    if (p2 && wi + 2 < SE_WORDS) atomicAdd(&wide[wi + 2], (unsigned long long)p2);
}
__device__ __forceinline__ int se_exp_shift(uint32_t key) {   // of the square of a significand
    const uint32_t E = key >> 23;
    return 2 * ((int)(E ? E : 1u) - 1);
}

// Per 256 bins: their ranks in descending order of their keys, classes, zones, thresholds that fall on bin edges.
__global__ __launch_bounds__(256) void k_se_scan(StopkArgs a) {
    __shared__ uint32_t s_scan[256 / 64 + 1];
    __shared__ uint32_t s_z0, s_off0, s_many, s_wide;
    __shared__ uint4 s_key[256];   // one-key bins with many boundaries: key, entries above, entries, boundaries
    __shared__ uint4 s_win[256];   // bins with many boundaries: lowest key, shift, entries above, entries
    __shared__ double s_apx[256];  // squares of the bins, added up by band from the workgroup's first one
    const int row = blockIdx.y, blk = blockIdx.x, tid = threadIdx.x;
    const int nbins = (int)a.se_nbins[row], nblk = (nbins + 255) / 256;
    if (blk >= nblk) return;
    const uint32_t s = (uint32_t)(a.s < a.d ? a.s : a.d), last_t = (uint32_t)a.L - 1u;   // boundaries 1 .. L - 1 at ranks t s
    const int bin = blk * 256 + 255 - tid;
    const uint32_t n = bin < nbins ? a.se_total[(size_t)row * SE_BINS + bin] : 0u;
    const uint2 in = bin < nbins ? a.se_info[(size_t)row * SE_BINS + bin] : make_uint2(0u, 0u);
    uint32_t above, mine;
    static_assert(SE_BLOCKS <= 256, "a thread takes a block's total");
    block_excl_scan<256>(tid > blk && tid < nblk ? a.se_bsum[row * SE_BLOCKS + tid] : 0u, s_scan, above);
    const uint32_t cum = above + block_excl_scan<256>(n, s_scan, mine);
    if (blk == 0 && tid == 0 && (int64_t)above + mine != a.d) atomicOr(a.dev_status, MLMC_DEV_INTERNAL);
    // boundaries strictly inside ranks [cum, cum + n): t0 .. t0 + nb - 1
    const uint32_t t0 = cum / s + 1u;
    uint32_t t1 = n ? (cum + n - 1u) / s : 0u;
    if (t1 > last_t) t1 = last_t;
    const uint32_t nb = t1 >= t0 ? t1 - t0 + 1u : 0u;
    const bool one_key = in.y == 0u || (a.bf16 && in.y <= 16u);
    const bool zone = nb && !one_key;
    uint32_t zones, zents;   // zones are numbered, and their lists placed, in any order
    const uint32_t z = block_excl_scan<256>(zone ? 1u : 0u, s_scan, zones);
    const uint32_t zoff = block_excl_scan<256>(zone ? n : 0u, s_scan, zents);
    if (tid == 0 && zones) {
        s_z0 = atomicAdd(&a.se_nz[SE_NZ * row], zones);
        s_off0 = atomicAdd(&a.se_nz[SE_NZ * row + 1], zents);
    }
    if (tid == 0) s_many = s_wide = 0;
    s_apx[tid] = 0.0;
    __syncthreads();
    uint2* thr = a.se_thr + (size_t)row * (a.L + 1);
    // For the forecast of the drawn segment: the keys of the bin that a boundary lies in, and the squares of the bins, each entry at the middle
    // of its bin (they choose what the second read marks, nothing else, so the order of the additions is free).
    const uint32_t band0 = above / s;
    uint2* win = a.se_win + (size_t)row * (a.L + 1);
    auto apx_add = [&](uint32_t band, double e) {
        if (band - band0 < 256u) unsafeAtomicAdd(&s_apx[band - band0], e);
        else unsafeAtomicAdd(&a.se_apx[(size_t)row * a.L + band], e);
    };
    auto mid_square = [&](uint32_t lo, uint32_t shift) -> double {
        const double v = (double)__uint_as_float(lo + ((1u << shift) >> 1));
        return __dmul_rn(v, v);
    };
    auto forecast_parts = [&](uint32_t lo, uint32_t shift, uint32_t above, uint32_t n, uint32_t u0, uint32_t step) {
        const double sq = mid_square(lo, shift);
        const uint32_t t0 = above / s + 1u;
        uint32_t t1 = (above + n - 1u) / s;
        if (t1 > last_t) t1 = last_t;
        for (uint32_t t = t0 + u0; t <= t1 + 1u; t += step) {   // the part in band t (from 1), the boundary below it
            const uint32_t r0 = t > t0 ? (t - 1u) * s - above : 0u, r1 = t <= t1 ? t * s - above : n;
            apx_add(t - 1u, __dmul_rn(sq, (double)(r1 - r0)));
            if (t <= t1) win[t] = make_uint2(lo, lo + ((1u << shift) - 1u));
        }
    };
    // parts u0, u0 + step, ... of a key's entries: the first t s - above of them (by index) are inside boundary t
    auto key_parts = [&](uint32_t key, uint32_t above, uint32_t n, uint32_t nb, uint32_t u0, uint32_t step) {
        const uint64_t sq = sig_square(key);
        const int sh = se_exp_shift(key);
        const uint32_t t0 = above / s + 1u;
        for (uint32_t u = u0; u <= nb; u += step) {
            const uint32_t r0 = u ? (t0 + u - 1u) * s - above : 0u, r1 = u < nb ? (t0 + u) * s - above : n;
            unsigned long long* wide = a.se_big + ((size_t)row * a.L + (t0 + u - 1u)) * SE_WORDS;
            se_add(wide, (sq & 0xFFFFFFFFull) * (r1 - r0), sh);
            se_add(wide, (sq >> 32) * (r1 - r0), sh + 32);
            if (u < nb) thr[t0 + u] = make_uint2(key, r1);
        }
    };
    uint32_t code = ((uint32_t)a.L + 255u) << a.se_rep;   // sums nobody reads: an empty bin, or one key with boundaries inside
    if (n && nb == 0) {
        // (255 - exponent) + band: one step at least whenever the exponent or the band changes
        const uint32_t group = 255u - (in.x >> 23) + (t0 - 1u);
        a.se_gtab[(size_t)row * (a.L + 256) + group] = (in.x >> 23) << 16 | (t0 - 1u);   // exponent, band (from 0)
        code = group << a.se_rep;
    } else if (zone) {
        code = (((uint32_t)a.L + 256u) << a.se_rep) + s_z0 + z;   // a zone holds a boundary: fewer than L <= SE_LMAX zones
        SZone zr;
        zr.cum = cum;
        zr.n = n;
        zr.lo = in.x;
        zr.shift = in.y;
        zr.t0 = t0;
        zr.nb = nb;
        zr.off = s_off0 + zoff;
        zr.bin = (uint32_t)bin;
        a.se_zone[(size_t)row * a.L + s_z0 + z] = zr;
        if (n > (uint32_t)SE_ZCAP) {   // work of k_se_wide
            uint32_t* nz = a.se_nz + SE_NZ * row;
            if (n <= (uint32_t)SE_ZBIG) {
                a.se_mid[(size_t)row * a.se_mids + atomicAdd(&nz[2], 1u)] = s_z0 + z;
            } else {
                a.se_bigz[(size_t)row * a.se_bigs + atomicAdd(&nz[3], 1u)] = s_z0 + z;
                const uint32_t ns = (n + SE_ZSLICE - 1u) / SE_ZSLICE, at = atomicAdd(&nz[4], ns);
                for (uint32_t i = 0; i < ns; ++i) a.se_item[(size_t)row * a.se_items + at + i] = make_uint2(s_z0 + z, i);
            }
        }
    } else if (nb) {
        if (nb <= 32u) key_parts(in.x, cum, n, nb, 0u, 1u);
        else s_key[atomicAdd(&s_many, 1u)] = make_uint4(in.x, cum, n, nb);
    }
    if (n && (cum + n) % s == 0u && (cum + n) / s <= last_t) thr[(cum + n) / s] = make_uint2(in.x, SE_ALL);   // a boundary at the bin's lower edge
    if (bin < nbins) a.se_class[(size_t)row * SE_BINS + bin] = (uint16_t)code;
    if (blk == 0 && tid == 0) {
        thr[0] = make_uint2(0xFFFFFFFFu, 0u);
        thr[a.L] = make_uint2(0u, SE_ALL);
    }
    if (a.se_marks) {   // uniform
        if (n && nb == 0) apx_add(t0 - 1u, __dmul_rn(mid_square(in.x, in.y), (double)n));
        else if (nb && nb <= 32u) forecast_parts(in.x, in.y, cum, n, 0u, 1u);
        else if (nb) s_win[atomicAdd(&s_wide, 1u)] = make_uint4(in.x, in.y, cum, n);
        if (n && (cum + n) % s == 0u && (cum + n) / s <= last_t) win[(cum + n) / s] = make_uint2(in.x, in.x);
        if (blk == 0 && tid == 0) {
            win[0] = make_uint2(0xFFFFFFFFu, 0xFFFFFFFFu);
            win[a.L] = make_uint2(0u, 0u);
        }
    }
    __syncthreads();
    for (uint32_t i = 0; i < s_many; ++i)   // (zeros; a row of one value has every boundary here)
        key_parts(s_key[i].x, s_key[i].y, s_key[i].z, s_key[i].w, (uint32_t)tid, 256u);
    if (a.se_marks) {
        for (uint32_t i = 0; i < s_wide; ++i) forecast_parts(s_win[i].x, s_win[i].y, s_win[i].z, s_win[i].w, (uint32_t)tid, 256u);
        __syncthreads();
        if (s_apx[tid] > 0.0 && band0 + tid < (uint32_t)a.L) unsafeAtomicAdd(&a.se_apx[(size_t)row * a.L + band0 + tid], s_apx[tid]);
    }
}

// The key window {lowest, highest} that holds the segment the draw will most likely take, from the squares that k_se_scan added up: the
// levels within 2^-12 of the whole of where the drawn word falls in the running sum.  By one workgroup, which leaves it in *win.
// What the forecast misses costs a read of the row (k_se_mark).
constexpr int SE_PER = SE_LMAX / SE_THREADS;
// The squares are read before the workgroup's other tables (se_forecast_read); the caller synchronizes before it reads *win.
__device__ __forceinline__ void se_forecast_read(const StopkArgs& a, int row, double (&e)[SE_PER]) {
#pragma unroll
    for (int i = 0; i < SE_PER; ++i) {
        const int l = (int)threadIdx.x * SE_PER + i;
        e[i] = l < a.L ? a.se_apx[(size_t)row * a.L + l] : 0.0;
    }
}
__device__ __forceinline__ void se_forecast(const StopkArgs& a, int row, const double (&e)[SE_PER], double* s_w /* SE_WAVES */, int* s_t /* 2 */, uint2* win) {
    const int tid = threadIdx.x;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    double v[SE_PER], sum = 0.0;
#pragma unroll
    for (int i = 0; i < SE_PER; ++i) {
        v[i] = sqrt(e[i]);
        sum += v[i];
    }
    double inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double u = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += u;
    }
    if (lane == 63) s_w[wave] = inc;
    if (tid == 0) s_t[0] = s_t[1] = a.L;
    __syncthreads();
    double before = 0.0, total = 0.0;
#pragma unroll
    for (int w = 0; w < SE_WAVES; ++w) {
        if (w == (int)wave) before = total;
        total += s_w[w];
    }
    double run = before + inc - sum;
    const double at = ((double)philox_word0(a.seed, a.step, (uint32_t)row) + 0.5) * 0x1p-32 * total, eps = total * 0x1p-12;
    int t0 = a.L, t1 = a.L;   // first levels whose running sums pass at - eps and at + eps
#pragma unroll
    for (int i = SE_PER - 1; i >= 0; --i) {
        double upto = run;
#pragma unroll
        for (int k = 0; k <= i; ++k) upto += v[k];
        const int l = tid * SE_PER + i + 1;
        if (l <= a.L && upto > at - eps) t0 = l;
        if (l <= a.L && upto > at + eps) t1 = l;
    }
    if (t0 < a.L) atomicMin(&s_t[0], t0);
    if (t1 < a.L) atomicMin(&s_t[1], t1);
    __syncthreads();
    if (tid == 0) {   // (a sum that is no number leaves the last level)
        const uint2* w = a.se_win + (size_t)row * (a.L + 1);
        *win = make_uint2(w[s_t[1]].x, w[s_t[0] - 1].y);
    }
}

// Second read: sums of the regions, lists of the zones, marks of the segment that the draw will most likely take.
struct SplitLds {
    uint32_t map[SE_CB];                  // first: its places are offsets of the reads
    unsigned long long slot[SE_SLOTS];
    uint16_t cls[SE_BINS];
    double fw[SE_WAVES];
    int ft[2];
    uint2 win;
};
static_assert(sizeof(SplitLds) <= 163840, "a CU's LDS");
template <int DT, bool STREAM, bool MARK>
__global__ __launch_bounds__(SE_THREADS) void k_se_split(StopkArgs a) {
    __shared__ __align__(16) SplitLds s;
    // Workgroups are dealt to the eight XCDs in turn: those of an XCD take slices that follow one another, so that the pieces of a zone's list that
    // they write meet in one L2 (130 -> 127 us, 8 rows of 1.17e7 entries).
    const uint32_t id = blockIdx.y * gridDim.x + blockIdx.x, all = gridDim.x * gridDim.y, xcd = id & 7u;
    const uint32_t at = xcd * (all >> 3) + (xcd < (all & 7u) ? xcd : all & 7u) + (id >> 3);
    const int row = (int)(at / gridDim.x), slice = (int)(at % gridDim.x), tid = threadIdx.x;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    double apx[SE_PER];
    if (MARK) se_forecast_read(a, row, apx);
    for (int i = tid; i < SE_CB / 4; i += SE_THREADS) ((uint4*)s.map)[i] = ((const uint4*)(a.se_map + (size_t)row * SE_CB))[i];
    for (int i = tid; i < SE_BINS / 8; i += SE_THREADS) ((uint4*)s.cls)[i] = ((const uint4*)(a.se_class + (size_t)row * SE_BINS))[i];
    const int rs = a.se_rep;
    const uint32_t groups = ((uint32_t)a.L + 256u) << rs;
    for (uint32_t i = tid; i < groups; i += SE_THREADS) s.slot[i] = 0ull;
    {
        const int nz = (int)a.se_nz[SE_NZ * row];
        const uint32_t* part = a.se_part + ((size_t)row * a.se_wgs + slice) * SE_BINS;
        const SZone* zr = a.se_zone + (size_t)row * a.L;
        for (int z = tid; z < nz; z += SE_THREADS) s.slot[groups + z] = zr[z].off + part[zr[z].bin];
        // the counts that k_se_wide adds to start at zero
        const uint32_t nbig = a.se_nz[SE_NZ * row + 3];
        for (uint32_t b = 0; b < nbig; ++b) {
            uint32_t* tab = a.se_list2 + (size_t)row * a.d + zr[a.se_bigz[(size_t)row * a.se_bigs + b]].off;
            for (uint32_t i = slice * SE_THREADS + tid; i <= (uint32_t)SE_ZBIG; i += gridDim.x * SE_THREADS) tab[i] = 0;
        }
    }
    if (MARK) se_forecast(a, row, apx, s.fw, s.ft, &s.win);
    __syncthreads();
    RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    const int64_t i0 = (int64_t)slice * a.se_slice, i1 = i0 + a.se_slice < a.d ? i0 + a.se_slice : a.d;
    uint32_t* list = a.se_list + (size_t)row * a.d;
    const uint32_t rlane = (lane & ((1u << rs) - 1u)) * 8u, nobody = ((uint32_t)a.L + 255u) << rs;
    // MARK: a bit per four entries, the key of one of them is in the window.  (Where one band has all of a row's norm, the window may reach from key 0 to
    // 2^32 - 1 and takes in the entries past the row's end too: their marks load nothing.)
    uint32_t wlo = 0, wspan = 0;
    uint32_t* cand = nullptr;
    if (MARK) {
        wlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.win.x);
        wspan = (uint32_t)__builtin_amdgcn_readfirstlane((int)s.win.y) - wlo;
        cand = a.se_cand + ((size_t)row * a.se_cblks + (size_t)(i0 >> 10) + wave) * 8 + lane;
        if (slice == 0 && tid == 0) a.se_got[row] = s.win;
    }
    stream_slice<DT, SE_WAVES, STREAM>(ld, i0, i1, wave, lane, [&](const uint32_t (&k)[4][4], const int (&nv)[4]) {
        uint32_t cl[4][4], words = 0;
        unsigned long long was[4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) cl[q][c] = s.map[k[q][c] >> SE_CSHIFT];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) cl[q][c] = s.cls[se_bin(cl[q][c], k[q][c])];
        if (MARK) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t u[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) u[c] = c < nv[q] ? k[q][c] - wlo : 0xFFFFFFFFu;
                const uint32_t u01 = u[0] < u[1] ? u[0] : u[1], u23 = u[2] < u[3] ? u[2] : u[3];
                const uint64_t m = __ballot((u01 < u23 ? u01 : u23) <= wspan);
                words = write_lane((uint32_t)m, 2 * q, words);
                words = write_lane((uint32_t)(m >> 32), 2 * q + 1, words);
            }
        }
        // One addition per entry, to its group's sum or its zone's cursor: an atomic of its own for the few zone entries is a branch, and a wait for
        // the LDS, per entry of the lane (8 rows of 1.17e7 entries 127 us against 119; of the reads, the lookups and the marks alone 78).
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (c >= nv[q]) cl[q][c] = nobody;
                const bool zone = cl[q][c] >= groups;
                const uint32_t key = k[q][c], sig = (zone ? 1u : key >= 0x800000u ? key | 0x800000u : key) & 0xFFFFFFu;
                was[q][c] = atomicAdd((unsigned long long*)((char*)s.slot + (cl[q][c] << 3) + (zone ? 0u : rlane)), (unsigned long long)sig * sig);
            }
        // (both halves of every result are kept until all are there: a register that is free again has to be waited for before it is used)
        asm volatile("" ::"v"(was[0][0]), "v"(was[0][1]), "v"(was[0][2]), "v"(was[0][3]), "v"(was[1][0]), "v"(was[1][1]), "v"(was[1][2]), "v"(was[1][3]),
                     "v"(was[2][0]), "v"(was[2][1]), "v"(was[2][2]), "v"(was[2][3]), "v"(was[3][0]), "v"(was[3][1]), "v"(was[3][2]), "v"(was[3][3]));
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (cl[q][c] >= groups) list[(uint32_t)was[q][c]] = k[q][c];
        if (MARK) {
            if (lane < 8) *cand = words;
            cand += SE_WAVES * 8;
        }
    });
    __syncthreads();
    unsigned long long* gsum = a.se_gsum + (size_t)row * (a.L + 256) * 2;
    for (int g = tid; g < a.L + 255; g += SE_THREADS) {
        unsigned long long lo = 0, hi = 0;
        for (int r = 0; r < (1 << rs); ++r) {
            const unsigned long long v = s.slot[(g << rs) + r];
            lo += v & 0xFFFFFFFFull;
            hi += v >> 32;
        }
        if (lo) atomicAdd(&gsum[2 * g], lo);
        if (hi) atomicAdd(&gsum[2 * g + 1], hi);
    }
}

// One workgroup per zone of up to SE_ZCAP entries.  Keys of a zone differ in their low `shift` bits only; they are counted in 256 buckets of the zone's key range.
// One boundary, as most zones have: it lies in one bucket, whose few keys are ranked; every other key is on one side of it by its bucket.
// A wave ranks the keys of such a zone by itself if they are at most one per lane, as the zones of long
// ladders and of shorter rows are: 8 rows of 300001 entries at 3001 levels 24 us, by the workgroup 46, all in order 39.
// More of them, or a crowded bucket: the keys are put in order in LDS, a bucket by a thread by insertion (a few keys); where a bucket holds many,
// all keys by a bitonic sort, which takes three times as long.  Bound by the LDS latency of those steps: 8 rows of 1.17e7 entries, 1000 levels, all in order
// 37 us, one boundary without it 22 (of the 15 saved nearly all were insertions: reads and writes of LDS that wait for one another).
constexpr int SZ_THREADS = 256;
constexpr uint32_t SZ_FEW = 32;
// Sum over the lanes of squares of up to 48 bits, from 16-bit parts
__device__ __forceinline__ uint64_t wave_sum_squares(uint64_t sq) {
    uint64_t all = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) all += (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan((uint32_t)(sq >> (16 * i)) & 0xFFFFu), 63) << (16 * i);
    return all;
}
__global__ __launch_bounds__(SZ_THREADS) void k_se_zone(StopkArgs a) {
    __shared__ uint32_t s_k[SE_ZCAP];
    __shared__ uint32_t s_h[256];
    __shared__ uint32_t s_scan[SZ_THREADS / 64 + 1];
    __shared__ uint32_t s_crowd, s_fill;
    __shared__ uint32_t s_cut[3];                     // the bucket of the one boundary, keys before it, in it; then the boundary's key, keys above it, and with its equals
    __shared__ uint32_t s_sums[SZ_THREADS / 64][6];   // per wave: squares by 16 bits, above the key and of all
    const int row = blockIdx.y, tid = threadIdx.x;
    if ((int)blockIdx.x >= a.L - 1) {   // the last workgroups of a row: sums of the regions to their bands
        const int g = ((int)blockIdx.x - (a.L - 1)) * SZ_THREADS + tid;
        if (g < a.L + 255) {
            const unsigned long long* gs = a.se_gsum + ((size_t)row * (a.L + 256) + g) * 2;
            const unsigned long long lo = gs[0], hi = gs[1];
            if (lo | hi) {
                const uint32_t t = a.se_gtab[(size_t)row * (a.L + 256) + g];
                const int sh = se_exp_shift((t >> 16) << 23);
                unsigned long long* wide = a.se_big + ((size_t)row * a.L + (t & 0xFFFFu)) * SE_WORDS;
                se_add(wide, lo, sh);
                se_add(wide, hi, sh + 32);
            }
        }
        return;
    }
    if (blockIdx.x >= a.se_nz[SE_NZ * row]) return;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const SZone zn = a.se_zone[(size_t)row * a.L + blockIdx.x];
    const uint32_t n = zn.n;
    if (n > (uint32_t)SE_ZCAP) return;   // k_se_wide
    const uint32_t* src = a.se_list + (size_t)row * a.d + zn.off;
    const uint32_t s = (uint32_t)(a.s < a.d ? a.s : a.d);
    const int esh = se_exp_shift(zn.lo);
    // part u lies in band t0 + u (from 1)
    auto part_from = [&](uint32_t u) -> uint32_t { return u ? (zn.t0 + u - 1u) * s - zn.cum : 0u; };
    auto part_to = [&](uint32_t u) -> uint32_t { return u < zn.nb ? (zn.t0 + u) * s - zn.cum : n; };
    auto part_add = [&](uint32_t u, uint64_t lo, uint64_t hi) {
        unsigned long long* wide = a.se_big + ((size_t)row * a.L + (zn.t0 + u - 1u)) * SE_WORDS;
        se_add(wide, lo, esh);
        se_add(wide, hi, esh + 32);
    };
    if (zn.nb == 1u && n <= 64u) {   // uniform
        if (wave) return;
        const uint32_t x = lane < n ? src[lane] : 0u, r1 = part_from(1u);
        uint32_t above = 0, upto = 0;
        for (uint32_t i = 0; i < n; ++i) {
            const uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)x, (int)i);
            above += y > x;
            upto += y >= x;
        }
        const int at = __builtin_ctzll(__ballot(lane < n && above < r1 && r1 <= upto));   // one of the keys equal to that of rank r1 - 1
        const uint32_t tau = (uint32_t)__builtin_amdgcn_readlane((int)x, at), over = (uint32_t)__builtin_amdgcn_readlane((int)above, at), with = (uint32_t)__builtin_amdgcn_readlane((int)upto, at);
        const uint64_t sq = lane < n ? sig_square(x) : 0u;   // 64 squares: 54 bits
        const uint32_t q = r1 - over;                        // equal keys inside
        const uint64_t in0 = q * sig_square(tau) + wave_sum_squares(x > tau ? sq : 0u), all0 = wave_sum_squares(sq);
        if (lane < 2) part_add(lane, lane ? all0 - in0 : in0, 0u);
        if (lane == 0) a.se_thr[(size_t)row * (a.L + 1) + zn.t0] = make_uint2(tau, with == r1 ? SE_ALL : q);
        return;
    }
    {
        constexpr int PER = SE_ZCAP / SZ_THREADS;
        const uint32_t dsh = zn.shift > 8u ? zn.shift - 8u : 0u;
        auto digit = [&](uint32_t k) -> uint32_t { return 255u - ((k - zn.lo) >> dsh); };
        uint32_t my[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t at = (uint32_t)(tid + i * SZ_THREADS);
            my[i] = at < n ? src[at] : 0u;   // a zone holds no zeros
        }
        s_h[tid] = 0;
        if (tid == 0) s_crowd = s_fill = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (my[i]) atomicAdd(&s_h[digit(my[i])], 1u);
        __syncthreads();
        const uint32_t c = s_h[tid];
        uint32_t all;
        const uint32_t start = block_excl_scan<SZ_THREADS>(c, s_scan, all);
        s_h[tid] = start;
        if (c > SZ_FEW) s_crowd = 1u;
        const uint32_t r1 = part_from(1u);   // keys inside the first boundary, 1 .. n - 1
        if (start < r1 && r1 <= start + c) { s_cut[0] = (uint32_t)tid; s_cut[1] = start; s_cut[2] = c; }
        __syncthreads();
        if (zn.nb == 1u && s_cut[2] <= 64u) {   // uniform
            const uint32_t b = s_cut[0], before = s_cut[1], in = s_cut[2];
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (my[i] && digit(my[i]) == b) s_k[atomicAdd(&s_fill, 1u)] = my[i];
            __syncthreads();
            if (wave == 0) {   // the key of rank r1 - 1
                const uint32_t x = lane < in ? s_k[lane] : 0u;
                uint32_t above = 0, upto = 0;
                for (uint32_t i = 0; i < in; ++i) {
                    const uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)x, (int)i);
                    above += y > x;
                    upto += y >= x;
                }
                if (lane < in && before + above < r1 && r1 <= before + upto) { s_cut[0] = x; s_cut[1] = before + above; s_cut[2] = before + upto; }   // equal keys agree
            }
            __syncthreads();
            const uint32_t tau = s_cut[0];
            uint32_t v[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if ((uint32_t)(i * SZ_THREADS) < n && my[i]) {
                    const uint64_t sq = sig_square(my[i]);
                    const uint32_t p0 = (uint32_t)sq & 0xFFFFu, p1 = (uint32_t)(sq >> 16) & 0xFFFFu, p2 = (uint32_t)(sq >> 32);   // 2048 of them: 27 bits
                    const bool in0 = my[i] > tau;
                    v[0] += in0 ? p0 : 0u;
                    v[1] += in0 ? p1 : 0u;
                    v[2] += in0 ? p2 : 0u;
                    v[3] += p0;
                    v[4] += p1;
                    v[5] += p2;
                }
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                v[i] = wave_incl_scan(v[i]);
                if (lane == 63) s_sums[wave][i] = v[i];
            }
            __syncthreads();
            if (tid < 2) {   // a part each
                uint64_t t[6];
#pragma unroll
                for (int i = 0; i < 6; ++i) t[i] = (uint64_t)s_sums[0][i] + s_sums[1][i] + s_sums[2][i] + s_sums[3][i];
                const uint32_t q = r1 - s_cut[1];   // equal keys inside
                const uint64_t sq = sig_square(tau);
                const uint64_t in0 = q * sq + t[0] + (t[1] << 16) + (t[2] << 32);             // at most 2048 squares: 59 bits
                const uint64_t all0 = t[3] + (t[4] << 16) + (t[5] << 32);
                part_add((uint32_t)tid, tid ? all0 - in0 : in0, 0u);
                if (tid == 0) a.se_thr[(size_t)row * (a.L + 1) + zn.t0] = make_uint2(tau, s_cut[2] == r1 ? SE_ALL : q);
            }
            return;
        }
        if (s_crowd == 0u) {   // uniform
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (my[i]) s_k[atomicAdd(&s_h[digit(my[i])], 1u)] = my[i];
            __syncthreads();
            for (uint32_t i = 1; i < c; ++i) {
                const uint32_t x = s_k[start + i];
                uint32_t j = i;
                for (; j > 0 && s_k[start + j - 1u] < x; --j) s_k[start + j] = s_k[start + j - 1u];
                s_k[start + j] = x;
            }
            __syncthreads();
        } else {
            uint32_t np2 = 64, other = 0;
            while (np2 < n) np2 <<= 1;
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if ((uint32_t)(tid + i * SZ_THREADS) < np2) s_k[tid + i * SZ_THREADS] = my[i];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < PER; ++i) other |= my[i] ? my[i] ^ s_k[0] : 0u;
            if (__syncthreads_or((int)other) == 0) np2 = 1;   // one key: in order as it is
            for (uint32_t k = 2; k <= np2; k <<= 1) {
                for (uint32_t j = k >> 1; j > 0; j >>= 1) {
                    for (uint32_t p = tid; p < (np2 >> 1); p += SZ_THREADS) {
                        const uint32_t i = ((p & ~(j - 1u)) << 1) | (p & (j - 1u)), l = i | j;
                        const uint32_t x = s_k[i], y = s_k[l];
                        if ((x < y) == ((i & k) == 0u)) { s_k[i] = y; s_k[l] = x; }
                    }
                    __syncthreads();
                }
            }
        }
    }
    for (uint32_t u = tid; u < zn.nb; u += SZ_THREADS) {
        const uint32_t r = (zn.t0 + u) * s - zn.cum;   // 1 .. n - 1 keys of the zone are inside
        const uint32_t tau = s_k[r - 1u];
        uint32_t q = SE_ALL;
        if (s_k[r] == tau) {   // its equal keys are split: how many are inside
            uint32_t lo = 0, hi = r - 1u;   // first position with a key <= tau
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (s_k[mid] > tau) lo = mid + 1u;
                else hi = mid;
            }
            q = r - lo;
        }
        a.se_thr[(size_t)row * (a.L + 1) + zn.t0 + u] = make_uint2(tau, q);
    }
    if (s <= 128u) {   // many short parts: a thread each (a wave needs 1.5 us to add up its lanes, whatever the part's length)
        for (uint32_t u = tid; u <= zn.nb; u += SZ_THREADS) {
            uint64_t lo = 0, hi = 0;
            for (uint32_t i = part_from(u), e = part_to(u); i < e; ++i) {
                const uint64_t sq = sig_square(s_k[i]);
                lo += sq & 0xFFFFFFFFull;
                hi += sq >> 32;
            }
            part_add(u, lo, hi);
        }
        return;
    }
    for (uint32_t u = wave; u <= zn.nb; u += SZ_THREADS / 64) {
        uint64_t lo = 0, hi = 0;
        for (uint32_t i = part_from(u) + lane, e = part_to(u); i < e; i += 64) {
            const uint64_t sq = sig_square(s_k[i]);
            lo += sq & 0xFFFFFFFFull;
            hi += sq >> 32;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            lo += (uint64_t)__shfl_xor((unsigned long long)lo, o, 64);
            hi += (uint64_t)__shfl_xor((unsigned long long)hi, o, 64);
        }
        if (lane == 0) part_add(u, lo, hi);
    }
}

// Zones of more than SE_ZCAP entries.  Nothing is put in order: the counts of 2^SE_ZBITS sub-bins of the zone's key range give
// their ranks; a sub-bin without a boundary belongs to one band, one with boundaries is counted key by key (at most 16 keys).
// PHASE 0: a zone of up to SE_ZBIG entries is resolved by one workgroup, its key range cut to the keys that are there (repeated keys
// make nearly all such zones: one key or a few); of a larger one, a workgroup adds the sub-bins of a slice to the zone's.
// PHASE 1: the slices of the larger ones again; the last workgroup of a zone resolves it from the counts.  Bound by LDS atomics
// on the words that many entries share; 8 rows of 1.17e7 entries at 1000 levels, compress: of one value 1031 us (a sort of the
// rows 3804, one workgroup per zone 19678), of two neighbouring values 1069 (3610, 90185), 16 values 693 (3457, 4226).
template <int PHASE>
__global__ __launch_bounds__(SE_THREADS) void k_se_wide(StopkArgs a) {
    __shared__ uint32_t s_tab[SE_ZSUB];             // counts of the sub-bins, then of the keys of those with boundaries
    __shared__ uint16_t s_cls[SE_ZSUB];             // part of the zone that a sub-bin lies in, or 0x8000 | its number among those with boundaries
    __shared__ unsigned long long s_sum[SE_LMAX];   // squares of the parts, in lane-interleaved copies
    __shared__ uint32_t s_rcum[SE_LMAX];            // sub-bins with boundaries: entries of the zone above
    __shared__ uint16_t s_rsub[SE_LMAX];            // which one
    __shared__ uint32_t s_scan[SE_THREADS / 64 + 1];
    __shared__ uint32_t s_min, s_max;
    const int row = blockIdx.y;
    const uint32_t tid = threadIdx.x, lane = lane_id();
    const uint32_t nmid = PHASE == 0 ? a.se_nz[SE_NZ * row + 2] : 0u, nwork = nmid + a.se_nz[SE_NZ * row + 4];
    const uint32_t s = (uint32_t)(a.s < a.d ? a.s : a.d);
    uint2* thr = a.se_thr + (size_t)row * (a.L + 1);
    for (uint32_t it = blockIdx.x; it < nwork; it += gridDim.x) {   // everything down to the end of the loop is uniform unless it says tid or lane
        const bool mid = it < nmid;
        const uint2 item = mid ? make_uint2(a.se_mid[(size_t)row * a.se_mids + it], 0u) : a.se_item[(size_t)row * a.se_items + (it - nmid)];
        const SZone zn = a.se_zone[(size_t)row * a.L + item.x];
        const uint32_t n = zn.n;
        const uint32_t* src = a.se_list + (size_t)row * a.d + zn.off;
        uint32_t* tab = mid ? nullptr : a.se_list2 + (size_t)row * a.d + zn.off;
        uint32_t lo = zn.lo, bits = zn.shift;
        __syncthreads();   // the work before this has been read
        if (mid) {
            if (tid == 0) { s_min = 0xFFFFFFFFu; s_max = 0; }
            __syncthreads();
            uint32_t mx = 0, mn_inv = 0;
            batched_loop<8, SE_THREADS>(0u, n, tid, [&](uint32_t i) { return src[i]; }, [&](uint32_t, uint32_t k) {
                mx = k > mx ? k : mx;
                mn_inv = ~k > mn_inv ? ~k : mn_inv;
            });
            mx = wave_max(mx);
            mn_inv = wave_max(mn_inv);
            if (lane == 0) { atomicMax(&s_max, mx); atomicMin(&s_min, ~mn_inv); }
            __syncthreads();
            lo = s_min;
            bits = s_max > lo ? 32u - (uint32_t)__clz((int)(s_max - lo)) : 0u;
        }
        const uint32_t b1 = bits < (uint32_t)SE_ZBITS ? bits : (uint32_t)SE_ZBITS, rest = bits - b1, nsub = 1u << b1, vmask = (1u << rest) - 1u;
        auto sub_of = [&](uint32_t k) -> uint32_t { return nsub - 1u - ((k - lo) >> rest); };   // descending keys
        const uint32_t i0 = mid ? 0u : item.y * SE_ZSLICE, i1 = mid || n - i0 < SE_ZSLICE ? n : i0 + SE_ZSLICE;
        // counts of the sub-bins
        if (mid || PHASE == 0) {
            for (uint32_t i = tid; i < nsub; i += SE_THREADS) s_tab[i] = 0;
            __syncthreads();
            if (bits == 0) {
                if (tid == 0) s_tab[0] = i1 - i0;
            } else {
                batched_loop<8, SE_THREADS>(i0, i1, tid, [&](uint32_t i) { return src[i]; }, [&](uint32_t, uint32_t k) { se_count_peeled(s_tab, sub_of(k), true); });
            }
        } else {
            for (uint32_t i = tid; i < nsub; i += SE_THREADS) s_tab[i] = tab[i];
        }
        __syncthreads();
        if (PHASE == 0 && !mid) {
            for (uint32_t i = tid; i < nsub; i += SE_THREADS)
                if (s_tab[i]) atomicAdd(&tab[i], s_tab[i]);
            continue;
        }
        if (rest == 0 && item.y != 0u) continue;   // the counts are of single keys: one workgroup has all it needs
        // classes of the sub-bins; thresholds of boundaries between two of them
        const uint32_t per = nsub > SE_THREADS ? nsub / SE_THREADS : 1u, f0 = tid * per, f1 = f0 < nsub ? f0 + per : f0;
        uint32_t mine = 0, nrec, total, flags = 0;
        for (uint32_t i = f0; i < f1; ++i) mine += s_tab[i];
        const uint32_t first = block_excl_scan<SE_THREADS>(mine, s_scan, total);
        if (total != n && tid == 0) atomicOr(a.dev_status, MLMC_DEV_INTERNAL);
        uint32_t run = first;
        uint64_t plo = 0, phi = 0;
        uint32_t pband = 0xFFFFFFFFu;
        auto band_add = [&](uint32_t band, uint64_t l, uint64_t h) {   // band from 0
            unsigned long long* wide = a.se_big + ((size_t)row * a.L + band) * SE_WORDS;
            se_add(wide, l, se_exp_shift(zn.lo));
            se_add(wide, h, se_exp_shift(zn.lo) + 32);
        };
        for (uint32_t i = f0; i < f1; ++i) {
            const uint32_t c = s_tab[i];
            if (!c) continue;
            const uint32_t g0 = zn.cum + run, g1 = g0 + c, b0 = g0 / s, be = (g1 - 1u) / s;
            if (b0 == be) {
                s_cls[i] = (uint16_t)(b0 + 1u - zn.t0);
                if (rest == 0) {   // c equal keys
                    if (b0 != pband) {
                        if (pband != 0xFFFFFFFFu) band_add(pband, plo, phi);
                        pband = b0;
                        plo = 0;
                        phi = 0;
                    }
                    const uint64_t sq = sig_square(lo + (nsub - 1u - i));
                    plo += (sq & 0xFFFFFFFFull) * c;
                    phi += (sq >> 32) * c;
                }
            } else {
                flags |= 1u << (i - f0);
            }
            run += c;
            if (item.y == 0u && run < n && (be + 1u) * s == g1) thr[be + 1u] = make_uint2(lo + ((nsub - 1u - i) << rest), SE_ALL);
        }
        if (pband != 0xFFFFFFFFu) band_add(pband, plo, phi);
        uint32_t j = block_excl_scan<SE_THREADS>((uint32_t)__popc(flags), s_scan, nrec);
        run = first;
        for (uint32_t i = f0; i < f1; ++i) {
            if (flags >> (i - f0) & 1u) {
                s_cls[i] = (uint16_t)(0x8000u | j);
                s_rsub[j] = (uint16_t)i;
                s_rcum[j++] = run;
            }
            run += s_tab[i];
        }
        __syncthreads();
        const uint32_t room = SE_ZSUB >> rest;   // sub-bins whose keys' counts LDS holds at a time
        // thresholds of the boundaries inside sub-bins j0 .. j0 + room - 1, and the parts on both sides of them
        auto resolve = [&](uint32_t j0) {
            for (uint32_t u = tid; u < zn.nb; u += SE_THREADS) {
                const uint32_t r = (zn.t0 + u) * s - zn.cum;   // entries of the zone inside boundary t0 + u
                uint32_t x = 0, y = nrec;                      // records [0, x) lie above r entries or fewer
                while (x < y) {
                    const uint32_t m = (x + y) >> 1;
                    if (s_rcum[m] < r) x = m + 1u;
                    else y = m;
                }
                if (x == 0u || x - 1u < j0 || x - 1u >= j0 + room) continue;
                const uint32_t rec = x - 1u, sub = s_rsub[rec], rr = r - s_rcum[rec], key0 = lo + ((nsub - 1u - sub) << rest);
                const uint32_t* cnt = rest ? s_tab + ((rec - j0) << rest) : s_tab + sub;
                uint32_t acc = 0, tau = 0, q = 0;
                for (uint32_t v = vmask + 1u; v-- > 0u;) {
                    const uint32_t c = cnt[v];
                    if (acc < rr && acc + c >= rr) {
                        tau = key0 + v;
                        q = acc + c == rr ? SE_ALL : rr - acc;
                    }
                    acc += c;
                }
                if (rr >= acc) continue;   // this boundary lies behind the sub-bin, or at its end
                thr[zn.t0 + u] = make_uint2(tau, q);
                auto part = [&](uint32_t from, uint32_t to, uint32_t band) {   // entries from .. to - 1 of the sub-bin
                    uint64_t l = 0, h = 0;
                    uint32_t at = 0;
                    for (uint32_t v = vmask + 1u; v-- > 0u;) {
                        const uint32_t e = at + cnt[v], x0 = at > from ? at : from, x1 = e < to ? e : to;
                        if (x1 > x0) {
                            const uint64_t sq = sig_square(key0 + v);
                            l += (sq & 0xFFFFFFFFull) * (x1 - x0);
                            h += (sq >> 32) * (x1 - x0);
                        }
                        at = e;
                    }
                    band_add(band, l, h);
                };
                part(u > 0u && rr > s ? rr - s : 0u, rr, zn.t0 + u - 1u);
                if (u + 1u >= zn.nb || rr + s >= acc) part(rr, acc, zn.t0 + u);
            }
        };
        if (rest == 0) {
            resolve(0u);
            continue;
        }
        uint32_t rep = 0;   // log2 of the copies of a part's sum
        while (rep < 4u && ((zn.nb + 1u) << (rep + 1u)) <= (uint32_t)SE_LMAX) ++rep;
        const uint32_t rlane = lane & ((1u << rep) - 1u);
        for (uint32_t i = tid; i < (uint32_t)SE_LMAX; i += SE_THREADS) s_sum[i] = 0ull;
        for (uint32_t j0 = 0; j0 == 0u || j0 < nrec; j0 += room) {
            for (uint32_t i = tid; i < SE_ZSUB; i += SE_THREADS) s_tab[i] = 0;
            __syncthreads();
            for (uint32_t p0 = i0; p0 < i1; p0 += SE_ZSLICE) {
                batched_loop<8, SE_THREADS>(p0, i1 - p0 < SE_ZSLICE ? i1 : p0 + SE_ZSLICE, tid, [&](uint32_t i) { return src[i]; }, [&](uint32_t, uint32_t k) {
                    const uint32_t c = s_cls[sub_of(k)];
                    if (c & 0x8000u) {
                        const uint32_t at = (c & 0x7FFFu) - j0;
                        if (at < room) atomicAdd(&s_tab[(at << rest) + ((k - lo) & vmask)], 1u);
                    } else if (j0 == 0u) {
                        atomicAdd(&s_sum[(c << rep) | rlane], (unsigned long long)sig_square(k));
                    }
                });
                if (j0 == 0u) {
                    __syncthreads();
                    for (uint32_t u = tid; u <= zn.nb; u += SE_THREADS) {
                        uint64_t l = 0, h = 0;
                        for (uint32_t i = 0; i < (1u << rep); ++i) {
                            const unsigned long long v = s_sum[(u << rep) + i];
                            l += v & 0xFFFFFFFFull;
                            h += v >> 32;
                            s_sum[(u << rep) + i] = 0ull;
                        }
                        band_add(zn.t0 + u - 1u, l, h);
                    }
                }
                __syncthreads();
            }
            const uint32_t here = nrec - j0 < room ? nrec - j0 : room;
            if (PHASE == 0) {
                resolve(j0);
            } else {
                for (uint32_t i = tid; i < (here << rest); i += SE_THREADS)
                    if (s_tab[i]) atomicAdd(&tab[SE_ZSUB + (j0 << rest) + i], s_tab[i]);
            }
            __syncthreads();
        }
        if (PHASE == 0) continue;
        // the last workgroup of the zone has everybody's counts
        __threadfence();
        __syncthreads();
        if (tid == 0) s_max = atomicAdd(&tab[SE_ZBIG], 1u);
        __syncthreads();
        if (s_max + 1u != (n + SE_ZSLICE - 1u) / SE_ZSLICE) continue;
        __threadfence();
        for (uint32_t j0 = 0; j0 < nrec; j0 += room) {
            const uint32_t here = nrec - j0 < room ? nrec - j0 : room;
            for (uint32_t i = tid; i < (here << rest); i += SE_THREADS)
                s_tab[i] = __hip_atomic_load(&tab[SE_ZSUB + (j0 << rest) + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            resolve(j0);
            __syncthreads();
        }
    }
}

// Delta_l of every band: carries, one rounding to fp64, sqrt.
__global__ __launch_bounds__(64) void k_se_norms(StopkArgs a) {
    __shared__ uint32_t s_big[64][SE_WORDS + 1];
    const int row = blockIdx.y;
    const int band = (int)(blockIdx.x * 64 + threadIdx.x);
    if (band >= a.L) return;
    const unsigned long long* wide = a.se_big + ((size_t)row * a.L + band) * SE_WORDS;
    unsigned long long carry = 0, w[SE_WORDS];
#pragma unroll
    for (int i = 0; i < SE_WORDS; ++i) w[i] = wide[i];
#pragma unroll
    for (int i = 0; i < SE_WORDS; ++i) {
        const unsigned long long t = w[i] + carry;
        s_big[threadIdx.x][i] = (uint32_t)t;
        carry = t >> 32;
    }
    BigAcc acc;
    acc.w = s_big[threadIdx.x];
    const double nrm = __dsqrt_rn(acc.to_double());
    a.norms[(size_t)row * a.L + band] = nrm;
    if (a.norms_user) a.norms_user[(size_t)row * a.L + band] = nrm;
}

// The drawn segment between its two boundaries: hi (boundary l - 1, its inside excluded) and lo (boundary l).
struct SegTest {
    uint32_t tau_hi, tau_lo, q_hi, q_lo;
    bool cut_hi, cut_lo, same;   // equal keys split at a boundary; both boundaries at one key
    __device__ __forceinline__ SegTest(const SSeg& r) {
        tau_hi = r.hi.x; q_hi = r.hi.y; tau_lo = r.lo.x; q_lo = r.lo.y;
        same = tau_hi == tau_lo;
        cut_hi = r.level > 1 && q_hi != SE_ALL;
        cut_lo = q_lo != SE_ALL && !same;
    }
    // 0: outside, 1: member, 2: equal to tau_hi and decided by rank, 3: equal to tau_lo and decided by rank
    __device__ __forceinline__ int kind(uint32_t key) const {
        if (key < tau_hi) return key > tau_lo || (key == tau_lo && !cut_lo) ? 1 : (key == tau_lo ? 3 : 0);
        return key == tau_hi && cut_hi ? 2 : 0;
    }
    __device__ __forceinline__ bool in_hi(uint32_t rank) const { return rank >= q_hi && (!same || q_lo == SE_ALL || rank < q_lo); }
    __device__ __forceinline__ bool in_lo(uint32_t rank) const { return rank < q_lo; }
    // how many of the equal keys of ranks [t, t + n) are members
    __device__ __forceinline__ uint32_t count_hi(uint32_t t, uint32_t n) const {
        const uint32_t top = same && q_lo != SE_ALL && q_lo < t + n ? q_lo : t + n, bot = q_hi > t ? q_hi : t;
        return top > bot ? top - bot : 0u;
    }
    __device__ __forceinline__ uint32_t count_lo(uint32_t t, uint32_t n) const { return q_lo > t ? (q_lo - t < n ? q_lo - t : n) : 0u; }
};

// The drawn segment's entries: a wave takes a tile of 4096 entries; its bitmap (members, and entries that a rank decides) and its counts.
// Where the window that the second read marked holds the segment, only the marked entries are loaded, four at a time, unless they lie in so many
// of a tile's lines that all of it is read as quickly.
constexpr uint32_t SE_DENSE = 128;
template <int DT, bool STREAM>
__global__ __launch_bounds__(256) void k_se_mark(StopkArgs a) {
    __shared__ uint32_t s_bm[4][TILE / 32];
    const int row = blockIdx.y;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = (int64_t)blockIdx.x * 4 + wave;
    if (tile >= a.ntiles) return;
    uint32_t m = 0;   // 64 consecutive entries, a bit per four
    if (tile * (TILE / 1024) + (lane >> 4) < a.se_cblks) m = ((const uint16_t*)(a.se_cand + ((size_t)row * a.se_cblks + tile * (TILE / 1024)) * 8))[lane];
    const SSeg sr = a.sseg[row];
    const SegTest st(sr);
    RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    ((uint2*)s_bm[wave])[lane] = make_uint2(0u, 0u);
    wave_lds_sync();
    const int64_t j0 = tile * TILE;
    uint32_t n1 = 0, n2 = 0, n3 = 0;
    auto test = [&](const uint32_t (&b)[4], int group, int nv) {   // four consecutive entries
        int kd[4];
        int any = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            kd[c] = c < nv ? st.kind(key_of_bits(b[c])) : 0;
            any |= kd[c];
        }
        if (any) {
            uint32_t nib = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                nib |= (kd[c] ? 1u : 0u) << c;
                n1 += kd[c] == 1;
                n2 += kd[c] == 2;
                n3 += kd[c] == 3;
            }
            const uint32_t rel = (uint32_t)group * 4u;
            atomicOr(&s_bm[wave][rel >> 5], nib << (rel & 31u));
        }
    };
    if (sr.few && (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan((uint32_t)__popc(m)), 63) <= SE_DENSE) {   // uniform
        while (__ballot(m != 0)) {
            int g[2], nv[2];
            uint32_t b[2][4];
            const int have = __popc(m);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                g[u] = (int)lane * 16 + (u < have ? __builtin_ctz(m) : 0);
                m &= m - 1;
                nv[u] = u < have ? ld.load4(j0 + g[u] * 4, b[u]) : 0;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) test(b[u], g[u], nv[u]);
        }
    } else if (j0 + TILE <= a.d) {   // uniform
        for (int h = 0; h < 2; ++h) {
            uint32_t b[8][4];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (STREAM) ld.load4_stream(j0 + (h * 8 + q) * 256 + lane * 4, b[q]);
                else ld.load4_full(j0 + (h * 8 + q) * 256 + lane * 4, b[q]);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) test(b[q], (h * 8 + q) * 64 + (int)lane, 4);
        }
    } else {
        for (int q = 0; q < 16; ++q) {
            uint32_t b[4];
            const int nv = ld.load4(j0 + q * 256 + lane * 4, b);
            test(b, q * 64 + (int)lane, nv);
        }
    }
    wave_lds_sync();
    const int64_t w0 = tile * (TILE / 32) + lane * 2;
    uint32_t* bm = a.bitmap + (size_t)row * a.bm_words;
    if (w0 < a.bm_words) *(uint2*)(bm + w0) = ((const uint2*)s_bm[wave])[lane];   // bm_words is a multiple of 4
    const uint32_t n12 = wave_incl_scan(n1 | n2 << 16);   // (at most 4096 each)
    n3 = wave_incl_scan(n3);
    if (lane == 63) {
        const size_t at = (size_t)row * a.ntiles + tile;
        a.tile_cnt[at] = n12 & 0xFFFFu;
        a.se_tie[at] = make_uint2(n12 >> 16, n3);
    }
}

// Per row: entries before every tile, equal keys before every tile, where the row's message starts.
__global__ __launch_bounds__(1024) void k_se_offsets(StopkArgs a) {
    __shared__ uint32_t s_scan[1024 / 64 + 1];
    const int row = blockIdx.x, tid = threadIdx.x;
    const SegTest st(a.sseg[row]);
    uint32_t* to = a.tile_off + (size_t)row * (a.ntiles + 1);
    const uint32_t* tc = a.tile_cnt + (size_t)row * a.ntiles;
    uint2* tie = a.se_tie + (size_t)row * a.ntiles;
    uint32_t carry = 0, carry2 = 0, carry3 = 0;
    for (int64_t j0 = 0; j0 < a.ntiles; j0 += 1024) {
        const int64_t t = j0 + tid;
        uint32_t c = t < a.ntiles ? tc[t] : 0u, round_total;
        if (st.cut_hi || st.cut_lo) {   // uniform
            const uint2 n = t < a.ntiles ? tie[t] : make_uint2(0u, 0u);
            uint2 before;
            uint32_t all2, all3;
            before.x = carry2 + block_excl_scan<1024>(n.x, s_scan, all2);
            before.y = carry3 + block_excl_scan<1024>(n.y, s_scan, all3);
            carry2 += all2;
            carry3 += all3;
            if (t < a.ntiles) tie[t] = before;
            c += st.count_hi(before.x, n.x) + st.count_lo(before.y, n.y);
        }
        const uint32_t ex = block_excl_scan<1024>(c, s_scan, round_total);
        if (t < a.ntiles) to[t] = carry + ex;
        carry += round_total;
    }
    if (tid == 0) {
        to[a.ntiles] = carry;
        if ((int64_t)carry != a.srow[row].count) atomicOr(a.dev_status, MLMC_DEV_INTERNAL);
        int64_t start = 0;
        for (int r = 0; r < row; ++r) start += a.srow[r].count;
        a.row_off[row] = start;
        if (row == a.M - 1) {
            a.row_off[a.M] = start + carry;
            if (start + (int64_t)carry > a.capacity) atomicOr(a.dev_status, MLMC_DEV_CAPACITY);
        }
    }
}

// The message in index order where equal keys may be split: a wave takes a tile, a lane two words of its bitmap.
template <int DT>
__global__ __launch_bounds__(256) void k_se_write(StopkArgs a) {
    const int row = blockIdx.y;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = (int64_t)blockIdx.x * 4 + wave;
    if (tile >= a.ntiles) return;
    const uint32_t* to = a.tile_off + (size_t)row * (a.ntiles + 1);
    const uint32_t* bm = a.bitmap + (size_t)row * a.bm_words;
    const int64_t w0 = tile * (TILE / 32) + lane * 2;
    const uint2 m = w0 < a.bm_words ? *(const uint2*)(bm + w0) : make_uint2(0u, 0u);
    const SSeg sr = a.sseg[row];
    if (to[tile + 1] == to[tile]) return;   // nothing of the segment in this tile
    const SegTest st(sr);
    RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    const float w = sr.weight;
    uint64_t bits = (uint64_t)m.y << 32 | m.x;
    // f(position, fp32 bits, ordinal) for the lane's entries in order, the loads of eight of them in flight (a run of equal entries
    // fills whole lanes: one load at a time, 64 in a row)
    auto each = [&](uint64_t b, auto f) {
        for (uint32_t n = 0; b; n += 8) {
            int at[8];
            uint32_t v[8];
            const int have = __popcll(b);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                at[u] = u < have ? __builtin_ctzll(b) : at[0];
                b &= b - 1;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = ld.load1(w0 * 32 + at[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (u < have) f(at[u], v[u], n + u);
        }
    };
    if (st.cut_hi || st.cut_lo) {   // uniform: entries decided by rank are kept or cleared
        uint64_t m2 = 0, m3 = 0;
        each(bits, [&](int at, uint32_t v, uint32_t) {
            const int kd = st.kind(key_of_bits(v));
            m2 |= (uint64_t)(kd == 2) << at;
            m3 |= (uint64_t)(kd == 3) << at;
        });
        const uint32_t n2 = (uint32_t)__popcll(m2), n3 = (uint32_t)__popcll(m3);
        uint32_t i2 = n2, i3 = n3;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u2 = __shfl_up(i2, o, 64), u3 = __shfl_up(i3, o, 64);
            if (lane >= (uint32_t)o) { i2 += u2; i3 += u3; }
        }
        const uint2 before = a.se_tie[(size_t)row * a.ntiles + tile];
        uint32_t r2 = before.x + i2 - n2, r3 = before.y + i3 - n3;
        for (; m2; m2 &= m2 - 1)
            if (!st.in_hi(r2++)) bits &= ~(m2 & (0 - m2));
        for (; m3; m3 &= m3 - 1)
            if (!st.in_lo(r3++)) bits &= ~(m3 & (0 - m3));
    }
    const uint32_t mine = (uint32_t)__popcll(bits);
    uint32_t inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(inc, o, 64);
        if (lane >= (uint32_t)o) inc += u;
    }
    const int64_t first = a.row_off[row] + to[tile] + (inc - mine);
    each(bits, [&](int at, uint32_t v, uint32_t n) {
        if (first + n < a.capacity) {
            a.idx[first + n] = (uint32_t)(w0 * 32 + at);
            a.val[first + n] = __fmul_rn(__uint_as_float(v), w);
        }
    });
}

template <int DT>
static mlmc_status launch_bins(const mlmc_plan_t* pl, const StopkArgs& a, bool message, hipStream_t st) {
    const int M = pl->M;
    // The rows are read twice, and the message's entries once or twice more: what the last cache (256 MB) holds is best left there.  compress, us, plain reads /
    // past the cache, with a third read, s = d / 100: 1 row of 4e6 fp32 (16 MB) 118 / 125, 8 of 5e6 (160 MB) 197 / 209, 8 of 1.1e7 bf16 (176 MB) 258 / 267, 8 of 8388608 fp32 (268 MB) 268 / 276,
    // 8 of 9e6 (288 MB) 309 / 312 (s = d / 1000: 322 / 323), 8 of 1e7 (320 MB) 336 / 334, 8 of 2.3e7 bf16 (368 MB) 471 / 462, 8 of 11689512 fp32 (374 MB) 380 / 369.
    const bool stream = (int64_t)M * a.d * (DT == MLMC_F32 ? 4 : 2) > ((int64_t)288 << 20);
    {
        const size_t n16 = a.clear_bytes / 16;   // coarse histograms and band sums
        int blocks = (int)((n16 + 255) / 256);
        if (blocks > 2048) blocks = 2048;
        MLMC_LAUNCH(K_ZERO, st, k_sb_clear<<<blocks, 256, 0, st>>>((uint4*)a.se_coarse, n16, a.dev_status));
    }
    {
        const int64_t ns = ((a.d + 1023) / 1024 + (1 << a.se_shift) - 1) >> a.se_shift;
        int64_t gx = ns <= 512 ? (ns + 15) / 16 : (ns + 63) / 64, cap = 1024 / M > 0 ? 1024 / M : 1;
        if (gx > cap) gx = cap;
        MLMC_LAUNCH(K_HIST, st, k_se_coarse<DT><<<dim3((unsigned)gx, M), 512, 0, st>>>(a));
    }
    MLMC_LAUNCH(K_SCAN, st, k_se_map<DT><<<M, 1024, 0, st>>>(a));
    if (stream) MLMC_LAUNCH(K_SE_COUNT, st, k_se_count<DT, true><<<dim3(a.se_wgs, M), SE_THREADS, 0, st>>>(a));
    else MLMC_LAUNCH(K_SE_COUNT, st, k_se_count<DT, false><<<dim3(a.se_wgs, M), SE_THREADS, 0, st>>>(a));
    MLMC_LAUNCH(K_SE_SCAN, st, k_se_reduce<<<dim3(SE_BLOCKS, M), 256, 0, st>>>(a));
    MLMC_LAUNCH(K_SE_SCAN, st, k_se_scan<<<dim3(SE_BLOCKS, M), 256, 0, st>>>(a));
    const dim3 sgrid(a.se_wgs, M);
    if (stream && a.se_marks) MLMC_LAUNCH(K_SE_SPLIT, st, k_se_split<DT, true, true><<<sgrid, SE_THREADS, 0, st>>>(a));
    else if (a.se_marks) MLMC_LAUNCH(K_SE_SPLIT, st, k_se_split<DT, false, true><<<sgrid, SE_THREADS, 0, st>>>(a));
    else if (stream) MLMC_LAUNCH(K_SE_SPLIT, st, k_se_split<DT, true, false><<<sgrid, SE_THREADS, 0, st>>>(a));
    else MLMC_LAUNCH(K_SE_SPLIT, st, k_se_split<DT, false, false><<<sgrid, SE_THREADS, 0, st>>>(a));
    MLMC_LAUNCH(K_SE_ZONE, st, k_se_zone<<<dim3(a.L - 1 + (a.L + 255 + SZ_THREADS - 1) / SZ_THREADS, M), SZ_THREADS, 0, st>>>(a));
    {
        const int64_t cap = 512 / M > 0 ? 512 / M : 1;   // about two workgroups per CU: nearly always they find nothing to do
        const int64_t w0 = (int64_t)a.se_mids + a.se_items, g0 = w0 < cap ? w0 : cap, g1 = a.se_items < cap ? a.se_items : cap;
        MLMC_LAUNCH(K_SE_ZONE, st, k_se_wide<0><<<dim3((unsigned)g0, M), SE_THREADS, 0, st>>>(a));
        if (a.d > SE_ZBIG) MLMC_LAUNCH(K_SE_ZONE, st, k_se_wide<1><<<dim3((unsigned)g1, M), SE_THREADS, 0, st>>>(a));
    }
    MLMC_LAUNCH(K_SB_NORMS, st, k_se_norms<<<dim3((a.L + 63) / 64, M), 64, 0, st>>>(a));
    if (!message) return MLMC_OK;
    const dim3 tgrid((unsigned)((a.ntiles + 3) / 4), M);
    MLMC_LAUNCH(K_SB_DRAW, st, k_sb_draw<<<M, 1024, 0, st>>>(a));
    if (stream) MLMC_LAUNCH(K_SB_MARK, st, k_se_mark<DT, true><<<tgrid, 256, 0, st>>>(a));
    else MLMC_LAUNCH(K_SB_MARK, st, k_se_mark<DT, false><<<tgrid, 256, 0, st>>>(a));
    MLMC_LAUNCH(K_SB_OFFSETS, st, k_se_offsets<<<M, 1024, 0, st>>>(a));
    MLMC_LAUNCH(K_SB_WRITE, st, k_se_write<DT><<<tgrid, 256, 0, st>>>(a));
    return MLMC_OK;
}

mlmc_status stopk_run(const mlmc_plan_t* pl, const StopkArgs& a, bool message, hipStream_t st) {
    if (pl->off_se_end) {
        if (pl->dtype == MLMC_F32) return launch_bins<MLMC_F32>(pl, a, message, st);
        return launch_bins<MLMC_BF16>(pl, a, message, st);
    }
    if (pl->dtype == MLMC_F32) return launch_stopk<MLMC_F32>(pl, a, message, st);
    return launch_stopk<MLMC_BF16>(pl, a, message, st);
}

}  // namespace mlmc
