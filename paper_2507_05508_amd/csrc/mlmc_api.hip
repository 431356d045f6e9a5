// C ABI of libmlmc: plan construction / validation on the host and the entry points that enqueue the
// kernels (see include/mlmc.h for the contract of every call).
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "mlmc_internal.h"

namespace mlmc {
mlmc_status topk_zero(const mlmc_plan_t* pl, void* ws, int32_t* dev_status, hipStream_t st);
mlmc_status topk_select(const mlmc_plan_t* pl, const TopkArgs& a, bool sums, bool vec, hipStream_t st);
mlmc_status topk_compact(const mlmc_plan_t* pl, const TopkArgs& a, bool vec, hipStream_t st);
mlmc_status topk16_run(const mlmc_plan_t* pl, const TopkArgs& a, bool message, hipStream_t st);
mlmc_status row_topk_run(const mlmc_plan_t* pl, const TopkArgs& a, bool message, hipStream_t st);
mlmc_status bits_compress(const mlmc_plan_t* pl, const BitsArgs& a, hipStream_t st);
mlmc_status rtn_compress(const mlmc_plan_t* pl, const BitsArgs& a, bool message, hipStream_t st);
mlmc_status agg_bits(const mlmc_plan_t* pl, const BitsArgs& b, const int32_t* level, const int32_t* scale_exp,
                     const uint64_t* planes, float alpha, float* out, float eta, float* x, hipStream_t st);
mlmc_status agg_sparse(const mlmc_plan_t* pl, const int64_t* row_off, const uint32_t* idx, const float* val, int64_t capacity,
                       const uint32_t* tile_off, uint32_t* tile_off_ws, float alpha, float* out, float eta, float* x,
                       hipStream_t st);
mlmc_status message_bits(const mlmc_plan_t* pl, const int32_t* level, unsigned long long* bits, hipStream_t st);
mlmc_status stopk_run(const mlmc_plan_t* pl, const StopkArgs& a, bool message, hipStream_t st);

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---- static device scratch for mlmc_compress_bits_static --------------------------------------------
// Every GPU that loads the library holds its own copy of this array until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress: the device address is looked up once per device and
// kept; kernels, like those of mlmc_compress_bits, take the address as an argument.
static __device__ __align__(256) unsigned char scratch[MLMC_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static void* g_scratch_ptr[MAX_DEVICES];
static std::mutex g_scratch_mutex;

static mlmc_status static_scratch_of_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return MLMC_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return MLMC_EHIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return MLMC_OK;
}

// ---- per-kernel HIP-event timing (off by default; not thread safe) ---------------------------------
bool g_prof_on = false;
static const char* const k_names[K_NUM] = {
    "k_zero", "k_hist", "k_scan", "k_main", "k_fhist", "k_finish", "k_finish_rank", "redo_pass", "k_norms", "k_bits_prep", "k_msgplan", "k_filter" /* or k_pick */, "k_write",
    "k_bits_smax", "k_bits_extract", "k_bits_redo", "k_agg_bits", "k_tileoff", "k_agg_sparse", "k_message_bits", "k_rtn_norms", "k_rtn_draw",
    "k_rs_hist", "k_rs_scan", "k_rs_scatter", "k_sb_norms", "k_sb_draw", "k_sb_mark", "k_sb_offsets", "k_sb_write", "k_se_count", "k_se_scan",
    "k_se_split", "k_se_zone", "k_row_select", "k_row_write", "k_c16_hist", "k_c16_reduce", "k_c16_scan", "k_c16_mark", "k_c16_offsets", "k_c16_write",
    "k_bits_extract_words", "k_agg_words", "k_scan_marks"};
struct ProfPair { int id; hipEvent_t e0, e1; };
static std::vector<ProfPair> g_pending;
static std::vector<ProfPair> g_free;
static bool g_open = false;   // the last entry of g_pending still waits for its end event
static double g_total_ms[K_NUM];
static int64_t g_launches[K_NUM];

static void prof_drain() {
    for (ProfPair& p : g_pending) {
        float ms = 0.f;
        if (hipEventSynchronize(p.e1) == hipSuccess && hipEventElapsedTime(&ms, p.e0, p.e1) == hipSuccess) {
            g_total_ms[p.id] += ms;
            g_launches[p.id] += 1;
        }
        g_free.push_back(p);
    }
    g_pending.clear();
}

void prof_begin(int id, hipStream_t st) {
    if (g_pending.size() >= 8192) prof_drain();
    ProfPair p;
    g_open = false;
    if (!g_free.empty()) {
        p = g_free.back();
        g_free.pop_back();
    } else {
        if (hipEventCreate(&p.e0) != hipSuccess) return;
        if (hipEventCreate(&p.e1) != hipSuccess) { (void)hipEventDestroy(p.e0); return; }
    }
    p.id = id;
    (void)hipEventRecord(p.e0, st);
    g_pending.push_back(p);
    g_open = true;
}

// Closes the pair that the matching prof_begin opened; when that call could not create its events there is no
// open pair and nothing is recorded (an older pair of the same kernel is never touched).
void prof_end(int id, hipStream_t st) {
    if (!g_open || g_pending.empty() || g_pending.back().id != id) return;
    (void)hipEventRecord(g_pending.back().e1, st);
    g_open = false;
}

// 32-bit rows can be read with aligned 16-byte loads
static bool vec_ok(const void* g, int64_t ld) { return ((uintptr_t)g % 16 == 0) && (ld % 4 == 0); }

static void fill_topk_args(const mlmc_plan_t* pl, TopkArgs& a, const void* g, int64_t ld, void* ws, int32_t* dev_status) {
    std::memset(&a, 0, sizeof(a));
    char* w = (char*)ws;
    a.g = g;
    a.ld = ld;
    a.d = pl->d;
    a.M = pl->M;
    a.L = pl->L;
    for (int t = 0; t <= pl->L; ++t) a.k[t] = pl->ladder[t];
    a.chunk = pl->chunk;
    a.chunks_per_row = pl->chunks_per_row;
    a.cchunk = pl->cchunk;
    a.csub = pl->csub;
    a.cchunks_per_row = pl->cchunks_per_row;
    a.sample_shift = pl->sample_shift;
    // Short rows are bound by the number of launches (5 to 6 us each), so what a launch saves there is less than it costs: a
    // zone of an exact histogram is one bucket, a few hundred candidates that one workgroup ranks without the two sliced
    // passes.  compress, us, with the passes / alone: 4 rows of 4096, fixed p 50 / 47, adaptive 68 / 62; 4 of 100000 60 / 56, 86 / 80; 32 of 100000 78 / 71, 127 / 118.
    // Longer rows keep the sliced passes for zones with many equal keys: adaptive rows with six in ten zero, 1 of 100000 161 / 161, 1 of 131072 162 / 171,
    // 1 of 200000 190 / 218, 4 of 200000 227 / 241.
    a.alone = pl->sample_shift == 0 && pl->d <= ((int64_t)1 << 17) ? 1 : 0;
    a.staging = pl->staging;
    {
        int fx = FIN_WGS;
        if (pl->M < 16) fx = 512 / pl->M < FIN_WGS_MAX ? 512 / pl->M : FIN_WGS_MAX;   // about 512 workgroups in all
        fx = fx / FIN_WGS * FIN_WGS;                                                 // a multiple of FIN_WGS (32, 64, 96, 128)
        a.fin_wgs = fx;
        a.fin_slice = FIN_SLICE * FIN_WGS / fx;
        a.fin_slices = FIN_SLICES * fx / FIN_WGS;
    }
    a.ntiles = pl->ntiles;
    a.racc = (RowAcc*)(w + pl->off_racc);
    a.hist = (uint32_t*)(w + pl->off_hist);
    a.hist2 = (uint32_t*)(w + pl->off_hist2);
    a.rinfo = (RowInfo*)(w + pl->off_rinfo);
    a.table = (uint32_t*)(w + pl->off_table);
    a.table8 = (uint8_t*)(w + pl->off_table8);
    a.chunk_cnt = (uint32_t*)(w + pl->off_chunk_cnt);
    a.chunk_zcnt = (uint32_t*)(w + pl->off_chunk_zcnt);
    a.zhist = (uint32_t*)(w + pl->off_zhist);
    a.zpacc = (unsigned long long*)(w + pl->off_zpacc);
    a.zcol = (unsigned long long*)(w + pl->off_zcol);
    a.tile_off = (uint32_t*)(w + pl->off_tileoff);
    a.norms = (double*)(w + pl->off_norms);
    a.cand = (uint2*)(w + pl->off_cand);
    a.cand2 = (uint2*)(w + pl->off_cand2);
    a.cand_priv = (uint2*)(w + pl->off_cand_priv);
    if (pl->off_marks && pl->staging) {
        a.marks = (uint64_t*)(w + pl->off_marks);
        a.mark_words = (int64_t)pl->chunks_per_row * pl->chunk / 256;
    }
    a.priv_cnt = (uint32_t*)(w + pl->off_priv_cnt);
    a.chunk_base = (uint32_t*)(w + pl->off_chunk_base);
    a.row_order = (int32_t*)(w + pl->off_row_order);
    a.row_part = (uint4*)(w + pl->off_row_part);
    a.c16_part = (uint32_t*)(w + pl->off_c16_part);
    a.c16_occ = (uint32_t*)(w + pl->off_c16_occ);
    a.c16_wgs = pl->c16_wgs;
    a.c16_slice = pl->c16_slice;
    if (pl->off_c16_list) {
        a.c16_list = (uint32_t*)(w + pl->off_c16_list);
        if (pl->off_c16_mark) a.c16_mark = (uint64_t*)(w + pl->off_c16_mark);
        a.c16_cnt = (uint4*)(w + pl->off_c16_cnt);
        a.c16_pre = (uint4*)(w + pl->off_c16_pre);
    }
    a.dev_status = dev_status;
}

static void fill_bits_args(const mlmc_plan_t* pl, BitsArgs& b, const void* g, int64_t ld, void* ws, int32_t* dev_status) {
    std::memset(&b, 0, sizeof(b));
    char* w = (char*)ws;
    b.g = g;
    b.ld = ld;
    b.d = pl->d;
    b.M = pl->M;
    b.L = pl->L;
    for (int t = 0; t <= pl->L; ++t) b.F[t] = (int32_t)pl->ladder[t];
    for (int l = 0; l < pl->L; ++l) b.p_fixed[l] = pl->p[l];
    b.flt = pl->kind == MLMC_FBITS ? 1 : 0;
    b.vmx = pl->kind == MLMC_VBITS ? 1 : 0;
    b.rtn = pl->kind == MLMC_RTN ? 1 : 0;
    b.adaptive = pl->adaptive ? 1 : 0;
    if (pl->kind == MLMC_RTN && ws) {
        b.rtn_sums = (unsigned long long*)(w + pl->off_rtn_sums);
        b.norms = (double*)(w + pl->off_norms);
        if (pl->rtn_wgs) {
            b.rtn_part = (uint32_t*)(w + pl->off_rtn_part);
            b.rtn_total = (uint32_t*)(w + pl->off_rtn_total);
            b.rtn_slice = pl->rtn_slice;
        }
    }
    b.nplanes = pl->nplanes;
    b.nwords = (pl->d + 63) / 64;
    b.chunk = pl->chunk;
    b.sample_shift = pl->sample_shift;
    b.rinfo = ws ? (RowInfo*)(w + pl->off_rinfo) : nullptr;
    b.racc = ws ? (RowAcc*)(w + pl->off_racc) : nullptr;
    b.dev_status = dev_status;
}
}  // namespace mlmc

using namespace mlmc;

extern "C" {

const char* mlmc_status_string(int status) {
    switch (status) {
        case MLMC_OK: return "MLMC_OK";
        case MLMC_EINVAL: return "MLMC_EINVAL: invalid argument";
        case MLMC_ENOMEM: return "MLMC_ENOMEM: host allocation failed";
        case MLMC_EHIP: return "MLMC_EHIP: HIP launch failed";
        case MLMC_ELIMIT: return "MLMC_ELIMIT: the plan needs more scratch than the static array holds";
        default: return "unknown mlmc status";
    }
}

void mlmc_profile_enable(int on) {
    if (!on) prof_drain();
    g_prof_on = on != 0;
}

void mlmc_profile_reset(void) {
    prof_drain();
    for (int i = 0; i < K_NUM; ++i) { g_total_ms[i] = 0.0; g_launches[i] = 0; }
}

int mlmc_profile_num_kernels(void) { return K_NUM; }

const char* mlmc_profile_kernel_name(int id) { return id >= 0 && id < K_NUM ? k_names[id] : ""; }

mlmc_status mlmc_profile_get(int id, double* total_ms, int64_t* launches) {
    if (id < 0 || id >= K_NUM || !total_ms || !launches) return MLMC_EINVAL;
    prof_drain();
    *total_ms = g_total_ms[id];
    *launches = g_launches[id];
    return MLMC_OK;
}

mlmc_status mlmc_geometric_p(int L, double* p) {
    if (L < 1 || L > 1000 || !p) return MLMC_EINVAL;
    const double norm = 1.0 - std::ldexp(1.0, -L);
    for (int l = 1; l <= L; ++l) p[l - 1] = std::ldexp(1.0, -l) / norm;
    return MLMC_OK;
}

// s-segmented Top-k (Sec. 2.2, Sec. 3.2): uniform ladder k_l = min(s l, d), L = ceil(d / s) levels, adaptive p only.
static mlmc_status plan_stopk(mlmc_plan_t** plan, int M, int64_t d, int in_dtype, int L, int64_t s, const double* p_fixed,
                              size_t* workspace_bytes, int64_t* sparse_capacity_worst) {
    if (in_dtype != MLMC_F32 && in_dtype != MLMC_BF16) return MLMC_EINVAL;
    if (M < 1 || M > MLMC_MAX_WORKERS || d < 1 || d >= ((int64_t)1 << 31) || s < 1 || p_fixed) return MLMC_EINVAL;
    const int64_t Lw = (d + s - 1) / s;
    if (Lw > MLMC_MAX_SLEVELS || (int64_t)L != Lw) return MLMC_EINVAL;
    mlmc_plan_t* pl = new (std::nothrow) mlmc_plan_t;
    if (!pl) return MLMC_ENOMEM;
    std::memset(pl, 0, sizeof(*pl));
    pl->kind = MLMC_STOPK;
    pl->M = M;
    pl->dtype = in_dtype;
    pl->L = L;
    pl->d = d;
    pl->s = s;
    pl->adaptive = true;
    pl->ntiles = (d + TILE - 1) / TILE;
    pl->nblk = (int)((d + 4096 - 1) / 4096);   // sort blocks: RS_TILE elements
    pl->bm_words = ((d + 31) / 32 + 3) / 4 * 4;   // whole 16-byte groups per row
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off = align_up(off + bytes, 256); return at; };
    // More levels: a boundary in every few bins, most entries would be zone entries.  Short rows: the tables of a row (0.8 MB) are not
    // worth it, a sort of a few blocks is a handful of short launches (at 16384 entries the bins are 20 us ahead).
    // 16-bit rows are sorted in two passes: with few of them the sort is the faster one up to some 2^22 entries in all (1 row of 1e6: 94 us
    // against 110, 4 of 524289: 112 against 112, or 129 against 152 where nine in ten are zero; 8 of 8192: 106 against 102).
    const bool bins = L <= SE_LMAX && d >= 8192 && (in_dtype == MLMC_F32 || M >= 8 || (int64_t)M * d >= ((int64_t)1 << 22));
    if (bins) {
        // The forecast of the drawn segment and the marks cost some 4 to 9 us (a sum and a window per bin, the draw in front of the second read) and spare most of the third read,
        // which comes from the last cache in smaller plans; segments of a thirtieth of a row or more have an entry in most of its lines.  Pass, us, without / with them, one scale
        // and many: 100 levels 8 of 16384 75 / 77 and 74 / 82, 8 of 300001 101 / 103 and 100 / 106, 8 of 1000001 119 / 120 and 120 / 123, 4 of 3000001 122 / 121 and 124 / 125, 1 of
        // 16000001 154 / 153 and 154 / 153, 8 of 4000001 176 / 165 and 176 / 172, 8 of 11689512 368 / 330 and 361 / 325; 1000 levels 8 of 300001 128 / 131 and 119 / 125, 2 of 4000001
        // 139 / 137 and 131 / 131, 8 of 4000001 204 / 193 and 195 / 188; 30 levels 8 of 4000001 176 / 180 and 190 / 187, 32 of 2000001 302 / 304 and 323 / 306; 10 levels 32 of 1000001
        // 227 / 235 and 270 / 271.  16 bits, 100 levels: 32 of 300001 111 / 110 and 115 / 120, 4 of 4000001 115 / 112 and 117 / 120, 8 of 4000001 148 / 142 and 149 / 147.
        pl->se_marks = L >= 32 && (int64_t)M * d >= ((int64_t)1 << 24) ? 1 : 0;
        pl->se_rep = L <= 1024 ? 2 : (L <= 2304 ? 1 : 0);   // (L + 256) << se_rep sums fill 40 KB of LDS
        // At least 2^19 entries of a row are sampled for the map.  Half as many as with 2^20 cost nothing where the map was the same and save their reads
        // (32 rows of 2e6 entries 296 -> 277 us, 16 of 4e6 in 16 bits 230 -> 224; 8 of 1.17e7 320 both).
        while (pl->se_shift < 4 && (d >> (pl->se_shift + 1)) >= (1 << 19)) ++pl->se_shift;
        // One workgroup per CU in one round.  A group's 64-bit sum has room for 2^16 squares: a band has at most s entries, a
        // copy gets its even share of the slice, so one of the two has to be that small.
        int64_t wgs = 256 / M > 0 ? 256 / M : 1;
        if (wgs > (d + 8191) / 8192) wgs = (d + 8191) / 8192;
        if (s > 65536) {
            const int64_t least = (d + (65536ll << pl->se_rep) - 1) / (65536ll << pl->se_rep);
            if (wgs < least) {
                const int64_t rounds = (least * M + 255) / 256;
                wgs = rounds * 256 / M > least ? rounds * 256 / M : least;
            }
        }
        pl->se_slice = ((d + wgs - 1) / wgs + 1023) / 1024 * 1024;
        if (s > 65536 && pl->se_slice > (65536ll << pl->se_rep)) pl->se_slice = 65536ll << pl->se_rep;
        pl->se_wgs = (int)((d + pl->se_slice - 1) / pl->se_slice);
        pl->off_se_coarse = take(sizeof(uint32_t) * 8192 * (size_t)M);
        pl->off_se_big = take(sizeof(uint64_t) * SE_WORDS * (size_t)L * M);
        pl->off_se_gsum = take(sizeof(uint64_t) * 2 * (size_t)(L + 256) * M);
        pl->off_se_nz = take(sizeof(uint32_t) * SE_NZ * (size_t)M);
        pl->off_se_apx = take(sizeof(double) * (size_t)L * M);
        pl->off_se_end = off;
        pl->off_se_bsum = take(sizeof(uint32_t) * ((SE_BINS + 255) / 256) * (size_t)M);
        pl->off_se_map = take(sizeof(uint32_t) * 8192 * (size_t)M);
        pl->off_se_info = take(sizeof(uint2) * SE_BINS * (size_t)M);
        pl->off_se_nbins = take(sizeof(uint32_t) * (size_t)M);
        pl->off_se_part = take(sizeof(uint32_t) * SE_BINS * (size_t)pl->se_wgs * M);
        pl->off_se_total = take(sizeof(uint32_t) * SE_BINS * (size_t)M);
        pl->off_se_class = take(sizeof(uint16_t) * SE_BINS * (size_t)M);
        pl->off_se_gtab = take(sizeof(uint32_t) * (size_t)(L + 256) * M);
        pl->off_se_thr = take(sizeof(uint2) * (size_t)(L + 1) * M);
        pl->off_se_zone = take(sizeof(SZone) * (size_t)L * M);
        // zones of more than 2048 entries; of more than SE_ZBIG; slices of 65536 entries of the latter
        pl->se_mids = (int)(d / 2049 + 1);
        pl->se_bigs = (int)(d / (SE_ZBIG + 1) + 1);
        pl->se_items = (int)(d / 32768 + 1);
        pl->off_se_mid = take(sizeof(uint32_t) * (size_t)pl->se_mids * M);
        pl->off_se_bigz = take(sizeof(uint32_t) * (size_t)pl->se_bigs * M);
        pl->off_se_item = take(sizeof(uint2) * (size_t)pl->se_items * M);
        pl->off_se_list = take(sizeof(uint32_t) * (size_t)d * M);
        if (d > SE_ZBIG) pl->off_se_list2 = take(sizeof(uint32_t) * (size_t)d * M);
        pl->off_se_tie = take(sizeof(uint2) * (size_t)pl->ntiles * M);
        pl->off_se_win = take(sizeof(uint2) * (size_t)(L + 1) * M);
        pl->off_se_got = take(sizeof(uint2) * (size_t)M);
        pl->off_se_cand = take(sizeof(uint32_t) * 8 * (size_t)((d + 1023) / 1024) * M);
    }
    pl->off_bitmap = off;
    off = align_up(off + sizeof(uint32_t) * (size_t)pl->bm_words * M + 16, 256);
    pl->off_tilecnt = off;
    off = align_up(off + sizeof(uint32_t) * (size_t)pl->ntiles * M, 256);
    pl->off_clear_end = off;
    pl->off_srow = off;
    off = align_up(off + sizeof(SRow) * (size_t)M, 256);
    if (bins) pl->off_sseg = take(sizeof(SSeg) * (size_t)M);
    pl->off_tileoff = off;
    off = align_up(off + sizeof(uint32_t) * (size_t)(pl->ntiles + 1) * M, 256);
    pl->off_norms = off;
    off = align_up(off + sizeof(double) * (size_t)L * M, 256);
    if (!bins) {
        pl->off_counts = take(sizeof(uint32_t) * 256 * (size_t)pl->nblk * M);
        pl->off_bintot = take(sizeof(uint32_t) * 256 * (size_t)M);
        pl->off_pa = take(sizeof(uint2) * (size_t)d * M);
        pl->off_pb = take(sizeof(uint2) * (size_t)d * M);
    }
    pl->ws_bytes = off;
    if (workspace_bytes) *workspace_bytes = off;
    if (sparse_capacity_worst) *sparse_capacity_worst = (int64_t)M * (s < d ? s : d);
    *plan = pl;
    return MLMC_OK;
}

static void fill_stopk_args(const mlmc_plan_t* pl, StopkArgs& a, const void* g, int64_t ld, void* ws, int32_t* dev_status) {
    std::memset(&a, 0, sizeof(a));
    char* w = (char*)ws;
    a.g = g;
    a.ld = ld;
    a.d = pl->d;
    a.M = pl->M;
    a.L = pl->L;
    a.s = pl->s;
    a.nblk = pl->nblk;
    a.ntiles = pl->ntiles;
    a.bm_words = pl->bm_words;
    a.pa = (uint2*)(w + pl->off_pa);
    a.pb = (uint2*)(w + pl->off_pb);
    a.counts = (uint32_t*)(w + pl->off_counts);
    a.bin_total = (uint32_t*)(w + pl->off_bintot);
    a.bitmap = (uint32_t*)(w + pl->off_bitmap);
    a.tile_cnt = (uint32_t*)(w + pl->off_tilecnt);
    a.clear_bytes = pl->off_clear_end - pl->off_bitmap;
    if (pl->off_se_end) {
        a.clear_bytes = pl->off_se_end - pl->off_se_coarse;
        a.bf16 = pl->dtype == MLMC_BF16 ? 1 : 0;
        a.se_shift = pl->se_shift;
        a.se_wgs = pl->se_wgs;
        a.se_rep = pl->se_rep;
        a.se_slice = pl->se_slice;
        a.se_coarse = (uint32_t*)(w + pl->off_se_coarse);
        a.se_big = (unsigned long long*)(w + pl->off_se_big);
        a.se_map = (uint32_t*)(w + pl->off_se_map);
        a.se_info = (uint2*)(w + pl->off_se_info);
        a.se_nbins = (uint32_t*)(w + pl->off_se_nbins);
        a.se_part = (uint32_t*)(w + pl->off_se_part);
        a.se_total = (uint32_t*)(w + pl->off_se_total);
        a.se_class = (uint16_t*)(w + pl->off_se_class);
        a.se_gtab = (uint32_t*)(w + pl->off_se_gtab);
        a.se_thr = (uint2*)(w + pl->off_se_thr);
        a.se_zone = (SZone*)(w + pl->off_se_zone);
        a.se_bsum = (uint32_t*)(w + pl->off_se_bsum);
        a.se_gsum = (unsigned long long*)(w + pl->off_se_gsum);
        a.se_nz = (uint32_t*)(w + pl->off_se_nz);
        a.se_mid = (uint32_t*)(w + pl->off_se_mid);
        a.se_bigz = (uint32_t*)(w + pl->off_se_bigz);
        a.se_item = (uint2*)(w + pl->off_se_item);
        a.se_mids = pl->se_mids;
        a.se_bigs = pl->se_bigs;
        a.se_items = pl->se_items;
        a.se_list = (uint32_t*)(w + pl->off_se_list);
        a.se_list2 = (uint32_t*)(w + pl->off_se_list2);
        a.se_tie = (uint2*)(w + pl->off_se_tie);
        a.se_apx = (double*)(w + pl->off_se_apx);
        a.se_win = (uint2*)(w + pl->off_se_win);
        a.se_got = (uint2*)(w + pl->off_se_got);
        a.se_cand = (uint32_t*)(w + pl->off_se_cand);
        a.se_cblks = (pl->d + 1023) / 1024;
        a.se_marks = pl->se_marks;
    }
    a.tile_off = (uint32_t*)(w + pl->off_tileoff);
    a.norms = (double*)(w + pl->off_norms);
    a.srow = (SRow*)(w + pl->off_srow);
    a.sseg = (SSeg*)(w + pl->off_sseg);
    a.dev_status = dev_status;
}

mlmc_status mlmc_plan(mlmc_plan_t** plan, int kind, int M, int64_t d, int in_dtype, int L, const int64_t* ladder,
                      const double* p_fixed, size_t* workspace_bytes, int64_t* sparse_capacity_worst) {
    if (plan) *plan = nullptr;
    if (!plan || !ladder) return MLMC_EINVAL;
    if (kind == MLMC_STOPK) return plan_stopk(plan, M, d, in_dtype, L, ladder[0], p_fixed, workspace_bytes, sparse_capacity_worst);
    if (kind != MLMC_TOPK && kind != MLMC_BITS && kind != MLMC_FBITS && kind != MLMC_VBITS && kind != MLMC_RTN) return MLMC_EINVAL;
    if (in_dtype != MLMC_F32 && in_dtype != MLMC_BF16) return MLMC_EINVAL;
    if (M < 1 || M > MLMC_MAX_WORKERS || d < 1 || d >= ((int64_t)1 << 31) || L < 1 || L > MLMC_MAX_LEVELS) return MLMC_EINVAL;
    if (ladder[0] < 0) return MLMC_EINVAL;
    for (int t = 0; t < L; ++t)
        if (ladder[t] >= ladder[t + 1]) return MLMC_EINVAL;
    if (kind == MLMC_TOPK && ladder[L] > d) return MLMC_EINVAL;
    if ((kind == MLMC_BITS || kind == MLMC_VBITS) && ladder[L] > 24) return MLMC_EINVAL;
    if (kind == MLMC_FBITS && ladder[L] > 23) return MLMC_EINVAL;
    if (kind == MLMC_RTN && (ladder[L] > 16 || L > MLMC_MAX_RTN_LEVELS)) return MLMC_EINVAL;
    if (kind != MLMC_TOPK && kind != MLMC_RTN && !p_fixed) return MLMC_EINVAL;  // Lemma 3.4 probabilities: rank bands and the Round-to-Nearest ladder
    if (p_fixed) {
        double s = 0.0;
        for (int l = 0; l < L; ++l) {
            if (!(p_fixed[l] > 0.0) || !(p_fixed[l] <= 1.0)) return MLMC_EINVAL;
            s += p_fixed[l];
        }
        if (std::fabs(s - 1.0) > 1e-9) return MLMC_EINVAL;
    }
    mlmc_plan_t* pl = new (std::nothrow) mlmc_plan_t;
    if (!pl) return MLMC_ENOMEM;
    std::memset(pl, 0, sizeof(*pl));
    pl->kind = kind;
    pl->M = M;
    pl->dtype = in_dtype;
    pl->L = L;
    pl->d = d;
    for (int t = 0; t <= L; ++t) pl->ladder[t] = ladder[t];
    pl->adaptive = p_fixed == nullptr;
    if (p_fixed)
        for (int l = 0; l < L; ++l) pl->p[l] = p_fixed[l];
    pl->ntiles = (d + TILE - 1) / TILE;
    pl->nplanes = 0;
    if (kind != MLMC_TOPK) {
        int maxw = 0;
        for (int l = 1; l <= L; ++l) {
            int w = (int)(ladder[l] - ladder[l - 1]);
            if (w > maxw) maxw = w;
        }
        pl->nplanes = (kind == MLMC_FBITS ? 9 : 1) + (int)ladder[0] + maxw;
        if (kind == MLMC_RTN) {   // the codes of the base, the previous and the drawn level
            int most = 0;
            for (int l = 1; l <= L; ++l) {
                const int n = (int)ladder[0] + (l > 1 ? (int)ladder[l - 1] : 0) + (int)ladder[l];
                if (n > most) most = n;
            }
            if (most > MAX_FPLANES) { delete pl; return MLMC_EINVAL; }
            pl->nplanes = most;
        }
    }
    // chunking of the streaming kernels: about 2048 workgroups over all rows, but chunks of at least some 96 K
    // elements (a workgroup of the selection read loads a table first), whole tiles, at most 2^18 elements
    // per workgroup (the LDS accumulators and the packed candidate offsets rely on that bound).  Rows that would leave CUs without a chunk are cut finer, down to
    // 32 K elements, but not into more than about 64 chunks each: 1 row of 8000001 in 123 chunks 23.0 / 11.4 and 27.4 / 9.1 (the search below goes a quarter further at most,
    // 1 row of 4000000 in 82).
    // Selection read / message from the staged lists, us, chunks of 96 K and this way: 8 rows of 1000001, adaptive 22.8 / 24.0 and 18.2 / 14.4, fixed p 14.3 / 10.2 and
    // 12.4 / 8.1; 8 of 300001 17.7 / 20.3 and 11.6 / 11.4; 4 of 4000001 30.4 / 29.4 and 31.4 / 22.8 (with chunks of 32 K 39.2 / 15.1).
    // Nor finer than the counters of a ranking workgroup reach when all thresholds lie in one zone, as in rows of few values: a zone whose counters do not fit is ranked by one
    // workgroup that reads its list again for the counts (1 row of one value, 32 levels inside it, compress, ms, 96 K / without this bound / with it: 2000001 entries
    // 38 / 55 / 39, 4000000 79 / 111 / 79).  Where they fit, they are in fewer copies than with 96 K: 2000001
    // entries of one value, 16 levels, 25.5 / 26.3 ms (normal ones 0.115 / 0.096).
    const int64_t most_chunks = ZC_CAP / (CSUB_MAX * (L + 2));
    int64_t least_chunk = (int64_t)M * d / 256;
    if (least_chunk < d / 64) least_chunk = d / 64;
    if (least_chunk < (d + most_chunks - 1) / most_chunks) least_chunk = (d + most_chunks - 1) / most_chunks;
    if (least_chunk < 8 * TILE) least_chunk = 8 * TILE;
    if (least_chunk > 98304) least_chunk = 98304;
    int64_t target_per_row = 2048 / M > 0 ? 2048 / M : 1;
    int64_t by_size = (d + least_chunk - 1) / least_chunk;
    if (by_size < 4) by_size = 4;   // a short row still spreads over a few CUs
    if (target_per_row > by_size) target_per_row = by_size;
    int64_t chunk = (d + target_per_row - 1) / target_per_row;
    chunk = (chunk + 4 * TILE - 1) / (4 * TILE) * (4 * TILE);
    if (chunk < 4 * TILE) chunk = 4 * TILE;
    if (chunk > CHUNK_MAX) chunk = CHUNK_MAX;
    // A workgroup of the selection read holds a whole CU, so its M * chunks workgroups run in rounds of one per
    // CU: among the chunk sizes within a quarter of the one above, take the one whose last round is the fullest
    // (rounds x chunk = the elements a CU streams through).
    {
        constexpr int64_t NUM_CUS = 256;   // MI355X
        int64_t best = chunk, best_cost = -1;
        for (int64_t c = chunk - chunk / 4; c <= chunk + chunk / 4; c += 4 * TILE) {
            const int64_t cc = (c + 4 * TILE - 1) / (4 * TILE) * (4 * TILE);
            if (cc < 4 * TILE || cc > CHUNK_MAX) continue;
            const int64_t n = (d + cc - 1) / cc;
            if (n > (least_chunk < 98304 ? most_chunks : CHUNKS_MAX / CSUB_MAX)) continue;
            const int64_t rounds = ((int64_t)M * n + NUM_CUS - 1) / NUM_CUS;
            const int64_t cost = rounds * (cc + 16384);   // + a workgroup's fixed part (table load, flush), in elements
            if (best_cost < 0 || cost < best_cost || (cost == best_cost && cc == chunk)) { best = cc; best_cost = cost; }
        }
        chunk = best;
    }
    pl->chunk = (int)chunk;
    pl->chunks_per_row = (int)((d + chunk - 1) / chunk);   // <= 2^31 / 2^18 = CHUNKS_MAX
    // message offsets are kept per count chunk, a quarter of a chunk (unless that would be too many per row):
    // the second read of a row, when one is needed, then has four times as many workgroups
    pl->csub = (pl->chunks_per_row * CSUB_MAX <= CHUNKS_MAX && chunk >= 8 * TILE) ? CSUB_MAX : 1;
    pl->cchunk = (int)(chunk / pl->csub);
    pl->cchunks_per_row = (int)((d + pl->cchunk - 1) / pl->cchunk);
    // rows long enough that a second full read matters get their thresholds from a sampled histogram
    pl->sample_shift = d >= ((int64_t)1 << 23) ? 4 : d >= ((int64_t)1 << 21) ? 2 : 0;
    if (kind == MLMC_VBITS || kind == MLMC_RTN) pl->sample_shift = 0;   // the largest entry itself is needed, not its binade
    // Small adaptive plans of several rows take the second read instead of the kernel that assembles staged lists (fp32 rows of 8192 to 65536 entries and
    // 16-bit rows have neither).  compress, us, second read / staged: 16 of 4096 65 / 69 (78 / 84 where keys repeat), 64 of 8000 108 / 115, 4 of 100000 80 / 79 (129 / 141).
    // One or two rows leave the second read too few workgroups (1 of 100000 78 / 76, 125 / 119; 2 of 200000 91 / 87, 176 / 180), and with fixed p it loses
    // where keys repeat (4 of 100000 59 / 56, 96 / 81).
    pl->staging = p_fixed == nullptr && M >= 4 && (int64_t)M * d <= ((int64_t)1 << 19) ? 0 : 1;
    // The fork and the join cost some twenty microseconds of stream operations, paid in every call, while the second read
    // has work in a call only when some row's band was not staged: worth it for many long rows (measured: -11 us per call
    // at 16 rows of 2.6e7 elements, +5 us at 4 rows of 1.2e8).
    pl->side_enable = M >= 8 && (int64_t)M * d >= ((int64_t)1 << 28) ? 1 : 0;

    size_t off = 0;
    pl->off_racc = off;
    off = align_up(off + sizeof(RowAcc) * (size_t)M, 256);
    // 16-bit rows have few enough magnitudes to count them all, at any size: compress, adaptive, us, against the way of the 32-bit rows, 4 rows of 1000
    // 68 -> 31, 1 of 16384 74 -> 33, 129 of 65536 210 -> 72, 255 of 300001 513 -> 173, 1024 of 32768 1032 -> 213; nine in ten zero, 129 of 65536, 790 -> 70.
    const bool counted = kind == MLMC_TOPK && in_dtype == MLMC_BF16;
    if (kind == MLMC_TOPK && !counted) {
        pl->off_hist = off;
        off = align_up(off + sizeof(uint32_t) * NB1 * (size_t)M, 256);
        pl->off_hist2 = off;
        off = align_up(off + sizeof(uint32_t) * NB1 * (size_t)M, 256);
        pl->off_chunk_zcnt = off;
        off = align_up(off + sizeof(uint32_t) * ZPMAX * (size_t)pl->cchunks_per_row * M, 256);
        pl->off_zhist = off;
        off = align_up(off + sizeof(uint32_t) * FH_BINS * ZMAX * (size_t)M, 256);
        pl->off_zpacc = off;
        off = align_up(off + sizeof(unsigned long long) * 2 * PIECE_CLASSES * ZMAX * (size_t)M, 256);
    }
    pl->zero_bytes = off;
    pl->off_rinfo = off;
    off = align_up(off + sizeof(RowInfo) * (size_t)M, 256);
    if (kind == MLMC_RTN) {
        pl->off_rtn_sums = off;
        off = align_up(off + sizeof(unsigned long long) * 2 * (size_t)L * M, 256);
        pl->off_norms = off;
        off = align_up(off + sizeof(double) * (size_t)L * M, 256);
        // Counting magnitudes costs a workgroup 128 KB to clear and to store and a row 128 KB of totals and 2^15 codes, whatever its length;
        // the two reads it replaces take about 1.2 us per 1e6 entries.  So the rows have to be long, not only many (us, four levels,
        // not counted / counted): 8 rows of 1048579 84 / 89, of 4194307 176 / 156; 64 of 524291 195 / 193; 128 of 262147 196 / 222,
        // of 524291 328 / 300; 256 of 524291 580 / 511; 512 of 131075 326 / 475; 1024 of 32771 217 / 645.
        if (in_dtype == MLMC_BF16 && (int64_t)M * d >= ((int64_t)1 << 25) && d >= ((int64_t)1 << 19)) {
            int64_t wgs = 256 / M > 0 ? 256 / M : 1;   // one workgroup per CU in one round
            if (wgs > (d + 8191) / 8192) wgs = (d + 8191) / 8192;
            pl->rtn_slice = ((d + wgs - 1) / wgs + 1023) / 1024 * 1024;
            pl->rtn_wgs = (int)((d + pl->rtn_slice - 1) / pl->rtn_slice);
            pl->off_rtn_part = off;
            off = align_up(off + sizeof(uint32_t) * 32768 * (size_t)pl->rtn_wgs * M, 256);
            pl->off_rtn_total = off;
            off = align_up(off + sizeof(uint32_t) * 32768 * (size_t)M, 256);
        }
    }
    // 32-bit rows of up to 65536 entries fit the registers of one workgroup.  The lower line is not one of speed: for rows of less than two tiles the staging hook is
    // kept, which decides what a call launches.  A workgroup per row would be the faster way there too: compress, us, general way / a workgroup per row,
    // 4 rows of 1000, fixed p 46 / 16, adaptive 61 / 23; 4 of 4096 47 / 16, 62 / 25; 64 of 8191 69 / 18, 110 / 28; 1024 of 4096 401 / 71, 865 / 107.
    // The workspace is that of the general way and 1 KB a row, though the two kernels touch a few MB of it at most: plans of this size were that large before.
    pl->row_mode = kind == MLMC_TOPK && in_dtype == MLMC_F32 && d >= ROW_MIN && d <= ROW_MAX ? 1 : 0;
    if (pl->row_mode) {
        pl->off_row_part = off;
        off = align_up(off + sizeof(uint4) * 64 * (size_t)M, 256);
    }
    if (counted) {
        // At most one workgroup per CU and whole slices for every row: 129 to 255 rows have one each and leave up to half the CUs idle, 257 need a second round.
        int64_t wgs = 256 / M > 0 ? 256 / M : 1;
        if (wgs > (d + 16383) / 16384) wgs = (d + 16383) / 16384;
        pl->c16_slice = ((d + wgs - 1) / wgs + TILE - 1) / TILE * TILE;
        pl->c16_wgs = (int)((d + pl->c16_slice - 1) / pl->c16_slice);
        pl->off_c16_part = off;
        off = align_up(off + sizeof(uint32_t) * 32768 * (size_t)(pl->c16_wgs + 1) * M, 256);
        pl->off_c16_occ = off;
        off = align_up(off + sizeof(uint32_t) * 8 * (size_t)pl->c16_wgs * M, 256);
        // The message read by slices (one launch) against the one by tiles (three), compress, 12 levels, us.  Rows whose stretches have scales of their own, adaptive: 32 rows of
        // 3000001 (slices of 376832) 142 / 154, 8 of 11689512 (368640) 135 / 141, 4 of 30000001 (471040) 173 / 167, 1 of 1e8 (393216) 127 / 138, 4 of 1.24e8 (1945600) 534 / 480;
        // with fixed p 123 / 122, 120 / 108, 145 / 135, 109 / 107, 449 / 379.  Rows of one distribution are faster by slices at these sizes too, with fixed p 123 / 129, 111 / 116,
        // 147 / 149, 101 / 117, but 440 / 423, adaptive 152 / 180, 138 / 165, 180 / 207, 135 / 200, 568 / 698, of one value, all of which may be in the message, 433 / 632.
        // Shorter slices: always faster (32 of 2000001 117 / 136 and 94 / 97).  So the line is where the stretches begin to gain with fixed p, not the best one for every row.
        if (pl->c16_slice >= (1 << 18)) {
            // A forecast of the message (k_c16_sample) costs some 30 us and a tenth of the first read, and spares most of the second one, which below this size
            // partly comes from the last cache.  Pass with the aggregate, 12 levels, us, without / with it, rows of many scales, adaptive: 8 of 11689512 161 / 167, 4 of 30000001
            // 211 / 217, 1 of 1.24e8 253 / 266, 2 of 7e7 231 / 234, 32 of 4000001 227 / 215, 4 of 50000001 293 / 267, 2 of 8e7 250 / 247, 4 of 4e7 223 / 214, 16 of 25557032 535 / 459, 4 of 1.24e8
            // (16 levels) 575 / 484; with fixed p 2 of 8e7 203 / 191, 32 of 5000001 197 / 174.  Rows of one distribution, whose lines nearly all have a member from bands of a thirtieth on: fixed p
            // 2 of 8e7 223 / 212, 4 of 50000001 261 / 231, 32 of 5000001 215 / 189, 4 of 1.2e8 552 / 453; adaptive, wide bands every other time, 8 of 2e7 306 / 301, 4 of 50000001 389 / 391, 32 of
            // 5000001 334 / 322, 4 of 1.2e8 868 / 845, but 2 of 8e7 332 / 339, 4 of 4e7 299 / 303.
            // These lose 2 % and gain 1 to 7 % with every other kind of row and draw.
            if ((int64_t)M * d >= 160000000) {
                pl->off_c16_mark = off;
                off = align_up(off + sizeof(uint64_t) * (TILE / 512) * (size_t)pl->ntiles * M, 256);
            }
            pl->off_c16_list = off;
            off = align_up(off + sizeof(uint32_t) * TILE * (size_t)pl->ntiles * M, 256);
            pl->off_c16_cnt = off;
            off = align_up(off + sizeof(uint4) * (size_t)pl->ntiles * M, 256);
            pl->off_c16_pre = off;
            off = align_up(off + sizeof(uint4) * (size_t)pl->ntiles * M, 256);
        }
        pl->off_tileoff = off;
        off = align_up(off + sizeof(uint32_t) * (size_t)(pl->ntiles + 1) * M, 256);
        pl->off_norms = off;
        off = align_up(off + sizeof(double) * (size_t)L * M, 256);
    } else if (kind == MLMC_TOPK) {
        pl->off_table = off;
        off = align_up(off + sizeof(uint32_t) * NB1 * (size_t)M, 256);
        pl->off_chunk_cnt = off;
        off = align_up(off + sizeof(uint32_t) * RMAX * (size_t)pl->cchunks_per_row * M, 256);
        pl->off_zcol = off;
        off = align_up(off + sizeof(unsigned long long) * COLLECT_CAP * ZMAX * (size_t)M, 256);
        pl->off_tileoff = off;
        off = align_up(off + sizeof(uint32_t) * (size_t)(pl->ntiles + 1) * M, 256);
        pl->off_norms = off;
        off = align_up(off + sizeof(double) * (size_t)L * M, 256);
        pl->off_cand = off;
        off = align_up(off + sizeof(uint2) * (size_t)d * M, 256);
        pl->off_cand2 = off;
        off = align_up(off + sizeof(uint2) * (size_t)d * M, 256);
        pl->off_cand_priv = off;
        off = align_up(off + sizeof(uint2) * 2 * (size_t)pl->chunk * pl->chunks_per_row * M, 256);   // room for twice a wave's even share
        pl->off_priv_cnt = off;
        off = align_up(off + sizeof(uint32_t) * 16 * (size_t)pl->chunks_per_row * M, 256);
        pl->off_chunk_base = off;
        off = align_up(off + sizeof(uint32_t) * (size_t)(pl->cchunks_per_row + 1) * M, 256);
        pl->off_row_order = off;
        off = align_up(off + sizeof(int32_t) * (size_t)M, 256);
        pl->off_table8 = off;
        off = align_up(off + (size_t)NB1 * M, 256);
        // Marks for the message (k_main2, k_pick) or its members in lists (k_filter)?  The marked entries are read again line by line, lists are written and read whatever
        // the lines are: rows of many scales have most lines without a member, rows of one scale hardly any.  Up to here the rows are in the last cache and the second
        // read costs little.  Pass, 12 levels, us, lists / marks, adaptive: many scales 8 of 300001 100 / 97, 32 of 1000001 220 / 197, 4 of 4000001 163 / 155, 4 of 8000001 205 / 189,
        // 2 of 16000001 213 / 194, 1 of 16777216 169 / 166; one scale 4 of 300001 92 / 91, 8 of 1000001 114 / 115, 32 of 1000001 210 / 207, 4 of 8000001 201 / 201, 2 of 16000001 208 / 212,
        // 1 of 16777216 178 / 183, 1 of 33000001 237 / 244.  Geometric p: many scales 32 of 1000001 131 / 127, 4 of 8000001 131 / 131, 1 of 16777216 110 / 109; one scale 4 of 300001
        // 64 / 63, 32 of 1000001 122 / 121, 4 of 8000001 122 / 123, 1 of 16777216 110 / 111.  Equal p: many scales 32 of 1000001 187 / 164, 4 of 8000001 170 / 161, 1 of 16777216 133 / 128;
        // one scale 32 of 1000001 163 / 160, 4 of 4000001 123 / 124, 4 of 8000001 151 / 152, 2 of 16000001 150 / 153, 1 of 16777216 125 / 129.  Larger, adaptive: many scales 16 of
        // 25557032 834 / 800, 8 of 11689512 334 / 307, but one scale 1047 / 1090 and 368 / 374, 4 of 6e7 723 / 762.
        if (pl->csub == CSUB_MAX && (int64_t)M * d <= ((int64_t)1 << 25) && d <= ((int64_t)1 << 24)) {
            pl->off_marks = off;
            off = align_up(off + sizeof(uint64_t) * ((size_t)pl->chunks_per_row * pl->chunk / 256) * (size_t)M, 256);
        }
    }
    pl->ws_bytes = off;
    if (workspace_bytes) *workspace_bytes = off;
    if (sparse_capacity_worst) {
        int64_t cap = 0;
        if (kind == MLMC_TOPK) {
            int64_t widest = 0;
            for (int l = 1; l <= L; ++l)
                if (ladder[l] - ladder[l - 1] > widest) widest = ladder[l] - ladder[l - 1];
            cap = (int64_t)M * (ladder[0] + widest);
        }
        *sparse_capacity_worst = cap;
    }
    *plan = pl;
    return MLMC_OK;
}

void mlmc_plan_destroy(mlmc_plan_t* plan) {
    if (!plan) return;
    // the side stream of the message step: its work was joined to the caller's stream, nothing is pending on it alone
    if (plan->side_stream) { (void)hipStreamSynchronize(plan->side_stream); (void)hipStreamDestroy(plan->side_stream); }
    if (plan->side_fork) (void)hipEventDestroy(plan->side_fork);
    if (plan->side_join) (void)hipEventDestroy(plan->side_join);
    delete plan;
}

mlmc_status mlmc_plan_set_overlap(mlmc_plan_t* plan, int enable) {
    if (!plan || plan->kind != MLMC_TOPK) return MLMC_EINVAL;
    plan->side_enable = enable ? 1 : 0;
    return MLMC_OK;
}

mlmc_status mlmc_plan_set_sampling(mlmc_plan_t* plan, int shift) {
    if (!plan || shift < 0 || shift > 12 || plan->kind == MLMC_VBITS || plan->kind == MLMC_RTN) return MLMC_EINVAL;
    plan->sample_shift = shift;
    return MLMC_OK;
}

mlmc_status mlmc_plan_set_staging(mlmc_plan_t* plan, int enable) {
    if (!plan || plan->kind != MLMC_TOPK) return MLMC_EINVAL;
    plan->staging = enable ? 1 : 0;
    return MLMC_OK;
}

int64_t mlmc_plan_num_tiles(const mlmc_plan_t* plan) { return plan ? plan->ntiles : 0; }
int64_t mlmc_plan_chunk(const mlmc_plan_t* plan) { return plan && plan->kind == MLMC_TOPK ? plan->chunk : 0; }
int mlmc_plan_num_planes(const mlmc_plan_t* plan) { return plan ? plan->nplanes : 0; }

mlmc_status mlmc_level_norms(const mlmc_plan_t* plan, const void* g, int64_t ld, double* norms, int32_t* dev_status,
                             void* ws, void* hip_stream) {
    if (!plan || (plan->kind != MLMC_TOPK && plan->kind != MLMC_STOPK && plan->kind != MLMC_RTN) || !g || !norms || !dev_status || !ws || ld < plan->d) return MLMC_EINVAL;
    if ((uintptr_t)ws % 256) return MLMC_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    if (plan->kind == MLMC_RTN) {
        BitsArgs b;
        fill_bits_args(plan, b, g, ld, ws, dev_status);
        b.norms_user = norms;
        return rtn_compress(plan, b, false, st);
    }
    if (plan->kind == MLMC_STOPK) {
        StopkArgs sa;
        fill_stopk_args(plan, sa, g, ld, ws, dev_status);
        sa.norms_user = norms;
        sa.se_marks = 0;
        return stopk_run(plan, sa, false, st);
    }
    TopkArgs a;
    fill_topk_args(plan, a, g, ld, ws, dev_status);
    a.all_thresholds = 1;
    a.draw_mode = -1;  // norms only, no draw
    a.marks = nullptr;
    a.norms_user = norms;
    if (plan->c16_wgs) return topk16_run(plan, a, false, st);
    if (plan->row_mode) return row_topk_run(plan, a, false, st);
    mlmc_status rc = topk_zero(plan, ws, dev_status, st);
    if (rc != MLMC_OK) return rc;
    return topk_select(plan, a, true, vec_ok(g, ld), st);
}

mlmc_status mlmc_compress_topk(const mlmc_plan_t* plan, const void* g, int64_t ld, const double* p, int p_is_norms,
                               uint64_t seed, uint64_t step, int32_t* level, int64_t* row_off, uint32_t* idx, float* val,
                               int64_t capacity, uint32_t* tile_off, double* norms_out, int32_t* dev_status, void* ws,
                               void* hip_stream) {
    if (!plan || (plan->kind != MLMC_TOPK && plan->kind != MLMC_STOPK) || !g || !level || !row_off || !idx || !val || !dev_status || !ws) return MLMC_EINVAL;
    if (ld < plan->d || capacity < 0 || (uintptr_t)ws % 256) return MLMC_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    if (plan->kind == MLMC_STOPK) {
        if (p || p_is_norms) return MLMC_EINVAL;   // Lemma 3.4 probabilities from the row itself, nothing else
        StopkArgs sa;
        fill_stopk_args(plan, sa, g, ld, ws, dev_status);
        sa.level = level;
        sa.row_off = row_off;
        sa.idx = idx;
        sa.val = val;
        sa.capacity = capacity;
        if (tile_off) sa.tile_off = tile_off;
        sa.norms_user = norms_out;
        sa.seed = seed;
        sa.step = step;
        return stopk_run(plan, sa, true, st);
    }
    const bool vec = vec_ok(g, ld);
    const bool internal_norms = plan->adaptive && p == nullptr;
    TopkArgs a;
    fill_topk_args(plan, a, g, ld, ws, dev_status);
    a.level = level;
    a.row_off = row_off;
    a.idx = idx;
    a.val = val;
    a.capacity = capacity;
    if (tile_off) a.tile_off = tile_off;
    a.norms_user = internal_norms ? norms_out : nullptr;
    a.all_thresholds = internal_norms ? 1 : 0;

    a.seed = seed;
    a.step = step;
    if (p) {
        a.draw_mode = p_is_norms ? 2 : 1;
        a.p_dev = p;
    } else if (!plan->adaptive) {
        a.draw_mode = 0;
        for (int l = 0; l < plan->L; ++l) a.p_fixed[l] = plan->p[l];
    } else {
        a.draw_mode = 3;
    }
    if (plan->c16_wgs) return topk16_run(plan, a, true, st);
    if (plan->row_mode) return row_topk_run(plan, a, true, st);
    mlmc_status rc = topk_zero(plan, ws, dev_status, st);
    if (rc != MLMC_OK) return rc;
    // draw_mode < 3: the level is drawn before the data is touched (inside the threshold scan), so only
    // three thresholds are resolved; draw_mode 3: all thresholds and band sums first, then the draw
    rc = topk_select(plan, a, internal_norms, vec, st);
    if (rc != MLMC_OK) return rc;
    return topk_compact(plan, a, vec, st);
}

mlmc_status mlmc_compress_bits(const mlmc_plan_t* plan, const void* g, int64_t ld, uint64_t seed, uint64_t step,
                               int32_t* level, int32_t* scale_exp, uint64_t* planes, int32_t* dev_status, void* ws,
                               void* hip_stream) {
    if (!plan || (plan->kind != MLMC_BITS && plan->kind != MLMC_FBITS && plan->kind != MLMC_VBITS) || !g || !level || !planes || !dev_status || !ws) return MLMC_EINVAL;
    if (plan->kind != MLMC_FBITS && !scale_exp) return MLMC_EINVAL;
    if (ld < plan->d || (uintptr_t)ws % 256) return MLMC_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    BitsArgs b;
    fill_bits_args(plan, b, g, ld, ws, dev_status);
    b.level = level;
    b.scale_exp = scale_exp;
    b.planes = planes;
    b.seed = seed;
    b.step = step;
    return bits_compress(plan, b, st);
}

mlmc_status mlmc_compress_rtn(const mlmc_plan_t* plan, const void* g, int64_t ld, uint64_t seed, uint64_t step, int32_t* level,
                              int32_t* scale, uint64_t* planes, double* norms_out, int32_t* dev_status, void* ws, void* hip_stream) {
    if (!plan || plan->kind != MLMC_RTN || !g || !level || !scale || !planes || !dev_status || !ws) return MLMC_EINVAL;
    if (ld < plan->d || (uintptr_t)ws % 256) return MLMC_EINVAL;
    BitsArgs b;
    fill_bits_args(plan, b, g, ld, ws, dev_status);
    b.level = level;
    b.scale_exp = scale;
    b.planes = planes;
    b.norms_user = norms_out;
    b.seed = seed;
    b.step = step;
    return rtn_compress(plan, b, true, (hipStream_t)hip_stream);
}

mlmc_status mlmc_compress_bits_static(const mlmc_plan_t* plan, const void* g, int64_t ld, uint64_t seed, uint64_t step,
                                      int32_t* level, int32_t* scale_exp, uint64_t* planes, int32_t* dev_status,
                                      void* hip_stream) {
    if (!plan || (plan->kind != MLMC_BITS && plan->kind != MLMC_FBITS && plan->kind != MLMC_VBITS)) return MLMC_EINVAL;
    if (plan->ws_bytes > (size_t)MLMC_STATIC_SCRATCH_BYTES) return MLMC_ELIMIT;   // before any HIP call
    void* ws = nullptr;
    const mlmc_status rc = static_scratch_of_current_device(&ws);
    if (rc != MLMC_OK) return rc;
    // same kernels as mlmc_compress_bits; the part of the scratch that must start at zero is cleared by the first of them
    return mlmc_compress_bits(plan, g, ld, seed, step, level, scale_exp, planes, dev_status, ws, hip_stream);
}

static mlmc_status aggregate_impl(const mlmc_plan_t* plan, const int32_t* level, const int64_t* row_off, const uint32_t* idx,
                                  const float* val, int64_t capacity, const uint32_t* tile_off, const int32_t* scale_exp,
                                  const uint64_t* planes, float alpha, float* out, float eta, float* x, void* ws, void* hip_stream) {
    if (!plan || (!out && !x)) return MLMC_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    if (plan->kind == MLMC_TOPK || plan->kind == MLMC_STOPK) {
        if (!row_off || !idx || !val || capacity < 0 || scale_exp || planes) return MLMC_EINVAL;
        if (!tile_off && (!ws || (uintptr_t)ws % 256)) return MLMC_EINVAL;
        uint32_t* tws = ws ? (uint32_t*)((char*)ws + plan->off_tileoff) : nullptr;
        return agg_sparse(plan, row_off, idx, val, capacity, tile_off, tws, alpha, out, eta, x, st);
    }
    if (!level || !planes || row_off || idx || val || tile_off) return MLMC_EINVAL;
    if (plan->kind != MLMC_FBITS && !scale_exp) return MLMC_EINVAL;
    BitsArgs b;
    fill_bits_args(plan, b, nullptr, plan->d, nullptr, nullptr);
    return agg_bits(plan, b, level, scale_exp, planes, alpha, out, eta, x, st);
}

mlmc_status mlmc_aggregate(const mlmc_plan_t* plan, const int32_t* level, const int64_t* row_off, const uint32_t* idx,
                           const float* val, int64_t capacity, const uint32_t* tile_off, const int32_t* scale_exp, const uint64_t* planes,
                           float alpha, float* out, void* ws, void* hip_stream) {
    if (!out) return MLMC_EINVAL;
    return aggregate_impl(plan, level, row_off, idx, val, capacity, tile_off, scale_exp, planes, alpha, out, 0.0f, nullptr, ws,
                          hip_stream);
}

mlmc_status mlmc_aggregate_update(const mlmc_plan_t* plan, const int32_t* level, const int64_t* row_off, const uint32_t* idx,
                                  const float* val, int64_t capacity, const uint32_t* tile_off, const int32_t* scale_exp,
                                  const uint64_t* planes, float alpha, float eta, float* x, float* out, void* ws,
                                  void* hip_stream) {
    if (!x || x == out) return MLMC_EINVAL;
    return aggregate_impl(plan, level, row_off, idx, val, capacity, tile_off, scale_exp, planes, alpha, out, eta, x, ws, hip_stream);
}

mlmc_status mlmc_message_bits(const mlmc_plan_t* plan, const int32_t* level, uint64_t* bits, void* hip_stream) {
    if (!plan || !level || !bits) return MLMC_EINVAL;
    return message_bits(plan, level, (unsigned long long*)bits, (hipStream_t)hip_stream);
}

}  // extern "C"
