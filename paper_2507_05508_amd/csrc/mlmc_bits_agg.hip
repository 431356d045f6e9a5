// Bit-wise MLMC (Sec. 3.1 fixed point, App. B floating point) and the server aggregate (Alg. 2 / Alg. 3) on gfx950.
//
//   k_bits_prep     level draw of every row (floating-point ladder; the other ladders draw in k_bits_smax)
//   k_bits_smax     largest |g| key of a sample of every row -> predicted power-of-two scale; level draw             [mlmc_extract.h]
//   k_bits_extract  the one full read: digits floor(|g_j| / s * 2^F), sign plane + field planes by bit transposes   [mlmc_extract.h]
//                   inside a lane, and the true row maximum; a row whose true maximum has a larger exponent than the
//                   sampled one is extracted again by a second launch (which returns at once for every other row)
//   k_agg_planes    out = alpha * sum_i decode_i, rows added in worker order (all plane messages, Round-to-Nearest included)
//   k_tileoff       (fallback) per-tile offsets of index-sorted sparse rows by binary search
//   k_agg_sparse    atomic-free segmented scatter-add: one workgroup owns one dense tile
//   k_message_bits  bits on the wire of every row's message
// The Round-to-Nearest ladder is launched from mlmc_vrtn.hip.
#include "mlmc_extract.h"

namespace mlmc {

// ---------------------------------------------------------------------------------------------------
// Level draw of every row (Alg. 2 "Sample l ~ p"), and the per-row state of the call set to its start values.
__global__ __launch_bounds__(1024) void k_bits_prep(BitsArgs a) {
    __shared__ double s_p[LMAX];
    const int r = threadIdx.x;
    if (r < a.L) s_p[r] = a.p_fixed[r];
    if (r == 0) *a.dev_status = 0;
    __syncthreads();
    for (int row = r; row < a.M; row += 1024) {
        const uint32_t x = philox_word0(a.seed, a.step, (uint32_t)row);
        const int level = draw_from_p(s_p, a.L, x);
        const double pl = s_p[level - 1];
        RowInfo* ri = a.rinfo + row;
        ri->level = level;
        ri->weight = pl == 0.0 ? 0.0f : (float)__ddiv_rn(1.0, pl);
        ri->draw_x = x;
        a.level[row] = level;
        a.racc[row].rowmax_key = 0u;
        a.racc[row].smpmax_key = 0u;
    }
}

// What a kernel of the aggregate does with the finished sum of entry j: g~_j = alpha * acc (Alg. 2 "Server
// aggregates"), written out and / or applied to the model, x_j <- x_j - eta * g~_j (Alg. 2 "Server updates": one
// multiply, one subtract).
__device__ __forceinline__ void finish_entry(float alpha, float acc, float* out, float eta, float* x, int64_t j) {
    const float gt = __fmul_rn(alpha, acc);
    if (out) __builtin_nontemporal_store(gt, &out[j]);   // written once, read by the caller later
    if (x) x[j] = __fsub_rn(x[j], __fmul_rn(eta, gt));
}

// the same for entries j .. j + 3
__device__ __forceinline__ void finish_four(float alpha, float4 acc, float* out, float eta, float* x, int64_t j) {
    typedef float f32x4_el __attribute__((ext_vector_type(4), aligned(4)));
    f32x4_el gt;
    gt.x = __fmul_rn(alpha, acc.x);
    gt.y = __fmul_rn(alpha, acc.y);
    gt.z = __fmul_rn(alpha, acc.z);
    gt.w = __fmul_rn(alpha, acc.w);
    if (out) __builtin_nontemporal_store(gt, (f32x4_el*)(out + j));
    if (x) {
        f32x4_el xv = *(const f32x4_el*)(x + j);
        xv.x = __fsub_rn(xv.x, __fmul_rn(eta, gt.x));
        xv.y = __fsub_rn(xv.y, __fmul_rn(eta, gt.y));
        xv.z = __fsub_rn(xv.z, __fmul_rn(eta, gt.z));
        xv.w = __fsub_rn(xv.w, __fmul_rn(eta, gt.w));
        *(f32x4_el*)(x + j) = xv;
    }
}

struct AggBitsArgs {
    BitsArgs b;
    const int32_t* level;
    const int32_t* scale_exp;
    float alpha, eta;
};

// out[j] = alpha * sum over rows (worker order) of the decoded messages: Alg. 2 "Server aggregates".
//
// The extraction's packing run backwards: a wave owns a block of EX_ELEMS elements, a lane 32 of them (half a word of every
// plane) and their sums in registers.  Eight planes of a row transposed (transpose8) are the low bytes of the lane's 32 values, so
// that a value costs an instruction or two to assemble whatever its width.  8 rows of 1.17e7 elements: 24 us at two or three planes
// (wave latency: a wave's rows come one after the other), 35 us at ten (0.16 GB, 4.6 TB/s), 31 us for Round-to-Nearest codes; 4 rows of
// 1.24e8 elements and 38 code planes in all 252 us (1.09 GB, 4.4 TB/s).  The vector instructions were two thirds of the time for the codes, so
// their residual integers come straight from dot products of the transposed bytes (before, with every code taken out and sign-extended and two
// 24-bit multiplications: 41 and 302 us), and the loads' addresses are scalar (a 64-bit multiplication per load in vector registers before: 27 us
// at two or three planes, 38 at ten).  A block per wave at a time and many of them: a grid that fits the chip and goes from block to
// block, the next one's planes in flight, took 8 % longer on the long rows.
// The next row's first planes (the low eight of both codes for Round-to-Nearest) are in flight while a row is decoded.  The sums leave through LDS in the order of the
// loads of the extraction, so that the dense vector is read and written 1 KB at a time.
// PK 0: fixed point (both scales), 1: floating point, 2: Round-to-Nearest.  BASE: the ladder has a base field (F_0 > 0).
struct AggRow {          // per row, in LDS
    float c0, cl;
    int32_t np;          // planes of the message
    int32_t w, fl;       // fixed point: width of the level field; floating point: and digits of the level; codes: width of the drawn and of the previous code
};

template <int PK, bool BASE>
__device__ __forceinline__ AggRow agg_row(const AggBitsArgs& a, int r) {
    const BitsArgs& b = a.b;
    const int F0 = BASE ? b.F[0] : 0;
    int lev = a.level[r];
    lev = lev < 1 ? 1 : (lev > b.L ? b.L : lev);
    const double pl = b.p_fixed[lev - 1];
    AggRow q;
    q.c0 = 0.0f;
    q.w = b.F[lev] - b.F[lev - 1];
    q.fl = b.F[lev];
    if (PK == 2) {          // c_0 = fp32(2c / D_0); the coefficient comes with the message
        const double c = key_to_double((uint32_t)a.scale_exp[2 * r] & 0x7FFFFFFFu);
        if (BASE) q.c0 = (float)__ddiv_rn(__dmul_rn(2.0, c), (double)((1 << F0) - 1));
        q.cl = __uint_as_float((uint32_t)a.scale_exp[2 * r + 1]);
        q.w = b.F[lev];                          // width of the drawn level's code
        q.fl = lev > 1 ? b.F[lev - 1] : 0;       // width of the previous level's code when it is sent
        q.np = F0 + q.fl + q.w;
    } else if (PK == 1) {   // the level's weight fp32(1 / p_l)
        q.cl = pl == 0.0 ? 0.0f : (float)__ddiv_rn(1.0, pl);
        q.np = 9 + F0 + q.w;
    } else {
        if (b.vmx) {        // the scale field carries the largest entry v: c_0 = fp32(v 2^-F_0), c_l = fp32(v 2^-F_l / p_l)
            const double vd = key_to_double((uint32_t)a.scale_exp[r] & 0x7FFFFFFFu);
            if (BASE) q.c0 = (float)ldexp(vd, -F0);
            q.cl = pl == 0.0 ? 0.0f : (float)__ddiv_rn(ldexp(vd, -b.F[lev]), pl);
        } else {
            const int e = a.scale_exp[r];
            if (BASE) q.c0 = (float)ldexp(1.0, e - F0);
            q.cl = pl == 0.0 ? 0.0f : (float)__ddiv_rn(ldexp(1.0, e - b.F[lev]), pl);
        }
        q.np = 1 + F0 + q.w;
    }
    return q;
}

// The same sum, a wave a word of 64 entries of every plane and an entry a lane: for rows that leave most of the chip idle with 2048 entries a wave (4 rows of 100003, fixed point: 8.4 -> 3.9 us).
// A lane loads a plane's word, four rows at a time, whatever the rows' levels are; the words then choose the bits of the lanes' entries.
template <int PK, bool BASE>
__global__ __launch_bounds__(EX_THREADS) void k_agg_words(AggBitsArgs a, const uint64_t* __restrict__ planes, float* __restrict__ out, float* __restrict__ x) {
    extern __shared__ __align__(16) unsigned char s_dyn_words[];
    AggRow* s_row = (AggRow*)s_dyn_words;
    const BitsArgs& b = a.b;
    const int F0 = BASE ? b.F[0] : 0;
    const uint32_t lane = lane_id();
    const int64_t word = (int64_t)blockIdx.x * (EX_THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t* mine = planes + (size_t)((int)lane < b.nplanes ? lane : 0u) * b.nwords + (word < b.nwords ? word : b.nwords - 1);
    constexpr int U = 4;
    uint64_t v[U];
    auto fetch = [&](int r0) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = mine[(size_t)(r0 + u < b.M ? r0 + u : b.M - 1) * b.nplanes * b.nwords];
    };
    fetch(0);
    for (int r = threadIdx.x; r < b.M; r += EX_THREADS) s_row[r] = agg_row<PK, BASE>(a, r);
    __syncthreads();
    if (word >= b.nwords) return;   // uniform
    float acc = 0.0f;
    for (int r0 = 0; r0 < b.M; r0 += U) {   // rows in worker order
        uint64_t cur[U];
#pragma unroll
        for (int u = 0; u < U; ++u) cur[u] = v[u];
        if (r0 + U < b.M) fetch(r0 + U);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r0 + u >= b.M) break;   // uniform
            const AggRow q = s_row[r0 + u];
            const int np = __builtin_amdgcn_readfirstlane(q.np);
            uint32_t y = 0;   // bit p: the entry's bit of plane p
            for (int p = 0; p < np; ++p) {   // uniform
                const uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(cur[u] >> 32), p) << 32 |
                                   (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)cur[u], p);
                y |= __builtin_amdgcn_inverse_ballot_w64(m) ? 1u << p : 0u;
            }
            float add;
            if (PK == 0) {
                const uint32_t n = y >> 1;
                if (!BASE) add = __fmul_rn((float)n, q.cl);
                else add = __fadd_rn(__fmul_rn((float)(n & ((1u << F0) - 1u)), q.c0), __fmul_rn((float)(n >> F0), q.cl));
                add = __uint_as_float(__float_as_uint(add) | y << 31);
            } else if (PK == 1) {
                const uint32_t se = y << 31 | ((y >> 1) & 0xFFu) << 23, lev = (y >> 9 >> F0) << (23 - q.fl);
                const float res = __fsub_rn(__uint_as_float(se | lev), __uint_as_float(se));
                const uint32_t base = BASE ? ((y >> 9) & ((1u << F0) - 1u)) << (23 - F0) : 0u;
                add = __fadd_rn(__uint_as_float(se | base), __fmul_rn(res, q.cl));
            } else {
                const int pw = q.fl > 0 ? q.fl : F0;         // level 1: the previous code is the base code
                const int32_t D = (1 << q.w) - 1, Dp = pw > 0 ? (1 << pw) - 1 : 1;
                const int32_t cur_n = __builtin_amdgcn_sbfe((int)y, F0 + q.fl, q.w);
                const int32_t prev_n = pw > 0 ? __builtin_amdgcn_sbfe((int)y, q.fl > 0 ? F0 : 0, pw) : 0;
                add = __fmul_rn((float)(int32_t)((uint32_t)cur_n * (uint32_t)Dp - (uint32_t)prev_n * (uint32_t)D), q.cl);
                if (BASE) add = __fadd_rn(__fmul_rn((float)(int32_t)__builtin_amdgcn_sbfe((int)y, 0, F0), q.c0), add);
            }
            acc = __fadd_rn(acc, add);
        }
    }
    const int64_t j = word * 64 + lane;
    if (j < b.d) finish_entry(a.alpha, acc, out, a.eta, x, j);
}

// The values of w <= 24 planes, v[0] the least significant, as numbers: u[e] for the lane's 32 elements.  G: groups of eight planes.
template <int G>
__device__ __forceinline__ uint32_t assemble(const uint32_t (&r)[3][8], int i, int k) {
    if (G == 1) return (r[0][i] >> (8 * k)) & 0xFFu;
    const uint32_t lo = __builtin_amdgcn_perm(r[1][i], r[0][i], 0x0C0C0400u + 0x0101u * (uint32_t)k);
    if (G == 2) return lo;
    return __builtin_amdgcn_perm(r[2][i], lo, 0x0C040100u + 0x010000u * (uint32_t)k);
}

template <int PK, bool BASE>
__global__ __launch_bounds__(EX_THREADS, 4) void k_agg_planes(AggBitsArgs a, const uint64_t* __restrict__ planes, float* __restrict__ out,
                                                              float* __restrict__ x) {
    extern __shared__ __align__(16) unsigned char s_dyn_planes[];   // the waves' blocks of sums on their way out, then the rows' records
    AggRow* s_row = (AggRow*)(s_dyn_planes + (EX_THREADS / 64) * EX_ELEMS * 4);
    const BitsArgs& b = a.b;
    const int F0 = BASE ? b.F[0] : 0;
    for (int r = threadIdx.x; r < b.M; r += EX_THREADS) s_row[r] = agg_row<PK, BASE>(a, r);
    __syncthreads();
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t blk = (int64_t)blockIdx.x * (EX_THREADS / 64) + wave;
    const int64_t nw2 = b.nwords * 2, h0 = blk * 64;   // half words of a plane; the block's first
    if (h0 >= nw2) return;
    const uint32_t last = nw2 - h0 < 64 ? (uint32_t)(nw2 - h0) - 1u : 63u;   // lanes past a plane's end read its last half word again
    const uint32_t off = (lane < last ? lane : last) * 4u;
    typedef const __attribute__((address_space(1))) char* GlobalBytes;
    const size_t step = (size_t)b.nwords * 8;
    const GlobalBytes base = (GlobalBytes)planes + h0 * 4;
    // n planes of the row from p0 on, q past the last of them: that one again.  The address is scalar and goes from plane to plane (opaque, or the
    // compiler keeps a vector of addresses for every load).
    auto planes_from = [&](GlobalBytes row, int p0, int have, auto n, uint32_t* r) {
        GlobalBytes at = row + (size_t)(uint32_t)p0 * step;
#pragma unroll
        for (int q = 0; q < decltype(n)::value; ++q) {
            r[q] = *(const __attribute__((address_space(1))) uint32_t*)(at + off);
            at += q + 1 < have ? step : (size_t)0;
            asm volatile("" : "+s"(at));
        }
    };
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    auto funi = [](float v) { return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v))); };

    float acc[32];
#pragma unroll
    for (int e = 0; e < 32; ++e) acc[e] = 0.0f;
    constexpr int AHEAD = PK == 2 ? 16 : PK == 1 ? 10 : 9;
    uint32_t ahead[AHEAD];
    auto look_ahead = [&](int r) {   // no branch between the loads: past the message's end its last plane is read again
        const GlobalBytes row = base + (size_t)r * b.nplanes * step;
        const int np = uni(s_row[r].np);
        if (PK == 2) {
            const int w = uni(s_row[r].w), pw = uni(s_row[r].fl);
            planes_from(row, np - w, w, std::integral_constant<int, 8>{}, ahead);
            if (pw > 0) planes_from(row, F0, pw, std::integral_constant<int, 8>{}, ahead + 8);
        } else {
            planes_from(row, 0, np, std::integral_constant<int, AHEAD>{}, ahead);
        }
    };
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) ahead[p] = 0;
    look_ahead(0);
    for (int r = 0; r < b.M; ++r) {   // rows in worker order
        const GlobalBytes row = base + (size_t)r * b.nplanes * step;
        const int np = uni(s_row[r].np), w = uni(s_row[r].w), fl = uni(s_row[r].fl);
        const float cl = funi(s_row[r].cl), c0 = BASE ? funi(s_row[r].c0) : 0.0f;
        uint32_t cur[AHEAD];
#pragma unroll
        for (int p = 0; p < AHEAD; ++p) cur[p] = ahead[p];
        if (r + 1 < b.M) look_ahead(r + 1);
        // planes p0 .. p0 + n - 1 (at most eight of them) of the row into r8, the rest of it zero, transposed
        auto group = [&](int p0, int n, uint32_t (&r8)[8]) {
#pragma unroll
            for (int q = 0; q < 8; ++q) r8[q] = 0;
                GlobalBytes at = row + (size_t)(uint32_t)p0 * step;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q < n) r8[q] = *(const __attribute__((address_space(1))) uint32_t*)(at + off);   // uniform
                at += step;
                asm volatile("" : "+s"(at));
            }
            transpose8(r8);
        };
        if (PK == 0) {
            const uint32_t sg = cur[0];
            auto add = [&](int e, float v) {   // v >= 0, its sign from the sign plane
                v = __uint_as_float(((sg << (31 - e)) & 0x80000000u) | __float_as_uint(v));
                acc[e] = __fadd_rn(acc[e], v);
            };
            if (!BASE && w == 1) {
                // f is 0 or 1: the entry is +-cl or absent (adding 0 of either sign leaves the sum as it is)
                const uint32_t fw = cur[1];
#pragma unroll
                for (int e = 0; e < 32; ++e)
                    acc[e] = __fadd_rn(acc[e], __uint_as_float((((sg << (31 - e)) & 0x80000000u) | __float_as_uint(cl)) & (uint32_t)__builtin_amdgcn_sbfe((int)fw, e, 1)));
            } else {
                uint32_t r8[3][8];
#pragma unroll
                for (int q = 0; q < 8; ++q) r8[0][q] = 1 + q < np ? cur[1 + q] : 0u;
                transpose8(r8[0]);
                auto all = [&](auto groups) {
                    constexpr int G = decltype(groups)::value;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const uint32_t u = assemble<G>(r8, i, k);
                            float v;
                            if (!BASE) v = __fmul_rn((float)u, cl);
                            else v = __fadd_rn(__fmul_rn((float)(u & ((1u << F0) - 1u)), c0), __fmul_rn((float)(u >> F0), cl));
                            add(8 * k + i, v);
                        }
                };
                if (np <= 9) {
                    all(std::integral_constant<int, 1>{});
                } else {
                    group(9, np - 9, r8[1]);
                    if (np <= 17) {
                        all(std::integral_constant<int, 2>{});
                    } else {
                        group(17, np - 17, r8[2]);
                        all(std::integral_constant<int, 3>{});
                    }
                }
            }
        } else if (PK == 1) {
            // App. B: sign, exponent field and base digits give C^{F_0}; the level digits, placed under the same sign and
            // exponent, minus the bare power of two give the residual (exact); weight, then one add
            uint32_t t[8];   // bits 24 .. 31 of the lane's fp32 words: the exponent's upper seven and the sign
#pragma unroll
            for (int q = 0; q < 7; ++q) t[q] = cur[2 + q];
            t[7] = cur[0];
            transpose8(t);
            const uint32_t e0 = cur[1];   // the exponent's lowest bit
            auto head = [&](int i, int k) -> uint32_t {   // sign and exponent of element 8 k + i
                const uint32_t hi = __builtin_amdgcn_perm(t[i], 0u, 0x040C0C0Cu + 0x01000000u * (uint32_t)k);
                return hi | (((e0 >> (8 * k + i)) & 1u) << 23);
            };
            auto finish = [&](int i, int k, uint32_t base_digits, uint32_t level_digits) {
                const uint32_t se = head(i, k);
                const float res = __fsub_rn(__uint_as_float(se | level_digits), __uint_as_float(se));
                const float v = __fadd_rn(__uint_as_float(se | base_digits), __fmul_rn(res, cl));
                acc[8 * k + i] = __fadd_rn(acc[8 * k + i], v);
            };
            const int pos = 23 - fl;
            if (!BASE && w == 1) {
                const uint32_t fw = cur[9];
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 8; ++i) finish(i, k, 0u, ((fw >> (8 * k + i)) & 1u) << pos);
            } else {
                uint32_t f8[3][8], b8[3][8];
                const int p0 = 9 + F0;
                group(p0, w, f8[0]);
                group(p0 + 8, w - 8, f8[1]);
                group(p0 + 16, w - 16, f8[2]);
                if (BASE) {
                    group(9, F0, b8[0]);
                    group(17, F0 - 8, b8[1]);
                    group(25, F0 - 16, b8[2]);
                }
                const int bpos = 23 - F0;
                // (a group past the field's end is zero; a base field of more than 8 or 16 digits ends inside its groups)
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const uint32_t fd = assemble<3>(f8, i, k) << pos;
                        uint32_t bd = 0;
                        if (BASE) bd = (assemble<3>(b8, i, k) & ((1u << F0) - 1u)) << bpos;
                        finish(i, k, bd, fd);
                    }
            }
        } else {
            // codes n_{b_0} (if any), n_{b_{l-1}} (if sent) and n_{b_l}; the residual integer k = n_cur D' - n_prev D;
            // value = fp32(n_0) c_0 + fp32(k) coefficient.
            // k comes out of dot products of small unsigned numbers: with u = n_cur + 2^(w-1) (its top bit turned) and
            // v = D' - (n_prev + 2^(pw-1)) (the other bits turned), k = u D' + v D + a constant, modulo 2^32.
            const int bp = fl, pw = bp > 0 ? bp : F0;         // level 1: the previous code is the base code
            const uint32_t D = (1u << w) - 1u, Dp = pw > 0 ? (1u << pw) - 1u : 1u;
            const uint32_t c = (pw > 0 ? D * (1u << (pw - 1)) - D * Dp : 0u) - (Dp << (w - 1));
            const uint32_t cturn = 1u << (w - 1), cmask = D, pturn = pw > 0 ? (1u << (pw - 1)) - 1u : 0u, pmask = pw > 0 ? Dp : 0u;
            constexpr uint32_t BYTES = 0x01010101u;
            uint32_t z8[3][8];
            if (BASE) {
                group(0, F0, z8[0]);
                if (F0 > 8) group(8, F0 - 8, z8[1]);
            }
            auto add = [&](int i, int k, uint32_t num) {
                float v = __fmul_rn((float)(int32_t)num, cl);
                if (BASE) {
                    const int n0 = F0 > 8 ? __builtin_amdgcn_sbfe((int)assemble<2>(z8, i, k), 0, F0) : __builtin_amdgcn_sbfe((int)z8[0][i], 8 * k, F0);
                    v = __fadd_rn(__fmul_rn((float)n0, c0), v);
                }
                acc[8 * k + i] = __fadd_rn(acc[8 * k + i], v);
            };
            auto masked = [&](uint32_t (&r8)[8], uint32_t turn, uint32_t mask) {   // bits of the byte, the same in every byte
#pragma unroll
                for (int q = 0; q < 8; ++q) r8[q] = (r8[q] ^ ((turn & 0xFFu) * BYTES)) & ((mask & 0xFFu) * BYTES);
            };
            // (an empty statement of its own at the end of every way: what they have in common is not moved behind them, which
            // would keep 32 values in registers and spill)
            if (w <= 4 && (!BASE || bp > 0)) {   // both codes in one byte: one transposition, one dot product of nibbles
                uint32_t r8[8];
#pragma unroll
                for (int q = 0; q < 4; ++q) { r8[q] = cur[q]; r8[4 + q] = cur[8 + q]; }
                transpose8(r8);
                masked(r8, cturn | pturn << 4, cmask | pmask << 4);
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 8; ++i) add(i, k, __builtin_amdgcn_udot8(r8[i], (Dp | D << 4) << (8 * k), c, false));
                asm volatile("; nibbles");
            } else {
                auto current = [&](uint32_t (&n0)[8]) {      // the low bytes of the codes
#pragma unroll
                    for (int q = 0; q < 8; ++q) n0[q] = cur[q];
                    transpose8(n0);
                    masked(n0, w > 8 ? 0u : cturn, cmask);
                };
                auto previous = [&](uint32_t (&p0)[8]) {
                    if (!BASE || bp > 0) {
#pragma unroll
                        for (int q = 0; q < 8; ++q) p0[q] = cur[8 + q];
                        transpose8(p0);
                    } else {
#pragma unroll
                        for (int q = 0; q < 8; ++q) p0[q] = z8[0][q];
                    }
                    masked(p0, pturn, pmask);
                };
                typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
                const u16x2 by = __builtin_bit_cast(u16x2, Dp | D << 16);
                if (w <= 8) {
                    uint32_t n8[8], p8[8];
                    current(n8);
                    if (pw > 0) {
                        previous(p8);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int i = 0; i < 8; ++i)
                                add(i, k, __builtin_amdgcn_udot4(p8[i], D << (8 * k), __builtin_amdgcn_udot4(n8[i], Dp << (8 * k), c, false), false));
                        asm volatile("; bytes");
                    } else {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int i = 0; i < 8; ++i) add(i, k, __builtin_amdgcn_udot4(n8[i], Dp << (8 * k), c, false));
                        asm volatile("; first bytes");
                    }
                } else {
                    uint32_t n8[8], h8[8];
                    group(F0 + bp + 8, w - 8, h8);
                    masked(h8, cturn >> 8, cmask >> 8);
                    current(n8);
                    if (pw == 0) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const uint32_t both = __builtin_amdgcn_perm(h8[i], n8[i], 0x0C0C0400u + 0x0101u * (uint32_t)k);
                                add(i, k, __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, both), by, c, false));
                            }
                        asm volatile("; first words");
                    } else if (pw <= 8) {
                        uint32_t p8[8];
                        previous(p8);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const uint32_t one = __builtin_amdgcn_perm(h8[i], n8[i], 0x0C0C0400u + 0x0101u * (uint32_t)k);
                                const uint32_t both = __builtin_amdgcn_perm(p8[i], one, 0x0C040100u + 0x010000u * (uint32_t)k);
                                add(i, k, __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, both), by, c, false));
                            }
                        asm volatile("; words and bytes");
                    } else {
                        uint32_t p8[8], q8[8];
                        if (bp > 0) {
                            group(F0 + 8, bp - 8, q8);
                        } else {
#pragma unroll
                            for (int q = 0; q < 8; ++q) q8[q] = BASE ? z8[1][q] : 0u;
                        }
                        masked(q8, pturn >> 8, pmask >> 8);
                        previous(p8);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const uint32_t one = __builtin_amdgcn_perm(h8[i], n8[i], 0x0C0C0400u + 0x0101u * (uint32_t)k);
                                const uint32_t both = one | __builtin_amdgcn_perm(q8[i], p8[i], 0x04000C0Cu + 0x01010000u * (uint32_t)k);
                                add(i, k, __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, both), by, c, false));
                            }
                        asm volatile("; words");
                    }
                }
            }
        }
    }
    // the lane's 32 sums into the wave's buffer, out of it 16 bytes at a time: chunk c of lane l in slot c ^ (l & 7)
    float* buf = (float*)(s_dyn_planes + wave * (EX_ELEMS * 4));
#pragma unroll
    for (int c = 0; c < 8; ++c)
        *(float4*)(buf + (lane * 8u + ((uint32_t)c ^ (lane & 7u))) * 4u) = make_float4(acc[4 * c], acc[4 * c + 1], acc[4 * c + 2], acc[4 * c + 3]);
    wave_lds_sync();
    const int64_t j0 = blk * EX_ELEMS;
    const uint32_t goff = (lane & ~7u) * 4u + ((lane & 7u) ^ ((lane >> 3) & 7u)) * 4u;   // element of this lane's first chunk
    if (j0 + EX_ELEMS <= b.d) {   // uniform
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float4 s4 = *(const float4*)(buf + (64 * k + lane) * 4u);
            finish_four(a.alpha, s4, out, a.eta, x, j0 + k * 256 + goff);
        }
    } else {
#pragma unroll 1
        for (uint32_t e = lane; e < EX_ELEMS && j0 + e < b.d; e += 64) {
            const uint32_t owner = e >> 5, c = (e & 31u) >> 2;
            finish_entry(a.alpha, buf[(owner * 8u + (c ^ (owner & 7u))) * 4u + (e & 3u)], out, a.eta, x, j0 + e);
        }
    }
}

// ---------------------------------------------------------------------------------------------------
struct AggSparseArgs {
    int32_t M;
    int64_t d, ntiles;
    const int64_t* row_off;
    const uint32_t* idx;
    const float* val;
    int64_t capacity;          // entries idx / val hold
    const uint32_t* tile_off;  // [M][ntiles + 1]
    uint32_t* tile_off_out;    // k_tileoff target
    float alpha;
    float* out;                // the dense update g~ (may be null when only x is wanted)
    float eta;
    float* x;                  // server update x <- x - eta * g~ (null: no update)
};

__global__ __launch_bounds__(256) void k_tileoff(AggSparseArgs a) {
    const int64_t n = (int64_t)a.M * (a.ntiles + 1);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int r = (int)(i / (a.ntiles + 1));
        const int64_t t = i % (a.ntiles + 1);
        int64_t s = a.row_off[r], e = a.row_off[r + 1];   // entries past the capacity were never written
        if (s > a.capacity) s = a.capacity;
        if (e > a.capacity) e = a.capacity;
        if (e < s) e = s;
        const uint64_t target = (uint64_t)t * TILE;
        int64_t lo = s, hi = e;  // first position with idx >= target
        while (lo < hi) {
            int64_t mid = lo + ((hi - lo) >> 1);
            if ((uint64_t)a.idx[mid] < target) lo = mid + 1; else hi = mid;
        }
        a.tile_off_out[i] = (uint32_t)(lo - s);
    }
}

// One workgroup per dense tile: LDS accumulators, rows added one after the other (indices within a row are
// distinct, so plain read-modify-write is race free), then one coalesced write of alpha * acc.  A row's step is the latency of LDS and a barrier, so
// where the tiles leave the CUs room a tile gets more threads, as far as a row has entries for them (agg_threads).  32 rows, 512 entries of each in a
// tile, us with 256 / 512 / 1024 threads: 245 tiles 34.1 / 21.6 / 13.8, 489 38.3 / 26.2 / 18.6, 977 44.3 / 32.8 / 34.9; 1024 entries 40.3 / 38.6 / 23.6, 41.5 / 42.9 / 30.7,
// 49.7 / 54.7 / 55.0; 16 rows, some 500 entries, 1954 tiles 28.5 / 32.3 / 43.2.  Of 32 entries or 128 a row's step is its barrier, which more waves make
// longer: 256 rows, 1 tile 73.5 / 72.9 / 76.8, 245 79.4 / 79.4 / 80.2, 489 83.8 / 84.7 / 102.8; 32 rows, 245 tiles 13.2 / 12.4 / 12.9, 977 14.9 / 16.7 / 29.1; with 4 rows
// there is nothing to lose (977 tiles 7.8 / 7.5 / 10.2), and what is drawn may be far longer than the mean (2048 entries 15.8 / 13.9 / 18.9).
template <int NT>
__global__ __launch_bounds__(NT) void k_agg_sparse(AggSparseArgs a) {
    // dynamic LDS, sized by the number of rows (M * 12 bytes), so that a CU holds as many workgroups as its wave
    // slots allow: the tile's accumulators, then every row's start and length inside the tile
    extern __shared__ __align__(16) unsigned char s_dyn_agg[];
    float* s_acc = (float*)s_dyn_agg;
    int64_t* s_beg = (int64_t*)(s_dyn_agg + TILE * sizeof(float));
    uint32_t* s_len = (uint32_t*)(s_dyn_agg + TILE * sizeof(float) + (size_t)a.M * sizeof(int64_t));
    const int64_t tile = blockIdx.x;
    const int64_t base = tile * TILE;
    for (int i = threadIdx.x; i < TILE / 4; i += NT) ((float4*)s_acc)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int r = threadIdx.x; r < a.M; r += NT) {
        const uint32_t* to = a.tile_off + (size_t)r * (a.ntiles + 1);
        // a tile holds at most TILE entries of a row and they lie inside the row's message: an offset table that
        // says otherwise (a failed compress call, a caller's own table) must not steer reads out of bounds
        const int64_t beg = a.row_off[r] + to[tile];
        uint32_t len = to[tile + 1] - to[tile];
        if (to[tile + 1] < to[tile] || len > (uint32_t)TILE || beg < a.row_off[r] || beg + len > a.row_off[r + 1] ||
            beg + len > a.capacity) len = 0;
        s_beg[r] = beg;
        s_len[r] = len;
    }
    __syncthreads();
    // rows in groups of eight: the first NT entries of every row of the group are fetched back to back (a thread's
    // entry, or the row's last one when it has fewer), then added in worker order
    constexpr int RG = 8, U = TILE / NT - 1 < 4 ? TILE / NT - 1 : 4;
    for (int r0 = 0; r0 < a.M; r0 += RG) {
        uint32_t pidx[RG];
        float pval[RG];
#pragma unroll
        for (int k = 0; k < RG; ++k) {
            const int r = r0 + k;
            const uint32_t len = r < a.M ? s_len[r] : 0u;
            pidx[k] = 0xFFFFFFFFu;
            pval[k] = 0.0f;
            if (len) {  // uniform
                const uint32_t e = threadIdx.x < len ? threadIdx.x : len - 1u;
                pidx[k] = a.idx[s_beg[r] + e];
                pval[k] = a.val[s_beg[r] + e];
            }
        }
#pragma unroll
        for (int k = 0; k < RG; ++k) {
            const int r = r0 + k;
            const uint32_t len = r < a.M ? s_len[r] : 0u;
            if (len) {  // uniform
                const int64_t beg = s_beg[r];
                if (threadIdx.x < len) {
                    const uint32_t off = pidx[k] - (uint32_t)base;
                    if (off < (uint32_t)TILE) s_acc[off] = __fadd_rn(s_acc[off], pval[k]);
                }
                // the rest of a long row: four (or all) loads per thread in flight (past the end: the last entry, discarded)
                for (uint32_t i0 = threadIdx.x + NT; i0 < len; i0 += U * NT) {
                    uint32_t qi[U];
                    float qv[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t i = i0 + (uint32_t)(u * NT);
                        const uint32_t e = i < len ? i : len - 1u;
                        qi[u] = a.idx[beg + e];
                        qv[u] = a.val[beg + e];
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t off = qi[u] - (uint32_t)base;
                        if (i0 + (uint32_t)(u * NT) < len && off < (uint32_t)TILE) s_acc[off] = __fadd_rn(s_acc[off], qv[u]);
                    }
                }
                __syncthreads();
            }
        }
    }
    // Whole tiles leave 16 bytes a thread, at any alignment of the vectors, but not dense updates that are all the launch moves: past some 4e7 entries few short messages
    // make it a fill, which 4 bytes a thread write faster.  us, 4 bytes / 16, out only, `per` message entries of all rows per tile: 2e7 entries, 1 or 8 rows, any per,
    // 16.3 / 14.9 and 19.5 / 18.7; 4e7, 2 or 4 rows, per 8 to 300, 27.6 to 31 / 27.6 to 30; 1 row of 6e7, 192 39.3 / 41.1, 384 44.3 / 41.1, of 1.24e8, 75.7 / 86.2 and
    // 84.1 / 80.4; 2 rows of 6e7, 8 to 128 39.6 / 42.6, 300 42.1 / 39.5, of 1.24e8, 384 78.5 / 81.7, 1024 120 / 112; 4 of 6e7, 8 41.2 / 42.6, 96 43.9 / 41.7, of 1.24e8, 8
    // 77.6 / 88.1, 300 83.3 / 85.9, 1024 118 / 113; 5 of 9e7, 70 64.7 / 60.5; 8 of 1.24e8, 8 84.6 / 86.3, 64 96.8 / 86.1; 16, 8 106 / 86.  With the update 1 of 1e7
    // 20.2 / 14.6, of 2e8 403 / 284, of 1e6 as fast.
    // Decided here: at the start of the kernel it cost 1 % at 16 rows of 2.56e7 and 256 of 131072.
    const bool beyond = a.ntiles > 16384;
    const int64_t per = a.M >= (beyond ? 5 : 4) ? 64 : beyond && a.M > 1 ? 512 : 256;
    const bool wide = base + TILE <= a.d && (a.x || a.ntiles <= 10240 || a.M >= 8 || a.row_off[a.M] >= per * a.ntiles);   // uniform
    if (wide) {
        for (int i = threadIdx.x; i < TILE / 4; i += NT) finish_four(a.alpha, ((const float4*)s_acc)[i], a.out, a.eta, a.x, base + 4 * i);
    } else {
        // Two forms of one loop: with the end of the row as its bound it is not unrolled, which a fill likes (2 rows of 1.24e8, 8 entries a tile, 76.5, unrolled 87.9), other launches
        // do not (4 rows, 96, 86.8 and 82.7).
        if (a.M <= 3) {   // uniform
            for (int i = threadIdx.x; i < TILE && base + i < a.d; i += NT) finish_entry(a.alpha, s_acc[i], a.out, a.eta, a.x, base + i);
        } else {
            for (int i = threadIdx.x; i < TILE; i += NT) {
                const int64_t j = base + i;
                if (j < a.d) finish_entry(a.alpha, s_acc[i], a.out, a.eta, a.x, j);
            }
        }
    }
}

// Bits that name one of n alternatives.
__device__ __forceinline__ int ceil_log2_dev(int64_t n) { return n <= 1 ? 0 : 64 - __clzll((unsigned long long)(n - 1)); }

// Bits every worker's message takes on the wire.  Rank bands (Sec. 3, Sec. 3.2): every entry as a 32-bit value and an
// index into d, plus the level.  Fixed-point ladder (Sec. 3.1): per entry the sign, the base bits and the bits of
// the level field, plus the 32-bit scale exponent and the level.
struct MsgBitsArgs {
    int32_t kind, M, L;
    int64_t d, s;
    int64_t ladder[TMAX];
    const int32_t* level;
    unsigned long long* bits;
};
__global__ __launch_bounds__(256) void k_message_bits(MsgBitsArgs a) {
    __shared__ int64_t s_lad[TMAX];
    if (a.kind != MLMC_STOPK && (int)threadIdx.x <= a.L) s_lad[threadIdx.x] = a.ladder[threadIdx.x];
    __syncthreads();
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= a.M) return;
    int lev = a.level[r];
    lev = lev < 1 ? 1 : (lev > a.L ? a.L : lev);
    unsigned long long n;
    if (a.kind == MLMC_STOPK) {   // the drawn segment: s entries, the last one what is left
        const int64_t lo = (int64_t)(lev - 1) * a.s;
        const int64_t cnt = lo + a.s < a.d ? a.s : a.d - lo;
        a.bits[r] = (unsigned long long)cnt * (unsigned long long)(32 + ceil_log2_dev(a.d)) + (unsigned long long)ceil_log2_dev(a.L);
        return;
    }
    const int64_t width = s_lad[lev] - s_lad[lev - 1];
    if (a.kind == MLMC_TOPK) n = (unsigned long long)(s_lad[0] + width) * (unsigned long long)(32 + ceil_log2_dev(a.d));
    else if (a.kind == MLMC_FBITS) n = (unsigned long long)a.d * (unsigned long long)(9 + s_lad[0] + width);
    else if (a.kind == MLMC_RTN) n = (unsigned long long)a.d * (unsigned long long)(s_lad[0] + (lev > 1 ? s_lad[lev - 1] : 0) + s_lad[lev]) + 64ull;
    else n = (unsigned long long)a.d * (unsigned long long)(1 + s_lad[0] + width) + 32ull;
    a.bits[r] = n + (unsigned long long)ceil_log2_dev(a.L);
}

mlmc_status message_bits(const mlmc_plan_t* pl, const int32_t* level, unsigned long long* bits, hipStream_t st) {
    MsgBitsArgs a;
    a.kind = pl->kind;
    a.M = pl->M;
    a.L = pl->L;
    a.d = pl->d;
    a.s = pl->s;
    if (pl->kind != MLMC_STOPK)
        for (int t = 0; t <= pl->L; ++t) a.ladder[t] = pl->ladder[t];
    a.level = level;
    a.bits = bits;
    MLMC_LAUNCH(K_MSGBITS, st, k_message_bits<<<(pl->M + 255) / 256, 256, 0, st>>>(a));
    return MLMC_OK;
}

// ---------------------------------------------------------------------------------------------------
// By words while that many waves still find room, which is up to other sizes for rows with a ragged last block, whose entries the blocks' kernel loads one by one (some 3 us),
// and for rows of whole blocks.  compress, us, 2048 entries a wave / words (graph replay).
// Ragged, fixed point: 4 rows of 100003 10.4 / 6.5, 128 of 12287 11.1 / 8.0 (16 bits 10.9 / 8.4), 1 of 1572863 11.2 / 7.6; largest entry 8 of 196607 11.7 / 7.4; floating point (up to
// 32 planes) 8 of 196607 11.3 / 9.3, 600 of 2049 10.7 / 10.6 (16 bits 10.9 / 10.9).
// Whole, fixed point: 1 of 16384 6.8 / 6.2, 4 of 262144 7.7 / 6.6, 1 of 1572864 7.8 / 7.6, 32 of 32768 7.4 / 7.2, but 32 of 49152 7.4 / 7.5, 128 of 2048 6.9 / 7.0 and of 8192 7.1 / 7.5; 16 bits 4 of 262144
// 7.1 / 6.9, 8 of 131072 7.0 / 7.0, 4 of 393216 7.1 / 7.4, 32 of 16384 6.9 / 7.3; largest entry the same to a tenth; floating point 1 of 16384 7.0 / 7.8, 4 of 262144 7.7 / 8.5.
static bool extract_by_words(const mlmc_plan_t* pl, const BitsArgs& a) {
    if (a.sample_shift != 0) return false;
    const int64_t all = (int64_t)pl->M * pl->d;
    if (pl->d % EX_ELEMS) return all <= 3 << 19;
    const bool f32 = pl->dtype == MLMC_F32;
    return !a.flt && pl->M <= (f32 ? 32 : 8) && all <= (f32 && pl->M <= 8 ? 3 << 19 : 1 << 20);
}
mlmc_status bits_compress(const mlmc_plan_t* pl, const BitsArgs& a0, hipStream_t st) {
    BitsArgs a = a0;
    if (a.flt) MLMC_LAUNCH(K_DRAW, st, k_bits_prep<<<1, 1024, 0, st>>>(a));
    const dim3 egrid = extract_grid(pl);
    const bool words = extract_by_words(pl, a);
    const dim3 wgrid((unsigned)((a.nwords + EW_WORDS * (EX_THREADS / 64) - 1) / (EW_WORDS * (EX_THREADS / 64))), pl->M);
#define MLMC_EXTRACT_B(ID, DT, REDO, KIND)                                                                               \
    do {                                                                                                                \
        if (words && a.F[0] == 0) MLMC_LAUNCH(K_BITS_WORDS, st, k_bits_extract_words<DT, KIND, false><<<wgrid, EX_THREADS, 0, st>>>(a)); \
        else if (words) MLMC_LAUNCH(K_BITS_WORDS, st, k_bits_extract_words<DT, KIND, true><<<wgrid, EX_THREADS, 0, st>>>(a));      \
        else if (a.F[0] == 0) MLMC_LAUNCH(ID, st, k_bits_extract<DT, REDO, KIND, false><<<egrid, EX_THREADS, 0, st>>>(a));    \
        else MLMC_LAUNCH(ID, st, k_bits_extract<DT, REDO, KIND, true><<<egrid, EX_THREADS, 0, st>>>(a));                 \
    } while (0)
#define MLMC_EXTRACT(ID, REDO, KIND)                                                                                     \
    do {                                                                                                                \
        if (pl->dtype == MLMC_F32) MLMC_EXTRACT_B(ID, MLMC_F32, REDO, KIND);                                             \
        else MLMC_EXTRACT_B(ID, MLMC_BF16, REDO, KIND);                                                                  \
    } while (0)
    if (a.flt) {
        // floating-point ladder (App. B): no scale, so nothing to find before the one read
        MLMC_EXTRACT(K_BITS_EXTRACT, false, 1);
        return MLMC_OK;
    }
    // sampled (or, for short rows, exact) row maxima
    const int64_t nblk = (pl->d + 1023) / 1024;
    const int64_t ns = (nblk >> a.sample_shift) > 0 ? (nblk >> a.sample_shift) : 1;
    int64_t sw = (ns + 7) / 8;   // a block per wave, up to four workgroups of eight waves on every CU
    const int64_t scap = 1024 / pl->M > 0 ? 1024 / pl->M : 1;
    if (sw > scap) sw = scap;
    if (sw < 1) sw = 1;
    const dim3 sgrid((unsigned)sw, pl->M);
    // the first launch of the call: its workgroups leave one maximum each (nothing to clear beforehand) and draw the levels
    static_assert(1024 <= SMAX_PARTS_MAX, "sw is at most 1024");
    a.smax_parts = (int32_t)sw;
    if (pl->dtype == MLMC_F32) MLMC_LAUNCH(K_BITS_MAX, st, k_bits_smax<MLMC_F32, true><<<sgrid, SMAX_THREADS, 0, st>>>(a));
    else MLMC_LAUNCH(K_BITS_MAX, st, k_bits_smax<MLMC_BF16, true><<<sgrid, SMAX_THREADS, 0, st>>>(a));
    if (a.vmx) {   // the maxima above are exact (every block was read): one extraction
        MLMC_EXTRACT(K_BITS_EXTRACT, false, 2);
        return MLMC_OK;
    }
    MLMC_EXTRACT(K_BITS_EXTRACT, false, 0);
    if (a.sample_shift > 0) MLMC_EXTRACT(K_BITS_REDO, true, 0);   // rows whose sampled maximum fell short (returns at once for the others)
#undef MLMC_EXTRACT
#undef MLMC_EXTRACT_B
    return MLMC_OK;
}

mlmc_status agg_bits(const mlmc_plan_t* pl, const BitsArgs& b, const int32_t* level, const int32_t* scale_exp,
                     const uint64_t* planes, float alpha, float* out, float eta, float* x, hipStream_t st) {
    AggBitsArgs a;
    a.b = b;
    a.level = level;
    a.scale_exp = scale_exp;
    a.alpha = alpha;
    a.eta = eta;
    const int64_t nblk = (b.d + EX_ELEMS - 1) / EX_ELEMS;
    const unsigned grid = (unsigned)((nblk + EX_THREADS / 64 - 1) / (EX_THREADS / 64));
    const size_t lds = (size_t)(EX_THREADS / 64) * EX_ELEMS * 4 + sizeof(AggRow) * (size_t)b.M;
    // By words: the rows come one after the other either way, so their length decides, and whether it leaves the blocks' kernel a ragged block (some 3 us).  us, 2048 entries a
    // wave / words (graph replay).  Ragged, fixed point: 4 rows of 100003 7.5 / 3.6, 1 of 524287 6.5 / 4.5, 32 of 524287 24.4 / 19.6, but 8 of 1000001 9.1 / 11.3; floating point 32 of
    // 100003 32.0 / 18.2, 1 of 262143 6.8 / 3.7, 32 of 262143 32.7 / 26.0; Round-to-Nearest (all planes of the widest message are loaded, whatever was sent) 32 of 100003 32.1 / 14.4,
    // 1 of 262143 6.6 / 4.1, 32 of 262143 34.2 / 28.6.  Whole: fixed point 1 of 262144 3.8 / 3.4, 2 of 393216 4.4 / 4.7, 1 of 524288 3.8 / 4.3, 4 of 524288 5.5 / 5.8, 8 of 524288 7.8 / 7.7,
    // 32 of 524288 22.2 / 19.5; floating point 1 of 262144 4.0 / 3.7, 32 30.2 / 25.9; Round-to-Nearest 1 of 196608 4.0 / 3.4, 1 of 262144 4.0 / 4.1 (equal probabilities 4 of 262144
    // 7.3 / 7.7), 8 of 262144 10.3 / 9.4.
    int64_t longest = b.flt || b.rtn ? 1 << 18 : 1 << 19;
    if (b.d % EX_ELEMS == 0 && b.M < 8 && !b.flt) longest = b.rtn ? 3 << 16 : 1 << 18;
    const bool words = b.d <= longest;
    const unsigned wgrid = (unsigned)((b.nwords + EX_THREADS / 64 - 1) / (EX_THREADS / 64));
    const size_t wlds = sizeof(AggRow) * (size_t)b.M;
#define MLMC_AGG(PK)                                                                                                     \
    do {                                                                                                                \
        if (words && b.F[0] == 0) MLMC_LAUNCH(K_AGG_WORDS, st, k_agg_words<PK, false><<<wgrid, EX_THREADS, wlds, st>>>(a, planes, out, x)); \
        else if (words) MLMC_LAUNCH(K_AGG_WORDS, st, k_agg_words<PK, true><<<wgrid, EX_THREADS, wlds, st>>>(a, planes, out, x)); \
        else if (b.F[0] == 0) MLMC_LAUNCH(K_AGG_BITS, st, k_agg_planes<PK, false><<<grid, EX_THREADS, lds, st>>>(a, planes, out, x)); \
        else MLMC_LAUNCH(K_AGG_BITS, st, k_agg_planes<PK, true><<<grid, EX_THREADS, lds, st>>>(a, planes, out, x));       \
    } while (0)
    if (b.rtn) MLMC_AGG(2);
    else if (b.flt) MLMC_AGG(1);
    else MLMC_AGG(0);
#undef MLMC_AGG
    return MLMC_OK;
}

// Threads of a tile, by the tiles and the mean entries of a row in one (adaptive plans: every level as likely as the next).
static int agg_threads(const mlmc_plan_t* pl) {
    double mean = 0.0;
    if (pl->kind == MLMC_STOPK) {
        mean = (double)pl->s;
    } else {
        mean = (double)pl->ladder[0];
        for (int l = 1; l <= pl->L; ++l) mean += (pl->adaptive ? 1.0 / pl->L : pl->p[l - 1]) * (double)(pl->ladder[l] - pl->ladder[l - 1]);
    }
    const bool short_rows = mean < 192.0 * (double)pl->ntiles;
    if (pl->ntiles <= 256) return short_rows && pl->M > 32 ? 512 : 1024;
    if (pl->ntiles <= 512) return 512;
    if (pl->ntiles <= 1024) return short_rows && pl->M >= 16 ? 256 : 512;
    return 256;
}

mlmc_status agg_sparse(const mlmc_plan_t* pl, const int64_t* row_off, const uint32_t* idx, const float* val, int64_t capacity,
                       const uint32_t* tile_off, uint32_t* tile_off_ws, float alpha, float* out, float eta, float* x,
                       hipStream_t st) {
    AggSparseArgs a;
    a.M = pl->M;
    a.d = pl->d;
    a.ntiles = pl->ntiles;
    a.row_off = row_off;
    a.idx = idx;
    a.val = val;
    a.capacity = capacity;
    a.tile_off = tile_off;
    a.tile_off_out = tile_off_ws;
    a.alpha = alpha;
    a.out = out;
    a.eta = eta;
    a.x = x;
    if (!tile_off) {
        int64_t n = (int64_t)pl->M * (pl->ntiles + 1);
        int blocks = (int)((n + 255) / 256);
        if (blocks > 4096) blocks = 4096;
        MLMC_LAUNCH(K_TILEOFF, st, k_tileoff<<<blocks, 256, 0, st>>>(a));
        a.tile_off = tile_off_ws;
    }
    const size_t lds = TILE * sizeof(float) + (size_t)pl->M * (sizeof(int64_t) + sizeof(uint32_t));
    const unsigned grid = (unsigned)pl->ntiles;
    const int nt = agg_threads(pl);
    if (nt == 1024) MLMC_LAUNCH(K_AGG_SPARSE, st, k_agg_sparse<1024><<<grid, 1024, lds, st>>>(a));
    else if (nt == 512) MLMC_LAUNCH(K_AGG_SPARSE, st, k_agg_sparse<512><<<grid, 512, lds, st>>>(a));
    else MLMC_LAUNCH(K_AGG_SPARSE, st, k_agg_sparse<256><<<grid, 256, lds, st>>>(a));
    return MLMC_OK;
}

}  // namespace mlmc
