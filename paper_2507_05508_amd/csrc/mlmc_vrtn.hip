// Round-to-Nearest MLMC (Sec. 3.3, App. G.2) on gfx950.
#include "mlmc_count16.h"
#include "mlmc_extract.h"

namespace mlmc {

// ---------------------------------------------------------------------------------------------------
// Round-to-Nearest MLMC.  k_rtn_prep clears the per-row state; k_bits_smax (every block) finds c; k_rtn_norms sums
// the squared residual integers of every level; k_rtn_draw turns them into norms, probabilities, the draw and the
// coefficient; k_rtn_extract writes the planes of the drawn message's codes.
static_assert(RTN_LMAX == 8, "launch_rtn_norms");
__global__ __launch_bounds__(256) void k_rtn_prep(BitsArgs a) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t == 0) *a.dev_status = 0;
    if (t < a.M) {
        a.racc[t].rowmax_key = 0u;
        a.racc[t].smpmax_key = 0u;
    }
    if (t < a.M * a.L * 2) a.rtn_sums[t] = 0ull;
}

// a uniform double in scalar registers
__device__ __forceinline__ double uniform_f64(double v) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)), __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ __forceinline__ uint32_t mul_u24(uint32_t a, uint32_t b) {   // of the low 24 bits
    uint32_t r;
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ uint32_t mad_u24(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Sums of squared residual integers, LV levels.  k_l = n_l D' - n_{l-1} D, so sum k_l^2 = D'^2 sum n_l^2 - 2 D D' sum n_l n_{l-1}
// + D^2 sum n_{l-1}^2: per entry and level two products of codes below 2^15 (signs cancel in them), 24-bit multiply-adds that
// meet in 32 bits for as many entries as fit, then in 64.  A code is the low word of |g| fl(D / 2c) + 1.5 2^52, formed with
// the multiplier moved towards and away from zero as in k_rtn_extract; where the two differ it is the even one.  Bound
// by instruction issue: with every code and residual in fp64 the kernel took 172 us for 8 rows of 1.17e7 at four levels, now 100
// (the bare read: 59).  Eight entries at a time and four waves per SIMD; sixteen, or two waves, took 10 % longer.
// CHAIN: every width of the ladder divides the widest, so D_L / D_l is an odd integer q and a code is rne(n_L / q): a boundary between
// two codes of level l is a half-integer in units of the widest level's, which n_L keeps the side of.  Where the entry lies on it, it ties at both levels:
// q = 1 (mod 4) for widths of two or more, so that the even n_L lies on the side of the even n_l.  Width 1 has q = 3 (mod 4) but one
// boundary only, at the largest entry: n_L / q stays below 1/2 and all its codes are zero, as the cut ones are.  One multiply-add
// per code instead of two and their comparison; n_L cut is n_l cut.
// With that and the next sixteen entries in flight 8 rows of 1.17e7 entries take 78 us (100 before, 82 with the multiply-adds alone), 4 of 4e7 133 (173), 8 of
// 1e6 17.5 (18.4); read past the cache it is no faster and the extraction behind it 8 us slower.
template <int DT, int LV, bool CHAIN>
__global__ __launch_bounds__(256, LV <= 4 ? 4 : 2) void k_rtn_norms(BitsArgs a) {
    const int row = blockIdx.y;
    const uint32_t ckey = a.racc[row].smpmax_key;
    if (ckey == 0u) return;   // a zero row: every residual is zero
    const double den = 2.0 * key_to_double(ckey);
    RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    double mul_in[LV + 1], mul_out[LV + 1];
#pragma unroll
    for (int t = 0; t <= LV; ++t) {
        const double mul = a.F[t] > 0 ? __ddiv_rn((double)((1 << a.F[t]) - 1), den) : 0.0;
        mul_in[t] = uniform_f64(__dmul_rn(mul, 1.0 - 0x1p-44));
        mul_out[t] = uniform_f64(__dmul_rn(mul, 1.0 + 0x1p-44));
    }
    double inv_q[LV];   // D_t / D_LV
    if (CHAIN) {
#pragma unroll
        for (int t = 0; t < LV; ++t) inv_q[t] = uniform_f64(__ddiv_rn((double)((1 << a.F[t]) - 1), (double)((1 << a.F[LV]) - 1)));
    }
    unsigned long long sqr[LV + 1], prod[LV + 1];   // sum n_t^2, sum n_t n_{t-1}
#pragma unroll
    for (int t = 0; t <= LV; ++t) { sqr[t] = 0; prod[t] = 0; }
    // x . y over eight entries, products of `bits` bits at most
    auto dot = [](const uint32_t (&x)[8], const uint32_t (&y)[8], int bits, unsigned long long& sum) {
        if (bits <= 29) {   // uniform
            uint32_t s = mul_u24(x[0], y[0]);
#pragma unroll
            for (int i = 1; i < 8; ++i) s = mad_u24(x[i], y[i], s);
            sum += s;
        } else {
#pragma unroll
            for (int q = 0; q < 8; q += 4)
                sum += mad_u24(x[q], y[q], mad_u24(x[q + 1], y[q + 1], mad_u24(x[q + 2], y[q + 2], mul_u24(x[q + 3], y[q + 3]))));
        }
    };
    auto batch_each = [&](const uint32_t* b) {
        double av[8];
        uint32_t prev[8], cur[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            av[i] = (double)fabsf(__uint_as_float(b[i]));
            prev[i] = 0;
        }
#pragma unroll
        for (int t = 0; t <= LV; ++t) {
            if (t == 0 && a.F[0] == 0) continue;   // uniform: no base code
            uint32_t differ = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                cur[i] = (uint32_t)__double2loint(__fma_rn(av[i], mul_in[t], 0x1.8p52));
                differ |= cur[i] ^ (uint32_t)__double2loint(__fma_rn(av[i], mul_out[t], 0x1.8p52));
            }
            if (__ballot(differ != 0u) != 0ull) {   // a tie: the even one; the largest entry's code is cut
                const uint32_t N = (1u << (a.F[t] - 1)) - 1u;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t out = (uint32_t)__double2loint(__fma_rn(av[i], mul_out[t], 0x1.8p52));
                    cur[i] = cur[i] & 1u ? out : cur[i];
                    cur[i] = cur[i] < N ? cur[i] : N;
                }
            }
            dot(cur, cur, 2 * a.F[t] - 2, sqr[t]);
            if (t > 0 && a.F[t - 1] > 0) dot(cur, prev, a.F[t] + a.F[t - 1] - 2, prod[t]);
#pragma unroll
            for (int i = 0; i < 8; ++i) prev[i] = cur[i];
        }
    };
    auto batch_chain = [&](const uint32_t* b) {
        double n[8];   // the widest level's codes
        uint32_t up[8], differ = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const double av = (double)fabsf(__uint_as_float(b[i])), in = __fma_rn(av, mul_in[LV], 0x1.8p52);
            up[i] = (uint32_t)__double2loint(in);
            n[i] = __dsub_rn(in, 0x1.8p52);
            differ |= up[i] ^ (uint32_t)__double2loint(__fma_rn(av, mul_out[LV], 0x1.8p52));
        }
        if (__ballot(differ != 0u) != 0ull) {   // a tie: the even one; the largest entry's code is cut
            const uint32_t N = (1u << (a.F[LV] - 1)) - 1u;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t out = (uint32_t)__double2loint(__fma_rn((double)fabsf(__uint_as_float(b[i])), mul_out[LV], 0x1.8p52));
                up[i] = up[i] & 1u ? out : up[i];
                up[i] = up[i] < N ? up[i] : N;
                n[i] = (double)up[i];
            }
        }
        dot(up, up, 2 * a.F[LV] - 2, sqr[LV]);
#pragma unroll
        for (int t = LV - 1; t >= 0; --t) {
            if (t == 0 && a.F[0] == 0) continue;   // uniform: no base code
            uint32_t low[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) low[i] = (uint32_t)__double2loint(__fma_rn(n[i], inv_q[t], 0x1.8p52));
            dot(low, low, 2 * a.F[t] - 2, sqr[t]);
            dot(up, low, a.F[t + 1] + a.F[t] - 2, prod[t + 1]);
#pragma unroll
            for (int i = 0; i < 8; ++i) up[i] = low[i];
        }
    };
    auto batch = [&](const uint32_t* b) {
        if constexpr (CHAIN) batch_chain(b);
        else batch_each(b);
    };
    // groups of four elements, four loads of a thread in flight
    const int64_t nq = (a.d + 3) / 4, qstride = (int64_t)gridDim.x * 256;
    int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    auto fetch = [&](int64_t at, uint32_t (&b)[16]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint32_t v[4];
            ld.load4_full((at + u * qstride) * 4, v);
#pragma unroll
            for (int e = 0; e < 4; ++e) b[4 * u + e] = v[e];
        }
    };
    auto whole = [&](int64_t at) -> bool { return at + 3 * qstride < nq - 1; };   // none of the four is the row's last (possibly partial) group
    uint32_t b[16];
    if (ckey >= 0x7F800000u) {   // uniform: Inf and NaN are the numbers their bit patterns spell, as in c; entry by entry
        for (; q < nq; q += qstride) {
            uint32_t v[4];
            const int nv = ld.load4(q * 4, v);
#pragma unroll 1
            for (int e = 0; e < nv; ++e) {
                const double av = key_to_double(key_of_bits(e == 0 ? v[0] : e == 1 ? v[1] : e == 2 ? v[2] : v[3]));
                uint32_t prev = 0;
#pragma unroll
                for (int t = 0; t <= LV; ++t) {
                    const uint32_t N = a.F[t] > 0 ? (1u << (a.F[t] - 1)) - 1u : 0u, in = (uint32_t)__double2loint(__fma_rn(av, mul_in[t], 0x1.8p52));
                    uint32_t cur = in & 1u ? (uint32_t)__double2loint(__fma_rn(av, mul_out[t], 0x1.8p52)) : in;
                    cur = cur < N ? cur : N;
                    sqr[t] += cur * cur;
                    if (t > 0) prod[t] += cur * prev;
                    prev = cur;
                }
            }
        }
    }
    if (whole(q)) {
        fetch(q, b);
        for (bool more = true; more; q += 4 * qstride) {
            more = whole(q + 4 * qstride);
            uint32_t next[16];
            fetch(more ? q + 4 * qstride : q, next);   // the last one again: a load without a condition
            batch(b);
            batch(b + 8);
#pragma unroll
            for (int i = 0; i < 16; ++i) b[i] = next[i];
        }
    }
    for (; q < nq; q += 4 * qstride) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            uint32_t v[4] = {0, 0, 0, 0};
            if (q + u * qstride < nq) ld.load4((q + u * qstride) * 4, v);   // past the end: +0, whose codes are 0
#pragma unroll
            for (int e = 0; e < 4; ++e) b[4 * u + e] = v[e];
        }
        batch(b);
        batch(b + 8);
    }
    // One pair of global atomics per workgroup and level (atomics of many waves on one address take turns): the waves'
    // sums meet in LDS first.
    __shared__ unsigned long long s_part[4][LV];
    const uint32_t wave = threadIdx.x >> 6;
#pragma unroll
    for (int l = 1; l <= LV; ++l) {
        const unsigned long long D = (1ull << a.F[l]) - 1, Dp = a.F[l - 1] > 0 ? (1ull << a.F[l - 1]) - 1 : 1ull;
        // modulo 2^64; the result, a sum of at most 2^16 squares below 2^36, is smaller
        unsigned long long v = Dp * Dp * sqr[l] - 2ull * D * Dp * prod[l] + D * D * sqr[l - 1];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane_id() == 0) s_part[wave][l - 1] = v;
    }
    __syncthreads();
    if ((int)threadIdx.x < LV) {
        const int l = threadIdx.x;
        const unsigned long long v = s_part[0][l] + s_part[1][l] + s_part[2][l] + s_part[3][l];   // < 2^60: no overflow
        if (v) {
            atomicAdd(&a.rtn_sums[((size_t)row * LV + l) * 2], v & 0xFFFFFFFFull);
            atomicAdd(&a.rtn_sums[((size_t)row * LV + l) * 2 + 1], v >> 32);
        }
    }
}
template <int DT, bool CHAIN>
static void launch_rtn_norms(int L, dim3 grid, hipStream_t st, const BitsArgs& a) {
    switch (L) {
        case 1: k_rtn_norms<DT, 1, CHAIN><<<grid, 256, 0, st>>>(a); break;
        case 2: k_rtn_norms<DT, 2, CHAIN><<<grid, 256, 0, st>>>(a); break;
        case 3: k_rtn_norms<DT, 3, CHAIN><<<grid, 256, 0, st>>>(a); break;
        case 4: k_rtn_norms<DT, 4, CHAIN><<<grid, 256, 0, st>>>(a); break;
        case 5: k_rtn_norms<DT, 5, false><<<grid, 256, 0, st>>>(a); break;
        case 6: k_rtn_norms<DT, 6, false><<<grid, 256, 0, st>>>(a); break;
        case 7: k_rtn_norms<DT, 7, false><<<grid, 256, 0, st>>>(a); break;
        default: k_rtn_norms<DT, 8, false><<<grid, 256, 0, st>>>(a); break;
    }
}
template <int DT>
static void launch_rtn_norms(int L, dim3 grid, hipStream_t st, const BitsArgs& a) {
    // with five levels or more (1, 2, 4, 8, 16 behind a base of 0; 1, 2, 3, 4, 6, 12) the way without it, whatever the widths
    bool chain = true;
    for (int t = 0; t < L; ++t) chain = chain && (a.F[t] == 0 || a.F[L] % a.F[t] == 0);
    if (chain) launch_rtn_norms<DT, true>(L, grid, st, a);
    else launch_rtn_norms<DT, false>(L, grid, st, a);
}

// 16-bit rows that are long enough: a row has at most 2^15 magnitudes, so one read that counts them (in LDS, one 32-bit atomic
// per entry) gives the largest entry and, a code per magnitude instead of one per entry, the exact sums: k_bits_smax and
// k_rtn_norms, two reads and the codes of every entry, took 154 + 440 us for 4 rows of 1.24e8 (773 before).
__global__ __launch_bounds__(C16_THREADS) void k_rtn_hist(BitsArgs a) {
    __shared__ __align__(16) uint32_t s_h[C16_LDS];
    const int row = blockIdx.y;
    const int64_t i0 = (int64_t)blockIdx.x * a.rtn_slice, i1 = i0 + a.rtn_slice < a.d ? i0 + a.rtn_slice : a.d;
    count16_slice<false>((const uint16_t*)a.g + (int64_t)row * a.ld, i0, i1, s_h, C16Window{}, nullptr);
    uint4* part = (uint4*)(a.rtn_part + ((size_t)row * gridDim.x + blockIdx.x) * C16_KEYS);
    for (int i = threadIdx.x; i < C16_KEYS / 4; i += C16_THREADS) part[i] = ((const uint4*)s_h)[i];
}
// Totals over the workgroups and the largest magnitude.
__global__ __launch_bounds__(256) void k_rtn_hmax(BitsArgs a, int wgs) {
    const int row = blockIdx.y;
    const uint32_t k = blockIdx.x * 256 + threadIdx.x;
    const uint32_t* p = a.rtn_part + (size_t)row * wgs * C16_KEYS + k;
    uint32_t n = 0;
#pragma unroll 8
    for (int g = 0; g < wgs; ++g) n += p[(size_t)g * C16_KEYS];
    a.rtn_total[(size_t)row * C16_KEYS + k] = n;
    const uint32_t m = wave_max(n ? k << 16 : 0u);
    if (m && lane_id() == 0) atomicMax(&a.racc[row].smpmax_key, m);
}
// A magnitude's residual integers, times how often it occurs.
__global__ __launch_bounds__(256) void k_rtn_hsum(BitsArgs a) {
    __shared__ unsigned long long s_lo[RTN_LMAX], s_hi[RTN_LMAX];
    const int row = blockIdx.y;
    const uint32_t ckey = a.racc[row].smpmax_key;
    if (ckey == 0u) return;   // a zero row: every residual is zero
    const uint32_t key = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x * 256u > ckey >> 16) return;   // uniform: no such magnitudes
    const double c = key_to_double(ckey), den = 2.0 * c, inv_den = __ddiv_rn(1.0, den);
    if (threadIdx.x < RTN_LMAX) { s_lo[threadIdx.x] = 0ull; s_hi[threadIdx.x] = 0ull; }
    __syncthreads();
    const unsigned long long n = a.rtn_total[(size_t)row * C16_KEYS + key];
    if (n) {
        const double x = key_to_double(key << 16);
        long long prev = a.F[0] > 0 ? rtn_code_abs(x, rtn_code_of(a.F[0]), c, den, inv_den) : 0;
        for (int l = 1; l <= a.L; ++l) {
            const long long D = (1ll << a.F[l]) - 1, Dp = a.F[l - 1] > 0 ? (1ll << a.F[l - 1]) - 1 : 1ll;
            const long long cur = rtn_code_abs(x, rtn_code_of(a.F[l]), c, den, inv_den), r = cur * Dp - prev * D;
            const unsigned long long sq = (unsigned long long)(r * r);   // < 2^36; n < 2^31: the product in two parts
            const unsigned long long lo = (sq & 0xFFFFFFFFull) * n, hi = (sq >> 32) * n + (lo >> 32);
            if (lo) atomicAdd(&s_lo[l - 1], lo & 0xFFFFFFFFull);
            if (hi) atomicAdd(&s_hi[l - 1], hi);
            prev = cur;
        }
    }
    __syncthreads();
    const int l = threadIdx.x;
    if (l < a.L) {
        if (s_lo[l]) atomicAdd(&a.rtn_sums[((size_t)row * a.L + l) * 2], s_lo[l]);
        if (s_hi[l]) atomicAdd(&a.rtn_sums[((size_t)row * a.L + l) * 2 + 1], s_hi[l]);
    }
}

// Per row (one thread each): Delta_l = (2c / (D D')) sqrt(S_l), S_l the integer sum converted to fp64 once;
// probabilities (Lemma 3.4, or the plan's), the draw (Alg. 2 / Alg. 3), level, c and the coefficient.
__global__ __launch_bounds__(64) void k_rtn_draw(BitsArgs a, int norms_only) {
    __shared__ double s_p[64][RTN_LMAX];
    __shared__ uint32_t s_big[64][20];
    const int row = blockIdx.x * 64 + threadIdx.x;
    if (row >= a.M) return;
    const int L = a.L;
    const uint32_t ckey = a.racc[row].smpmax_key;
    if (ckey >= 0x7F800000u) atomicOr(a.dev_status, MLMC_DEV_NONFINITE);
    const double c = key_to_double(ckey);
    double* p = s_p[threadIdx.x];
    double factor[RTN_LMAX];
#pragma unroll
    for (int l = 0; l < RTN_LMAX; ++l) factor[l] = 0.0;
    for (int l = 1; l <= L; ++l) {
        const unsigned long long lo = a.rtn_sums[((size_t)row * L + (l - 1)) * 2], hi = a.rtn_sums[((size_t)row * L + (l - 1)) * 2 + 1];
        // S = hi 2^32 + lo as 32-bit words
        uint32_t* w = s_big[threadIdx.x];
        for (int i = 0; i < 20; ++i) w[i] = 0u;
        const unsigned long long w1 = (lo >> 32) + (hi & 0xFFFFFFFFull);
        w[0] = (uint32_t)lo;
        w[1] = (uint32_t)w1;
        const unsigned long long w2 = (w1 >> 32) + (hi >> 32);
        w[2] = (uint32_t)w2;
        w[3] = (uint32_t)(w2 >> 32);
        BigAcc big;
        big.w = w;
        const double Sd = ldexp(big.to_double(), 298);
        const double D = (double)((1 << a.F[l]) - 1), Dp = a.F[l - 1] > 0 ? (double)((1 << a.F[l - 1]) - 1) : 1.0;
        const double f = __ddiv_rn(__dmul_rn(2.0, c), __dmul_rn(D, Dp));
        const double nrm = __dmul_rn(f, __dsqrt_rn(Sd));
#pragma unroll
        for (int q = 0; q < RTN_LMAX; ++q) if (q == l - 1) factor[q] = f;
        p[l - 1] = nrm;
        a.norms[(size_t)row * L + (l - 1)] = nrm;
        if (a.norms_user) a.norms_user[(size_t)row * L + (l - 1)] = nrm;
    }
    if (norms_only) return;
    if (a.adaptive) {
        double tot = 0.0;
        for (int l = 0; l < L; ++l) tot = __dadd_rn(tot, p[l]);
        for (int l = 0; l < L; ++l) p[l] = tot == 0.0 ? __ddiv_rn(1.0, (double)L) : __ddiv_rn(p[l], tot);
    } else {
        for (int l = 0; l < L; ++l) p[l] = a.p_fixed[l];
    }
    const uint32_t x = philox_word0(a.seed, a.step, (uint32_t)row);
    const int level = draw_from_p(p, L, x);
    const double pl = p[level - 1];
    double f = 0.0;
#pragma unroll
    for (int q = 0; q < RTN_LMAX; ++q) if (q == level - 1) f = factor[q];
    a.rinfo[row].level = level;
    a.rinfo[row].draw_x = x;
    a.level[row] = level;
    a.scale_exp[2 * row] = (int32_t)ckey;
    a.scale_exp[2 * row + 1] = (int32_t)__float_as_uint(pl == 0.0 ? 0.0f : (float)__ddiv_rn(f, pl));
}

struct RtnPlaneCode {    // one of the (up to three) codes of a row's message
    double mul_in, mul_out;   // D / 2c, moved towards and away from zero
    RtnCode code;
};
// Code planes of the drawn message.  A code n = rne(a D / 2c) comes from one fused multiply-add: a * fl(D / 2c) plus
// 1.5 2^52 leaves the rounded integer, sign included, in the low word.  Rounding the multiplier can only matter at an
// exact half-integer (the exact quotient is otherwise at least 2^-40 of itself away from one: its numerator is an
// integer below 2^40), so the product is formed twice, with the multiplier moved 2^-44 towards and away from zero:
// where the two agree the code is exact; they differ at a tie and only there, and the code is the even one of them (at the
// largest entry itself, D / 2, it is cut).  A block with a tie is formed twice; rows with few significant bits (16-bit ones, or such
// widened) may tie in every block: 8 rows of 1.17e7 fp32 entries, compress, 245 us, 260 with ties everywhere (1829 with a division each).
// The codes of an element meet in one word, pushed in from its top, one instruction each (alignbit); masked and shifted into place it was two,
// and the kernel, bound by instruction issue and short of registers, took 88 us for those rows instead of 69 (5.6 TB/s).  16-bit rows go at
// the rate of a copy either way: 4 rows of 1.24e8, 38 planes in all, 300 us (5.3 TB/s).
// A block's elements stay in LDS and are read once per code, so that the codes in the making are all the registers hold.
template <int DT>
__global__ __launch_bounds__(EX_THREADS, 4) void k_rtn_extract(BitsArgs a) {
    typedef BlockLoader<DT> Loader;
    __shared__ __align__(16) unsigned char s_buf[EX_THREADS / 64][EX_ELEMS * 4];
    __shared__ RtnPlaneCode s_code[3];
    const int row = blockIdx.y;
    const int level = a.rinfo[row].level;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
    const int64_t nblk = (a.d + EX_ELEMS - 1) / EX_ELEMS, nwhole = a.d / EX_ELEMS;
    const int64_t stride = (int64_t)gridDim.x * (EX_THREADS / 64);
    const int64_t blk = (int64_t)extract_place() * (EX_THREADS / 64) + wave;
    const Loader ld(a.g, a.ld, a.d, row);
    const uint32_t ckey = a.racc[row].smpmax_key;
    const double c = key_to_double(ckey), den = 2.0 * c;
    // the codes of the message in plane order: the base's (b_0 > 0), the previous level's (l > 1), the drawn level's
    const int b0 = a.F[0], b1 = level > 1 ? a.F[level - 1] : 0, b2 = a.F[level];
    const int nc = (b0 > 0 ? 1 : 0) + (b1 > 0 ? 1 : 0) + 1, np = b0 + b1 + b2;
    if (threadIdx.x < 3) {
        const int b = threadIdx.x == 0 ? b0 : threadIdx.x == 1 ? b1 : b2;
        if (b > 0) {
            RtnPlaneCode& k = s_code[threadIdx.x == 0 ? 0 : threadIdx.x == 1 ? nc - 2 : nc - 1];
            k.code = rtn_code_of(b);
            const double mul = c > 0.0 ? __ddiv_rn(k.code.D, den) : 0.0;   // a zero row has only zero codes
            k.mul_in = __dmul_rn(mul, 1.0 - 0x1p-44);
            k.mul_out = __dmul_rn(mul, 1.0 + 0x1p-44);
        }
    }
    __syncthreads();
    unsigned char* buf = s_buf[wave];
    const bool nonfinite = ckey >= 0x7F800000u;
    for_blocks(ld, buf, blk, stride, nblk, nwhole, [&](int64_t at_blk) {
        uint32_t x[32], tie = nonfinite ? 1u : 0u;
#pragma unroll
        for (int i = 0; i < 32; ++i) asm volatile("" : "=v"(x[i]));   // what the codes do not fill is not looked at
#pragma unroll 1
        for (int k = 0; k < nc; ++k) {
            const double mul_in = s_code[k].mul_in, mul_out = s_code[k].mul_out;
            const uint32_t width = (uint32_t)s_code[k].code.b;
            wave_lds_sync();   // the elements are read again for every code (kept, their doubles would take 64 registers)
            const uint32_t from = ld.take_at(wave * (EX_ELEMS * 4));
#pragma unroll
            for (int h = 0; h < Loader::CPL; ++h) {
                uint32_t b[Loader::EPC];
                ld.take_chunk(&s_buf[0][0], from, h, b);
#pragma unroll
                for (int i = 0; i < Loader::EPC; ++i) {
                    const double av = (double)__uint_as_float(b[i]);
                    const int n = __double2loint(__fma_rn(av, mul_in, 0x1.8p52)), m = __double2loint(__fma_rn(av, mul_out, 0x1.8p52));
                    tie = __builtin_amdgcn_bitop3_b32(tie, (uint32_t)n, (uint32_t)m, 0xF6);   // tie | (n ^ m)
                    x[h * Loader::EPC + i] = __builtin_amdgcn_alignbit((uint32_t)n, x[h * Loader::EPC + i], width);
                }
            }
        }
        if (__ballot(tie != 0u) != 0ull) {
            // again, four of a lane's elements at a time: in LDS they take the place of the block, the codes theirs
            wave_lds_sync();
            const uint32_t from = ld.take_at(wave * (EX_ELEMS * 4));
#pragma unroll
            for (int h = 0; h < Loader::CPL; ++h) {
                uint32_t b[Loader::EPC];
                ld.take_chunk(&s_buf[0][0], from, h, b);
#pragma unroll
                for (int i = 0; i < Loader::EPC; ++i) x[h * Loader::EPC + i] = b[i];
            }
            wave_lds_sync();   // every lane has read its elements
            uint32_t* mine = (uint32_t*)buf + lane;
            auto slot = [&](int i) -> uint32_t& { return mine[64 * i]; };
#pragma unroll
            for (int i = 0; i < 32; ++i) slot(i) = x[i];
#pragma unroll 1
            for (int i = 0; i < 32; i += 4) {
                double av[4];
                uint32_t v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t bits = slot(i + u);
                    av[u] = (double)__uint_as_float(bits);
                    if (nonfinite) {   // uniform: Inf and NaN are the numbers their bit patterns spell, as in c
                        av[u] = key_to_double(key_of_bits(bits));
                        av[u] = (int32_t)bits < 0 ? -av[u] : av[u];
                    }
                    v[u] = 0;
                }
#pragma unroll 1
                for (int k = 0; k < nc; ++k) {
                    const double mul_in = s_code[k].mul_in, mul_out = s_code[k].mul_out;
                    const uint32_t width = (uint32_t)s_code[k].code.b;
                    const int N = s_code[k].code.N;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        int n = __double2loint(__fma_rn(av[u], mul_in, 0x1.8p52));
                        const int m = __double2loint(__fma_rn(av[u], mul_out, 0x1.8p52));
                        n = n & 1 ? m : n;
                        n = n < -N ? -N : n > N ? N : n;
                        v[u] = __builtin_amdgcn_alignbit((uint32_t)n, v[u], width);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) slot(i + u) = v[u];
            }
#pragma unroll
            for (int i = 0; i < 32; ++i) x[i] = slot(i);
        }
        if (at_blk * 64 + lane < a.nwords * 2) {   // a plane's half words end inside the row's last block
            PlaneWriter w(a, row, at_blk);
            uint32_t r[8];
            auto put = [&](auto byte) {
                constexpr int B = decltype(byte)::value;
                gather_bytes<B>(x, r);
                transpose8(r);
#pragma unroll
                for (int p = 0; p < 8; ++p)
                    if (8 * B + p >= 32 - np) w.put(r[p]);   // uniform
            };
            if (np > 24) put(std::integral_constant<int, 0>{});
            if (np > 16) put(std::integral_constant<int, 1>{});
            if (np > 8) put(std::integral_constant<int, 2>{});
            put(std::integral_constant<int, 3>{});
        }
    });
}

// Round-to-Nearest MLMC: largest entry, residual sums, draw, codes.  message == false: norms only.
mlmc_status rtn_compress(const mlmc_plan_t* pl, const BitsArgs& a, bool message, hipStream_t st) {
    const int M = pl->M;
    int pb = (M * pl->L * 2 + 255) / 256;
    if (pb < (M + 255) / 256) pb = (M + 255) / 256;
    MLMC_LAUNCH(K_DRAW, st, k_rtn_prep<<<pb, 256, 0, st>>>(a));
    const int64_t nblk = (pl->d + 1023) / 1024;
    int64_t sw = (nblk + 7) / 8;
    const int64_t scap = 1024 / M > 0 ? 1024 / M : 1;
    if (sw > scap) sw = scap;
    if (sw < 1) sw = 1;
    const dim3 sgrid((unsigned)sw, M);
    int64_t nw = (pl->d + 4 * 256 * 8 - 1) / (4 * 256 * 8);   // a thread takes at least about eight groups of four elements
    const int64_t ncap = 2048 / M > 0 ? 2048 / M : 1;          // eight workgroups per CU in all: few atomics per sum
    if (nw > ncap) nw = ncap;
    const int64_t nmin = (pl->d + ((int64_t)1 << 24) - 1) >> 24;   // a thread adds at most 2^16 squares below 2^36, a workgroup 2^60 in all
    if (nw < nmin) nw = nmin;
    if (nw < 1) nw = 1;
    const dim3 ngrid((unsigned)nw, M);
    const dim3 egrid = extract_grid(pl);
    // with the plan's own probabilities the draw needs no norms: that read of the input is made only when they are asked for
    const bool need_norms = pl->adaptive || !message || a.norms_user != nullptr;
#define MLMC_RTN_STEPS(DT)                                                                                               \
    do {                                                                                                                \
        MLMC_LAUNCH(K_BITS_MAX, st, k_bits_smax<DT, false><<<sgrid, SMAX_THREADS, 0, st>>>(a));                            \
        if (need_norms) MLMC_LAUNCH(K_RTN_NORMS, st, launch_rtn_norms<DT>(pl->L, ngrid, st, a));                     \
        MLMC_LAUNCH(K_RTN_DRAW, st, k_rtn_draw<<<(M + 63) / 64, 64, 0, st>>>(a, message ? 0 : 1));                        \
        if (message) MLMC_LAUNCH(K_BITS_EXTRACT, st, k_rtn_extract<DT><<<egrid, EX_THREADS, 0, st>>>(a));                  \
    } while (0)
    if (need_norms && a.rtn_part) {
        MLMC_LAUNCH(K_RTN_NORMS, st, k_rtn_hist<<<dim3(pl->rtn_wgs, M), C16_THREADS, 0, st>>>(a));
        MLMC_LAUNCH(K_RTN_NORMS, st, k_rtn_hmax<<<dim3(C16_KEYS / 256, M), 256, 0, st>>>(a, pl->rtn_wgs));
        MLMC_LAUNCH(K_RTN_NORMS, st, k_rtn_hsum<<<dim3(C16_KEYS / 256, M), 256, 0, st>>>(a));
        MLMC_LAUNCH(K_RTN_DRAW, st, k_rtn_draw<<<(M + 63) / 64, 64, 0, st>>>(a, message ? 0 : 1));
        if (message) MLMC_LAUNCH(K_BITS_EXTRACT, st, k_rtn_extract<MLMC_BF16><<<egrid, EX_THREADS, 0, st>>>(a));
        return MLMC_OK;
    }
    if (pl->dtype == MLMC_F32) MLMC_RTN_STEPS(MLMC_F32);
    else MLMC_RTN_STEPS(MLMC_BF16);
#undef MLMC_RTN_STEPS
    return MLMC_OK;
}

}  // namespace mlmc
