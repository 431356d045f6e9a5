// Round-to-Nearest MLMC (Sec. 3.3, App. G.2) on gfx950.
#include "mlmc_extract.h"

namespace mlmc {

// ---------------------------------------------------------------------------------------------------
// Round-to-Nearest MLMC.  k_rtn_prep clears the per-row state; k_bits_smax (every block) finds c; k_rtn_norms sums
// the squared residual integers of every level; k_rtn_draw turns them into norms, probabilities, the draw and the
// coefficient; k_rtn_extract writes the planes of the drawn message's codes.
__global__ __launch_bounds__(256) void k_rtn_prep(BitsArgs a) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t == 0) *a.dev_status = 0;
    if (t < a.M) {
        a.racc[t].rowmax_key = 0u;
        a.racc[t].smpmax_key = 0u;
    }
    if (t < a.M * a.L * 2) a.rtn_sums[t] = 0ull;
}

template <int DT>
__global__ __launch_bounds__(256) void k_rtn_norms(BitsArgs a) {
    const int row = blockIdx.y;
    const uint32_t ckey = a.racc[row].smpmax_key;
    if (ckey == 0u) return;   // a zero row: every residual is zero
    const double c = key_to_double(ckey), den = 2.0 * c, inv_den = __ddiv_rn(1.0, den);
    RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    const int L = a.L;
    // Everything below is fp64 arithmetic on integers that fp64 holds exactly: |g| D has 40 bits, a code 16, a residual
    // integer k fewer than 18, k^2 fewer than 36, and a thread adds far fewer than 2^17 of them per level.
    RtnCode code[RTN_LMAX + 1];
    double Dcur[RTN_LMAX + 1], Dprev[RTN_LMAX + 1];   // D of level t; D' of level t (1 when the previous width is 0)
#pragma unroll
    for (int t = 0; t <= RTN_LMAX; ++t) {
        code[t] = rtn_code_of(t <= L ? a.F[t] : 0);
        Dcur[t] = code[t].D;
        Dprev[t] = t >= 1 && t <= L && a.F[t - 1] > 0 ? (double)((1 << a.F[t - 1]) - 1) : 1.0;
    }
    double acc[RTN_LMAX];
#pragma unroll
    for (int l = 0; l < RTN_LMAX; ++l) acc[l] = 0.0;
    auto code_of = [&](double av, int t) -> double { return rtn_code_f64(av, code[t], c, den, inv_den); };
    auto one = [&](uint32_t bits) {
        const double av = key_to_double(key_of_bits(bits));
        double nprev = code[0].b > 0 ? code_of(av, 0) : 0.0;
#pragma unroll
        for (int l = 1; l <= RTN_LMAX; ++l) {
            if (l <= L) {   // uniform
                const double ncur = code_of(av, l);
                const double k = __fma_rn(ncur, Dprev[l], -__dmul_rn(nprev, Dcur[l]));
                acc[l - 1] = __fma_rn(k, k, acc[l - 1]);
                nprev = ncur;
            }
        }
    };
    // groups of four elements, four loads of a thread in flight
    const int64_t nq = (a.d + 3) / 4, qstride = (int64_t)gridDim.x * 256;
    int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (; q + 3 * qstride < nq - 1; q += 4 * qstride) {   // none of the four is the row's last (possibly partial) group
        uint32_t b[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) ld.load4_full((q + u * qstride) * 4, b[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) one(b[u][e]);
    }
    for (; q < nq; q += qstride) {
        uint32_t b[4];
        const int nv = ld.load4(q * 4, b);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u < nv) one(b[u]);
    }
    // One pair of global atomics per workgroup and level (atomics of many waves on one address take turns): the waves'
    // sums meet in LDS first.
    __shared__ unsigned long long s_part[4][RTN_LMAX];
    const uint32_t wave = threadIdx.x >> 6;
#pragma unroll
    for (int l = 0; l < RTN_LMAX; ++l) {
        if (l < L) {
            unsigned long long v = (unsigned long long)acc[l];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
            if (lane_id() == 0) s_part[wave][l] = v;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < L) {
        const int l = threadIdx.x;
        const unsigned long long v = s_part[0][l] + s_part[1][l] + s_part[2][l] + s_part[3][l];   // < 2^53 + 2: no overflow
        if (v) {
            atomicAdd(&a.rtn_sums[((size_t)row * L + l) * 2], v & 0xFFFFFFFFull);
            atomicAdd(&a.rtn_sums[((size_t)row * L + l) * 2 + 1], v >> 32);
        }
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
    int32_t at;               // its first plane
};
// Code planes of the drawn message.  A code n = rne(a D / 2c) comes from one fused multiply-add: a * fl(D / 2c) plus
// 1.5 2^52 leaves the rounded integer, sign included, in the low word.  Rounding the multiplier can only matter at an
// exact half-integer (the exact quotient is otherwise at least 2^-40 of itself away from one: its numerator is an
// integer below 2^40), so the product is formed twice, with the multiplier moved 2^-44 towards and away from zero:
// where the two agree the code is exact; a block where they differ anywhere (a tie; always at the largest entry itself,
// whose code is cut) and a row of non-finite numbers have their codes computed the long way.
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
    int64_t blk = (int64_t)blockIdx.x * (EX_THREADS / 64) + wave;
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
            k.at = threadIdx.x == 0 ? 0 : threadIdx.x == 1 ? b0 : b0 + b1;
        }
    }
    __syncthreads();
    unsigned char* buf = s_buf[wave];
    for_blocks(ld, buf, blk, stride, nblk, nwhole, [&](int64_t at_blk) {
        uint32_t x[32], tie = ckey >= 0x7F800000u ? 1u : 0u;
#pragma unroll
        for (int i = 0; i < 32; ++i) x[i] = 0;
#pragma unroll 1
        for (int k = 0; k < nc; ++k) {
            const double mul_in = s_code[k].mul_in, mul_out = s_code[k].mul_out;
            const uint32_t mask = (1u << s_code[k].code.b) - 1u, at = (uint32_t)s_code[k].at;
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
                    tie |= (uint32_t)(n ^ m);
                    x[h * Loader::EPC + i] |= ((uint32_t)n & mask) << at;
                }
            }
        }
        if (__builtin_expect(__ballot(tie != 0u) != 0ull, 0)) {
            RowLoader<DT, false> ld1(a.g, a.ld, a.d, row);
            const int64_t j0 = at_blk * EX_ELEMS + 32 * (int64_t)lane;
            const double inv_den = c > 0.0 ? __ddiv_rn(1.0, den) : 0.0;
            wave_lds_sync();   // every lane has read its elements: their place takes the codes
            uint32_t* mine = (uint32_t*)buf + 32 * lane;
#pragma unroll 1
            for (int i = 0; i < 32; ++i) {
                uint32_t v = 0;
                const uint32_t bits = j0 + i < a.d ? ld1.load1(j0 + i) : 0u;
#pragma unroll 1
                for (int k = 0; k < nc; ++k) {
                    const RtnCode kc = s_code[k].code;
                    int32_t n = c > 0.0 ? rtn_code_abs(key_to_double(key_of_bits(bits)), kc, c, den, inv_den) : 0;
                    n = (int32_t)bits < 0 ? -n : n;
                    v |= ((uint32_t)n & ((1u << kc.b) - 1u)) << s_code[k].at;
                }
                mine[i] = v;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint4 v = ((const uint4*)mine)[i];
                x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
            }
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
                    if (8 * B + p < np) w.put(r[p]);   // uniform
            };
            put(std::integral_constant<int, 0>{});
            if (np > 8) put(std::integral_constant<int, 1>{});
            if (np > 16) put(std::integral_constant<int, 2>{});
            if (np > 24) put(std::integral_constant<int, 3>{});
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
    const int64_t nmin = (pl->d + ((int64_t)1 << 24) - 1) >> 24;   // a thread adds at most 2^16 squares below 2^36: exact in fp64
    if (nw < nmin) nw = nmin;
    if (nw < 1) nw = 1;
    const dim3 ngrid((unsigned)nw, M);
    const dim3 egrid = extract_grid(pl);
    // with the plan's own probabilities the draw needs no norms: that read of the input is made only when they are asked for
    const bool need_norms = pl->adaptive || !message || a.norms_user != nullptr;
#define MLMC_RTN_STEPS(DT)                                                                                               \
    do {                                                                                                                \
        MLMC_LAUNCH(K_BITS_MAX, st, k_bits_smax<DT, false><<<sgrid, SMAX_THREADS, 0, st>>>(a));                            \
        if (need_norms) MLMC_LAUNCH(K_RTN_NORMS, st, k_rtn_norms<DT><<<ngrid, 256, 0, st>>>(a));                     \
        MLMC_LAUNCH(K_RTN_DRAW, st, k_rtn_draw<<<(M + 63) / 64, 64, 0, st>>>(a, message ? 0 : 1));                        \
        if (message) MLMC_LAUNCH(K_BITS_EXTRACT, st, k_rtn_extract<DT><<<egrid, EX_THREADS, 0, st>>>(a));                  \
    } while (0)
    if (pl->dtype == MLMC_F32) MLMC_RTN_STEPS(MLMC_F32);
    else MLMC_RTN_STEPS(MLMC_BF16);
#undef MLMC_RTN_STEPS
    return MLMC_OK;
}

}  // namespace mlmc
