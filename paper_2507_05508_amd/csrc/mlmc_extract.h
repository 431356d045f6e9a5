// Extraction of bit-plane messages on gfx950, shared by the translation units that launch it: the row maximum
// (k_bits_smax), the packing of a block into plane words (BlockLoader, transpose8) and the extraction kernel of the
// bit-wise ladders (k_bits_extract).  Sec. 3.1 (fixed point), App. B (floating point), Sec. 3.3 / App. G.2 (Round-to-Nearest codes).
#pragma once
#include <type_traits>

#include "mlmc_device.h"

namespace mlmc {

// Largest |g| key of the sampled blocks of every row (block b of 1024 elements is sampled when b % S == S / 2,
// S = 2^sample_shift; S = 1 reads the whole row and the result is the row maximum itself).
// PARTS: nothing is cleared beforehand, so no launch precedes this one: every workgroup stores its own maximum (the
// readers take the largest of a row's, row_smpmax), and the first workgroup of a row draws the row's level (Alg. 2
// "Sample l ~ p") and sets the state that the extraction accumulates into to its start values.
constexpr int SMAX_THREADS = 512;
template <int DT, bool PARTS>
__global__ __launch_bounds__(SMAX_THREADS) void k_bits_smax(BitsArgs a) {
    const int row = blockIdx.y;
    if (PARTS && blockIdx.x == 0) {   // uniform over the workgroup
        __shared__ double s_p[LMAX];
        if ((int)threadIdx.x < a.L) s_p[threadIdx.x] = a.p_fixed[threadIdx.x];
        __syncthreads();
        if (threadIdx.x == 0) {
            if (row == 0) *a.dev_status = 0;   // no workgroup of this launch reports through it
            const uint32_t x = philox_word0(a.seed, a.step, (uint32_t)row);
            const int level = draw_from_p(s_p, a.L, x);
            const double pl = s_p[level - 1];
            RowInfo* ri = a.rinfo + row;
            ri->level = level;
            ri->weight = pl == 0.0 ? 0.0f : (float)__ddiv_rn(1.0, pl);
            ri->draw_x = x;
            a.level[row] = level;
            a.racc[row].rowmax_key = 0u;
        }
    }
    const int64_t S = (int64_t)1 << a.sample_shift, first = S >> 1;
    const int64_t nblk = (a.d + 1023) / 1024;
    const int64_t ns = nblk > first ? (nblk - first + S - 1) / S : 0;
    RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t maxkey = 0;
    // a wave's blocks, the loads of the next one in flight while the current one is reduced
    const int64_t i0 = (int64_t)blockIdx.x * (SMAX_THREADS / 64) + wave, istride = (int64_t)gridDim.x * (SMAX_THREADS / 64);
    auto fetch = [&](int64_t i, uint32_t (&b)[4][4]) {
        const int64_t blk = first + i * S;
        const int64_t base = blk * 1024 + lane * 4;
        if ((blk + 1) * 1024 <= a.d) {   // a whole block: four loads in flight
#pragma unroll
            for (int q = 0; q < 4; ++q) ld.load4_stream(base + q * 256, b[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) ld.load4(base + q * 256, b[q]);   // past the end: +0
        }
    };
    auto reduce = [&](const uint32_t (&b)[4][4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t key = key_of_bits(b[q][c]);
                maxkey = key > maxkey ? key : maxkey;
            }
    };
    uint32_t b0[4][4], b1[4][4];
    int64_t i = i0;
    if (i < ns) fetch(i, b0);
    for (; i < ns; i += 2 * istride) {
        const bool more1 = i + istride < ns, more2 = i + 2 * istride < ns;   // uniform
        if (more1) fetch(i + istride, b1);
        reduce(b0);
        if (more2) fetch(i + 2 * istride, b0);
        if (more1) reduce(b1);
    }
    // the waves' maxima meet in LDS: atomics of many waves on one address take turns
    maxkey = wave_max(maxkey);
    __shared__ uint32_t s_wmax[SMAX_THREADS / 64];
    if (lane == 0) s_wmax[wave] = maxkey;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t m = 0;
#pragma unroll
        for (int w = 0; w < SMAX_THREADS / 64; ++w) m = s_wmax[w] > m ? s_wmax[w] : m;
        if (PARTS) {
            ((uint32_t*)a.racc[row].gsum)[blockIdx.x] = m;   // a non-finite entry is reported by the extraction, which sees every entry
        } else if (m) {
            atomicMax(&a.racc[row].smpmax_key, m);
            if (m >= 0x7F800000u) atomicOr(a.dev_status, MLMC_DEV_NONFINITE);
        }
    }
}

// The largest key k_bits_smax found in a row (every lane of the calling wave gets it).
__device__ __forceinline__ uint32_t row_smpmax(const BitsArgs& a, int row) {
    const RowAcc* ra = a.racc + row;
    if (a.smax_parts == 0) return ra->smpmax_key;
    const uint32_t* part = (const uint32_t*)ra->gsum;
    uint32_t m = 0;
    for (int i = (int)lane_id(); i < a.smax_parts; i += 64) {
        const uint32_t v = part[i];
        m = v > m ? v : m;
    }
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max(m));
}

// ---------------------------------------------------------------------------------------------------
// Round-to-Nearest ladder (Sec. 3.3, App. G.2).  Code of magnitude a at width b: n = rne(a D / (2c)), D = 2^b - 1, cut
// at N = 2^(b-1) - 1.  a D is an exact double (40 bits); n0 = rint(a D * (1 / 2c)) is off by at most one, and the
// remainder a D - n0 2c, exact in one fused multiply-add, decides: beyond +-c the neighbour, exactly +-c the even one.
struct RtnCode {
    double D;     // 2^b - 1 (0: no such code)
    int32_t N;    // 2^(b-1) - 1
    int32_t b;    // width in bits
};
__device__ __forceinline__ int32_t rtn_code_abs(double a, const RtnCode& k, double c, double den, double inv_den) {
    const double num = __dmul_rn(a, k.D);
    double n = rint(__dmul_rn(num, inv_den));
    const double rem = __fma_rn(-n, den, num);
    n += rem > c ? 1.0 : 0.0;
    n -= rem < -c ? 1.0 : 0.0;
    int32_t ni = (int32_t)n;
    if ((rem == c || rem == -c) && (ni & 1)) ni += rem > 0.0 ? 1 : -1;
    return ni < k.N ? ni : k.N;
}
__device__ __forceinline__ RtnCode rtn_code_of(int b) {
    RtnCode k;
    k.b = b;
    k.D = b > 0 ? (double)((1 << b) - 1) : 0.0;
    k.N = b > 0 ? (1 << (b - 1)) - 1 : 0;
    return k;
}
// |g| as an exact double from its key
__device__ __forceinline__ double key_to_double(uint32_t key) {
    const uint32_t E = key >> 23;
    return ldexp((double)(E ? (key & 0x7FFFFFu) | 0x800000u : key), (int)(E ? E : 1u) - 150);
}
// ---------------------------------------------------------------------------------------------------
// Packing a block of EX_ELEMS elements into plane words, one wave per block.
//
// A lane owns the block's elements 32 l .. 32 l + 31, i.e. half a plane word of every plane, so that planes are made
// inside a lane: bytes of four elements share a register, eight such registers are an 8 x 8 bit matrix per byte
// column, and three exchange steps transpose it (transpose8).  That is 2.3 instructions per element for eight planes,
// about 12 for the whole extraction, and leaves it to the memory: 8 rows of 1.17e7 fp32 elements take 75 us at two or three planes
// (0.41 GB, 5.4 TB/s) and 83 us at the floating-point ladder's ten (0.49 GB, 5.9 TB/s; without its stores the kernel takes 61 and 60).
// A wave ballot per plane with its two lane writes took three instructions per element and plane: 94 and 175 us.
//
// The loads stay coalesced (a wave's load instruction covers 1 KB of consecutive elements) and are dealt to the lanes through LDS.
// Chunk c of lane l lies in slot c ^ s(l) of the lane's part of the buffer, so that the 16-byte reads of eight neighbouring lanes
// meet all banks; the permutation is applied to the addresses of the loads (inside a lane's 128 or 64 bytes), the writes are linear.
// Rows may start at any element: 80.3 us for odd fp32 rows as against 79.7; bf16 rows of twice the length 96 against 83 us.
constexpr int EX_ELEMS = 2048;
constexpr int EX_THREADS = 256;

typedef uint32_t u32x4_el2 __attribute__((ext_vector_type(4), aligned(2)));

template <int DT>
struct BlockLoader {
    static constexpr int EB = DT == MLMC_F32 ? 4 : 2;    // bytes of an element
    static constexpr int EPC = 16 / EB;                  // elements of a 16-byte chunk
    static constexpr int CPL = 32 / EPC;                 // chunks of a lane
    static constexpr int LDS_BYTES = EX_ELEMS * EB;
    const char* row;
    int64_t d;
    uint32_t lane;
    uint32_t goff;      // where this lane's first load lies in the block; the k-th is 1 KB further on each time
    __device__ __forceinline__ BlockLoader(const void* g, int64_t ld, int64_t d_, int r) : d(d_), lane(lane_id()) {
        row = (const char*)g + (int64_t)r * ld * EB;
        // slot 64 k + lane of the buffer holds chunk c ^ s(l) of its owner l = slot / CPL; s(l) does not depend on k
        goff = ((lane & ~(uint32_t)(CPL - 1)) | ((lane & (CPL - 1)) ^ swz(lane / CPL))) * 16u;
    }
    static __device__ __forceinline__ uint32_t swz(uint32_t l) { return DT == MLMC_F32 ? (l & 7u) : ((l >> 1) & 3u); }
    __device__ __forceinline__ void fetch(int64_t blk, uint4 (&q)[CPL]) const {   // a whole block
        const char* base = row + blk * (int64_t)LDS_BYTES;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
            if (DT == MLMC_F32) {
                const u32x4_f32 v = __builtin_nontemporal_load((const u32x4_f32*)(base + k * 1024 + goff));
                q[k] = make_uint4(v.x, v.y, v.z, v.w);
            } else {
                const u32x4_el2 v = __builtin_nontemporal_load((const u32x4_el2*)(base + k * 1024 + goff));
                q[k] = make_uint4(v.x, v.y, v.z, v.w);
            }
        }
    }
    // the registers of a fetch that is not made: no value, and none kept from before (an old one would be copied around the loop)
    static __device__ __forceinline__ void skip(uint4 (&q)[CPL]) {
#pragma unroll
        for (int k = 0; k < CPL; ++k) asm volatile("" : "=v"(q[k].x), "=v"(q[k].y), "=v"(q[k].z), "=v"(q[k].w));
    }
    // the loaded chunks into the wave's LDS buffer
    __device__ __forceinline__ void put(const uint4 (&q)[CPL], unsigned char* buf) const {
#pragma unroll
        for (int k = 0; k < CPL; ++k) *(uint4*)(buf + k * 1024 + lane * 16u) = q[k];
    }
    // the row's last block when it is not a whole one, straight into the buffer; past the end +0
    __device__ __forceinline__ void put_part(int64_t blk, unsigned char* buf) const {
        const int64_t e0 = blk * EX_ELEMS;
#pragma unroll 1
        for (uint32_t e = lane; e < EX_ELEMS; e += 64) {
            const uint32_t owner = e >> 5, c = (e & 31u) / EPC;
            unsigned char* p = buf + (owner * CPL + (c ^ swz(owner))) * 16u + (e & (EPC - 1)) * EB;
            const bool in = e0 + e < d;
            if (DT == MLMC_F32) *(uint32_t*)p = in ? ((const uint32_t*)row)[e0 + e] : 0u;
            else *(uint16_t*)p = in ? ((const uint16_t*)row)[e0 + e] : (uint16_t)0;
        }
    }
    // where this lane's chunks lie in the workgroup's buffers (chunk c: 16 c flipped in); hidden from the compiler anew for every
    // block, which would otherwise keep all of a lane's addresses in registers across the loop
    __device__ __forceinline__ uint32_t take_at(uint32_t wave_offset) const {
        uint32_t at = wave_offset + lane * (CPL * 16u) + swz(lane) * 16u;
        asm volatile("" : "+v"(at));
        return at;
    }
    // chunk c of what the buffer holds for this lane, as fp32 bits (elements 32 lane + EPC c ...)
    __device__ __forceinline__ void take_chunk(const unsigned char* bufs, uint32_t at, int c, uint32_t (&b)[EPC]) const {
        const uint4 v = *(const uint4*)(bufs + (at ^ (uint32_t)(16 * c)));
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            if (DT == MLMC_F32) {
                b[h] = w[h];
            } else {
                b[(2 * h) % EPC] = w[h] << 16;
                b[(2 * h + 1) % EPC] = w[h] & 0xFFFF0000u;
            }
        }
    }
};

// A wave's blocks first, first + stride, ...: proc(block) finds the block in the LDS buffer while the loads of the next one are in
// flight.  The first turn only loads, so that there is one place that does: with a second one before the loop the
// compiler gave its registers a second home and, unable to tell which loads were out, waited for half of them in every turn.
template <class Loader, class Proc>
__device__ __forceinline__ void for_blocks(const Loader& ld, unsigned char* buf, int64_t first, int64_t stride, int64_t nblk,
                                           int64_t nwhole, Proc proc) {
    uint4 q[Loader::CPL];
    int64_t cur = first - stride;   // all uniform
    for (;;) {
        const int64_t next = cur + stride;
        const bool have = next != first;
        if (have) {
            if (cur < nwhole) ld.put(q, buf);
            else ld.put_part(cur, buf);
        }
        if (next < nwhole) ld.fetch(next, q);
        else ld.skip(q);
        if (have) {
            wave_lds_sync();
            proc(cur);
            wave_lds_sync();   // the next writes come after these reads
        }
        if (next >= nblk) break;
        cur = next;
    }
}

// r[i], byte k = byte B of element 8 k + i
template <int B>
__device__ __forceinline__ void gather_bytes(const uint32_t (&x)[32], uint32_t (&r)[8]) {
    constexpr uint32_t sel = 0x0C0C0400u + 0x0101u * B;   // byte B of the second operand, byte B of the first, two zero bytes
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t lo = __builtin_amdgcn_perm(x[8 + i], x[i], sel);
        const uint32_t hi = __builtin_amdgcn_perm(x[24 + i], x[16 + i], sel);
        r[i] = (hi << 16) | lo;
    }
}
// Bit q of r[i]'s byte k <-> bit i of r[q]'s byte k, in all four byte columns (its own inverse).
__device__ __forceinline__ void transpose8(uint32_t (&r)[8]) {
    auto swap_bits = [&](int i, int j, int s, uint32_t m) {   // m: the bits of r[i] that stay
        const uint32_t lo = r[i], hi = r[j];
        r[i] = (lo & m) | ((hi << s) & ~m);
        r[j] = ((lo >> s) & m) | (hi & ~m);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) swap_bits(i, i + 4, 4, 0x0F0F0F0Fu);
#pragma unroll
    for (int i = 0; i < 8; ++i) if (!(i & 2)) swap_bits(i, i + 2, 2, 0x33333333u);
#pragma unroll
    for (int i = 0; i < 8; ++i) if (!(i & 1)) swap_bits(i, i + 1, 1, 0x55555555u);
}

// Which of a row's workgroups this one is.  Workgroups are dealt to the eight XCDs in turn; where their number is a multiple of eight, those of one XCD
// take consecutive blocks here, so that the lines in which the words of neighbouring blocks meet (planes start at any word) are whole in one L2
// before they leave it.
__device__ __forceinline__ uint32_t extract_place() {
    return (gridDim.x & 7u) == 0u ? (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;
}

// Writes this lane's half words of a block, plane after plane in ascending order.  The position of the next plane is one running
// pointer for the wave (hidden from the compiler, which would otherwise keep thirty plane offsets in scalar registers
// across the loop and spill them), the lane's offset one register.
struct PlaneWriter {
    typedef __attribute__((address_space(1))) char* GlobalBytes;
    GlobalBytes at;      // uniform: this block's words of the next plane
    size_t step;         // bytes of a plane
    uint32_t off;        // this lane's half word
    __device__ __forceinline__ PlaneWriter(const BitsArgs& a, int row, int64_t blk)
        : at((GlobalBytes)(a.planes + (size_t)row * a.nplanes * a.nwords) + blk * (EX_ELEMS / 8)), step((size_t)a.nwords * 8), off(lane_id() * 4u) {}
    __device__ __forceinline__ void put(uint32_t v) {
        *(__attribute__((address_space(1))) uint32_t*)(at + off) = v;
        at += step;
        asm volatile("" : "+s"(at));
    }
};

// The exact multiplier of the largest-entry ladder: trunc(|g| r) = floor(|g| 2^Q / v) for every |g| <= v, Q <= 24.
// Let q be the exact quotient.  |g| and v have 24-bit significands, so a q that is no integer lies at least q 2^-49 away from
// the next integer above (q < 2^(s+1) when the significands' quotient is scaled by 2^s, and its distance is a multiple of 1 / significand
// of v; s <= Q), and a q below 1 at least 2^-25.  r = fl(fl(2^Q / v) (1 + 2^-50)) and the product carry three roundings, 3 2^-53 in all, less than the
// 2^-50 they are raised by, and 2^-50 + 3 2^-53 < 2^-49: an integer q is never missed, no other one is passed.
__device__ __forceinline__ double largest_entry_multiplier(double v, int Q) {
    return v > 0.0 ? __dmul_rn(__ddiv_rn(ldexp(1.0, Q), v), 1.0 + 0x1p-50) : 0.0;
}

// How an element becomes the value whose bits are the row's planes after the sign plane (KIND as in k_bits_extract).
// A row that holds Inf or NaN is scaled by its own largest bit pattern: its keys are taken one binade down (`halve`,
// whole-row uniform), so that every pattern is a finite number again; what that shifts out has only zero digits there.
struct ExtractRow {
    int np, F0;
    uint32_t halve;      // 0, or one exponent step for a row whose largest key is not finite
    int shl, sh0;        // fixed point: |g| 2^shl and |g| 2^sh0 cut to integers are the level's and the base's digits
    double mul;          // largest entry: largest_entry_multiplier
    uint32_t cap, vsl, vs0, mask0;
};
template <int KIND, bool BASE>
__device__ __forceinline__ uint32_t digits_of(const ExtractRow& e, uint32_t key) {
    const float v = __uint_as_float(__builtin_elementwise_sub_sat(key, e.halve));
    if (KIND == 0) {
        // floor(|g| / s 2^F): the scaling by a power of two is exact (or underflows below 1), the conversion truncates
        const uint32_t x = (uint32_t)__builtin_ldexpf(v, e.shl);
        if (!BASE) return x;
        return (uint32_t)__builtin_ldexpf(v, e.sh0) | (x << e.F0);
    }
    uint32_t n = (uint32_t)__dmul_rn((double)v, e.mul);
    n = n < e.cap ? n : e.cap;
    const uint32_t x = n >> e.vsl;
    if (!BASE) return x;
    return ((n >> e.vs0) & e.mask0) | (x << e.F0);
}

// The planes of one block.  KIND 0: fixed point, 1: floating point, 2: fixed point of |g| / max|g|.
template <int KIND, bool BASE>
__device__ __forceinline__ void write_block(const BitsArgs& a, const ExtractRow& e, int level, const uint32_t (&x)[32], uint32_t sign, PlaneWriter w) {
    uint32_t r[8];
    if (KIND == 1) {
        // App. B: the planes are bits of the fp32 word itself: sign, exponent, the base's digits, the level's digits
        const int Fl = a.F[level], Fp = a.F[level - 1], F0 = e.F0;
        gather_bytes<3>(x, r);
        transpose8(r);
        w.put(r[7]);
        uint32_t hi[8];
        gather_bytes<2>(x, hi);
        transpose8(hi);
        w.put(hi[7]);
#pragma unroll
        for (int q = 0; q < 7; ++q) w.put(r[q]);
        // fraction bits lo .. 22, least significant first (uniform bounds)
        auto field = [&](auto byte, const uint32_t (&v)[8], int lo, int end) {
            constexpr int B = decltype(byte)::value;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int bit = 8 * B + q;
                if (bit < 23 && bit >= lo && bit < end) w.put(v[q]);
            }
        };
        auto digits = [&](int lo, int end) {
            if (lo < 8) {
                gather_bytes<0>(x, r);
                transpose8(r);
                field(std::integral_constant<int, 0>{}, r, lo, end);
            }
            if (lo < 16 && end > 8) {
                gather_bytes<1>(x, r);
                transpose8(r);
                field(std::integral_constant<int, 1>{}, r, lo, end);
            }
            if (end > 16) field(std::integral_constant<int, 2>{}, hi, lo, end);
        };
        if (BASE) digits(23 - F0, 23);
        digits(23 - Fl, 23 - Fp);
        return;
    }
    w.put(sign);
    auto put = [&](auto byte) {
        constexpr int B = decltype(byte)::value;
        gather_bytes<B>(x, r);
        transpose8(r);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (1 + 8 * B + q < e.np) w.put(r[q]);   // uniform
    };
    put(std::integral_constant<int, 0>{});
    if (e.np > 9) put(std::integral_constant<int, 1>{});
    if (e.np > 17) put(std::integral_constant<int, 2>{});
}

// The row's record under the largest key `smpmax` of its sample and the exponent `Ex` that its scale is taken from.
template <int KIND>
__device__ __forceinline__ ExtractRow extract_row(const BitsArgs& a, int row, int level, uint32_t smpmax, uint32_t Ex, bool store) {
    ExtractRow e;
    const int Emax = Ex ? (int)Ex : 1;
    e.F0 = a.F[0];
    e.np = (KIND == 1 ? 9 : 1) + e.F0 + (a.F[level] - a.F[level - 1]);   // planes written for this row
    if (KIND == 0) {
        e.halve = Emax == 255 ? 0x800000u : 0u;
        const int down = Emax - 126 - (Emax == 255 ? 1 : 0);
        e.shl = a.F[level] - down;
        e.sh0 = e.F0 - down;
        if (store) a.scale_exp[row] = Emax - 126;
    } else if (KIND == 2) {
        const int Q = a.F[a.L];
        e.halve = smpmax >= 0x7F800000u ? 0x800000u : 0u;
        const double vd = (double)__uint_as_float(smpmax - e.halve);   // the largest |g| of the row
        e.mul = largest_entry_multiplier(vd, Q);
        e.cap = vd > 0.0 ? (1u << Q) - 1u : 0u;   // a zero row has only zero digits
        e.vsl = (uint32_t)(Q - a.F[level]);
        e.vs0 = (uint32_t)(Q - e.F0);
        e.mask0 = (1u << e.F0) - 1u;
        if (store) a.scale_exp[row] = (int32_t)smpmax;
    }
    return e;
}

// The row's message under the scale taken from the sampled maximum; the true maximum of the row is tracked on the
// way.  REDO (second launch, only when the maximum was sampled): rows whose true maximum has a larger exponent than
// the sampled one are extracted again with the true one; every other row is already final and is skipped.
// KIND 0: fixed-point ladder (Sec. 3.1): |g| = sig 2^(E - 150), scale s = 2^(Emax - 126), digits floor(|g| / s 2^F).
// KIND 1: floating-point ladder (no scale).  KIND 2: fixed-point ladder of |g| / v: the row maximum was read exactly
// beforehand (sample of every block).  Planes: sign, base field, level field (floating point: the exponent after the sign).
// A wave takes its blocks in turn (extract_grid: one or three, or more in the kinds with a row maximum, 6 at 8 rows of 1.17e7, 30 at 4 of 1.24e8) with the next one's
// loads in flight; 8 KB (4 KB) of LDS per wave.
// BASE: the ladder has a base field (F_0 > 0).  Four waves per SIMD (128 registers).
template <int DT, bool REDO, int KIND, bool BASE>
__global__ __launch_bounds__(EX_THREADS, 4) void k_bits_extract(BitsArgs a) {
    typedef BlockLoader<DT> Loader;
    __shared__ __align__(16) unsigned char s_buf[EX_THREADS / 64][Loader::LDS_BYTES];
    const int row = blockIdx.y;
    RowAcc* ra = a.racc + row;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t nblk = (a.d + EX_ELEMS - 1) / EX_ELEMS, nwhole = a.d / EX_ELEMS;
    const int64_t stride = (int64_t)gridDim.x * (EX_THREADS / 64);
    const int64_t blk = (int64_t)extract_place() * (EX_THREADS / 64) + wave;
    const Loader ld(a.g, a.ld, a.d, row);
    const uint32_t smpmax = KIND == 1 ? 0u : row_smpmax(a, row);
    const uint32_t Es = smpmax >> 23;
    uint32_t Ex = Es;
    if (REDO) {
        Ex = ra->rowmax_key >> 23;
        if (Ex <= Es) return;
    }
    const int level = a.rinfo[row].level;
    ExtractRow e = extract_row<KIND>(a, row, level, smpmax, Ex, blockIdx.x == 0 && threadIdx.x == 0);
    asm volatile("" : "+s"(e.halve));   // a number to subtract, not a choice to make for every element
    uint32_t maxkey = 0;
    const uint32_t lane = lane_id();
    unsigned char* buf = s_buf[wave];
    uint32_t x[32];
    for_blocks(ld, buf, blk, stride, nblk, nwhole, [&](int64_t b0) {
        uint32_t sign = 0;
        const uint32_t at = ld.take_at(wave * Loader::LDS_BYTES);
#pragma unroll
        for (int c = Loader::CPL - 1; c >= 0; --c) {
            uint32_t b[Loader::EPC];
            ld.take_chunk(&s_buf[0][0], at, c, b);
#pragma unroll
            for (int i = Loader::EPC - 1; i >= 0; --i) {
                const uint32_t key = key_of_bits(b[i]);
                maxkey = key > maxkey ? key : maxkey;
                if (KIND != 1) sign = __builtin_amdgcn_alignbit(sign, b[i], 31);   // (sign << 1) | bit 31: element 0 ends lowest
                x[c * Loader::EPC + i] = KIND == 1 ? b[i] : digits_of<KIND, BASE>(e, key);
            }
            if (KIND != 1 && (c & 1) == 0) __builtin_amdgcn_sched_barrier(0);   // keeps the raw elements of few chunks alive
        }
        if (b0 * 64 + lane < a.nwords * 2)   // a plane's half words end inside the row's last block
            write_block<KIND, BASE>(a, e, level, x, sign, PlaneWriter(a, row, b0));
    });
    if (!REDO) {
        maxkey = wave_max(maxkey);
        __shared__ uint32_t s_max[EX_THREADS / 64];
        if (lane == 0) s_max[wave] = maxkey;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t m = s_max[0];
#pragma unroll
            for (int w = 1; w < EX_THREADS / 64; ++w) m = s_max[w] > m ? s_max[w] : m;
            // Only a key above the sampled maximum's binade is reported: with every workgroup's, the atomics of a single long row met on the line
            // that all its workgroups read the sampled maxima from (1 row of 5e7 fp32 entries: 81 us, 41 now; 1 row of 1e8: 122, 83).
            if (KIND == 0 && (m >> 23) > Es) atomicMax(&ra->rowmax_key, m);
            if (m >= 0x7F800000u) atomicOr(a.dev_status, MLMC_DEV_NONFINITE);
        }
    }
}

// The same message, a wave a few words of 64 entries of every plane, an entry a lane: for plans that leave most of the chip idle with 2048 entries a wave, which is
// bound by the instructions of its one wave a SIMD (4 rows of 100003, fixed point: 8.5 -> 4.3 us).  Rows whose maximum is exact (no second launch).  The planes' words are ballots.
constexpr int EW_WORDS = 4;
template <int DT, int KIND, bool BASE>
__global__ __launch_bounds__(EX_THREADS) void k_bits_extract_words(BitsArgs a) {
    const int row = blockIdx.y;
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t w0 = ((int64_t)blockIdx.x * (EX_THREADS / 64) + wave) * EW_WORDS;
    const RowLoader<DT, true> ld(a.g, a.ld, a.d, row);
    uint32_t b[EW_WORDS];
#pragma unroll
    for (int i = 0; i < EW_WORDS; ++i) {
        const int64_t j = (w0 + i) * 64 + lane;
        b[i] = j < a.d ? ld.load1(j) : 0u;
    }
    const int level = a.rinfo[row].level;
    const uint32_t smpmax = KIND == 1 ? 0u : row_smpmax(a, row);
    const ExtractRow e = extract_row<KIND>(a, row, level, smpmax, smpmax >> 23, blockIdx.x == 0 && threadIdx.x == 0);
    const int Fl = a.F[level], Fp = a.F[level - 1];
    uint64_t* out = a.planes + ((size_t)row * a.nplanes + lane) * a.nwords + w0;   // this lane's plane
#pragma unroll
    for (int i = 0; i < EW_WORDS; ++i) {
        if (w0 + i >= a.nwords) break;   // uniform
        const uint32_t key = key_of_bits(b[i]);
        uint32_t y;   // bit p: the entry's bit of plane p
        if (KIND == 1) {   // sign, exponent, the base's digits, the level's digits
            const uint32_t frac = b[i] & 0x7FFFFFu, lev = (frac >> (23 - Fl)) & ((1u << (Fl - Fp)) - 1u);
            y = b[i] >> 31 | (key >> 23) << 1 | (BASE ? (frac >> (23 - e.F0)) << 9 : 0u) | lev << (9 + e.F0);
        } else {
            y = b[i] >> 31 | digits_of<KIND, BASE>(e, key) << 1;
        }
        uint32_t lo = 0, hi = 0;
        for (int p = 0; p < e.np; ++p) {   // uniform
            const uint64_t m = __ballot((y >> p) & 1u);
            lo = write_lane((uint32_t)m, p, lo);
            hi = write_lane((uint32_t)(m >> 32), p, hi);
        }
        if ((int)lane < e.np) out[i] = (uint64_t)hi << 32 | lo;
        if (__ballot(key >= 0x7F800000u) && lane == 0) atomicOr(a.dev_status, MLMC_DEV_NONFINITE);
    }
}

// Workgroups of an extraction.  Every wave of a row takes the same number of blocks, give or take the last (the loads run ahead from block to block): three,
// or one where that leaves fewer than four workgroups per CU.  The kinds with a row maximum begin every workgroup with a reduction over the maxima of
// its row, so they get about 2048 workgroups in all however long the rows are.  A multiple of eight per row: extract_place.
// us, grids without that and with at most 2048 or 4096 workgroups in all / now: 4 rows of 1.24e8 bf16 entries, Round-to-Nearest, 327 / 300 and the
// aggregate after it 267 / 249; 8 rows of 1.17e7 fp32, Round-to-Nearest 77 / 73, floating point 84.8 / 83.1, fixed point 76.7 / 74.4, largest entry 81.1 / 78.1;
// the last two with three blocks a wave 76.9 and 82.2, 3 rows of 1.24e8 bf16 entries, fixed point, 176 as against 152.
inline dim3 extract_grid(const mlmc_plan_t* pl) {
    const int64_t wgs = ((pl->d + EX_ELEMS - 1) / EX_ELEMS + EX_THREADS / 64 - 1) / (EX_THREADS / 64);
    int64_t per = 3;
    if ((pl->kind == MLMC_BITS || pl->kind == MLMC_VBITS) && wgs * pl->M > per * 2048) per = (wgs * pl->M + 2047) / 2048;
    int64_t gx = (wgs + per - 1) / per;
    if (gx * pl->M < 1024) gx = wgs;
    if (gx >= 64) gx = (gx + 7) / 8 * 8;
    return dim3((unsigned)gx, pl->M);
}

}  // namespace mlmc
