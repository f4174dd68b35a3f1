// Device helpers shared by the kernels: operand vector types, the exact quantizer's fast path, reductions over the lanes
// of a wavefront that hold one row, byte-to-fp16 conversion (gfx950 only).
#pragma once
#include "taq_internal.h"

namespace taq {

typedef int int32x4_t __attribute__((ext_vector_type(4)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

#define TAQ_NEG_INF (-__builtin_inff())

__device__ __forceinline__ int symq_code_f(float x, float qmaxf, float amax) {
    float t = x * qmaxf;
    float q = t / amax;  // correctly rounded float32 division
    float r = __builtin_rintf(q);
    r = fminf(fmaxf(r, -qmaxf), qmaxf);
    return (int)r;
}

__device__ __forceinline__ unsigned pack4(int a, int b, int c, int d) {
    return (unsigned)(a & 0xFF) | ((unsigned)(b & 0xFF) << 8) | ((unsigned)(c & 0xFF) << 16) | ((unsigned)(d & 0xFF) << 24);
}

// x / d for a grid's largest code d = 127 or 7, correctly rounded, x >= 0: the quotient by the rounded reciprocal, its remainder (exact) and one
// correction. Compared with the division for every float x from 0 to infinity (tests/host/grid_quotients.cpp; the minimum is for infinity, whose
// remainder is taken of the largest finite quotient). The division itself is 11 dependent instructions, a reciprocal among them, and a
// block has four or five of them in its chain.
__host__ __device__ __forceinline__ float div_grid(float x, float d) {
    const float r = __builtin_bit_cast(unsigned, d) == 0x40e00000u ? 1.0f / 7.0f : 1.0f / 127.0f, q = x * r;
    return __builtin_fmaf(__builtin_fmaf(-fminf(q, 3.402823466e+38f), d, x), r, q);
}

// 1 / pmax, correctly rounded, of the grids' 255, 15 and 256 (the same for all lanes: scalar instructions).
__device__ __forceinline__ float inv_pmax(float pmax) {
    return __float_as_uint(pmax) == 0x41700000u ? 1.0f / 15.0f : __float_as_uint(pmax) == 0x43800000u ? 1.0f / 256.0f : 1.0f / 255.0f;
}

// qmax / amax, refined once: within 0.5 ulp and a little (6.1e-8, relatively).
__device__ __forceinline__ float quant_mult(float qmaxf, float amax) {
    const float r = __builtin_amdgcn_rcpf(amax), c = qmaxf * r;
    return __builtin_fmaf(__builtin_fmaf(-c, amax, qmaxf), r, c);
}

// Settles the values of four whose bytes are flagged by the definition code = rint(fl(t / amax)), t = fl(y * qmax), without the
// division: such a quotient lies beside H = n + copysign(0.5, e) (n: the inner candidate, in pk), so only its side of H matters,
// or whether it rounds to H itself, in which case the even neighbour is taken. s = fma(-H, amax, t) has the exact sign of
// t / amax - H, and the quotient rounds to H while |s| <= amax * (half a unit in the last place of H; half of that on
// the inner side of a power of two, here only 0.5; the end points round to H too, whose last bit is 0).
// A value in 10^5 gets here, but then its whole wavefront waits. One value after the other, in a loop (a lane rarely has
// two at once), keeps the code small.
__device__ __forceinline__ unsigned quant4_ties(unsigned pk, unsigned flags, float x0, float x1, float x2, float x3, float f, float fc, float amax,
                                                float qmaxf) {
#pragma unroll 1
    do {
        const int i = __builtin_ctz(flags) >> 3;
        const float x = i & 2 ? (i & 1 ? x3 : x2) : (i & 1 ? x1 : x0);
        const float n = (float)((int)(pk << (24 - 8 * i)) >> 24);
        const float e = __builtin_fmaf(x, fc, -n);
        const float h = n + copysignf(0.5f, e);
        const float t = (x * f) * qmaxf;
        const float s = __builtin_fmaf(-h, amax, t);
        const float out = h < 0.f ? -s : s;  // positive: beyond H, away from zero
        const float ah = fabsf(h);
        const float u = amax * __uint_as_float((__float_as_uint(ah) & 0x7f800000u) - (24u << 23));
        const int inner = (int)(ah - 0.5f), outer = inner + 1;
        int code = (inner & 1) ? outer : inner;
        code = out > u ? outer : code;
        code = out < -(ah == 0.5f ? 0.5f * u : u) ? inner : code;
        code = h < 0.f ? -code : code;
        const unsigned m = 0xFFu << (8 * i);
        pk = (pk & ~m) | (((unsigned)code << (8 * i)) & m);
        flags &= ~m;
    } while (flags);
    return pk;
}

// Symmetric 8-bit codes of four values y = x * f of one row, packed into a dword (low byte first).
//   exact definition: code = rint((y * qmax) / amax) with IEEE float32 operations (qmax = 127, or 7 for 4-bit Q~).
//   fast path: the defined quotient is within 3 * 2^-24 of y * qmax / amax, relatively (y, where f is not 1, its product and
//   the division, rounded once each), x times fc = f * quant_mult(qmax, amax) within 2^-23 and a little: together less than
//   3.1e-7. The inner and outer products x fc (1 -+ 2^-21) lie 4.1e-7 and more to either side of it; rounding is monotone, so where both round
//   to the same integer the quotient does. fma(x, inner factor, 1.5 * 2^23) rounds the inner one half-to-even to an integer, the constant's low
//   mantissa byte: the code, unless the outer one rounds to another (quant4_fast); then quant4_ties decides. The doubtful zone narrows with
//   the magnitude.
struct QuantRow {
    float f, c, amax;  // c = quant_mult(qmax, amax)
};
__device__ __forceinline__ unsigned quant4_at(float x0, float x1, float x2, float x3, float m) {
    const float magic = 12582912.0f;
    const unsigned lo = __builtin_amdgcn_perm(__float_as_uint(__builtin_fmaf(x1, m, magic)), __float_as_uint(__builtin_fmaf(x0, m, magic)), 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm(__float_as_uint(__builtin_fmaf(x3, m, magic)), __float_as_uint(__builtin_fmaf(x2, m, magic)), 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
// The inner candidates. The outer product less the inner result (the constant plus n), rounded to an integer, is minus the constant, unless it is
// beyond n + 1/2: then a neighbour of it. (On n + 1/2 itself it counts as n: the quotient is on the inner side by more than 1e-7 of it.)
// `doubt`, the OR of them, starts as TAQ_SURE and stays that while no value is in doubt: 13 instructions per four values, two less than
// packing the outer candidates and comparing.
#define TAQ_SURE 0xCB400000u
__device__ __forceinline__ unsigned quant4_fast(float x0, float x1, float x2, float x3, QuantRow r, unsigned& doubt) {
    const float fc = r.f * r.c, magic = 12582912.0f;
    const float in = __builtin_fmaf(fc, -4.76837158203125e-07f, fc), out = __builtin_fmaf(fc, 4.76837158203125e-07f, fc);
    const float t0 = __builtin_fmaf(x0, in, magic), t1 = __builtin_fmaf(x1, in, magic), t2 = __builtin_fmaf(x2, in, magic), t3 = __builtin_fmaf(x3, in, magic);
    doubt |= __float_as_uint(__builtin_fmaf(x0, out, -t0)) | __float_as_uint(__builtin_fmaf(x1, out, -t1));
    doubt |= __float_as_uint(__builtin_fmaf(x2, out, -t2)) | __float_as_uint(__builtin_fmaf(x3, out, -t3));
    const unsigned lo = __builtin_amdgcn_perm(__float_as_uint(t1), __float_as_uint(t0), 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm(__float_as_uint(t3), __float_as_uint(t2), 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
__device__ __forceinline__ unsigned quant4_settle(unsigned pk, float x0, float x1, float x2, float x3, QuantRow r, float qmaxf) {
    const float fc = r.f * r.c;
    const unsigned flags = pk ^ quant4_at(x0, x1, x2, x3, __builtin_fmaf(fc, 4.76837158203125e-07f, fc));
    return flags ? quant4_ties(pk, flags, x0, x1, x2, x3, r.f, fc, r.amax, qmaxf) : pk;
}

// Codes of a row of fp16 values (amax one of them): for most rows one product settles them. |x| 127 / amax = 127 X / (A 2^s) with integer
// significands X, A < 2^11 and s >= 0 is either half an integer H or, relatively, at least 1 / (2 * 127 * 2047) = 1.9e-6 away from one, further
// than c (1 + 2^-21) is from 127 / amax (at most 6e-7). And it is H itself only if 254 X = (2 k + 1) A 2^s: where the prime 127 does not
// divide A, it divides 2 k + 1 <= 254, so H = 63.5, whose even neighbour is the outer one, which that product rounds to. Rows with
// 127 | A, one in 128, are those whose scale amax / 127 is exact; their outer candidates go on to half_row_settle. (Every fp16 amax against
// every fp16 value below it gives the definition's codes: tests/host/grid_quotients.cpp.) 7 instructions per four values instead of 13:
// with div_grid 61.9 -> 60.7 us at 16 requests of 4096 x 320, 10.86 -> 10.78 at 2 x 4096 x 320.
struct HalfRow {
    float m;      // the product's factor
    bool doubt;   // 127 | A
};
__host__ __device__ __forceinline__ HalfRow half_row(float c, float scale, float amax) {  // c = quant_mult(127, amax), scale = amax / 127
    return {__builtin_fmaf(c, 4.76837158203125e-07f, c), __builtin_fmaf(-scale, 127.f, amax) == 0.f};
}

// Four codes of a row with 127 | A from its outer candidates `pk`: the inner ones, and the ties where they differ. (The quantizer begun
// anew for such rows, by quant4_fast and quant4_settle: 73 registers instead of 50 in rowquant_op_kernel, six wavefronts to a SIMD instead of
// eight; 2 x 4096 x 640, us, 5.59 and 5.49 on normal values, 6.44 and 5.72 where every row is one.)
__device__ __forceinline__ unsigned half_row_settle(unsigned pk, float x0, float x1, float x2, float x3, QuantRow r) {
    const unsigned in = quant4_at(x0, x1, x2, x3, __builtin_fmaf(r.c, -4.76837158203125e-07f, r.c)), flags = in ^ pk;
    return flags ? quant4_ties(in, flags, x0, x1, x2, x3, 1.f, r.c, r.amax, 127.f) : pk;
}

// Whether any lane of the wavefront is in doubt: one test for as many values as a wavefront has at hand, and a branch out of line
// that is hardly ever taken. (A test for every four, each jumping over the rare code, cut the arithmetic into pieces of one
// dependent chain each: 15.72 -> 15.37 us at 64 tokens of 1280 channels, 11.48 -> 11.35 us at 2 x 4096 x 320.)
#define TAQ_DOUBT(doubt) __builtin_expect(__builtin_amdgcn_ballot_w64(doubt) != 0ull, 0)

// N dwords of codes, four values x(i) of the row row(i) each; one test for every G of them.
template <int G, int N, typename X, typename R>
__device__ __forceinline__ void quant4_group(unsigned (&pk)[N], X x, R row, float qmaxf = 127.f) {
#pragma unroll
    for (int i0 = 0; i0 < N; i0 += G) {
        unsigned doubt = TAQ_SURE;
#pragma unroll
        for (int i = i0; i < (i0 + G < N ? i0 + G : N); ++i) {
            const float4 v = x(i);
            pk[i] = quant4_fast(v.x, v.y, v.z, v.w, row(i), doubt);
        }
        if (TAQ_DOUBT(doubt != TAQ_SURE)) {
#pragma unroll
            for (int i = i0; i < (i0 + G < N ? i0 + G : N); ++i) {
                const float4 v = x(i);
                pk[i] = quant4_settle(pk[i], v.x, v.y, v.z, v.w, row(i), qmaxf);
            }
        }
    }
}

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

// Wait states between 32-deep fp16 products and the 16-deep ones that go on with their sums `a`. The compiler places none, as if a
// 16-deep product could take such a sum over while it is being formed; on gfx950 one that came 1 to 3 instructions behind found, now and
// then, only part of it: two of the four rows of a lane without the last product, 1e-4 of the result. 5 instructions were enough wherever
// they stood; these are 8, as many as the compiler places in front of every other reader of a 32-deep product (a vector instruction, an A or B
// operand). They stand in front of every such product, also where today's compiler leaves more instructions than that in
// between: it promises none of them. At 2 x 4096 x 640, ten heads, they cost 0.1 of 21 us, elsewhere nothing measurable.
// tests/test_sum_depth.py looks at the generated code.
template <int M, int N>
__device__ __forceinline__ void sums_settle(floatx4_t (&a)[M][N]) {
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) asm volatile("" : "+v"(a[i][j]));
    asm volatile("s_nop 7");
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j) asm volatile("" : "+v"(a[i][j]));
}

// All-reduce over the four quarter-wave lanes that hold one image token (l, l^16, l^32, l^48) with the
// gfx950 row / half-wave swaps: no LDS round trip.
__device__ __forceinline__ float quad_allmax(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_allsum(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// Maximum over 8 neighbouring lanes (DPP: xor 1, xor 2, mirror within 8), and over the 16 of a row (mirror within 16).
__device__ __forceinline__ float row8_allmax(float x) {
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0xB1, 0xF, 0xF, true)));
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x4E, 0xF, 0xF, true)));
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x141, 0xF, 0xF, true)));
    return x;
}
__device__ __forceinline__ float row16_allmax(float x) {
    x = row8_allmax(x);
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x140, 0xF, 0xF, true)));
    return x;
}

// x, and the compiler does not know it: what is computed from it is computed here and not kept from elsewhere.
__device__ __forceinline__ int opaque(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Two values in [0, 1] as fp16 high parts (truncated) and remainders, at i and i + 1 of two operands. (High parts by the conversion
// intrinsic: the value that enters the MFMA is the one subtracted, whatever the compiler would pick for a plain cast.)
__device__ __forceinline__ void split_half2(float e0, float e1, half4_t& hi, half4_t& lo, int i) {
    const auto w = __builtin_amdgcn_cvt_pkrtz(e0, e1);
    const _Float16 h0 = (_Float16)w[0], h1 = (_Float16)w[1];
    typedef float float2_t __attribute__((ext_vector_type(2)));
    const half2_t l = __builtin_convertvector((float2_t){e0 - (float)h0, e1 - (float)h1}, half2_t);
    hi[i] = h0;
    hi[i + 1] = h1;
    lo[i] = l[0];
    lo[i + 1] = l[1];
}

// Four biased bytes (code + 128) -> four fp16 codes: 0x6400 | byte is the fp16 number 1152 + code.
__device__ __forceinline__ void biased4_to_half(unsigned w, half2_t& a, half2_t& b) {
    const unsigned lo = __builtin_amdgcn_perm(0x64646464u, w, 0x04010400u);
    const unsigned hi = __builtin_amdgcn_perm(0x64646464u, w, 0x04030402u);
    const half2_t off = {(_Float16)1152.0f, (_Float16)1152.0f};
    a = *reinterpret_cast<const half2_t*>(&lo) - off;
    b = *reinterpret_cast<const half2_t*>(&hi) - off;
}

// Integer sums that become floats: started at the bits of 1.5 * 2^23, a sum below 2^22 is, read as a float, that constant plus the sum, and a
// subtraction leaves the sum. With two or more wavefronts to a SIMD, additions, products and bit operations on float32 registers and literals
// take 2.2 clocks of it, conversions, maxima, comparisons, selects, permutations, packed fp16 and anything with a scalar register operand 4
// (selects by vcc in a row 22), exponentials and lane swaps 8. Sums of scores stay below 127 * 127 * TAQ_MAX_D < 2^22; those of projections need
// not. This, no selects for rows past a head and protected rows by bounds-checked loads, us: 16 requests of 4096 x 320 59.4 -> 58.6,
// 2 x 4096 x 640 20.8 -> 20.7, the layers of a UNet step of 8 x 96 x 64 649 -> 642.
static_assert(127 * 127 * TAQ_MAX_D < 1 << 22, "sums of scores as the mantissa of a float");
__device__ __forceinline__ int32x4_t sum_start() { return (int32x4_t){0x4B400000, 0x4B400000, 0x4B400000, 0x4B400000}; }
__device__ __forceinline__ float sum_float(int s) { return __int_as_float(s) - 12582912.0f; }

// 4 x 4 transpose of dwords between four registers and the four quarters of the wavefront: afterwards register k of a lane
// in quarter q holds what register q of the same lane in quarter k held.
__device__ __forceinline__ void quad_transpose(unsigned (&r)[4]) {
    const auto s02 = __builtin_amdgcn_permlane32_swap(r[0], r[2], false, false);
    const auto s13 = __builtin_amdgcn_permlane32_swap(r[1], r[3], false, false);
    const auto r01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
    const auto r23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
    r[0] = r01[0];
    r[1] = r01[1];
    r[2] = r23[0];
    r[3] = r23[1];
}

// Maximum over all 64 lanes.
__device__ __forceinline__ float wave_allmax(float x) { return quad_allmax(row16_allmax(x)); }

// Q~ codes of a (token tile, head), TPH dwords a lane, lie in units of as many 16-channel blocks as a wavefront of to_q holds at least:
// within a unit four blocks by four, a lane's four dwords together, then the one to three that are left. Both sides move whole pieces of
// memory with the widest accesses (blocks of one dword a lane: 10 loads at 160 channels; units cut by a wavefront's share: 1 us more
// for to_q there).
template <int TPH>
struct QPlace {
    static constexpr int UNIT = TPH == 4 ? 2 : TPH >= 6 && TPH % 2 == 0 ? TPH / 2 : TPH;
    static __device__ __forceinline__ int at(int j, int lane) {
        const int u = j / UNIT * UNIT, k = j - u, full = UNIT & ~3, rest = UNIT & 3;
        return 64 * u + (k < full ? (k & ~3) * 64 + lane * 4 + (k & 3) : full * 64 + lane * rest + (k - full));
    }
};

}  // namespace taq
