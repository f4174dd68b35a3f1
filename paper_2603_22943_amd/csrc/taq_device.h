// Device helpers shared by the kernels: operand vector types, the exact quantizer's fast path, reductions over the lanes
// of a wavefront that hold one row, byte-to-fp16 conversion (gfx950 only).
#pragma once
#include "taq_internal.h"

namespace taq {

typedef int int32x4_t __attribute__((ext_vector_type(4)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
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

// Symmetric 8-bit codes of four values of one row, packed into a dword (low byte first).
//   exact definition: code = rint((x * qmax) / amax) with IEEE float32 multiply and divide (qmax = 127, or 7 for
//   4-bit Q~; the bounds below are stated for 127 and only shrink for 7).
//   fast path: with c = quant_mult(qmax, amax) (within 0.5 ulp and a little of qmax / amax: 6.1e-8, relatively),
//   m = fma(x, c, 1.5 * 2^23) is the EXACT product x * c rounded half-to-even to an integer (plus the magic constant,
//   whose low mantissa byte is then the code's byte), and e = fma(x, c, -(m - magic)) is the distance of that exact
//   product from the integer. x * c lies within 7.7e-6 of the exact ratio (|ratio| <= 127), the defined quotient within
//   7.6e-6 (its product, rounded once; exact where x is fp16 and qmax 127) + 3.8e-6 (half a last place below 128), so
//   both round to the same integer unless x * c is within 1.9e-5 (fp16 rows: 1.15e-5) of a half-integer; values beyond
//   TAQ_TIE (TAQ_TIE_F16) are settled by quant4_ties.
#define TAQ_TIE 0.49997f
#define TAQ_TIE_F16 0.49998f

__device__ __forceinline__ float quant_mult(float qmaxf, float amax) {  // qmax / amax, refined once
    const float r = __builtin_amdgcn_rcpf(amax), c = qmaxf * r;
    return __builtin_fmaf(__builtin_fmaf(-c, amax, qmaxf), r, c);
}

// Settles the flagged values of four by the definition code = rint(fl(t / amax)), t = fl(y * qmax), without the division:
// such a quotient lies beside H = n + copysign(0.5, e) (n: the fast path's integer), so only its side of H matters, or
// whether it rounds to H itself, in which case the even neighbour is taken. s = fma(-H, amax, t) has the exact sign of
// t / amax - H, and the quotient rounds to H while |s| <= amax * (half a unit in the last place of H; half of that on
// the inner side of a power of two, here only 0.5; the end points round to H too, whose last bit is 0).
// A value in 2 * 10^4 gets here, but then its whole wavefront waits. One value after the other, in a loop (a lane rarely has
// two at once), keeps the code small.
__device__ __forceinline__ unsigned quant4_ties(unsigned pk, bool f0, bool f1, bool f2, bool f3, float x0, float x1, float x2, float x3,
                                                float f, float fc, float amax, float qmaxf) {
    unsigned flags = (f0 ? 1u : 0u) | (f1 ? 2u : 0u) | (f2 ? 4u : 0u) | (f3 ? 8u : 0u);
#pragma unroll 1
    do {
        const int i = __builtin_ctz(flags);
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
        flags &= flags - 1;
    } while (flags);
    return pk;
}

__device__ __forceinline__ unsigned quant4_i8(float x0, float x1, float x2, float x3, float c, float amax,
                                              float qmaxf = 127.f, float tie = TAQ_TIE) {
    const float magic = 12582912.0f;
    const float m0 = __builtin_fmaf(x0, c, magic), m1 = __builtin_fmaf(x1, c, magic);
    const float m2 = __builtin_fmaf(x2, c, magic), m3 = __builtin_fmaf(x3, c, magic);
    const float e0 = __builtin_fmaf(x0, c, magic - m0), e1 = __builtin_fmaf(x1, c, magic - m1);
    const float e2 = __builtin_fmaf(x2, c, magic - m2), e3 = __builtin_fmaf(x3, c, magic - m3);
    const unsigned lo = __builtin_amdgcn_perm(__float_as_uint(m1), __float_as_uint(m0), 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm(__float_as_uint(m3), __float_as_uint(m2), 0x0c0c0400u);
    unsigned pk = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    if (fmaxf(fmaxf(fabsf(e0), fabsf(e1)), fmaxf(fabsf(e2), fabsf(e3))) > tie)
        pk = quant4_ties(pk, fabsf(e0) > tie, fabsf(e1) > tie, fabsf(e2) > tie, fabsf(e3) > tie, x0, x1, x2, x3, 1.f, c, amax, qmaxf);
    return pk;
}

// The same for values x_i * f whose products have not been formed yet (f > 0 common to the four): the fast path rounds
// the exact product x * (f * c), f * c rounded once, which adds 7.6e-6, as does the rounding in y = fl(x * f): the two
// agree unless the product is within 3.5e-5 of a half-integer.
__device__ __forceinline__ unsigned quant4_i8_scaled(float x0, float x1, float x2, float x3, float f, float c, float amax) {
    constexpr float tie = 0.49996f;
    const float magic = 12582912.0f;
    const float fc = f * c;
    const float m0 = __builtin_fmaf(x0, fc, magic), m1 = __builtin_fmaf(x1, fc, magic);
    const float m2 = __builtin_fmaf(x2, fc, magic), m3 = __builtin_fmaf(x3, fc, magic);
    const float e0 = __builtin_fmaf(x0, fc, magic - m0), e1 = __builtin_fmaf(x1, fc, magic - m1);
    const float e2 = __builtin_fmaf(x2, fc, magic - m2), e3 = __builtin_fmaf(x3, fc, magic - m3);
    const unsigned lo = __builtin_amdgcn_perm(__float_as_uint(m1), __float_as_uint(m0), 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm(__float_as_uint(m3), __float_as_uint(m2), 0x0c0c0400u);
    unsigned pk = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    if (fmaxf(fmaxf(fabsf(e0), fabsf(e1)), fmaxf(fabsf(e2), fabsf(e3))) > tie)
        pk = quant4_ties(pk, fabsf(e0) > tie, fabsf(e1) > tie, fabsf(e2) > tie, fabsf(e3) > tie, x0, x1, x2, x3, f, fc, amax, 127.f);
    return pk;
}

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

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
// Maximum over the 16 lanes of a row (DPP: xor 1, xor 2, mirror within 8, mirror within 16).
__device__ __forceinline__ float row16_allmax(float x) {
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0xB1, 0xF, 0xF, true)));
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x4E, 0xF, 0xF, true)));
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x141, 0xF, 0xF, true)));
    x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x140, 0xF, 0xF, true)));
    return x;
}

// Four biased bytes (code + 128) -> four fp16 codes: 0x6400 | byte is the fp16 number 1152 + code.
__device__ __forceinline__ void biased4_to_half(unsigned w, half2_t& a, half2_t& b) {
    const unsigned lo = __builtin_amdgcn_perm(0x64646464u, w, 0x04010400u);
    const unsigned hi = __builtin_amdgcn_perm(0x64646464u, w, 0x04030402u);
    const half2_t off = {(_Float16)1152.0f, (_Float16)1152.0f};
    a = *reinterpret_cast<const half2_t*>(&lo) - off;
    b = *reinterpret_cast<const half2_t*>(&hi) - off;
}

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

}  // namespace taq
