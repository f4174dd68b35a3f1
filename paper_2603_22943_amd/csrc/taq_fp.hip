// Full-precision stages of libtaq (gfx950): what runs when shape.bits_proj, bits_q or bits_prob is 16, i.e. when a
// projection, Q~ or the probabilities of PersonalQ's Eq. (2) / Eq. (3) are to stay unquantized. These modes exist for
// reference runs (Eq. (1): "all other parameters and activations in full precision"; the identity "every row protected,
// nothing quantized = plain softmax attention"): float32 arithmetic, one simple kernel per stage.
#include "taq_device.h"

namespace taq {

typedef float fp_floatx4_t __attribute__((ext_vector_type(4)));
typedef int fp_int4_t __attribute__((ext_vector_type(4)));
typedef __bf16 fp_bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 fp_half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 fp_half8_t __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- out[m][n] = sum_k A[m][k] * W[n][k]  (+ bias[n])
// A: f16 or f32 [M][K]; W: f16 [N][K] (out x in, as the projections are stored); float32 accumulation.

// fp16 rows whose sums feed a quantizer: one float32 FMA chain per output in K order, so that a sum, and with it a code,
// is the same number whatever the tiling (products of fp16 numbers are exact; v_fma_mix reads the fp16 operands as they
// are). 8 TM x 64 outputs per workgroup, TM x 2 per thread (columns tx, tx + 32). Chunks of 64 k in two LDS buffers, rows of 144 bytes: a
// thread reads eight k of a row at a time, without conflicts, TM + 2 reads for 16 TM FMAs. The next chunk travels in registers.
// Bound by vector issue. One wavefront of a SIMD issues an instruction every 8.6 clocks, two and more one in 4.3, so with few rows the
// tile is the small one, TM = 2: 154 x 2 x 1280 x 768 are 400 workgroups, 1.6 wavefronts to a SIMD, 19.2 us; with TM = 4 200 workgroups and 26.3.
// With many rows TM = 4 reads less per FMA (gemm_seq_rows: where the line lies); 128 columns instead of twice the rows, 4 x 64 outputs to
// a wavefront and 132 registers, are 1 to 20 % slower from 500 small workgroups to 11000.
// With TM = 2 half of the threads load a row of A that another holds already, and the last two chunks are loaded for nothing: behind a
// condition the loads no longer lie between the FMAs (154 x 1280 x 1280 20.6 and 24.9 us, 4096 x 320 x 320 17.1 and 17.4, equal from 2500
// workgroups on).
// blockIdx.z = 1: a second matrix W1 of the same size, results `N` columns further (K and V of a context in one launch).
template <int TM>
__global__ __launch_bounds__(256) void gemm_nt_seq_kernel(const __half* __restrict__ A, const __half* __restrict__ W0,
                                                          const __half* __restrict__ W1, const float* __restrict__ bias, int M,
                                                          int N, int K, float* __restrict__ out_f32, __half* __restrict__ out_f16,
                                                          int ldo) {
    constexpr int TN = 2, KC = 64, RS = KC + 8;
    __shared__ __align__(16) __half As[2][8 * TM * RS], Ws[2][32 * TN * RS];
    const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5;
    const int m0 = blockIdx.x * 8 * TM, n0 = blockIdx.y * 32 * TN;
    const __half* W = blockIdx.z ? W1 : W0;
    const int cz = blockIdx.z ? N : 0;
    const int lr = tid >> 3, ls = (tid & 7) * 8;  // staging: rows lr and lr + 32 of W, eight halves from ls
    const int la = lr % (8 * TM);  // its row of A
    const __half* ag = A + (size_t)(m0 + la < M ? m0 + la : M - 1) * K;
    const __half* wg[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) wg[j] = W + (size_t)(n0 + 32 * j + lr < N ? n0 + 32 * j + lr : N - 1) * K;
    fp_int4_t av, wv[TN];
    auto fetch = [&](int k0) {  // (K % 32 == 0: the last chunk may be half; what lies past the end is not read back)
        const int k = k0 + ls < K ? k0 + ls : 0;
        av = *reinterpret_cast<const fp_int4_t*>(ag + k);
#pragma unroll
        for (int j = 0; j < TN; ++j) wv[j] = *reinterpret_cast<const fp_int4_t*>(wg[j] + k);
    };
    auto store = [&](int s) {
        if (TM == 4 || tid < 128) *reinterpret_cast<fp_int4_t*>(&As[s][lr * RS + ls]) = av;
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<fp_int4_t*>(&Ws[s][(32 * j + lr) * RS + ls]) = wv[j];
    };
    float acc[TM][TN] = {};
    fetch(0);
    store(0);
    fetch(KC);
    for (int k0 = 0, s = 0; k0 < K; k0 += KC, s ^= 1) {
        __syncthreads();  // chunk s is in LDS, and everybody is done with the other one
        if (k0 + KC < K) store(s ^ 1);
        fetch(k0 + 2 * KC);
#pragma unroll
        for (int k = 0; k < KC; k += 8) {
            if (k == KC / 2 && k0 + k >= K) break;
            fp_half8_t a[TM], w[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const fp_half8_t*>(&As[s][(ty + 8 * i) * RS + k]);
#pragma unroll
            for (int j = 0; j < TN; ++j) w[j] = *reinterpret_cast<const fp_half8_t*>(&Ws[s][(tx + 32 * j) * RS + k]);
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_fmaf((float)a[i][e], (float)w[j][e], acc[i][j]);
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + ty + 8 * i;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + tx + 32 * j;
            if (n >= N) continue;
            const float y = acc[i][j] + (bias ? bias[n] : 0.f);
            if (out_f32) out_f32[(size_t)m * ldo + cz + n] = y;
            if (out_f16) out_f16[(size_t)m * ldo + cz + n] = __float2half_rn(y);
        }
    }
}

static void launch_gemm_seq(const __half* A, const __half* W0, const __half* W1, const float* bias, int M, int N, int K, float* out_f32,
                            __half* out_f16, int ldo, hipStream_t st) {
    const unsigned ny = (N + 63) / 64, z = W1 ? 2 : 1;
    if (gemm_seq_rows(M, N, z) == 16)
        hipLaunchKernelGGL(gemm_nt_seq_kernel<2>, dim3((M + 15) / 16, ny, z), dim3(256), 0, st, A, W0, W1, bias, M, N, K, out_f32, out_f16, ldo);
    else
        hipLaunchKernelGGL(gemm_nt_seq_kernel<4>, dim3((M + 31) / 32, ny, z), dim3(256), 0, st, A, W0, W1, bias, M, N, K, out_f32, out_f16, ldo);
}

// Matrix-core versions, for sums that feed no quantizer. All stage rows of A and of W through LDS, in K steps of KC, the
// next step in registers while the current one is multiplied: loaded in operand order straight from
// row-major memory (lane = row + 16 * segment) every lane of a load is a cache access of its own, 64 instead of 16 per KiB,
// and that, not the matrix cores, was the time (512 x 1280 per head slice, 8 heads: 45 us so, 24 us through LDS).

// fp16 rows: V_MFMA_F32_16X16X32_F16 (products of fp16 numbers are exact in float32). 32 MI x 32 MI outputs per workgroup of four
// wavefronts, 16 MI x 16 MI each; every output is one chain of products in K order, whatever the tile. K % 32 == 0.
// A step is as long as a load takes, so with few outputs small tiles and long steps: 512 x 1280 x 1280 as 640 workgroups of
// 32 x 32 and ten steps 10.1 us, as 160 of 64 x 64 and twenty steps 12.0 (gemm_f16_small: where the line lies).
template <int MI, int KC>
__global__ __launch_bounds__(256) void gemm_nt_f16_kernel(const __half* __restrict__ A, const __half* __restrict__ W, int M, int N, int K,
                                                          float* __restrict__ out) {
    // row stride in halves: 144 or 272 bytes (with 272 a third of the LDS clocks are conflicts, 320 of a wavefront's 960 at 512 x 1280 x 1280)
    constexpr int TILE = 32 * MI, RS = KC + 8;
    constexpr int TR = KC / 8, RPP = 256 / TR, NL = TILE / RPP;  // staging: threads per row, rows at a time, loads per thread and operand
    static_assert(TILE % RPP == 0, "whole loads");
    __shared__ __align__(16) __half As[2][TILE * RS], Ws[2][TILE * RS];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.x * TILE, n0 = blockIdx.y * TILE;
    const int lr = tid / TR, ls = (tid % TR) * 8;  // rows lr, lr + RPP, ..., eight halves from ls
    const __half* ag[NL];
    const __half* wg[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {  // rows past the end re-read the last one; their results are dropped
        const int m = m0 + lr + RPP * i, n = n0 + lr + RPP * i;
        ag[i] = A + (size_t)(m < M ? m : M - 1) * K;
        wg[i] = W + (size_t)(n < N ? n : N - 1) * K;
    }
    fp_int4_t av[NL], wv[NL];
    bool in;
    auto fetch = [&](int k0) {  // (the last step may be partly filled: zeros past the end, set when the step is stored)
        in = k0 + ls < K;
        const int k = in ? k0 + ls : 0;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            av[i] = *reinterpret_cast<const fp_int4_t*>(ag[i] + k);
            wv[i] = *reinterpret_cast<const fp_int4_t*>(wg[i] + k);
        }
    };
    const fp_int4_t zero = {0, 0, 0, 0};  // (a vector: selects; of a struct of four they become branches around the stores, 0.1 to 1.2 us a call)
    auto store = [&](int s) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            *reinterpret_cast<fp_int4_t*>(&As[s][(lr + RPP * i) * RS + ls]) = in ? av[i] : zero;
            *reinterpret_cast<fp_int4_t*>(&Ws[s][(lr + RPP * i) * RS + ls]) = in ? wv[i] : zero;
        }
    };
    const int wm = (wave & 1) * 16 * MI, wn = (wave >> 1) * 16 * MI;
    fp_floatx4_t acc[MI][MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) acc[i][j] = (fp_floatx4_t){0.f, 0.f, 0.f, 0.f};
    fetch(0);
    store(0);
    fetch(KC);
    for (int k0 = 0, s = 0; k0 < K; k0 += KC, s ^= 1) {
        __syncthreads();  // step s is in LDS, and everybody is done with the other one
        if (k0 + KC < K) store(s ^ 1);
        fetch(k0 + 2 * KC);
#pragma unroll
        for (int u = 0; u < KC / 32; ++u) {
            fp_half8_t a[MI], w[MI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                a[i] = *reinterpret_cast<const fp_half8_t*>(&As[s][(wm + 16 * i + r16) * RS + 32 * u + 8 * q]);
                w[i] = *reinterpret_cast<const fp_half8_t*>(&Ws[s][(wn + 16 * i + r16) * RS + 32 * u + 8 * q]);
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < MI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[i], a[j], acc[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < MI; ++j) {
        const int m = m0 + wm + 16 * j + r16;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int n = n0 + wn + 16 * i + 4 * q;  // N % 4 == 0: the four channels are in or out together
            if (m < M && n < N)
                *reinterpret_cast<float4*>(out + (size_t)m * N + n) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        }
    }
}

// float32 rows: V_MFMA_F32_16X16X4_F32, float32 operands throughout. 64 rows x 64 channels per workgroup, a wavefront
// owns 16 rows. The contraction order within 16 consecutive k is free, so a lane takes four of them with one read and
// feeds them to four MFMAs. K % 8 == 0.
__global__ __launch_bounds__(256) void gemm_nt_f32_kernel(const float* __restrict__ A, const __half* __restrict__ W,
                                                          const float* __restrict__ bias, int M, int N, int K,
                                                          float* __restrict__ out_f32, __half* __restrict__ out_f16, size_t ldo) {
    constexpr int KC = 32, RA = KC + 4, RW = KC + 4;  // row strides: 144 bytes of floats, 72 bytes of halves
    __shared__ __align__(16) float As[2][64 * RA];
    __shared__ __align__(16) __half Ws[2][64 * RW];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    const int lr = tid >> 3, ls = (tid & 7) * 4;  // staging: rows lr, lr + 32, four values from ls
    const float* ag[2];
    const __half* wg[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = m0 + lr + 32 * i, n = n0 + lr + 32 * i;
        ag[i] = A + (size_t)(m < M ? m : M - 1) * K;
        wg[i] = W + (size_t)(n < N ? n : N - 1) * K;
    }
    float4 av[2];
    uint2 wv[2];
    bool in;
    auto fetch = [&](int k0) {
        in = k0 + ls < K;
        const int k = in ? k0 + ls : 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            av[i] = *reinterpret_cast<const float4*>(ag[i] + k);
            wv[i] = *reinterpret_cast<const uint2*>(wg[i] + k);
        }
    };
    auto store = [&](int s) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *reinterpret_cast<float4*>(&As[s][(lr + 32 * i) * RA + ls]) = in ? av[i] : make_float4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<uint2*>(&Ws[s][(lr + 32 * i) * RW + ls]) = in ? wv[i] : make_uint2(0u, 0u);
        }
    };
    fp_floatx4_t acc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = (fp_floatx4_t){0.f, 0.f, 0.f, 0.f};
    fetch(0);
    store(0);
    fetch(KC);
    for (int k0 = 0, s = 0; k0 < K; k0 += KC, s ^= 1) {
        __syncthreads();
        if (k0 + KC < K) store(s ^ 1);
        fetch(k0 + 2 * KC);
#pragma unroll
        for (int u = 0; u < KC / 16; ++u) {
            if (k0 + 16 * u >= K) break;
            const float4 a4 = *reinterpret_cast<const float4*>(&As[s][(16 * wave + r16) * RA + 16 * u + 4 * q]);
            const float ae[4] = {a4.x, a4.y, a4.z, a4.w};
            float we[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint2 w = *reinterpret_cast<const uint2*>(&Ws[s][(16 * i + r16) * RW + 16 * u + 4 * q]);
                const float2 w01 = __half22float2(*reinterpret_cast<const __half2*>(&w.x));
                const float2 w23 = __half22float2(*reinterpret_cast<const __half2*>(&w.y));
                we[i][0] = w01.x; we[i][1] = w01.y; we[i][2] = w23.x; we[i][3] = w23.y;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(we[i][e], ae[e], acc[i], 0, 0, 0);
        }
    }
    const int m = m0 + 16 * wave + r16;
    if (m >= M) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int n = n0 + 16 * i + 4 * q;
        if (n >= N) continue;
        float4 y = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
        if (bias) {
            const float4 b4 = *reinterpret_cast<const float4*>(bias + n);
            y = make_float4(y.x + b4.x, y.y + b4.y, y.z + b4.z, y.w + b4.w);
        }
        const size_t at = (size_t)m * ldo + n;
        if (out_f32) *reinterpret_cast<float4*>(out_f32 + at) = y;
        if (out_f16) {
            __half2* o = reinterpret_cast<__half2*>(out_f16 + at);
            o[0] = __floats2half2_rn(y.x, y.y);
            o[1] = __floats2half2_rn(y.z, y.w);
        }
    }
}

// The same products, a slice of the contraction per head, for finite float32 rows and without bias, on V_MFMA_F32_16X16X32_BF16. Three bfloat16
// numbers hold the 24 bits of a float32 and two the 11 bits of an fp16 weight (each the leading 8 bits of what the ones before left: no
// rounding), so six exact products stand for each product of before: 96 clocks of the matrix core for 16 x 16 x 32, against 256 of
// V_MFMA_F32_16X16X4_F32, and no conversions beside the products. Sums are float32 as before, the small products of a step first.
// 64 x 64 outputs per workgroup of four wavefronts, 32 x 32 each; what a step of 32 k needs is split when it is stored in LDS (80 bytes to
// a row). Half of the LDS clocks are conflicts, 400 of a wavefront's 800 at 512 x 1280 in heads of 160: the stores, eight bytes a lane, wrap
// the last of four rows, which lie 20 dwords apart, onto the first one's banks. One buffer of 25 KiB, so that five workgroups share a compute unit:
// 512 x 1280, eight heads of 160, are 1280 of them, all at once. 24.5 -> 17.0 us (with two buffers, three to a unit, 19.7). Relative error against
// float64 at heads of 32, 40, 80 and 160: 1.0e-7, 1.1e-7, 1.6e-7, 2.3e-7 before, 0.4e-7, 0.6e-7, 1.0e-7, 1.6e-7 so; largest, over the sum of
// magnitudes, 3.3e-7 and 2.4e-7.
__global__ __launch_bounds__(256) void gemm_nt_split_kernel(const float* __restrict__ A, const __half* __restrict__ W, int M, int N, int K, int Kz,
                                                            float* __restrict__ out, size_t ldo) {
    constexpr int KC = 32, RS = KC + 8;
    __shared__ __align__(16) unsigned short As[3][64 * RS], Ws[2][64 * RS];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    const int lr = tid >> 3, ls = (tid & 7) * 4;  // staging: rows lr, lr + 32, four values from ls
    const float* ag[2];
    const __half* wg[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {  // rows past the end re-read the last one; their results are dropped
        const int m = m0 + lr + 32 * i, n = n0 + lr + 32 * i;
        ag[i] = A + (size_t)(m < M ? m : M - 1) * K + blockIdx.z * Kz;
        wg[i] = W + (size_t)(n < N ? n : N - 1) * K + blockIdx.z * Kz;
    }
    fp_floatx4_t av[2];
    fp_half4_t wv[2];
    bool in;
    auto fetch = [&](int k0) {
        in = k0 + ls < Kz;
        const int k = in ? k0 + ls : 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            av[i] = *reinterpret_cast<const fp_floatx4_t*>(ag[i] + k);
            wv[i] = *reinterpret_cast<const fp_half4_t*>(wg[i] + k);
        }
    };
    // the leading 8 bits of four numbers, which become what they leave
    auto lead = [](float (&x)[4]) {
        unsigned u[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            u[e] = __float_as_uint(x[e]);
            x[e] -= __uint_as_float(u[e] & 0xffff0000u);
        }
        return make_uint2(__builtin_amdgcn_perm(u[1], u[0], 0x07060302u), __builtin_amdgcn_perm(u[3], u[2], 0x07060302u));
    };
    auto store = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            float x[4], w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] = in ? av[i][e] : 0.f;
                w[e] = in ? (float)wv[i][e] : 0.f;
            }
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<uint2*>(&As[p][(lr + 32 * i) * RS + ls]) = lead(x);
#pragma unroll
            for (int p = 0; p < 2; ++p) *reinterpret_cast<uint2*>(&Ws[p][(lr + 32 * i) * RS + ls]) = lead(w);
        }
    };
    const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
    fp_floatx4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (fp_floatx4_t){0.f, 0.f, 0.f, 0.f};
    fetch(0);
    for (int k0 = 0; k0 < Kz; k0 += KC) {
        if (k0 > 0) __syncthreads();  // everybody is done with the step before
        store();
        fetch(k0 + KC);
        __syncthreads();
        fp_bf16x8_t a[3][2], w[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int p = 0; p < 3; ++p) a[p][i] = *reinterpret_cast<const fp_bf16x8_t*>(&As[p][(wm + 16 * i + r16) * RS + 8 * q]);
#pragma unroll
            for (int p = 0; p < 2; ++p) w[p][i] = *reinterpret_cast<const fp_bf16x8_t*>(&Ws[p][(wn + 16 * i + r16) * RS + 8 * q]);
        }
#pragma unroll
        for (int o = 3; o >= 0; --o)  // a[pa] w[pw], pa + pw = o
#pragma unroll
            for (int pw = 1; pw >= 0; --pw) {
                const int pa = o - pw;
                if (pa < 0 || pa > 2) continue;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[pw][i], a[pa][j], acc[i][j], 0, 0, 0);
            }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int m = m0 + wm + 16 * j + r16;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int n = n0 + wn + 16 * i + 4 * q;  // N % 4 == 0: the four channels are in or out together
            if (m < M && n < N) *reinterpret_cast<fp_floatx4_t*>(out + (size_t)m * ldo + (size_t)blockIdx.z * N + n) = acc[i][j];
        }
    }
}

hipError_t launch_gemm_fp(const void* A, bool a_is_f32, const __half* W, const float* bias, int M, int N, int K,
                          float* out_f32, __half* out_f16, int ldo, hipStream_t st) {
    const dim3 grid((M + 63) / 64, (N + 63) / 64), block(256);
    if (a_is_f32)
        hipLaunchKernelGGL(gemm_nt_f32_kernel, grid, block, 0, st, static_cast<const float*>(A), W, bias, M, N, K, out_f32, out_f16, (size_t)ldo);
    else
        launch_gemm_seq(static_cast<const __half*>(A), W, nullptr, bias, M, N, K, out_f32, out_f16, ldo, st);
    return hipGetLastError();
}

hipError_t launch_gemm_kv_rows(const __half* context, const __half* Wk, const __half* Wv, int M, int C, int K, float* rows_f, hipStream_t st) {
    launch_gemm_seq(context, Wk, Wv, nullptr, M, C, K, rows_f, nullptr, 2 * C, st);
    return hipGetLastError();
}

hipError_t launch_gemm_f16(const __half* A, const __half* W, int M, int N, int K, float* out, hipStream_t st) {
    if (gemm_f16_small(M, N))
        hipLaunchKernelGGL((gemm_nt_f16_kernel<1, 128>), dim3((M + 31) / 32, (N + 31) / 32), dim3(256), 0, st, A, W, M, N, K, out);
    else
        hipLaunchKernelGGL((gemm_nt_f16_kernel<2, 64>), dim3((M + 63) / 64, (N + 63) / 64), dim3(256), 0, st, A, W, M, N, K, out);
    return hipGetLastError();
}

hipError_t launch_gemm_f32_heads(const float* A, const __half* W, int M, int N, int K, int H, float* out, hipStream_t st) {
    hipLaunchKernelGGL(gemm_nt_split_kernel, dim3((M + 63) / 64, (N + 63) / 64, H), dim3(256), 0, st, A, W, M, N, K, K / H, out, (size_t)H * N);
    return hipGetLastError();
}

// ---------------------------------------------------------------- protected rows from float32 projection rows
// rows_f [B*T][2C] (K channels then V channels of every text token) -> K16, V16 (compacted by slot) and the transposed
// V16T [B][C][96], one rounding to fp16; unused slots and the padding of V16T read as zeros. One workgroup per
// (slot, batch element).
__global__ __launch_bounds__(256) void kv_rows_from_f32_kernel(const float* __restrict__ rows_f, const int* __restrict__ ntrig,
                                                               const int* __restrict__ trig_idx, int T, int C,
                                                               __half* __restrict__ k16, __half* __restrict__ v16,
                                                               __half* __restrict__ v16t) {
    const int slot = blockIdx.x, b = blockIdx.y;
    const bool live = slot < ntrig[b];
    const int t = live ? trig_idx[b * T + slot] : 0;
    for (int c = threadIdx.x; c < 2 * C; c += 256) {
        const __half y = live ? __float2half_rn(rows_f[((size_t)b * T + t) * 2 * C + c]) : __float2half(0.f);
        if (c < C) {
            k16[((size_t)b * T + slot) * C + c] = y;
        } else {
            v16[((size_t)b * T + slot) * C + (c - C)] = y;
            v16t[((size_t)b * C + (c - C)) * 96 + slot] = y;
            if (slot == T - 1)
                for (int sp = T; sp < 96; ++sp) v16t[((size_t)b * C + (c - C)) * 96 + sp] = __float2half(0.f);
        }
    }
}

hipError_t launch_kv_rows_from_f32(const float* rows_f, const int* ntrig, const int* trig_idx, int B, int T, int C,
                                   __half* k16, __half* v16, __half* v16t, hipStream_t st) {
    hipLaunchKernelGGL(kv_rows_from_f32_kernel, dim3(T, B), dim3(256), 0, st, rows_f, ntrig, trig_idx, T, C, k16, v16, v16t);
    return hipGetLastError();
}

// ---------------------------------------------------------------- attention with unquantized Q and / or probabilities
// A = softmax(Q~ K~^T * sigma), Eq. (3), O = A^ V~ in float32, for any mix of bits_q in {4, 8, 16} and bits_prob in
// {4, 8, 16} and the three probability grids. K~ and V~ (Eq. 2) are expanded to float32 in LDS: s * code for unprotected
// rows, the fp16 row for protected ones. One workgroup per (16 image tokens, head, batch element); a wavefront takes four
// tokens in turn, lanes over text tokens for the scores and the softmax, lanes over channels for A^ V~.
struct FpAttnArgs {
    const float* q_f;       // [B*N][C]  unquantized Q (bits_q = 16)
    const int8_t* q_code;   // [B*N][C]  Q~ codes and scales otherwise
    const float* s_q;       // [B*N][H]
    const uint8_t* packed;
    KvLayout L;
    float* o_f;             // [B*N][C]
    uint8_t* p_code;        // [B*N][H][T] tap or NULL
    int N, C, H, T, bits_kv, bits_q, bits_prob, grid;
    float sigma;
};

__device__ __forceinline__ float fp_wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__global__ __launch_bounds__(256) void attn_fp_kernel(FpAttnArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int b = blockIdx.z, h = blockIdx.y, n0 = blockIdx.x * 16;
    const int N = a.N, C = a.C, H = a.H, T = a.T, d = C / H;
    float* Kd = reinterpret_cast<float*>(smem);   // [T][d]
    float* Vd = Kd + (size_t)T * d;               // [T][d]
    float* qs = Vd + (size_t)T * d;               // [4 wavefronts][d]
    float* ah = qs + 4 * d;                       // [4 wavefronts][96]
    int* prot = reinterpret_cast<int*>(ah + 4 * 96);  // [96]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const uint8_t* pk = a.packed;
    const int* slot_of = reinterpret_cast<const int*>(pk + a.L.slot_of) + b * T;
    const float* s_k = reinterpret_cast<const float*>(pk + a.L.s_k) + ((size_t)b * H + h) * T;
    const float* s_v = reinterpret_cast<const float*>(pk + a.L.s_v) + ((size_t)b * H + h) * T;
    const __half* k16 = reinterpret_cast<const __half*>(pk + a.L.k16);
    const __half* v16 = reinterpret_cast<const __half*>(pk + a.L.v16);
    auto code_at = [&](const uint8_t* codes, int t, int c) -> float {
        if (a.bits_kv == 8) return (float)(int8_t)codes[((size_t)b * T + t) * C + c];
        const int nib = (codes[((size_t)b * T + t) * (C >> 1) + (c >> 1)] >> (4 * (c & 1))) & 0xF;
        return (float)((nib ^ 8) - 8);
    };
    for (int i = tid; i < T * d; i += 256) {
        const int t = i / d, j = i % d, slot = slot_of[t];
        if (slot >= 0) {
            Kd[i] = __half2float(k16[((size_t)b * T + slot) * C + h * d + j]);
            Vd[i] = __half2float(v16[((size_t)b * T + slot) * C + h * d + j]);
        } else {
            Kd[i] = code_at(pk + a.L.k_code, t, h * d + j) * s_k[t];
            Vd[i] = code_at(pk + a.L.v_code, t, h * d + j) * s_v[t];
        }
    }
    for (int t = tid; t < 96; t += 256) prot[t] = (t < T && slot_of[t] >= 0) ? 1 : 0;
    __syncthreads();
    const float pmax = a.bits_prob == 4 ? 15.f : 255.f;
    for (int it = 0; it < 4; ++it) {
        const int n = n0 + wave * 4 + it;
        const bool nvalid = n < N;
        const size_t tok = (size_t)b * N + (nvalid ? n : N - 1);
        for (int j = lane; j < d; j += 64)
            qs[wave * d + j] = a.bits_q == 16 ? a.q_f[tok * C + h * d + j]
                                              : (float)a.q_code[tok * C + h * d + j] * a.s_q[tok * H + h];
        __syncthreads();
        float sc[2], A[2];
        float mx = -__builtin_inff();
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int t = lane + 64 * r;
            sc[r] = -__builtin_inff();
            if (t < T) {
                float s = 0.f;
                for (int j = 0; j < d; ++j) s = __builtin_fmaf(qs[wave * d + j], Kd[t * d + j], s);
                sc[r] = s * a.sigma;
            }
            mx = fmaxf(mx, sc[r]);
        }
        mx = wave_allmax(mx);
        float Z = 0.f;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            A[r] = (lane + 64 * r < T) ? __expf(sc[r] - mx) : 0.f;
            Z += A[r];
        }
        Z = fp_wave_sum(Z);
        float amax = 0.f;  // row-range grid: largest unprotected probability
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int t = lane + 64 * r;
            A[r] = A[r] / Z;
            if (t < T && !prot[t]) amax = fmaxf(amax, A[r]);
        }
        amax = wave_allmax(amax);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int t = lane + 64 * r;
            if (t >= T) continue;
            float ahat = A[r], code = 0.f;
            if (a.bits_prob != 16 && !prot[t]) {  // Eq. (3): Q_a on unprotected columns
                if (a.grid == TAQ_PROB_LOG2) {
                    code = A[r] > 0.f ? fminf(fmaxf(__builtin_rintf(-__log2f(A[r])), 0.f), pmax) : pmax;
                    ahat = exp2f(-code);
                } else if (a.grid == TAQ_PROB_ROWMAX) {
                    const float safe = amax == 0.f ? 1.f : amax;
                    const float scale = amax == 0.f ? 1.f : amax / pmax;
                    code = fminf(fmaxf(__builtin_rintf((A[r] * pmax) / safe), 0.f), pmax);
                    ahat = code * scale;
                } else {
                    code = __builtin_rintf(A[r] * pmax);
                    ahat = code / pmax;
                }
            }
            ah[wave * 96 + t] = ahat;
            if (a.p_code && nvalid) a.p_code[(tok * H + h) * (size_t)T + t] = (uint8_t)(int)code;
        }
        __syncthreads();
        for (int j = lane; j < d; j += 64) {
            float o = 0.f;
            for (int t = 0; t < T; ++t) o = __builtin_fmaf(ah[wave * 96 + t], Vd[t * d + j], o);
            if (nvalid) a.o_f[tok * C + h * d + j] = o;
        }
        __syncthreads();
    }
}

hipError_t launch_attn_fp(const float* q_f, const int8_t* q_code, const float* s_q, const uint8_t* packed, const taq_shape& s,
                          float* o_f, uint8_t* p_code, hipStream_t st) {
    FpAttnArgs a;
    a.q_f = q_f;
    a.q_code = q_code;
    a.s_q = s_q;
    a.packed = packed;
    a.L = kv_layout(s);
    a.o_f = o_f;
    a.p_code = p_code;
    a.N = s.N;
    a.C = s.C;
    a.H = s.H;
    a.T = s.T;
    a.bits_kv = s.bits_kv;
    a.bits_q = s.bits_q;
    a.bits_prob = s.bits_prob;
    a.grid = s.prob_grid;
    const int d = s.C / s.H;
    a.sigma = s.softmax_scale != 0.f ? s.softmax_scale : 1.0f / sqrtf((float)d);
    const size_t bytes = ((size_t)2 * s.T * d + 4 * d + 4 * 96) * 4 + 96 * 4;
    static std::atomic<unsigned long long> lds_set{0};
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&attn_fp_kernel), 160 * 1024, lds_set);
    if (e != hipSuccess) return e;
    if (bytes > 160 * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(attn_fp_kernel, dim3((s.N + 15) / 16, s.H, s.B), dim3(256), bytes, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------- mean squared difference of two fp16 arrays
// The loss of the token-sensitivity experiment (Section III-B, Eq. 1) on block outputs. One workgroup; float64 sum.
// (Eight values per thread and load: one workgroup reads 2.6 MB in about 30 us instead of 200.)
__global__ __launch_bounds__(1024) void mse_f16_kernel(const __half* __restrict__ x, const __half* __restrict__ y, size_t n,
                                                       double* __restrict__ out) {
    __shared__ double part[1024];
    double s = 0.0;
    auto add = [&](__half a, __half b) {
        const double dlt = (double)__half2float(a) - (double)__half2float(b);
        s += dlt * dlt;
    };
    const bool wide = ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) & 15u) == 0;
    const size_t nv = wide ? n / 8 : 0;
    constexpr int U = 4;  // loads of each array in flight per thread
    for (size_t v0 = threadIdx.x; v0 < nv; v0 += 1024 * U) {
        uint4 a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t v = v0 + 1024 * u;
            a[u] = b[u] = make_uint4(0u, 0u, 0u, 0u);
            if (v < nv) {
                a[u] = reinterpret_cast<const uint4*>(x)[v];
                b[u] = reinterpret_cast<const uint4*>(y)[v];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const __half* ha = reinterpret_cast<const __half*>(&a[u]);
            const __half* hb = reinterpret_cast<const __half*>(&b[u]);
#pragma unroll
            for (int e = 0; e < 8; ++e) add(ha[e], hb[e]);
        }
    }
    for (size_t i = 8 * nv + threadIdx.x; i < n; i += 1024) add(x[i], y[i]);
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = part[0] / (double)n;
}

hipError_t launch_mse_f16(const __half* x, const __half* y, size_t n, double* out, hipStream_t st) {
    hipLaunchKernelGGL(mse_f16_kernel, dim3(1), dim3(1024), 0, st, x, y, n, out);
    return hipGetLastError();
}

}  // namespace taq
