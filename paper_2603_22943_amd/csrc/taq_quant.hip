// Quantizer kernels of libtaq (gfx950): per-row / per-(row, head) symmetric codes,
// K~/V~ packing (Eq. 2 of PersonalQ, Section III-B), protected-row projection.
//
// The symmetric quantizer is a fixed float32 sequence so that codes are reproducible
// bit for bit:  amax = max|x|;  scale = amax/qmax;  code = clamp(rint((x*qmax)/amax)).
// The build disables FMA contraction and keeps IEEE-correct float32 division.
#include "taq_device.h"

namespace taq {

__device__ __forceinline__ void unpack_half8(const uint4& u, float f[8]) {
    const __half2* h = reinterpret_cast<const __half2*>(&u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float2 p = __half22float2(h[i]);
        f[2 * i] = p.x;
        f[2 * i + 1] = p.y;
    }
}

// ---------------------------------------------------------------- fp16 rows -> int8
// One wavefront per row, K % 8 == 0. Rows of up to 2048 values (every projection of the configured backbones) stay in
// registers between the maximum and the codes: one pass over memory, all of a row's loads in flight at once; the maximum
// is taken on the fp16 values, two per instruction (exact in any precision). Bound by the latency of that one round
// trip: 1280 x 1280 weights 6.0 -> 3.8 us per launch with the two-pass loop and a division per value before.
// `put(v, codes)` stores the eight codes of values 8v .. 8v+7.
template <typename Put>
__device__ __forceinline__ void rowquant_f16_exact(const uint4* __restrict__ xr, int nv, float amax, int lane, Put put) {
#pragma unroll 1
    for (int v = lane; v < nv; v += 64) {
        const __half* x = reinterpret_cast<const __half*>(xr + v);
        unsigned w[2] = {0u, 0u};
#pragma unroll 1
        for (int e = 0; e < 8; ++e) w[e >> 2] |= (unsigned)(symq_code_f(__half2float(x[e]), 127.f, amax) & 0xFF) << (8 * (e & 3));
        put(v, make_uint2(w[0], w[1]));
    }
}

template <int NV, typename Put>
__device__ __forceinline__ void rowquant_f16_held(const uint4* __restrict__ xr, int nv, float* scale, int lane, Put put) {
    uint4 u[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int v = lane + 64 * i;
        u[i] = make_uint4(0u, 0u, 0u, 0u);
        if (v < nv) u[i] = xr[v];
    }
    half2_t am2 = {(_Float16)0.f, (_Float16)0.f};
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const unsigned w[4] = {u[i].x & 0x7fff7fffu, u[i].y & 0x7fff7fffu, u[i].z & 0x7fff7fffu, u[i].w & 0x7fff7fffu};
#pragma unroll
        for (int e = 0; e < 4; ++e) am2 = __builtin_elementwise_max(am2, *reinterpret_cast<const half2_t*>(&w[e]));
    }
    const float amax = wave_allmax(fmaxf((float)am2[0], (float)am2[1]));
    const bool zero = amax == 0.f;
    const float safe = zero ? 1.f : amax;
    const float c = quant_mult(127.f, safe), sc = zero ? 1.f : div_grid(amax, 127.f);
    if (lane == 0) *scale = sc;
    const HalfRow half = half_row(c, sc, amax);
    unsigned pk[2 * NV];
    auto values = [&](int i) {
        const half2_t* x = reinterpret_cast<const half2_t*>(&u[i >> 1]) + 2 * (i & 1);
        return make_float4((float)x[0][0], (float)x[0][1], (float)x[1][0], (float)x[1][1]);
    };
#pragma unroll
    for (int i = 0; i < 2 * NV; ++i) {
        const float4 f = values(i);
        pk[i] = quant4_at(f.x, f.y, f.z, f.w, half.m);
    }
    if (TAQ_DOUBT(half.doubt)) {
#pragma unroll
        for (int i = 0; i < 2 * NV; ++i) {
            const float4 f = values(i);
            pk[i] = half_row_settle(pk[i], f.x, f.y, f.z, f.w, QuantRow{1.f, c, safe});
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int v = lane + 64 * i;
        if (v < nv) put(v, make_uint2(pk[2 * i], pk[2 * i + 1]));
    }
}

template <typename Put>
__device__ __forceinline__ void rowquant_f16_row(const __half* __restrict__ x, int K, float* scale, int lane, Put put) {
    const uint4* xr = reinterpret_cast<const uint4*>(x);
    const int nv = K >> 3;
    if (nv <= 64) return rowquant_f16_held<1>(xr, nv, scale, lane, put);
    if (nv <= 128) return rowquant_f16_held<2>(xr, nv, scale, lane, put);
    if (nv <= 256) return rowquant_f16_held<4>(xr, nv, scale, lane, put);
    float amax = 0.f;
    for (int v = lane; v < nv; v += 64) {
        float f[8];
        unpack_half8(xr[v], f);
#pragma unroll
        for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(f[i]));
    }
    amax = wave_allmax(amax);
    const bool zero = amax == 0.f;
    const float safe = zero ? 1.f : amax;
    if (lane == 0) *scale = zero ? 1.f : div_grid(amax, 127.f);
    rowquant_f16_exact(xr, nv, safe, lane, put);
}

__global__ __launch_bounds__(256) void rowquant_f16_kernel(const __half* __restrict__ x, int M, int K,
                                                           int8_t* __restrict__ code,
                                                           float* __restrict__ scale) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wave;
    if (row >= M) return;
    uint2* cr = reinterpret_cast<uint2*>(code + (size_t)row * K);
    rowquant_f16_row(x + (size_t)row * K, K, scale + row, lane, [&](int v, uint2 c) { cr[v] = c; });
}

// Kernel-per-stage path: per-token codes of hidden in the order to_q's token operand is read (tiles of 16 tokens, per K step
// of 64 codes one KiB, lane = token + 16 * quarter). C % 64 == 32: the second half of the last step is cleared. Tiles go to
// the XCDs in the eighths of gemm_op_kernel, four workgroups each.
__global__ __launch_bounds__(256) void rowquant_op_kernel(const __half* __restrict__ x, StageChunk c, int N, int C,
                                                          int8_t* __restrict__ tap_code, float* __restrict__ tap_scale) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int slot = (int)blockIdx.x >> 3;
    const int lt = XcdShare::item((blockIdx.x & 7) + 8 * (slot >> 2), c.tile1 - c.tile0), r = (slot & 3) * 4 + wave;  // tile of the chunk, token of the tile
    if (lt < 0) return;
    const int tile = c.tile0 + lt, b = tile / c.NT, n = (tile - b * c.NT) * 16 + r;
    if (n >= N) return;  // (codes past the last token are never used)
    const int KC = (C + 63) >> 6;
    const size_t row = (size_t)b * N + n;
    int8_t* code = c.code + (size_t)lt * KC * 1024 + r * 16;
    rowquant_f16_row(x + row * C, C, c.s + lt * 16 + r, lane, [&](int v, uint2 w) {
        *reinterpret_cast<uint2*>(code + (size_t)(v >> 3) * 1024 + ((v >> 1) & 3) * 256 + (v & 1) * 8) = w;
        if (tap_code) *reinterpret_cast<uint2*>(tap_code + row * C + 8 * v) = w;
    });
    if ((C & 63) && lane < 4) {
        const int v = (C >> 3) + lane;
        *reinterpret_cast<uint2*>(code + (size_t)(v >> 3) * 1024 + ((v >> 1) & 3) * 256 + (v & 1) * 8) = make_uint2(0u, 0u);
    }
    if (tap_scale && lane == 0) tap_scale[row] = c.s[lt * 16 + r];
}

hipError_t launch_rowquant_op(const StageChunk& c, const taq_shape& s, const __half* hidden, const taq_debug* dbg, hipStream_t st) {
    hipLaunchKernelGGL(rowquant_op_kernel, dim3(4 * XcdShare::grid(c.tile1 - c.tile0)), dim3(256), 0, st, hidden, c, s.N, s.C, dbg ? dbg->h_code : nullptr,
                       dbg ? dbg->s_h : nullptr);
    return hipGetLastError();
}

// Kernel-per-stage path: per-token codes of A^ V~ from its float32 values in accumulator order and the largest magnitudes
// per head (one pass: the row maximum is there already). A wavefront forms one K step of a tile of 16 tokens, a lane the 16
// codes of one token and 16-channel segment: four groups of four channels, each a 16-byte load of a contiguous 256-byte
// piece. With one workgroup per tile, its wavefronts walking the steps, a call was as long as one wavefront's five dependent
// rounds: 7.1 us at 64 tokens and 8.4 us at 2048 (C = 1280), 4.2 and 5.4 us this way; from 8192 tokens on both are bound by
// memory (10 to 11 us). Tiles go to the XCD whose L2 holds them, as in gemm_op_kernel.
__global__ __launch_bounds__(256) void oquant_op_kernel(StageChunk c, int N, int C, int H, int d, int tph, unsigned inv_d,
                                                        int8_t* __restrict__ tap_code, float* __restrict__ tap_scale) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int lt = XcdShare::item(blockIdx.x, c.tile1 - c.tile0);
    const int ks = blockIdx.y * 4 + wave, KC = (C + 63) >> 6;
    if (lt < 0 || ks >= KC) return;
    const int c0 = 64 * ks + 16 * q;
    const float4* o = reinterpret_cast<const float4*>(c.o_op) + (size_t)lt * H * tph * 64 + r16;
    float4 x[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int ch = c0 + 4 * g < C ? c0 + 4 * g : 0;
        const int h = (int)__umulhi((unsigned)ch, inv_d), cl = ch - h * d;  // (ch / d: exact while ch * d < 2^32)
        x[g] = o[(size_t)(h * tph + (cl >> 4)) * 64 + 16 * ((cl >> 2) & 3)];
    }
    float amax = 0.f;
    for (int h = q; h < H; h += 4) amax = fmaxf(amax, c.o_max[((size_t)lt * H + h) * 16 + r16]);
    amax = quad_allmax(amax);
    const bool zero = amax == 0.f;
    const float safe = zero ? 1.f : amax, cq = quant_mult(127.f, safe);
    unsigned w[4];
    quant4_group<4>(w, [&](int g) { return x[g]; }, [&](int) { return QuantRow{1.f, cq, safe}; });
    if (c0 >= C) w[0] = w[1] = w[2] = w[3] = 0u;
    const uint4 w4 = make_uint4(w[0], w[1], w[2], w[3]);
    *reinterpret_cast<uint4*>(c.code + ((size_t)lt * KC + ks) * 1024 + lane * 16) = w4;
    const int tile = c.tile0 + lt, b = tile / c.NT, n = (tile - b * c.NT) * 16 + r16;
    if (tap_code && n < N && c0 < C) *reinterpret_cast<uint4*>(tap_code + ((size_t)b * N + n) * C + c0) = w4;
    if (ks == 0 && q == 0) {
        const float sc = zero ? 1.f : div_grid(amax, 127.f);
        c.s[lt * 16 + r16] = sc;
        if (tap_scale && n < N) tap_scale[(size_t)b * N + n] = sc;
    }
}

hipError_t launch_oquant_op(const StageChunk& c, const taq_shape& s, const taq_debug* dbg, hipStream_t st) {
    const int d = s.C / s.H;
    hipLaunchKernelGGL(oquant_op_kernel, dim3(XcdShare::grid(c.tile1 - c.tile0), ((s.C + 63) / 64 + 3) / 4), dim3(256), 0, st, c, s.N, s.C, s.H, d, (d + 15) / 16,
                       (unsigned)(0x100000000ull / d + 1), dbg ? dbg->o_code : nullptr, dbg ? dbg->s_o : nullptr);
    return hipGetLastError();
}

// First launch of taq_quantize_kv: the per-row codes of up to three fp16 matrices that share the row length K (the
// context rows and, unless cached, the rows of Wk and Wv), and the protected-token list, each part on workgroups of
// its own: one launch instead of four.
struct KvPrepJob {
    const __half* x;   // rows to quantize (NULL: none)
    int M;             // number of rows
    int8_t* code;
    float* scale;
};

// Codes of the context in the order the projection's B operand reads them (K % 64 == 0): tiles of 16 tokens, per K step
// of 64 codes one KiB, lane = token + 16 * quarter of the step. Byte offset of code k of text token t.
__host__ __device__ static inline size_t ctx_code_at(int T, int K, int b, int t, int k) {
    const int nt = (T + 15) >> 4;
    return ((((size_t)b * nt + (t >> 4)) * (K >> 6) + (k >> 6)) * 64 + (t & 15) + 16 * ((k >> 4) & 3)) * 16 + (k & 15);
}

__global__ __launch_bounds__(256) void kv_prep_kernel(KvPrepJob j0, KvPrepJob j1, KvPrepJob j2, int K,
                                                      const uint8_t* __restrict__ mask, int B, int T, int bits,
                                                      int* __restrict__ ntrig, int* __restrict__ trig_idx,
                                                      int* __restrict__ slot_of) {
    __shared__ int flag[128];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int blk = blockIdx.x;
    if (blk < B) {  // protected-token list of batch element blk (T <= 96: a direct count is cheaper than a scan)
        const int t = threadIdx.x;
        const bool prot = t < T && (bits == 16 || mask[blk * T + t] != 0);
        if (t < 128) flag[t] = prot ? 1 : 0;
        __syncthreads();
        if (t >= 128) return;
        int before = 0, total = 0;
        for (int u = 0; u < T; ++u) {
            before += (u < t) ? flag[u] : 0;
            total += flag[u];
        }
        if (t < T) {
            slot_of[blk * T + t] = prot ? before : -1;
            if (prot) trig_idx[blk * T + before] = t;
            if (t >= total) trig_idx[blk * T + t] = -1;
        }
        if (t == 0) ntrig[blk] = total;
        return;
    }
    blk -= B;
    const bool operand_order = (K & 63) == 0;
    // which matrix, and which of its rows (selected without a branch per matrix: one copy of the quantizer in the kernel)
    const int n0 = (j0.M + 3) / 4, n1 = (j1.M + 3) / 4;
    const int k = blk < n0 ? 0 : blk < n0 + n1 ? 1 : 2;
    const KvPrepJob j = k == 0 ? j0 : k == 1 ? j1 : j2;
    const int row = (blk - (k == 0 ? 0 : k == 1 ? n0 : n0 + n1)) * 4 + wave;
    if (!j.x || row >= j.M) return;
    const bool oo = k == 0 && operand_order;
    const int b = oo ? row / T : 0, t = oo ? row - b * T : 0;
    rowquant_f16_row(j.x + (size_t)row * K, K, j.scale + row, lane, [&](int v, uint2 c) {
        *reinterpret_cast<uint2*>(j.code + (oo ? ctx_code_at(T, K, b, t, 8 * v) : (size_t)row * K + 8 * v)) = c;
    });
}

hipError_t launch_kv_prep(const __half* context, int M, int8_t* x_code, float* s_x, const __half* Wk, const __half* Wv,
                          int C, int8_t* w_code, float* s_w, int K, const uint8_t* mask, int B, int T, int bits,
                          int* ntrig, int* trig_idx, int* slot_of, hipStream_t st) {
    KvPrepJob j0 = {context, context ? M : 0, x_code, s_x};
    KvPrepJob j1 = {Wk, Wk ? C : 0, w_code, s_w};
    KvPrepJob j2 = {Wv, Wv ? C : 0, w_code + (size_t)C * K, s_w + C};
    const int blocks = B + (j0.M + 3) / 4 + (j1.M + 3) / 4 + (j2.M + 3) / 4;
    hipLaunchKernelGGL(kv_prep_kernel, dim3(blocks), dim3(256), 0, st, j0, j1, j2, K, mask, B, T, bits, ntrig, trig_idx,
                       slot_of);
    return hipGetLastError();
}

hipError_t launch_rowquant_f16(const __half* x, int M, int K, int8_t* code, float* scale, hipStream_t st) {
    if (M <= 0) return hipSuccess;
    hipLaunchKernelGGL(rowquant_f16_kernel, dim3((M + 3) / 4), dim3(256), 0, st, x, M, K, code, scale);
    return hipGetLastError();
}

// ---------------------------------------------------------------- f32 rows -> int8
// One wavefront per row. K % 4 == 0.
__global__ __launch_bounds__(256) void rowquant_f32_kernel(const float* __restrict__ x, int M, int K,
                                                           int8_t* __restrict__ code,
                                                           float* __restrict__ scale) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wave;
    if (row >= M) return;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)row * K);
    const int nv = K >> 2;
    float amax = 0.f;
    for (int v = lane; v < nv; v += 64) {
        float4 f = xr[v];
        amax = fmaxf(amax, fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w))));
    }
    amax = wave_allmax(amax);
    const bool zero = amax == 0.f;
    const float sc = zero ? 1.f : amax / 127.f;
    const float safe = zero ? 1.f : amax;
    if (lane == 0) scale[row] = sc;
    unsigned* cr = reinterpret_cast<unsigned*>(code + (size_t)row * K);
    for (int v = lane; v < nv; v += 64) {
        float4 f = xr[v];
        cr[v] = pack4(symq_code_f(f.x, 127.f, safe), symq_code_f(f.y, 127.f, safe),
                         symq_code_f(f.z, 127.f, safe), symq_code_f(f.w, 127.f, safe));
    }
}

hipError_t launch_rowquant_f32(const float* x, int M, int K, int8_t* code, float* scale, hipStream_t st) {
    if (M <= 0) return hipSuccess;
    hipLaunchKernelGGL(rowquant_f32_kernel, dim3((M + 3) / 4), dim3(256), 0, st, x, M, K, code, scale);
    return hipGetLastError();
}

// ---------------------------------------------------------------- f32 rows -> int8 per head
// One wavefront per row; per-head maxima through LDS atomics on the bit pattern of |x|
// (non-negative floats order like unsigned integers). d % 4 == 0, H <= TAQ_MAX_H.
__global__ __launch_bounds__(256) void headquant_f32_kernel(const float* __restrict__ x, int M, int C, int H,
                                                            float qmaxf, int8_t* __restrict__ code,
                                                            float* __restrict__ scale) {
    __shared__ unsigned smax[4][TAQ_MAX_H];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wave;
    const bool live = row < M;
    const int d = C / H;
    for (int h = lane; h < H; h += 64) smax[wave][h] = 0u;
    __syncthreads();
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)(live ? row : 0) * C);
    const int nv = C >> 2;
    if (live) {
        for (int v = lane; v < nv; v += 64) {
            float4 f = xr[v];
            float a = fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w)));
            atomicMax(&smax[wave][(v * 4) / d], __float_as_uint(a));
        }
    }
    __syncthreads();
    if (!live) return;
    for (int h = lane; h < H; h += 64) {
        float amax = __uint_as_float(smax[wave][h]);
        scale[(size_t)row * H + h] = amax == 0.f ? 1.f : amax / qmaxf;
    }
    unsigned* cr = reinterpret_cast<unsigned*>(code + (size_t)row * C);
    for (int v = lane; v < nv; v += 64) {
        float4 f = xr[v];
        float amax = __uint_as_float(smax[wave][(v * 4) / d]);
        float safe = amax == 0.f ? 1.f : amax;
        cr[v] = pack4(symq_code_f(f.x, qmaxf, safe), symq_code_f(f.y, qmaxf, safe),
                         symq_code_f(f.z, qmaxf, safe), symq_code_f(f.w, qmaxf, safe));
    }
}

hipError_t launch_headquant_f32(const float* x, int M, int C, int H, int bits, int8_t* code, float* scale,
                                hipStream_t st) {
    if (M <= 0) return hipSuccess;
    hipLaunchKernelGGL(headquant_f32_kernel, dim3((M + 3) / 4), dim3(256), 0, st, x, M, C, H, bits == 4 ? 7.f : 127.f,
                       code, scale);
    return hipGetLastError();
}

// ---------------------------------------------------------------- K~/V~ codes, Eq. (2)
// One wavefront per (batch, token). rows_f holds that token's K channels then V channels;
// each head's d channels are one quantization row. Protected tokens get zero codes/scales.
__global__ __launch_bounds__(64) void kv_pack_kernel(const float* __restrict__ rows_f,
                                                     const int* __restrict__ slot_of, int T, int C, int H,
                                                     int bits, uint8_t* __restrict__ k_code,
                                                     uint8_t* __restrict__ v_code, float* __restrict__ s_k,
                                                     float* __restrict__ s_v) {
    __shared__ unsigned smax[2 * TAQ_MAX_H];
    const int bt = blockIdx.x, b = bt / T, t = bt % T, lane = threadIdx.x;
    const int d = C / H;
    const bool prot = slot_of[bt] >= 0;
    const float qmaxf = bits == 4 ? 7.f : 127.f;
    for (int g = lane; g < 2 * H; g += 64) smax[g] = 0u;
    __syncthreads();
    const float4* xr = reinterpret_cast<const float4*>(rows_f + (size_t)bt * 2 * C);
    const int nv = (2 * C) >> 2;
    if (!prot) {
        for (int v = lane; v < nv; v += 64) {
            float4 f = xr[v];
            float a = fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w)));
            atomicMax(&smax[(v * 4) / d], __float_as_uint(a));
        }
    }
    __syncthreads();
    for (int g = lane; g < 2 * H; g += 64) {
        float amax = __uint_as_float(smax[g]);
        float sc = prot ? 0.f : (amax == 0.f ? 1.f : amax / qmaxf);
        float* dst = g < H ? s_k : s_v;
        dst[((size_t)b * H + (g % H)) * T + t] = sc;
    }
    if (bits == 16) return;  // every row protected: there is no code section
    for (int v = lane; v < nv; v += 64) {
        const int ch = v * 4;  // channel within the 2C-wide row
        int c0 = 0, c1 = 0, c2 = 0, c3 = 0;
        if (!prot) {
            float4 f = xr[v];
            float amax = __uint_as_float(smax[ch / d]);
            float safe = amax == 0.f ? 1.f : amax;
            c0 = symq_code_f(f.x, qmaxf, safe);
            c1 = symq_code_f(f.y, qmaxf, safe);
            c2 = symq_code_f(f.z, qmaxf, safe);
            c3 = symq_code_f(f.w, qmaxf, safe);
        }
        uint8_t* base = ch < C ? k_code : v_code;
        const int c = ch < C ? ch : ch - C;
        if (bits == 8) {
            *reinterpret_cast<unsigned*>(base + (size_t)bt * C + c) = pack4(c0, c1, c2, c3);
        } else {
            unsigned short w = (unsigned short)((c0 & 0xF) | ((c1 & 0xF) << 4) | ((c2 & 0xF) << 8) |
                                                ((c3 & 0xF) << 12));
            *reinterpret_cast<unsigned short*>(base + (size_t)bt * (C / 2) + c / 2) = w;
        }
    }
}

hipError_t launch_kv_pack(const float* rows_f, const int* slot_of, int B, int T, int C, int H, int bits,
                          uint8_t* k_code, uint8_t* v_code, float* s_k, float* s_v, hipStream_t st) {
    hipLaunchKernelGGL(kv_pack_kernel, dim3(B * T), dim3(64), 0, st, rows_f, slot_of, T, C, H, bits, k_code,
                       v_code, s_k, s_v);
    return hipGetLastError();
}

// ---------------------------------------------------------------- protected K/V rows, bits_kv = 16 (every row protected)
// One workgroup (512 threads) per (slot, batch, 128 output channels): y[c] = s_w[c] * sum_k ctx[t][k] * w_code[c][k].
// Four threads share an output channel, each summing every fourth 16-code piece of the row in float32 (four
// partial sums per thread), combined by two shuffles; one rounding to fp16. Cc % 16 == 0, Cc <= 4096.
__device__ __forceinline__ void kv_trigger_rows_block(float* xs, int slot, int b, int cblk, const __half* __restrict__ context,
                                                      const int8_t* __restrict__ w_code, const float* __restrict__ s_w,
                                                      const int* __restrict__ ntrig, const int* __restrict__ trig_idx,
                                                      int T, int C, int Cc, __half* __restrict__ k16,
                                                      __half* __restrict__ v16, __half* __restrict__ v16t) {
    const int c = cblk * 128 + (threadIdx.x >> 2), part = threadIdx.x & 3;  // output channel in [0, 2C)
    // unused slots of all three copies read as zeros: the padding slots T..95 of the transposed copy ...
    if (slot == T - 1 && c >= C && c < 2 * C && part == 0)
        for (int sp = T; sp < 96; ++sp) v16t[((size_t)b * C + (c - C)) * 96 + sp] = __float2half(0.f);
    if (slot >= ntrig[b]) {  // ... and every slot past the protected tokens
        if (c < 2 * C && part == 0) {
            if (c < C) {
                k16[((size_t)b * T + slot) * C + c] = __float2half(0.f);
            } else {
                v16[((size_t)b * T + slot) * C + (c - C)] = __float2half(0.f);
                v16t[((size_t)b * C + (c - C)) * 96 + slot] = __float2half(0.f);
            }
        }
        return;
    }
    const int t = trig_idx[b * T + slot];
    const __half* xr = context + ((size_t)b * T + t) * Cc;
    for (int k = threadIdx.x; k < Cc; k += 512) xs[k] = __half2float(xr[k]);
    __syncthreads();
    float sum = 0.f;
    if (c < 2 * C) {
        const int4* wr = reinterpret_cast<const int4*>(w_code + (size_t)c * Cc);
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        for (int kv = part; kv < (Cc >> 4); kv += 4) {
            const int4 w = wr[kv];
            const int wd[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float wf = (float)(int)(int8_t)((wd[qd] >> (8 * e)) & 0xFF);
                    acc[e] = __builtin_fmaf(xs[kv * 16 + qd * 4 + e], wf, acc[e]);
                }
            }
        }
        sum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    }
    sum += __shfl_xor(sum, 1);
    sum += __shfl_xor(sum, 2);
    if (c < 2 * C && part == 0) {
        const __half yh = __float2half_rn(sum * s_w[c]);
        if (c < C) {
            k16[((size_t)b * T + slot) * C + c] = yh;
        } else {
            v16[((size_t)b * T + slot) * C + (c - C)] = yh;
            v16t[((size_t)b * C + (c - C)) * 96 + slot] = yh;  // transposed copy, slot along the row
        }
    }
}

__global__ __launch_bounds__(512) void kv_trigger_rows_kernel(const __half* __restrict__ context,
                                                              const int8_t* __restrict__ w_code,
                                                              const float* __restrict__ s_w,
                                                              const int* __restrict__ ntrig,
                                                              const int* __restrict__ trig_idx, int T, int C,
                                                              int Cc, __half* __restrict__ k16,
                                                              __half* __restrict__ v16,
                                                              __half* __restrict__ v16t) {
    __shared__ float xs[4096];
    kv_trigger_rows_block(xs, blockIdx.x, blockIdx.y, blockIdx.z, context, w_code, s_w, ntrig, trig_idx, T, C, Cc, k16, v16, v16t);
}

hipError_t launch_kv_trigger_rows(const __half* context, const int8_t* w_code, const float* s_w,
                                  const int* ntrig, const int* trig_idx, int B, int T, int C, int Cc,
                                  __half* k16, __half* v16, __half* v16t, hipStream_t st) {
    hipLaunchKernelGGL(kv_trigger_rows_kernel, dim3(T, B, (2 * C + 127) / 128), dim3(512), 0, st, context, w_code, s_w,
                       ntrig, trig_idx, T, C, Cc, k16, v16, v16t);
    return hipGetLastError();
}

// ---------------------------------------------------------------- K/V projection + Eq. (2) codes + image, per head
// Second launch of taq_quantize_kv for 4/8-bit rows. One workgroup per (head, batch element, K or V), one wavefront per
// 16-token column tile, or per two of them and a part of the channels (at most six of the eight; the last one stores the scales): the integer projection of the head's K (or V) channels (acc = x_code .
// w_code over Cc, 16x16x64 int8 MFMA, channels as rows and tokens as columns), the float32 dequantisation float(acc) *
// (s_x * s_w), the per-(head, token) symmetric quantizer of Eq. (2) (zero codes and scales on protected tokens), and the
// plain code / scale sections of qkv_packed and this head's block of the operand-ordered image.
// Further workgroups of the launch, a few per 128 output channels and batch element: the protected rows (kvh_protected).
// WLDS: the head's weight slice (16*TPH rows x Cc codes, Cc % 64 == 0) is fetched once per workgroup, straight into LDS
// (one KiB per 16 rows x 64 codes, LDS address = base + lane * 16), and every wavefront reads its A operands from there;
// otherwise each wavefront fetches the slice itself. d % 8 == 0, Cc % 32 == 0.
// Bound by the latency chain (weights into LDS, then the K loop, then the quantizer) on 2 H B compute units. Before, every
// slot of the protected rows had workgroups of its own, used or not: 3080 of them at C = 1280, one per compute unit
// beside 140 KiB of LDS, and that was most of the launch (C = 1280, batch 2: 20.8 -> 10.3 us).

// What the epilogue reads from memory, requested ahead of the K loop: the lane's token of a column tile, and the scales of its channels
// 16*(j0 + j) + 4*q .. +3 of the head.
struct KvhTok {
    float sx;
    int slot;  // its slot among the protected tokens, -1 if unprotected
};
template <int NJ>
struct KvhChan {
    float4 sw[NJ];
};
template <int NJ, int NT>
__device__ __forceinline__ void kvh_row_load(KvhChan<NJ>& S, KvhTok (&tok)[NT], int j0, int st, int b, int d, int r16, int q, int T,
                                             const float* __restrict__ s_x, const float* __restrict__ s_w_head, const int* __restrict__ slot_of) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        const int t = 16 * (st + n) + r16, tc = t < T ? t : T - 1;
        tok[n].slot = slot_of[tc];
        tok[n].sx = s_x[(size_t)b * T + tc];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int cl = 16 * (j0 + j) + 4 * q;
        S.sw[j] = *reinterpret_cast<const float4*>(s_w_head + (cl < d ? cl : 0));
    }
}

typedef unsigned uint4_a8 __attribute__((ext_vector_type(4), aligned(8)));
typedef unsigned uint2_a4 __attribute__((ext_vector_type(2), aligned(4)));

// float32 dequantisation of the integer sums of NJ channel tiles and one column tile; returns the largest magnitude of the lane's token.
template <int NJ>
__device__ __forceinline__ float kvh_values(float (&v)[NJ][4], const int32x4_t (&acc)[NJ], const KvhChan<NJ>& S, const KvhTok& tok, int j0, int d, int q) {
    float amax = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const bool valid = 16 * (j0 + j) + 4 * q < d;
        const float swv[4] = {S.sw[j].x, S.sw[j].y, S.sw[j].z, S.sw[j].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float sc = tok.sx * swv[i];
            v[j][i] = valid ? (float)acc[j][i] * sc : 0.f;
            amax = fmaxf(amax, fabsf(v[j][i]));
        }
    }
    return quad_allmax(amax);
}

// Epilogue of channel tiles J0 .. J0 + NJ - 1 (of TPH; J0 a multiple of 4) and one 16-token column tile: Eq. (2) quantizer per (head, token),
// plain code / scale sections and the head's image block. Four tiles at a time are transposed between the four quarters of the wavefront, so
// that a lane stores the 16 contiguous channels of one tile (a dword per tile and lane otherwise: four times the stores, each 64 cache accesses).
// amax: of the token's row of this head, over all its tiles.
template <int TPH, int J0, int NJ>
__device__ __forceinline__ void kvh_finish(const float (&v)[NJ][4], float amax, int slot, int st, int h, int b, int side, int d, int r16,
                                           int q, int T, int C, int bits, float qmaxf, uint8_t* codes, uint8_t* img, const KvImage& I) {
    const int t = 16 * st + r16;
    const bool tv = t < T, prot = !tv || slot >= 0;  // protected or past the last token: zero codes, zero scale
    const float safe = amax == 0.f ? 1.f : amax;
    const float cq = quant_mult(qmaxf, safe);  // (a non-zero |v| is at least 2e-19: s_x and s_w come from fp16 rows)
    constexpr int TP4 = (NJ + 3) & ~3;
    unsigned pk[TP4], codes4[NJ];
    quant4_group<NJ>(codes4, [&](int j) { return make_float4(v[j][0], v[j][1], v[j][2], v[j][3]); }, [&](int) { return QuantRow{1.f, cq, safe}; }, qmaxf);
#pragma unroll
    for (int j = 0; j < TP4; ++j) pk[j] = j < NJ && !prot && 16 * (J0 + j) + 4 * q < d ? codes4[j < NJ ? j : 0] : 0u;
    const int pos = vt_pos(t & ~3, I.nt16);  // place of this lane's group of four tokens in a V^T row
    const unsigned sel1 = (r16 & 1) ? 0x03070105u : 0x06020400u, sel2 = (r16 & 2) ? 0x03020706u : 0x05040100u;
    if (side) {
        // Vt[channel][pos], stored with the sign bit flipped. The four lanes of a quad hold four channels of four
        // neighbouring tokens each: transposed (two exchanges), a lane stores four tokens of one channel.
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const unsigned w0 = pk[j] ^ 0x80808080u;
            const unsigned w1 = __builtin_amdgcn_perm(__builtin_amdgcn_update_dpp(0u, w0, 0xB1, 0xF, 0xF, true), w0, sel1);
            const unsigned w2 = __builtin_amdgcn_perm(__builtin_amdgcn_update_dpp(0u, w1, 0x4E, 0xF, 0xF, true), w1, sel2);
            if (16 * (J0 + j) + 4 * q < d) *reinterpret_cast<unsigned*>(img + I.vt + (size_t)(16 * (J0 + j) + 4 * q + (r16 & 3)) * I.cols_v + pos) = w2;
        }
    }
#pragma unroll
    for (int j = 0; j < NJ; j += 4) {
        if (!side && TPH % 4 == 0 && t < I.rows_k)  // Kp, heads of a multiple of 4 tiles: [t][tile/4][q][tile%4][4]
            *reinterpret_cast<uint4*>(img + I.kp + kp_offset(TPH, t, J0 + j, q)) = make_uint4(pk[j], pk[j + 1], pk[j + 2], pk[j + 3]);
        unsigned w[4] = {pk[j], pk[j + 1], pk[j + 2], pk[j + 3]};
        quad_transpose(w);  // this lane now: tile j + q, its 16 channels in order
        const int tl = J0 + j + q;
        const bool own = tl < J0 + NJ, full = own && 16 * tl + 16 <= d, half = own && !full && 16 * tl < d;  // (d % 8 == 0)
        if (!side && TPH % 4 != 0 && t < I.rows_k && own)  // Kp[t][tile][quarter][4]
            *reinterpret_cast<uint4*>(img + I.kp + kp_offset(TPH, t, tl, 0)) = make_uint4(w[0], w[1], w[2], w[3]);
        if (tv) {
            if (bits == 8) {
                uint8_t* o = codes + ((size_t)b * T + t) * C + h * d + 16 * tl;
                if (full) *reinterpret_cast<uint4_a8*>(o) = (uint4_a8){w[0], w[1], w[2], w[3]};
                if (half) *reinterpret_cast<uint2*>(o) = make_uint2(w[0], w[1]);
            } else {
                unsigned n[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    n[i] = w[i] & 0x0F0F0F0Fu;
                    n[i] = (n[i] | (n[i] >> 4)) & 0x00FF00FFu;
                    n[i] = (n[i] | (n[i] >> 8)) & 0xFFFFu;
                }
                uint8_t* o = codes + ((size_t)b * T + t) * (C / 2) + (h * d) / 2 + 8 * tl;
                if (full) *reinterpret_cast<uint2_a4*>(o) = (uint2_a4){n[0] | (n[1] << 16), n[2] | (n[3] << 16)};
                if (half) *reinterpret_cast<unsigned*>(o) = n[0] | (n[1] << 16);
            }
        }
    }
}

// Scales of a head's tokens from their largest magnitudes (amax_l[part][token]): the plain section, and the image's per-token scales, the 0 /
// -inf bias and the power-of-two prescale of V. One wavefront, a lane for tokens lane and lane + 64, whose slots among the protected are slot.
// Beside the others' codes and stores: behind them and a second barrier, with the largest scale by an LDS atomic, it stood in the chain (us per call,
// Cc = 768, batch 2, before and now: C = 320 8.65 and 8.05, 640 10.2 and 9.3, 1280 13.3 and 12.55).
template <int PARTS>
__device__ __forceinline__ void kvh_scales(const float (*amax_l)[96], const int (&slot)[2], int side, int lane, int T, float qmaxf,
                                           float* scales, uint8_t* img, const KvImage& I) {
    float sc[2];
    unsigned scmax = 0u;  // (of non-negative floats)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = lane + 64 * i;
        const bool in = t < I.ntok, tv = t < T, prot = !tv || slot[i] >= 0;
        float amax = in ? amax_l[0][t] : 0.f;
        if (PARTS > 1 && in) amax = fmaxf(amax, amax_l[PARTS - 1][t]);
        sc[i] = prot ? 0.f : (amax == 0.f ? 1.f : div_grid(amax, qmaxf));
        scmax = __float_as_uint(sc[i]) > scmax ? __float_as_uint(sc[i]) : scmax;
        if (tv) scales[t] = sc[i];
        if (!side && in) {
            reinterpret_cast<float*>(img + I.s_k)[t] = sc[i];
            reinterpret_cast<float*>(img + I.bias)[t] = prot ? TAQ_NEG_INF : 0.f;
        }
    }
    if (!side) return;
#pragma unroll
    for (int m = 32; m; m >>= 1) {
        const unsigned o = (unsigned)__shfl_xor((int)scmax, m);
        scmax = o > scmax ? o : scmax;
    }
    // the largest |s_V * code| goes to [256, 512)
    int kexp = 0;
    const float dmax = __uint_as_float(scmax) * qmaxf;
    if (dmax > 0.f) {
        int e;
        (void)frexpf(dmax, &e);
        kexp = 9 - e;
    }
    const float vpre = ldexpf(1.0f, kexp);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = lane + 64 * i;
        if (t < I.ntok) {  // s' = s_V * 2^kexp as two fp16 numbers, high part and remainder
            const float sp = sc[i] * vpre;
            const __half hi = __float2half_rn(sp);
            reinterpret_cast<__half*>(img + I.s_vp)[t] = hi;
            reinterpret_cast<__half*>(img + I.s_vp)[I.ntok + t] = __float2half_rn(sp - __half2float(hi));
        }
    }
    if (lane == 0) {
        reinterpret_cast<float*>(img + I.vpre)[0] = vpre;
        reinterpret_cast<float*>(img + I.oscale)[0] = ldexpf(1.0f, -kexp);
    }
}

// Protected rows, y[c] = s_w[c] * sum_k ctx[t][k] * w_code[c][k], one rounding to fp16: 128 output channels (of K, then V) per
// workgroup, protected slots group, group + groups, ... Four threads share an output channel, each summing every fourth 16-code piece
// of the row in float32 (four partial sums per thread, combined by two exchanges): the same sums in the same order as
// kv_trigger_rows_block. Up to KVH_SLOTS rows at a time share a pass over the weight codes.
// Slots past the protected tokens are zero in the transposed V copy (they meet zero weights there) and unspecified in
// the other two.
//
// A chain of round trips to memory with almost no work in between: the list and its length at once, then the first weight pieces with the
// context rows; and the zeros of the unused slots are stored last, by the groups with the fewest slots (a load behind a store waits for
// it). With the length, the list, the rows and the weights one after the other behind the zeros, these workgroups were the launch's last
// at C = 320 and Cc = 2048: 9.9 -> 8.9 us of a call at C = 320, Cc = 768, B = 2, and
// 17.7 -> 14.1 at C = 640 or 1280, Cc = 2048 (2 protected tokens; 8.9 and 13.9 with none). Twelve pieces at a time instead of four are no
// faster and leave a compute unit one workgroup.
#define KVH_SLOTS 4
#define KVH_PIECES 4
struct KvhPieces {  // of this thread's row of weight codes: every fourth, 16 codes each
    int4 w[KVH_PIECES];
    __amdgpu_buffer_rsrc_t codes;
    int at, np, part;  // byte of the thread's first piece; pieces of a row; the thread's place among the four
    __device__ __forceinline__ void request(int p) {  // pieces p + part + 4 u of the row (past its end: the next row's, or zeros; not used)
#pragma unroll
        for (int u = 0; u < KVH_PIECES; ++u) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(codes, at + 64 * u, 16 * p, 0);
            w[u] = make_int4(v[0], v[1], v[2], v[3]);
        }
    }
};
template <int S>
__device__ __forceinline__ void kvh_protected_rows(const __half* xs, KvhPieces& W, int c, int slot0, int step, int ntrig, int b,
                                                   const float* __restrict__ s_w, uint8_t* __restrict__ packed, const KvLayout& L, int T, int C, int Cc) {
    float acc[S][4] = {};
    const int np = W.np, part = W.part;
    for (int p0 = 0;; p0 += 4 * KVH_PIECES) {
        const __half* xp = xs + (p0 + part) * 16;
#pragma unroll
        for (int u = 0; u < KVH_PIECES; ++u) {
            if (p0 + part + 4 * u < np) {
                const int wd[4] = {W.w[u].x, W.w[u].y, W.w[u].z, W.w[u].w};
#pragma unroll
                for (int qh = 0; qh < 2; ++qh) {
                    uint4 x[S];
#pragma unroll
                    for (int i = 0; i < S; ++i) x[i] = *reinterpret_cast<const uint4*>(xp + i * Cc + 64 * u + qh * 8);
#pragma unroll
                    for (int i = 0; i < S; ++i) {
                        const half2_t* xh = reinterpret_cast<const half2_t*>(&x[i]);  // (v_fma_mix reads the fp16 values as they are)
#pragma unroll
                        for (int q2 = 0; q2 < 2; ++q2)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                acc[i][e] = __builtin_fmaf((float)xh[2 * q2 + (e >> 1)][e & 1],
                                                           (float)(int)(int8_t)((wd[2 * qh + q2] >> (8 * e)) & 0xFF), acc[i][e]);
                    }
                }
            }
        }
        if (p0 + 4 * KVH_PIECES >= np) break;
        W.request(p0 + 4 * KVH_PIECES);
    }
#pragma unroll
    for (int i = 0; i < S; ++i) {
        float sum = (acc[i][0] + acc[i][1]) + (acc[i][2] + acc[i][3]);
        sum += __shfl_xor(sum, 1);
        sum += __shfl_xor(sum, 2);
        const int slot = slot0 + step * i;
        if (c < 2 * C && part == 0 && slot < ntrig) {
            // product and conversion in one rounding, spelled out so that the row and its transposed copy hold the same number
            // (left to itself the compiler may round twice in one of the two uses)
            unsigned yb = 0u;
            asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "+v"(yb) : "v"(sum), "v"(s_w[c]));
            const __half yh = __ushort_as_half((unsigned short)yb);
            if (c < C) {
                reinterpret_cast<__half*>(packed + L.k16)[((size_t)b * T + slot) * C + c] = yh;
            } else {
                reinterpret_cast<__half*>(packed + L.v16)[((size_t)b * T + slot) * C + (c - C)] = yh;
                reinterpret_cast<__half*>(packed + L.v16t)[((size_t)b * C + (c - C)) * 96 + slot] = yh;
            }
        }
    }
}

__device__ __forceinline__ void kvh_protected(unsigned char* lds, int cblk, int group, int groups, int b, const __half* __restrict__ context,
                                              const int8_t* __restrict__ w_code, const float* __restrict__ s_w,
                                              uint8_t* __restrict__ packed, const KvLayout& L, int T, int C, int Cc) {
    __half* xs = reinterpret_cast<__half*>(lds);  // [KVH_SLOTS][Cc]
    const int tid = threadIdx.x;
    const int c = cblk * 128 + (tid >> 2), part = tid & 3;
    const int* trig_idx = reinterpret_cast<const int*>(packed + L.trig_idx) + b * T;
    const int ntrig = reinterpret_cast<const int*>(packed + L.ntrig)[b];
    int token[KVH_SLOTS];  // of slots group, group + groups, ... (past the protected tokens: -1)
    auto tokens_of = [&](int slot) {
#pragma unroll
        for (int i = 0; i < KVH_SLOTS; ++i) token[i] = trig_idx[slot + groups * i < T ? slot + groups * i : T - 1];
    };
    tokens_of(group);
    KvhPieces W;
    W.codes = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(w_code), 0, 2 * C * Cc, 0x00020000);  // (C <= 64 * 160, Cc <= 4096)
    W.at = (c < 2 * C ? c : 2 * C - 1) * Cc + 16 * part;
    W.np = Cc >> 4;
    W.part = part;
    for (int slot = group; slot < ntrig; slot += groups * KVH_SLOTS) {
        const int left = (ntrig - slot + groups - 1) / groups, n = left < KVH_SLOTS ? left : KVH_SLOTS;  // slots slot, slot + groups, ...
        if (slot > group) __syncthreads();  // the rows of the turn before are done with
        W.request(0);
        for (int v = tid; v < n * (Cc >> 3); v += 512) {
            const int i = v / (Cc >> 3), k = 8 * (v - i * (Cc >> 3));
            const int t = i == 0 ? token[0] : i == 1 ? token[1] : i == 2 ? token[2] : token[3];
            *reinterpret_cast<uint4*>(xs + (size_t)i * Cc + k) = *reinterpret_cast<const uint4*>(context + ((size_t)b * T + t) * Cc + k);
        }
        __syncthreads();
        tokens_of(slot + groups * KVH_SLOTS);  // of the next turn
        if (n == 1) kvh_protected_rows<1>(xs, W, c, slot, groups, ntrig, b, s_w, packed, L, T, C, Cc);
        else if (n == 2) kvh_protected_rows<2>(xs, W, c, slot, groups, ntrig, b, s_w, packed, L, T, C, Cc);
        else  // (of three rows the fourth is whatever the LDS holds; its slot is past the protected tokens and not stored)
            kvh_protected_rows<4>(xs, W, c, slot, groups, ntrig, b, s_w, packed, L, T, C, Cc);
    }
    // unused slots of the transposed V copy, eight of one channel at a time (the last groups, which have the fewest slots)
    for (int i = tid + 512 * (groups - 1 - group); i < 128 * 12; i += 512 * groups) {
        const int vc = cblk * 128 + i / 12 - C, s0 = 8 * (i % 12);
        if (vc < 0 || vc >= C) continue;
        __half* p = reinterpret_cast<__half*>(packed + L.v16t) + ((size_t)b * C + vc) * 96 + s0;
        if (s0 >= ntrig) *reinterpret_cast<uint4*>(p) = make_uint4(0u, 0u, 0u, 0u);
        else
            for (int e = ntrig - s0; e < 8; ++e) p[e] = __float2half(0.f);
    }
}

// (heads of up to five tiles: registers for two workgroups per compute unit, which the protected rows of many batch elements fill; with 148
// registers a call at B = 8, C = 640 took 15.5 us instead of 12.6)
template <int TPH, bool WLDS>
__global__ __launch_bounds__(512, WLDS && TPH <= 5 ? 4 : 2) void kv_head_kernel(const int8_t* __restrict__ x_code, const float* __restrict__ s_x,
                                                      const int8_t* __restrict__ w_code, const float* __restrict__ s_w,
                                                      uint8_t* __restrict__ packed, KvLayout L, KvImage I, int T, int C,
                                                      int H, int d, int Cc, int bits, const __half* __restrict__ context) {
    __shared__ float amax_l[TPH > 8 ? 2 : 1][96];  // largest magnitudes of the tokens' rows of this head and side, over each part of the channel tiles
    extern __shared__ __align__(16) unsigned char kvh_w[];  // WLDS: [TPH][Cc/64][64 lanes][16 bytes]
    const int b = (int)blockIdx.y;
    if ((int)blockIdx.x >= 2 * H) {
        const int p = (int)blockIdx.x - 2 * H, nc = (2 * C + 127) >> 7;
        kvh_protected(kvh_w, p % nc, p / nc, ((int)gridDim.x - 2 * H) / nc, b, context, w_code, s_w, packed, L, T, C, Cc);
        return;
    }
    const int h = (int)blockIdx.x >> 1, side = (int)blockIdx.x & 1;  // side 0: K, 1: V
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r16 = lane & 15, q = lane >> 4;
    const int nsub = (T + 15) / 16;  // 16-token column tiles
    const int ksteps = (Cc + 63) / 64;  // K steps of 64 (the last one may be half: Cc % 32 == 0)
    const bool operand_order = (Cc & 63) == 0;  // of the context codes
    if constexpr (WLDS) {
        // all eight wavefronts: piece f = j * ksteps + ks of the slice (rows 16*j .. 16*j+15, codes 64*ks .. 64*ks+63)
        // Four consecutive lanes fetch the 64 bytes of one row (a lane per row and segment in operand order would make every
        // lane a cache access of its own), the segments of a row swizzled so that the operand reads meet no bank conflicts.
        const int lr = lane >> 2, seg = (lane & 3) ^ ((lr >> 1 ^ lr >> 2) & 3);
        for (int f = wave, j = 0, ks = wave; f < TPH * ksteps; f += 8, ks += 8) {
            while (ks >= ksteps) {
                ks -= ksteps;
                ++j;
            }
            int c = side * C + h * d + 16 * j + lr;  // rows past the head are computed and dropped; stay inside [0, 2C)
            c = c < 2 * C ? c : 2 * C - 1;
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(w_code + (size_t)c * Cc + 64 * ks + 16 * seg),
                (__attribute__((address_space(3))) void*)(kvh_w + (size_t)f * 1024), 16, 0, 0);
        }
    }
    const int w_off = r16 * 64 + ((q ^ ((r16 >> 1 ^ r16 >> 2) & 3)) << 4);
    // weight codes of tile j, K step ks: this lane's row 16*j + r16 of the head, codes 64*ks + 16*q .. +15
    auto load_w = [&](int j, int ks) -> int32x4_t {
        if constexpr (WLDS) {
            return *reinterpret_cast<const int32x4_t*>(kvh_w + (size_t)(j * ksteps + ks) * 1024 + w_off);
        } else {
            int c = side * C + h * d + 16 * j + r16;
            c = c < 2 * C ? c : 2 * C - 1;
            return 64 * ks + 16 * q < Cc ? *reinterpret_cast<const int32x4_t*>(w_code + (size_t)c * Cc + 64 * ks + 16 * q)
                                         : (int32x4_t){0, 0, 0, 0};
        }
    };
    const float qmaxf = bits == 4 ? 7.f : 127.f;
    const int* slot_of = reinterpret_cast<const int*>(packed + L.slot_of) + b * T;
    uint8_t* codes = packed + (side ? L.v_code : L.k_code);
    float* scales = reinterpret_cast<float*>(packed + (side ? L.s_v : L.s_k)) + ((size_t)b * H + h) * T;
    uint8_t* img = packed + L.image + (size_t)b * L.image_bytes + (size_t)h * I.head_bytes;
    // A wavefront's share: channel tiles J0 .. J0 + NJ - 1 and NT column tiles from st on. Heads of up to eight channel tiles: one column tile
    // each. Larger ones: two column tiles share the weights read from LDS (600 KB a workgroup otherwise, 2 us of them), and the channel tiles are
    // split behind the fourth; the third pair has one column tile as a rule, and its larger part goes where a smaller one runs. A call at
    // C = 1280 (8 heads), Cc = 768: 13.4 us with one column tile each, 13.3 in pairs (batch 1: 12.25 and 12.15); with heads of 5 tiles the
    // pairs' registers leave a compute unit one workgroup: 10.1 and 11.2.
    constexpr bool PAIR = TPH > 8;
    constexpr int NT = PAIR ? 2 : 1, J1 = PAIR ? 4 : TPH;
    const int pair = wave >> 1, part = PAIR ? (wave & 1) ^ (pair != 2) : 0;
    const int st = PAIR ? 2 * pair : wave;
    const bool two = PAIR && st + 1 < nsub;
    auto unit = [&](auto j0) {
        constexpr int J0 = j0(), NJ = J0 ? TPH - J1 : J1;
        KvhTok tok[NT];
        KvhChan<NJ> S;
        kvh_row_load(S, tok, J0, st, b, d, r16, q, T, s_x, s_w + side * C + h * d, slot_of);
        int32x4_t acc[NT][NJ];
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[n][j] = (int32x4_t){0, 0, 0, 0};
        if constexpr (WLDS) {
            // the token codes of the first K steps travel with the weight slice; then everybody waits for the slice
            const int8_t* xrow = x_code + (size_t)(b * nsub + st) * ksteps * 1024 + lane * 16;
            const size_t second = two ? (size_t)ksteps * 1024 : 0;
            constexpr int XG = PAIR ? 2 : TPH == 5 ? 3 : 4;  // groups of four K steps of token codes in flight per wavefront (as the registers allow)
            int32x4_t xb[XG][4][NT];
            auto load_x = [&](int32x4_t (&x)[4][NT], int k0) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int8_t* p = xrow + 1024 * (k0 + u < ksteps ? k0 + u : ksteps - 1);
#pragma unroll
                    for (int n = 0; n < NT; ++n) x[u][n] = *reinterpret_cast<const int32x4_t*>(p + (n ? second : 0));
                }
            };
            auto load_all = [&](int k0) {
#pragma unroll
                for (int g = 0; g < XG; ++g) load_x(xb[g], k0 + 4 * g);
            };
            load_all(0);
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's pieces of the slice are in LDS
            __syncthreads();                     // ... and so are everybody else's
            // (token codes past the end become zeros here and not where they are loaded: setting a register waits for the loads before its own;
            // weights past the end are whatever the LDS holds)
            auto steps = [&](auto nt, int32x4_t (&x)[4][NT], int k0) {
                if (k0 + 4 > ksteps) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int n = 0; n < NT; ++n)
                            if (k0 + u >= ksteps) x[u][n] = (int32x4_t){0, 0, 0, 0};
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const int32x4_t w = load_w(J0 + j, k0 + u);
#pragma unroll
                        for (int n = 0; n < nt(); ++n) acc[n][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, x[u][n], acc[n][j], 0, 0, 0);
                    }
            };
            for (int k0 = 0; k0 < ksteps; k0 += 4 * XG) {
                if (!PAIR && k0 > 0) load_all(k0);
#pragma unroll
                for (int g = 0; g < XG; ++g) {
                    const int k = k0 + 4 * g;
                    if (k < ksteps) {
                        if (NT == 2 && two)
                            steps(std::integral_constant<int, NT>(), xb[g], k);
                        else
                            steps(std::integral_constant<int, 1>(), xb[g], k);
                        if (PAIR && k + 4 * XG < ksteps) load_x(xb[g], k + 4 * XG);
                    }
                }
            }
        } else {
            __syncthreads();
            const int xstep = operand_order ? 1024 : 64;
            const int8_t* xrow[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int sn = st + (n && two), t = 16 * sn + r16, tc = t < T ? t : T - 1;
                xrow[n] = operand_order ? x_code + (size_t)(b * nsub + sn) * ksteps * 1024 + lane * 16 : x_code + ((size_t)b * T + tc) * Cc + 16 * q;
            }
            // K steps of 64 codes, KB at a time: all their loads are issued before the first MFMA consumes one
            constexpr int KB = PAIR ? (NJ <= 4 ? 6 : 4) : NJ <= 3 ? 8 : NJ <= 5 ? 6 : 2;  // (NJ + NT) * KB * 4 operand registers in flight
            for (int k0 = 0; k0 < ksteps; k0 += KB) {
                int32x4_t xb[KB][NT], wa[KB][NJ];
#pragma unroll
                for (int u = 0; u < KB; ++u) {
                    const bool in = 64 * (k0 + u) + 16 * q < Cc;  // past the end of the row (its length need not divide)
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        xb[u][n] = (int32x4_t){0, 0, 0, 0};
                        if (in) xb[u][n] = *reinterpret_cast<const int32x4_t*>(xrow[n] + xstep * (k0 + u));
                    }
#pragma unroll
                    for (int j = 0; j < NJ; ++j) wa[u][j] = load_w(J0 + j, k0 + u);
                }
#pragma unroll
                for (int u = 0; u < KB; ++u)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
#pragma unroll
                        for (int n = 0; n < NT; ++n) acc[n][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[u][j], xb[u][n], acc[n][j], 0, 0, 0);
            }
        }
        float v[NT][NJ][4], amax[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            amax[n] = kvh_values(v[n], acc[n], S, tok[n], J0, d, q);
            if (q == 0) amax_l[J0 ? 1 : 0][16 * (st + n) + r16] = amax[n];
        }
        __syncthreads();
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            if constexpr (PAIR) amax[n] = fmaxf(amax[n], amax_l[J0 ? 0 : 1][16 * (st + n) + r16]);
            if (n == 0 || two)
                kvh_finish<TPH, J0, NJ>(v[n], amax[n], tok[n].slot, st + n, h, b, side, d, r16, q, T, C, bits, qmaxf, codes, img, I);
        }
    };
    if (st < nsub && wave < 6) {
        if (part == 0)
            unit(std::integral_constant<int, 0>());
        else if constexpr (PAIR)
            unit(std::integral_constant<int, J1>());
    } else {  // the barriers of the others; the last wavefront, which has no column tile, then stores what the scales go into, beside them
        int slot[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) slot[i] = slot_of[lane + 64 * i < T ? lane + 64 * i : T - 1];
        if constexpr (WLDS) __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        __syncthreads();
        if (wave == 7) kvh_scales<PAIR ? 2 : 1>(amax_l, slot, side, lane, T, qmaxf, scales, img, I);
    }
}

template <int TPH, bool WLDS>
static hipError_t launch_kv_head_cfg(const int8_t* x_code, const float* s_x, const int8_t* w_code, const float* s_w,
                                     uint8_t* packed, const __half* context, const taq_shape& s, size_t lds, hipStream_t st) {
    const KvLayout L = kv_layout(s);
    const KvImage I = kv_image(s);
    {
        static std::atomic<unsigned long long> lds_set{0};
        const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&kv_head_kernel<TPH, WLDS>), 144 * 1024, lds_set);
        if (e != hipSuccess) return e;
    }
    const size_t xs = (size_t)KVH_SLOTS * s.Cc * 2;  // context rows of the protected-row workgroups
    if (WLDS) lds += 3 * 1024;  // up to three K steps past the end are read
    if (lds < xs) lds = xs;
    // Workgroups that share the protected rows of 128 channels (slots g, g + groups, ...): as many as run beside the others in
    // one round of the 256 compute units (LDS and 2048 threads per unit), at least 2, at most 16: a prompt has a few
    // protected rows, but any number is allowed.
    const int nc = (2 * s.C + 127) / 128;
    const int per_cu = lds > 80 * 1024 ? 1 : lds > 53 * 1024 ? 2 : lds > 40 * 1024 ? 3 : 4;
    int groups = (256 * per_cu - 2 * s.H * s.B) / (nc * s.B);
    groups = groups < 2 ? 2 : groups > 16 ? 16 : groups;
    const dim3 grid(2 * s.H + groups * nc, s.B), block(512);
    hipLaunchKernelGGL((kv_head_kernel<TPH, WLDS>), grid, block, lds, st, x_code, s_x, w_code, s_w, packed, L, I, s.T, s.C, s.H,
                       s.C / s.H, s.Cc, s.bits_kv, context);
    return hipGetLastError();
}

hipError_t launch_kv_head(const int8_t* x_code, const float* s_x, const int8_t* w_code, const float* s_w, uint8_t* packed,
                          const __half* context, const taq_shape& s, hipStream_t st) {
    const int tph = (s.C / s.H + 15) / 16;
    // weight slice of a head in LDS (one KiB per 16 rows x 64 codes) when the row length allows whole K steps and the
    // slice fits
    const size_t slice = (size_t)tph * (s.Cc / 64) * 1024;
    const bool wlds = s.Cc % 64 == 0 && slice <= 140 * 1024;
#define TAQ_KVH(N)                                                                                                       \
    case N:                                                                                                              \
        return wlds ? launch_kv_head_cfg<N, true>(x_code, s_x, w_code, s_w, packed, context, s, slice, st)               \
                    : launch_kv_head_cfg<N, false>(x_code, s_x, w_code, s_w, packed, context, s, 0, st);
    switch (tph) {
        TAQ_KVH(1) TAQ_KVH(2) TAQ_KVH(3) TAQ_KVH(4) TAQ_KVH(5) TAQ_KVH(6) TAQ_KVH(7) TAQ_KVH(8) TAQ_KVH(9) TAQ_KVH(10)
        default: return hipErrorInvalidValue;
    }
#undef TAQ_KVH
}

// ---------------------------------------------------------------- expansion for tests
__global__ __launch_bounds__(256) void kv_unpack_kernel(const uint8_t* __restrict__ packed, KvLayout L, int T,
                                                        int C, int H, int bits, int8_t* k_codes,
                                                        int8_t* v_codes, float* k_scales, float* v_scales,
                                                        __half* k_trig, __half* v_trig) {
    const int bt = blockIdx.x, b = bt / T, t = bt % T;
    const int slot = reinterpret_cast<const int*>(packed + L.slot_of)[bt];
    const float* s_k = reinterpret_cast<const float*>(packed + L.s_k);
    const float* s_v = reinterpret_cast<const float*>(packed + L.s_v);
    for (int h = threadIdx.x; h < H; h += 256) {
        size_t i = ((size_t)b * H + h) * T + t;
        if (k_scales) k_scales[i] = s_k[i];
        if (v_scales) v_scales[i] = s_v[i];
    }
    for (int side = 0; side < 2; ++side) {
        const uint8_t* codes = packed + (side ? L.v_code : L.k_code);
        const __half* full = reinterpret_cast<const __half*>(packed + (side ? L.v16 : L.k16));
        int8_t* oc = side ? v_codes : k_codes;
        __half* ot = side ? v_trig : k_trig;
        for (int c = threadIdx.x; c < C; c += 256) {
            int code = 0;
            if (slot < 0 && bits == 8) code = (int8_t)codes[(size_t)bt * C + c];
            if (slot < 0 && bits == 4) {
                int nib = (codes[(size_t)bt * (C / 2) + c / 2] >> (4 * (c & 1))) & 0xF;
                code = (nib ^ 8) - 8;  // sign-extend the two's-complement nibble
            }
            if (oc) oc[(size_t)bt * C + c] = (int8_t)code;
            if (ot) ot[(size_t)bt * C + c] = slot >= 0 ? full[((size_t)b * T + slot) * C + c] : __float2half(0.f);
        }
    }
}

hipError_t launch_kv_unpack(const uint8_t* packed, const taq_shape& s, int8_t* k_codes, int8_t* v_codes,
                            float* k_scales, float* v_scales, __half* k_trig, __half* v_trig, hipStream_t st) {
    KvLayout L = kv_layout(s);
    hipLaunchKernelGGL(kv_unpack_kernel, dim3(s.B * s.T), dim3(256), 0, st, packed, L, s.T, s.C, s.H, s.bits_kv,
                       k_codes, v_codes, k_scales, v_scales, k_trig, v_trig);
    return hipGetLastError();
}

}  // namespace taq
