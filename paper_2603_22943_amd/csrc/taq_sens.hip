// The token-sensitivity experiment (PersonalQ, Section III-B, Eq. 1) on block outputs, as one call: for every swept text
// token i and bit width b, the mean squared change of the block output when only the K and V rows of token i are
// quantized to b bits and everything else stays in full precision.
//
// Running the block once per (i, b) repeats almost all of its work. With p = A[n, i] of head h, u = 1 - p as the sum of the other
// tokens' weights (a difference from 1 would be all rounding where token i dominates), r = exp(sigma q.(k' - k)) and
// g = u + p r, replacing row i by (k', v') moves the head's attention output by
//     dO = alpha (O - v) + beta (v' - v),      alpha = p (1 - r) / g,   beta = p r / g
// (1 - r taken from expm1: no cancellation), and to_out is linear, so with P[n, h] = Wo_h O[n, h], a[i, h] = Wo_h v and
// D[i, h] = Wo_h (v' - v), each formed once,
//     y'(i, b)[n] = y[n] + sum_h ( alpha (P[n, h] - a[i, h]) + beta D[i, h] ),
// H multiply-adds per output element and term instead of the whole block. Everything is float32 (float64 in the sums of
// squares); the outputs are rounded to fp16 on both sides before the difference is taken, as the block stores them.
//
// Where token i dominates its row and its score falls, alpha is large (up to p / u) and O - v = u (m - v) is small, m being the
// mean of V over the other tokens by their weights: a difference of nearly equal numbers, enlarged. From alpha = 16 on, where
// the 2^-24 of O would be 2^-20 in dO (a 512th of the fp16 rounding of y'), the row's term is taken from m itself,
//     dO = (p - beta) (m - v) + beta (v' - v).
// alpha > 16 needs u < 1/16, so it is one token of a (row, head) at most, the one of the largest score: `dom` says which swept
// token that is, md holds m - v and dcoef p - beta, and sens_main_kernel adds that term apart from the others.
#include "taq_internal.h"

namespace taq {

typedef float sens_floatx4_t __attribute__((ext_vector_type(4)));

struct SensDims {
    int B, N, C, H, d, T;
    int Np;             // image tokens per batch element, padded to a multiple of 32 (rows of the chunked arrays)
    int nk;             // swept tokens
    float sigma;        // softmax scale
    float qmax[2];      // grids of the widths: 127 or 7
    unsigned char tok[TAQ_MAX_T];  // swept tokens
    signed char slot[TAQ_MAX_T];   // place of text token t among them, or -1
};

// ---------------------------------------------------------------- K, V rows: fp16 rows and the change quantization makes
// rows_f [B*T][2C] -> plane 0 = the row as the block stores it (fp16), plane 1 + j = code * s - that row (Eq. 2 at width
// j). V: vx[plane][b*T + t][C]. K in the order the score MFMAs read it, zero past the head and past the last token:
// kx[b][h][d/16 step][plane][tile of 16 tokens][lane = token + 16 * quarter][4 channels], one KiB per operand.
// One workgroup per (text token, batch element), tokens padded to whole tiles; per-head maxima through LDS atomics.
__device__ __forceinline__ size_t sens_kx_at(const SensDims& D, int nplanes, int b, int h, int k, int plane, int t) {
    const int S = (D.d + 15) >> 4, MT = (D.T + 15) >> 4;
    return ((((((size_t)b * D.H + h) * S + (k >> 4)) * nplanes + plane) * MT + (t >> 4)) * 64 + (t & 15) + 16 * ((k & 15) >> 2)) * 4;
}

template <int NB>
__global__ __launch_bounds__(256) void sens_rows_kernel(const float* __restrict__ rows_f, SensDims D, float* __restrict__ kx,
                                                        float* __restrict__ vx) {
    __shared__ unsigned smax[2 * TAQ_MAX_H];
    const int t = blockIdx.x, b = blockIdx.y;
    const int d16 = (D.d + 15) & ~15;
    const bool live = t < D.T;
    for (int v = threadIdx.x; v < D.H * d16 / 4; v += 256) {  // padding of the K operands
        const int h = v / (d16 / 4), k = 4 * (v % (d16 / 4));
        if (!live || k >= D.d)
#pragma unroll
            for (int j = 0; j <= NB; ++j)
                *reinterpret_cast<float4*>(kx + sens_kx_at(D, 1 + NB, b, h, k, j, t)) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (!live) return;
    for (int g = threadIdx.x; g < 2 * D.H; g += 256) smax[g] = 0u;
    __syncthreads();
    const int bt = b * D.T + t;
    const float4* xr = reinterpret_cast<const float4*>(rows_f + (size_t)bt * 2 * D.C);
    const int nv = D.C >> 1;
    for (int v = threadIdx.x; v < nv; v += 256) {
        const float4 f = xr[v];
        atomicMax(&smax[(v * 4) / D.d], __float_as_uint(fmaxf(fmaxf(fabsf(f.x), fabsf(f.y)), fmaxf(fabsf(f.z), fabsf(f.w)))));
    }
    __syncthreads();
    const size_t plane = (size_t)D.B * D.T * D.C;
    for (int v = threadIdx.x; v < nv; v += 256) {
        const int ch = v * 4;
        const bool isk = ch < D.C;
        const float4 f = xr[v];
        const float fv[4] = {f.x, f.y, f.z, f.w};
        const float amax = __uint_as_float(smax[ch / D.d]), safe = amax == 0.f ? 1.f : amax;
        auto put = [&](int j, float4 o) {
            if (isk) *reinterpret_cast<float4*>(kx + sens_kx_at(D, 1 + NB, b, ch / D.d, ch % D.d, j, t)) = o;
            else *reinterpret_cast<float4*>(vx + (size_t)j * plane + (size_t)bt * D.C + ch - D.C) = o;
        };
        float st[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) st[i] = __half2float(__float2half_rn(fv[i]));
        put(0, make_float4(st[0], st[1], st[2], st[3]));
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const float s = amax == 0.f ? 1.f : amax / D.qmax[j];
            float o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float code = fminf(fmaxf(__builtin_rintf((fv[i] * D.qmax[j]) / safe), -D.qmax[j]), D.qmax[j]);
                o[i] = __builtin_fmaf(code, s, -st[i]);
            }
            put(1 + j, make_float4(o[0], o[1], o[2], o[3]));
        }
    }
}

__device__ __forceinline__ float sens_quad_max(float x) {  // over the lanes l, l^16, l^32, l^48
    x = fmaxf(x, __shfl_xor(x, 16));
    return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float sens_quad_sum(float x) {
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// ---------------------------------------------------------------- attention of the reference block and the sweep's factors
// One workgroup of WV = 1 or 4 wavefronts per (16 image tokens, head): S^T = K Q^T and the score changes (k' - k) Q^T of every text token,
// softmax, O^T = V^T A^T, all with V_MFMA_F32_16X16X4_F32 (text tokens or channels along the rows, image tokens along the columns: the
// accumulator registers of the scores are the B operand of the last product). Each step's operands are requested while the step before is
// multiplied. Four wavefronts share out the operand tiles of the scores, the text tokens' factors (element i of each accumulator) and
// the channel blocks of O; scores and weights pass through LDS. One wavefront by itself on a SIMD issues an instruction every 8.6
// clocks, and 5000 of them were the time: 34 -> 18.9 us at 512 tokens of eight heads of 160 (256 workgroups), same bits. Where there are
// wavefronts enough without, the maxima and sums that all four form cost more (sens_wavefronts: where the line lies).
// o, md [row][C], ab [row][nk][NB][H]{alpha, beta}, dom [row][H] (swept token or -1), dcoef [row][H][NB], rows counted from row0 over all
// batch elements, D.Np of them each; md is written by workgroups with a dom >= 0 only. MT: tiles of 16 text tokens.
template <int NB, int MT, int WV>
__global__ __launch_bounds__(64 * WV) void sens_attn_kernel(const float* __restrict__ q_f, const float* __restrict__ kx,
                                                        const float* __restrict__ vx, SensDims D, int row0,
                                                        float* __restrict__ o, float* __restrict__ ab, int* __restrict__ dom,
                                                        float* __restrict__ dcoef, float* __restrict__ md) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int tile = blockIdx.x, h = blockIdx.y;
    const int row = tile * 16 + r16;  // of the chunk
    const int b = (row0 + tile * 16) / D.Np, np = (row0 + row) % D.Np, n = np < D.N ? np : D.N - 1;
    const int d = D.d, C = D.C, T = D.T, S16 = (d + 15) >> 4;
    constexpr int NP = (1 + NB) * MT, NW = (NP + WV - 1) / WV;  // operands of a step, of a wavefront: wave, wave + WV, ...
    __shared__ sens_floatx4_t sS[WV > 1 ? NP : 1][64];    // scores and their changes, as the accumulators hold them
    __shared__ __align__(16) float sp[WV > 1 ? MT : 1][64][4];        // weights
    __shared__ int sflag[4][16];
    sens_floatx4_t acc[NW];
#pragma unroll
    for (int u = 0; u < NW; ++u) acc[u] = (sens_floatx4_t){0.f, 0.f, 0.f, 0.f};
    const float* qr = q_f + ((size_t)b * D.N + n) * C + h * d;
    const float4* kr = reinterpret_cast<const float4*>(kx) + ((size_t)b * D.H + h) * S16 * NP * 64 + lane;
    float4 kv[NW], qv;
    auto fetch = [&](int s) {
        const int sc = s < S16 ? s : S16 - 1, k = 16 * sc + 4 * q;
        qv = *reinterpret_cast<const float4*>(qr + (k < d ? k : 0));  // (meets zeros of K past the head)
#pragma unroll
        for (int u = 0; u < NW; ++u) kv[u] = kr[((size_t)sc * NP + (wave + WV * u < NP ? wave + WV * u : NP - 1)) * 64];
    };
    fetch(0);
    for (int s = 0; s < S16; ++s) {
        float4 kc[NW];
#pragma unroll
        for (int u = 0; u < NW; ++u) kc[u] = kv[u];
        const float qe[4] = {qv.x, qv.y, qv.z, qv.w};
        fetch(s + 1);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int u = 0; u < NW; ++u) {
                const float ke[4] = {kc[u].x, kc[u].y, kc[u].z, kc[u].w};
                acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ke[e], qe[e], acc[u], 0, 0, 0);
            }
    }
    sens_floatx4_t S[MT], pw[MT];
    if constexpr (WV > 1) {
#pragma unroll
        for (int u = 0; u < NW; ++u)
            if (wave + WV * u < NP) sS[wave + WV * u][lane] = acc[u];
        __syncthreads();
    }
#pragma unroll
    for (int tt = 0; tt < MT; ++tt) {
        if constexpr (WV > 1) S[tt] = sS[tt][lane];
        else S[tt] = acc[tt];
    }
    auto change = [&](int j, int tt, int i) -> float {  // of the score by width j
        if constexpr (WV > 1) return reinterpret_cast<const float*>(&sS[(1 + j) * MT + tt][lane])[i];
        else return acc[(1 + j) * MT + tt][i];
    };
    // this lane: text tokens 16*tt + 4*q + i of image token r16
    float mx = -__builtin_inff();
#pragma unroll
    for (int tt = 0; tt < MT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool live = 16 * tt + 4 * q + i < T;
            S[tt][i] = live ? S[tt][i] * D.sigma : -__builtin_inff();
            mx = fmaxf(mx, S[tt][i]);
        }
    mx = sens_quad_max(mx);
    int top = TAQ_MAX_T;  // the first token of the largest score
#pragma unroll
    for (int tt = 0; tt < MT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = 16 * tt + 4 * q + i;
            if (S[tt][i] == mx && t < top) top = t;
        }
    top = min(top, __shfl_xor(top, 16));
    top = min(top, __shfl_xor(top, 32));
    float mr = -__builtin_inff();  // the largest of the others
#pragma unroll
    for (int tt = 0; tt < MT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (16 * tt + 4 * q + i != top) mr = fmaxf(mr, S[tt][i]);
    const bool alone = T == 1;
    mr = alone ? mx : sens_quad_max(mr);
    float Z = 0.f, R2 = 0.f;  // sum over all tokens beside the largest score, over the others beside theirs (>= 1 both)
#pragma unroll
    for (int tt = 0; tt < MT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            Z += __expf(S[tt][i] - mx);
            R2 += 16 * tt + 4 * q + i == top ? 0.f : __expf(S[tt][i] - mr);
        }
    Z = sens_quad_sum(Z);
    R2 = sens_quad_sum(R2);
    const float inv_z = 1.f / Z, u_top = R2 * __expf(mr - mx) * inv_z;
    int flagged = -1;
#pragma unroll
    for (int tt = 0; tt < MT; ++tt)
#pragma unroll
        for (int ii = 0; ii < 4 / WV; ++ii) {  // element `wave` of each tile, or all four
            const int i = WV > 1 ? wave : ii, t = 16 * tt + 4 * q + i;
            const float s0 = WV == 1 ? S[tt][ii] : wave == 0 ? S[tt][0] : wave == 1 ? S[tt][1] : wave == 2 ? S[tt][2] : S[tt][3];
            const float e = __expf(s0 - mx), p = e / Z;
            const int k = t < T ? D.slot[t] : -1;
            if (k >= 0) {
                const bool is_top = t == top;
                const float R = is_top ? R2 : Z - e;                     // the others' sum, >= 1 but for rounding ...
                const float lead = s0 - (is_top ? mr : mx);    // ... and this token's score beside the same reference
                const float u = is_top ? u_top : R * inv_z;
                float al[NB], be[NB], w[NB], Rc[NB];
                bool hv[NB], heavy = false;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const float dl = alone ? 0.f : change(j, tt, i) * D.sigma;
                    const float x = lead + dl, c = fmaxf(x, 0.f);
                    w[j] = __expf(x - c);
                    Rc[j] = R * __expf(-c);
                    be[j] = w[j] * __builtin_amdgcn_rcpf(w[j] + Rc[j]);  // (the sum is between 1 and T + 1)
                    const float em = expm1f(-fabsf(dl));               // e^-|dl| - 1
                    const float num = -p * em, g = u + p * (1.f + em);  // (of a score that falls)
                    hv[j] = dl <= 0.f && num > 16.f * g;
                    heavy |= hv[j];
                    al[j] = dl > 0.f ? be[j] * em : num / g;           // (p (1 - r) / g = beta (1 - r) / r)
                }
                if (heavy) {
                    flagged = k;
#pragma unroll
                    for (int j = 0; j < NB; ++j) {  // p - beta
                        dcoef[((size_t)row * D.H + h) * NB + j] = hv[j] ? Rc[j] / (w[j] + Rc[j]) - u : al[j] * u;
                        al[j] = 0.f;
                    }
                }
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    reinterpret_cast<float2*>(ab)[(((size_t)row * D.nk + k) * NB + j) * D.H + h] = make_float2(al[j], be[j]);
            }
            if constexpr (WV > 1) sp[tt][lane][i] = p;
            else pw[tt][ii] = p;
        }
    flagged = max(flagged, __shfl_xor(flagged, 16));
    flagged = max(flagged, __shfl_xor(flagged, 32));
    if constexpr (WV > 1) {
        if (q == 0) sflag[wave][r16] = flagged;
        __syncthreads();
        flagged = max(max(sflag[0][r16], sflag[1][r16]), max(sflag[2][r16], sflag[3][r16]));
#pragma unroll
        for (int tt = 0; tt < MT; ++tt) pw[tt] = *reinterpret_cast<const sens_floatx4_t*>(sp[tt][lane]);
    }
    if (wave == 0 && q == 0) dom[(size_t)row * D.H + h] = flagged;
    const bool sharp = __any(flagged >= 0);
    if (sharp) {  // m - v as weights of the V rows
        const float inv = 1.f / R2;
#pragma unroll
        for (int tt = 0; tt < MT; ++tt)
#pragma unroll
            for (int i = 0; i < 4; ++i) S[tt][i] = 16 * tt + 4 * q + i == top ? -1.f : __expf(S[tt][i] - mr) * inv;
    }
    float va[MT][4];
    auto fetch_v = [&](int j0) {
        const int c = j0 + r16 < d ? j0 + r16 : d - 1;
#pragma unroll
        for (int tt = 0; tt < MT; ++tt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = 16 * tt + 4 * q + i;
                va[tt][i] = vx[((size_t)b * T + (t < T ? t : T - 1)) * C + h * d + c];  // (weight 0 past the last token)
            }
    };
    fetch_v(16 * wave);
    for (int j0 = 16 * wave; j0 < d; j0 += 16 * WV) {
        float vc[MT][4];
#pragma unroll
        for (int tt = 0; tt < MT; ++tt)
#pragma unroll
            for (int i = 0; i < 4; ++i) vc[tt][i] = va[tt][i];
        fetch_v(j0 + 16 * WV);
        sens_floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tt = 0; tt < MT; ++tt)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(vc[tt][i], pw[tt][i], acc, 0, 0, 0);
        if (j0 + 4 * q < d)
            *reinterpret_cast<float4*>(o + (size_t)row * C + h * d + j0 + 4 * q) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        if (sharp) {
            sens_floatx4_t m = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int tt = 0; tt < MT; ++tt)
#pragma unroll
                for (int i = 0; i < 4; ++i) m = __builtin_amdgcn_mfma_f32_16x16x4f32(vc[tt][i], S[tt][i], m, 0, 0, 0);
            if (j0 + 4 * q < d)
                *reinterpret_cast<float4*>(md + (size_t)row * C + h * d + j0 + 4 * q) = make_float4(m[0], m[1], m[2], m[3]);
        }
    }
}

// One output channel's slice of a head (d % 8 == 0, 16-byte aligned) times a row's vector.
__device__ __forceinline__ float sens_dot(const __half* w, const float* m, int d) {
    float t = 0.f;
#pragma unroll 2
    for (int c = 0; c < d; c += 8) {
        const uint4 v = *reinterpret_cast<const uint4*>(w + c);
        const unsigned x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float2 f = __half22float2(*reinterpret_cast<const __half2*>(&x[i]));
            t = __builtin_fmaf(f.x, m[c + 2 * i], t);
            t = __builtin_fmaf(f.y, m[c + 2 * i + 1], t);
        }
    }
    return t;
}

// ---------------------------------------------------------------- outputs of every (token, width) and their squared changes
// A wavefront owns NR rows x 64 channels: P of all heads sits in registers (NR * HT of them), the factors alpha, beta of a
// row are wave-uniform (scalar loads), a and D come one coalesced load per head and are shared by the NR rows; the four
// wavefronts of a workgroup take neighbouring rows of the same channels, so that those loads meet in the compute unit's
// cache. Bound by vector issue: HT * (1 + 2 NB) multiply-adds per output element and swept token.
// Sums of squares in float64: per lane over the rows, then across lanes through LDS, 16 (token, width) pairs at a time.
// Workgroups with a row whose largest token needs its own term (dom) take a second form of the loop; the term is one dot
// product over the head's channels, for one token of a (row, head) at most.
template <int HT, int NR, int NB, bool EXACT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HT <= 8 ? 4 : 2))) void sens_main_kernel(const float* __restrict__ P, const float* __restrict__ ab,
                                                        const float* __restrict__ va, const float* __restrict__ bias,
                                                        const int* __restrict__ dom, const float* __restrict__ dcoef,
                                                        const float* __restrict__ md, const __half* __restrict__ Wo, SensDims D,
                                                        int row0, int kper, double* __restrict__ part, int part0, int npart) {
    constexpr int CHUNK = 16;
    __shared__ double red[4][CHUNK][65];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int H = EXACT ? HT : D.H, C = D.C;
    const int c = blockIdx.y * 64 + lane, cc = c < C ? c : C - 1;
    const int row = ((int)blockIdx.x * 4 + wave) * NR;  // first row of this wavefront, within the chunk
    const int b = (row0 + row) / D.Np, np0 = (row0 + row) % D.Np;
    const float bc = bias[cc];
    const int k0 = blockIdx.z * kper, k1 = k0 + kper < D.nk ? k0 + kper : D.nk;
    const size_t plane = (size_t)D.B * D.T * H * C;
    const bool cin = c < C;
    bool sharp = false;  // of the workgroup's rows
    for (int i = threadIdx.x; i < 4 * NR * H; i += 256) sharp |= dom[(size_t)blockIdx.x * (4 * NR) * H + i] >= 0;
    sharp = __syncthreads_or(sharp);
    // sums(k, a, dl, s): squared changes of token k over this wavefront's rows, given its a and D
    auto sweep = [&](auto sums) {
        for (int kb = k0; kb < k1; kb += CHUNK / NB) {
#pragma unroll 1
            for (int kk = 0; kk < CHUNK / NB && kb + kk < k1; ++kk) {
                const int k = kb + kk;
                const float* vr = va + ((size_t)b * D.T + D.tok[k]) * H * C + cc;
                float a[HT], dl[NB][HT];
#pragma unroll
                for (int h = 0; h < HT; ++h) {
                    const bool in = EXACT || h < H;
                    a[h] = in ? vr[(size_t)h * C] : 0.f;
#pragma unroll
                    for (int j = 0; j < NB; ++j) dl[j][h] = in ? vr[(size_t)(1 + j) * plane + (size_t)h * C] : 0.f;
                }
                double s[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) s[j] = 0.0;
                sums(k, a, dl, s);
#pragma unroll
                for (int j = 0; j < NB; ++j) red[wave][kk * NB + j][lane] = s[j];
            }
            __syncthreads();
            {
                int e = lane >> 2;  // four lanes per (token, width) pair
                asm volatile("" : "+v"(e));  // (addresses formed here, not held in registers over the loop)
                const int k = kb + e / NB;
                double t = 0.0;
#pragma unroll
                for (int u = 0; u < 16; ++u) t += red[wave][e][(lane & 3) * 16 + u];
                t += __shfl_xor(t, 1);
                t += __shfl_xor(t, 2);
                if ((lane & 3) == 0 && k < k1)
                    part[((size_t)(e % NB) * D.nk + k) * npart + part0 + ((int)blockIdx.x * 4 + wave) * (int)gridDim.y + (int)blockIdx.y] = t;
            }
            __syncthreads();
        }
    };
    auto row_of_p = [&](int r, float (&p)[HT], float& y, float& y16) {
        y = 0.f;
#pragma unroll
        for (int h = 0; h < HT; ++h) {
            p[h] = (EXACT || h < H) ? P[((size_t)(row + r) * H + h) * C + cc] : 0.f;
            y += p[h];
        }
        y += bc;
        y16 = __half2float(__float2half_rn(y));
    };
    auto changed = [&](int r, int k, const float (&p)[HT], const float (&a)[HT], const float (&dl)[NB][HT], float (&y)[NB]) {
        const float* fr = ab + ((size_t)(row + r) * D.nk + k) * NB * H * 2;
#pragma unroll
        for (int h = 0; h < HT; ++h) {
            if (EXACT || h < H) {
                const float pm = p[h] - a[h];
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    y[j] = __builtin_fmaf(fr[(j * H + h) * 2], pm, y[j]);
                    y[j] = __builtin_fmaf(fr[(j * H + h) * 2 + 1], dl[j][h], y[j]);
                }
            }
        }
    };
    auto square = [&](int r, const float (&y)[NB], float y16, double (&s)[NB]) {
        if (np0 + r < D.N && cin) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const double df = (double)(__half2float(__float2half_rn(y[j])) - y16);  // (exact: both are fp16 numbers)
                s[j] = __builtin_fma(df, df, s[j]);
            }
        }
    };
    if (!sharp) {
        float p[NR][HT], ys[NR], y16[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) row_of_p(r, p[r], ys[r], y16[r]);
        sweep([&](int k, const float (&a)[HT], const float (&dl)[NB][HT], double (&s)[NB]) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                float y[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) y[j] = ys[r];
                changed(r, k, p[r], a, dl, y);
                square(r, y, y16[r], s);
            }
        });
    } else {  // a row at a time, P read again for each token: with the rows' P in registers this form would spill
        sweep([&](int k, const float (&a)[HT], const float (&dl)[NB][HT], double (&s)[NB]) {
#pragma unroll 1
            for (int r = 0; r < NR; ++r) {
                float p[HT], ref, y16, y[NB];
                row_of_p(r, p, ref, y16);
#pragma unroll
                for (int j = 0; j < NB; ++j) y[j] = ref;
                changed(r, k, p, a, dl, y);
#pragma unroll 1
                for (int h = 0; h < H; ++h) {
                    const size_t rh = (size_t)(row + r) * H + h;
                    if (dom[rh] != k) continue;
                    const float t = sens_dot(Wo + (size_t)cc * C + h * D.d, md + (size_t)(row + r) * C + h * D.d, D.d);
#pragma unroll
                    for (int j = 0; j < NB; ++j) y[j] = __builtin_fmaf(dcoef[rh * NB + j], t, y[j]);
                }
                square(r, y, y16, s);
            }
        });
    }
}

__global__ __launch_bounds__(256) void sens_reduce_kernel(const double* __restrict__ part, int npart, double count, double* __restrict__ out) {
    __shared__ double red[256];
    const double* p = part + (size_t)blockIdx.x * npart;
    double s = 0.0;
    for (int i = threadIdx.x; i < npart; i += 256) s += p[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = red[0] / count;
}

// ---------------------------------------------------------------- host side
namespace {
int rows_per_wave(int H) { return H <= 8 ? 8 : H <= 16 ? 4 : 2; }
}  // namespace

SensWorkspace sens_workspace(const taq_shape& s, int ntok, int nbits) {
    SensWorkspace W;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    const size_t BT = (size_t)s.B * s.T, C = s.C, H = s.H;
    W.np = (int)align_up(s.N, 32);
    const size_t rows = (size_t)s.B * W.np;
    // rows per pass: P and the factors of a chunk stay within 128 MiB (whole 64-row GEMM tiles)
    const size_t per_row = (H * C + 2 * C + (size_t)ntok * nbits * H * 2 + H * (1 + nbits)) * 4;
    size_t chunk = ((size_t)128 << 20) / per_row / 64 * 64;
    chunk = chunk < 64 ? 64 : chunk;
    W.chunk = (int)(chunk < rows ? chunk : rows);
    W.rows_f = take(BT * 2 * C * 4);
    W.kx = take((1 + nbits) * s.B * align_up(s.T, 16) * H * align_up(C / H, 16) * 4);
    W.vx = take((1 + nbits) * BT * C * 4);
    W.va = take((1 + nbits) * BT * H * C * 4);
    W.q_f = take((size_t)s.B * s.N * C * 4);
    W.o = take((size_t)W.chunk * C * 4);
    W.p = take((size_t)W.chunk * H * C * 4);
    W.ab = take((size_t)W.chunk * ntok * nbits * H * 2 * 4);
    W.dom = take((size_t)W.chunk * H * 4);
    W.dcoef = take((size_t)W.chunk * H * nbits * 4);
    W.md = take((size_t)W.chunk * C * 4);
    W.npart = (int)(rows / rows_per_wave(s.H) * ((C + 63) / 64));
    W.part = take((size_t)W.npart * ntok * nbits * 8);
    W.total = off;
    return W;
}

template <int NB>
static hipError_t sens_run(const void* hidden, const void* context, const __half* Wk, const __half* Wv, const __half* Wq,
                           const __half* Wo, const float* bias, const int* tokens, int ntok, const int* bits, const taq_shape& s,
                           double* out, uint8_t* ws, hipStream_t st) {
    const SensWorkspace W = sens_workspace(s, ntok, NB);
    SensDims D;
    D.B = s.B; D.N = s.N; D.C = s.C; D.H = s.H; D.d = s.C / s.H; D.T = s.T;
    D.Np = W.np;
    D.nk = ntok;
    D.sigma = s.softmax_scale != 0.f ? s.softmax_scale : 1.0f / sqrtf((float)D.d);
    for (int j = 0; j < 2; ++j) D.qmax[j] = bits[j < NB ? j : 0] == 4 ? 7.f : 127.f;
    for (int t = 0; t < TAQ_MAX_T; ++t) { D.slot[t] = -1; D.tok[t] = 0; }
    for (int k = 0; k < ntok; ++k) {
        D.tok[k] = (unsigned char)tokens[k];
        D.slot[tokens[k]] = (signed char)k;
    }
    float* rows_f = reinterpret_cast<float*>(ws + W.rows_f);
    float* kx = reinterpret_cast<float*>(ws + W.kx);
    float* vx = reinterpret_cast<float*>(ws + W.vx);
    float* va = reinterpret_cast<float*>(ws + W.va);
    float* q_f = reinterpret_cast<float*>(ws + W.q_f);
    float* o = reinterpret_cast<float*>(ws + W.o);
    float* P = reinterpret_cast<float*>(ws + W.p);
    float* ab = reinterpret_cast<float*>(ws + W.ab);
    int* dom = reinterpret_cast<int*>(ws + W.dom);
    float* dcoef = reinterpret_cast<float*>(ws + W.dcoef);
    float* md = reinterpret_cast<float*>(ws + W.md);
    double* part = reinterpret_cast<double*>(ws + W.part);
    const int BT = s.B * s.T, C = s.C, H = s.H, rows = s.B * W.np, NR = rows_per_wave(H);
    hipError_t e;
    if ((e = launch_gemm_kv_rows(static_cast<const __half*>(context), Wk, Wv, BT, C, s.Cc, rows_f, st)) != hipSuccess) return e;
    if ((e = launch_gemm_f16(static_cast<const __half*>(hidden), Wq, s.B * s.N, C, C, q_f, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(sens_rows_kernel<NB>, dim3((s.T + 15) / 16 * 16, s.B), dim3(256), 0, st, rows_f, D, kx, vx);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = launch_gemm_f32_heads(vx, Wo, (1 + NB) * BT, C, C, H, va, st)) != hipSuccess) return e;
    for (int r0 = 0; r0 < rows; r0 += W.chunk) {
        const int nr = rows - r0 < W.chunk ? rows - r0 : W.chunk;  // a multiple of 32
#define TAQ_SENS_ATTN(MT) \
    case MT: \
        if (sens_wavefronts(nr / 16 * H) == 4) \
            hipLaunchKernelGGL((sens_attn_kernel<NB, MT, 4>), dim3(nr / 16, H), dim3(256), 0, st, q_f, kx, vx, D, r0, o, ab, dom, dcoef, md); \
        else hipLaunchKernelGGL((sens_attn_kernel<NB, MT, 1>), dim3(nr / 16, H), dim3(64), 0, st, q_f, kx, vx, D, r0, o, ab, dom, dcoef, md); \
        break;
        switch ((s.T + 15) / 16) {
            TAQ_SENS_ATTN(1) TAQ_SENS_ATTN(2) TAQ_SENS_ATTN(3) TAQ_SENS_ATTN(4) TAQ_SENS_ATTN(5) TAQ_SENS_ATTN(6)
            default: return hipErrorInvalidValue;
        }
#undef TAQ_SENS_ATTN
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = launch_gemm_f32_heads(o, Wo, nr, C, C, H, P, st)) != hipSuccess) return e;
        const int gx = nr / (4 * NR), gy = (C + 63) / 64;
        // split the swept tokens so that about four workgroups per compute unit are there, at least 8 tokens each (every
        // part loads its rows of P again)
        int split = 1024 / (gx * gy);
        split = split < 1 ? 1 : split > (ntok + 7) / 8 ? (ntok + 7) / 8 : split;
        const int kper = (ntok + split - 1) / split;
        const dim3 grid(gx, gy, (ntok + kper - 1) / kper);
        const int part0 = r0 / NR * gy;
#define TAQ_SENS_MAIN(HT, R, EX)                                                                                              \
    hipLaunchKernelGGL((sens_main_kernel<HT, R, NB, EX>), grid, dim3(256), 0, st, P, ab, va, bias, dom, dcoef, md, Wo, D, r0, kper, part, \
                       part0, W.npart)
        if (H == 8) TAQ_SENS_MAIN(8, 8, true);
        else if (H == 4) TAQ_SENS_MAIN(4, 8, true);
        else if (H < 8) TAQ_SENS_MAIN(8, 8, false);
        else if (H <= 16) TAQ_SENS_MAIN(16, 4, false);
        else TAQ_SENS_MAIN(32, 2, false);
#undef TAQ_SENS_MAIN
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(sens_reduce_kernel, dim3(ntok * NB), dim3(256), 0, st, part, W.npart, (double)s.B * s.N * s.C, out);
    return hipGetLastError();
}

hipError_t launch_token_sensitivity(const void* hidden, const void* context, const __half* Wk, const __half* Wv, const __half* Wq,
                                    const __half* Wo, const float* bias, const int* tokens, int ntok, const int* bits, int nbits,
                                    const taq_shape& s, double* out, uint8_t* ws, hipStream_t st) {
    if (s.H > TAQ_SENS_MAX_H || ntok < 1 || ntok > s.T) return hipErrorInvalidValue;
    if (nbits == 1) return sens_run<1>(hidden, context, Wk, Wv, Wq, Wo, bias, tokens, ntok, bits, s, out, ws, st);
    if (nbits == 2) return sens_run<2>(hidden, context, Wk, Wv, Wq, Wo, bias, tokens, ntok, bits, s, out, ws, st);
    return hipErrorInvalidValue;
}

}  // namespace taq
