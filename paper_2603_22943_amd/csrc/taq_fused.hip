// Dispatch of the fused TAQ cross-attention block (PersonalQ, Section III-B), the K~/V~ image and weight re-layout
// kernels, and the to_out tail kernel of the head-group path. The block kernel itself is in taq_fused_kernel.h.
#include "taq_fused_kernel.h"
#include "taq_heads_kernel.h"

namespace taq {

// ------------------------------------------------------------------------------------------
// K~/V~ image builder: rearranges the codes of qkv_packed into the order the fused kernel's MFMA
// operands are read in, and precomputes the per-head power-of-two prescale of V.
//   per head h:  Kp[t][tile][q][e] = k_code[t][h*d + 16*tile + 4*q + e]         (0 outside d / T; heads with a
//                multiple of 4 tiles use the order [t][tile/4][q][tile%4][e])
//                Vt[j][vt_pos(t)] = v_code[t][h*d + j] ^ 0x80   (vt_pos: 32*s + 8*q + 4*a + e for t = 32*s + 16*a + 4*q + e)
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int code_at(const uint8_t* codes, size_t row, int C, int c, int bits) {
    if (bits == 8) return (int8_t)codes[row * C + c];
    const int nib = (codes[row * (C >> 1) + (c >> 1)] >> (4 * (c & 1))) & 0xF;
    return (nib ^ 8) - 8;
}

__global__ __launch_bounds__(256) void kv_image_kernel(uint8_t* __restrict__ packed, KvLayout L, KvImage I, int T, int C,
                                                       int H, int bits) {
    const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x + 256 * blockIdx.z, nth = 256 * gridDim.z;
    const int d = C / H;
    const int* slot_of = reinterpret_cast<const int*>(packed + L.slot_of) + b * T;
    const float* s_k = reinterpret_cast<const float*>(packed + L.s_k) + ((size_t)b * H + h) * T;
    const float* s_v = reinterpret_cast<const float*>(packed + L.s_v) + ((size_t)b * H + h) * T;
    const uint8_t* k_code = packed + L.k_code;
    const uint8_t* v_code = packed + L.v_code;
    uint8_t* img = packed + L.image + (size_t)b * L.image_bytes + (size_t)h * I.head_bytes;  // this head's block
    __shared__ float vpre_s;
    if (threadIdx.x == 0) {  // (every z-slice recomputes it; only slice 0 stores it)  // per-head prescale: the largest |s_V * code| goes to [256, 512)
        float smax = 0.f;
        for (int t = 0; t < T; ++t)
            if (slot_of[t] < 0) smax = fmaxf(smax, s_v[t]);
        int kexp = 0;
        const float dmax = smax * (bits == 4 ? 7.f : 127.f);
        if (dmax > 0.f) {
            int e;
            (void)frexpf(dmax, &e);
            kexp = 9 - e;
        }
        vpre_s = ldexpf(1.0f, kexp);
        if (blockIdx.z == 0) {
            reinterpret_cast<float*>(img + I.vpre)[0] = ldexpf(1.0f, kexp);
            reinterpret_cast<float*>(img + I.oscale)[0] = ldexpf(1.0f, -kexp);
        }
    }
    __syncthreads();
    for (int t = tid; t < I.ntok; t += nth) {
        const bool isint = t < T && slot_of[t] < 0;
        reinterpret_cast<float*>(img + I.s_k)[t] = isint ? s_k[t] : 0.f;
        const float sp = isint ? s_v[t] * vpre_s : 0.f;  // s' = s_V * 2^kexp as two fp16 numbers, high part and remainder
        const __half sph = __float2half_rn(sp);
        reinterpret_cast<__half*>(img + I.s_vp)[t] = sph;
        reinterpret_cast<__half*>(img + I.s_vp)[I.ntok + t] = __float2half_rn(sp - __half2float(sph));
        reinterpret_cast<float*>(img + I.bias)[t] = isint ? 0.f : TAQ_NEG_INF;
    }
    const int rowb = I.tph * 16;  // bytes per (head, token) row of Kp
    for (int i = tid; i < I.rows_k * rowb; i += nth) {
        const int e = i & 3, q = (i >> 2) & 3, tile = (i % rowb) >> 4, t = i / rowb;
        const int cl = 16 * tile + 4 * q + e;
        int v = 0;
        if (t < T && cl < d && slot_of[t] < 0) v = code_at(k_code, (size_t)b * T + t, C, h * d + cl, bits);
        img[I.kp + kp_offset(I.tph, t, tile, q) + e] = (uint8_t)(v & 0xFF);
    }
    for (int i = tid; i < d * I.cols_v; i += nth) {
        const int t = i % I.cols_v, j = i / I.cols_v;  // token t of channel j goes to position vt_pos(t)
        int v = 0;
        if (t < T && slot_of[t] < 0) v = code_at(v_code, (size_t)b * T + t, C, h * d + j, bits);
        // stored with the sign bit flipped (code + 128 as an unsigned byte): 0x6400 | byte is then the
        // fp16 number 1024 + 128 + code, one packed subtraction away from the code itself
        img[I.vt + (size_t)j * I.cols_v + vt_pos(t, I.nt16)] = (uint8_t)((v & 0xFF) ^ 0x80);
    }
}

hipError_t launch_kv_image(uint8_t* packed, const taq_shape& s, hipStream_t st) {
    const KvLayout L = kv_layout(s);
    const KvImage I = kv_image(s);
    hipLaunchKernelGGL(kv_image_kernel, dim3(s.H, s.B, 8), dim3(256), 0, st, packed, L, I, s.T, s.C, s.H, s.bits_kv);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Weight re-layout for the fused kernel (optional, shape.w_layout = 1)
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_weight_kernel(const int8_t* __restrict__ codes, int C, int d, int tph, int kc,
                                                          size_t pack_off, int8_t* __restrict__ out) {
    // one 16-byte vector per thread: first the row-major copy, then the operand-ordered copy
    const size_t nrow = (size_t)C * C / 16;
    const size_t npack = (size_t)(C / d) * tph * kc * 64;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nrow + npack; i += (size_t)gridDim.x * 256) {
        if (i < nrow) {
            if (codes != out) reinterpret_cast<uint4*>(out)[i] = reinterpret_cast<const uint4*>(codes)[i];
        } else {
            const size_t v = i - nrow;
            const int lane = (int)(v & 63), r = lane & 15, q = lane >> 4;
            const size_t blk = v >> 6;  // (h * tph + j) * kc + ks
            const int ks = (int)(blk % kc), j = (int)((blk / kc) % tph), h = (int)(blk / ((size_t)kc * tph));
            int row = h * d + 16 * j + r;
            row = row < C ? row : C - 1;
            reinterpret_cast<uint4*>(out + pack_off)[v] =
                *reinterpret_cast<const uint4*>(codes + (size_t)row * C + 64 * ks + 16 * q);
        }
    }
}

hipError_t launch_pack_weight(const int8_t* codes, const taq_shape& s, int8_t* out, hipStream_t st) {
    const int d = s.C / s.H;
    hipLaunchKernelGGL(pack_weight_kernel, dim3(256), dim3(256), 0, st, codes, s.C, d, (d + 15) / 16, s.C / 64,
                       weight_pack_offset(s), out);
    return hipGetLastError();
}

// Per-token quantization of A^ V~ and to_out for the head-group shapes (C = 1280 and 640):
// Y^T[c][n] = Wo[c][:] . o_code[n][:]. A workgroup owns 16 image tokens and OT output tiles of 16 channels; KS wavefronts share an output
// tile by K range. A^ V~ and its largest magnitudes come from the workspace in operand order (StageTile), a lane's four channels at a
// time, and every workgroup of a token tile forms the same int8 codes in LDS: one kernel less. Same operand layout and epilogue as the
// last phase of the fused kernel. An eighth of the (tile, output tiles) pairs to an XCD, tile after tile, as in heads_kernel, whose
// A^ V~ is then in the XCD's own L2.
// What bounds it: what the busiest compute unit pulls through its path, 80 KB of rows and 20 KB of weights per output tile at C = 1280
// (41 and 10 at 640). So: the smallest OT of 2, 4, 8, 10 with which all workgroups run at once, one to a unit (tail_ot, where the timings
// are). Before, OT = 8 throughout and all weights in front of the barrier, us per layer at d = 160: 64 tokens 12.7, 128 13.2, 256 13.3, 512 15.0,
// 700 18.3.
// Registers: at most 128 with eight wavefronts, 96 with ten, 80 with C = 640, for two and three workgroups to a unit (C = 640, 2048
// tokens: 16.95 -> 15.95 us).
struct TailReq {
    const int8_t* wo;
    const float* scales;  // s_wo | bias
    __half* out;
};
struct TailArgs {
    TailReq rq;
    const float* o_op;
    const float* o_max;
    int8_t* tap_code;
    float* tap_scale;
    size_t w_off;
    int N, NT, tile0, tiles, H;
};
struct TailManyArgs {  // several requests in a launch, as HeadsManyArgs
    TailArgs a;
    size_t ws_step;
    TailReq req[TAQ_MAX_REQ];
};

template <int C, int OT, int KS, bool ROWMAJ, bool MANY>
__global__ __launch_bounds__(64 * OT * KS) __attribute__((amdgpu_waves_per_eu(OT == 10 ? 5 : C == 640 ? 6 : 4)))
void to_out_tail_kernel(std::conditional_t<MANY, TailManyArgs, TailArgs> args) {
    const TailArgs& a = [&]() -> const TailArgs& {
        if constexpr (MANY) return args.a;
        else return args;
    }();
    constexpr int NW = OT * KS, KC = C / 64, KW = KC / KS, TILE_RS = C + 16, NG = C / 16 / OT;
    static_assert(C % (16 * NW) == 0 && KC % KS == 0, "whole groups of output tiles, whole shares of a row");
    constexpr int CH = C / 16 / NW;  // float4 pieces of the tile per thread
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r16 = lane & 15, q = lane >> 4;
    const unsigned ri = MANY ? blockIdx.y : 0u;
    TailReq rq = a.rq;
    size_t ws_at = 0;
    if constexpr (MANY) {
        rq = args.req[ri];
        ws_at = ri * args.ws_step;
    }
    asm volatile("" ::"s"(a.o_op), "s"(a.o_max), "s"(rq.wo), "s"(a.w_off), "s"(a.tiles), "s"(a.H), "s"(a.tile0), "s"(a.NT), "s"(a.N));
    const int item = XcdShare::item(blockIdx.x, (unsigned)(a.tiles * NG));
    if (item < 0) return;
    const int lt = item / NG, gt = (item - lt * NG) * OT + wave % OT;  // tile of the chunk; output tile of the layer: channels 16*gt .. 16*gt+15
    const int k0 = wave / OT * KW;                                     // first K step
    const float* o_op = reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.o_op) + ws_at);
    const float* o_max = reinterpret_cast<const float*>(reinterpret_cast<const char*>(a.o_max) + ws_at);
    int8_t* tileq = reinterpret_cast<int8_t*>(smem);               // [16][C+16]
    unsigned char* slot = smem + 16 * TILE_RS + wave * 1024;       // row-major weights only
    // The rows of the tile are requested first: they are needed first (quantizer), and loads return in order.
    const int wrow = !ROWMAJ ? (int)a.w_off + (gt * KC + k0) * 1024 + lane * 16 : (16 * gt + (lane >> 2)) * C + 64 * k0 + 16 * (lane & 3);
    constexpr int wstep = ROWMAJ ? 64 : 1024;
    int32x4_t wa[KW];
    float4 xv[CH];
    const float4* xr = reinterpret_cast<const float4*>(o_op) + (size_t)lt * (C / 16) * 64 + tid;
#pragma unroll
    for (int it = 0; it < CH; ++it) xv[it] = xr[it * 64 * NW];
    float amax = 0.f;
    for (int h = q; h < a.H; h += 4) amax = fmaxf(amax, o_max[((size_t)lt * a.H + h) * 16 + r16]);
    __builtin_amdgcn_sched_barrier(0);
    amax = quad_allmax(amax);
    const bool zero = amax == 0.f;
    const float so = zero ? 1.f : div_grid(amax, 127.f);
    const float safe = zero ? 1.f : amax;
    const float cq = quant_mult(127.f, safe);
    const int tile = a.tile0 + lt, b = tile / a.NT, n = (tile - b * a.NT) * 16 + r16;
    const size_t row = (size_t)b * a.N + (n < a.N ? n : a.N - 1);
    const bool tap = gt < OT && n < a.N;
    if (tap && a.tap_scale && tid < 16) a.tap_scale[row] = so;
    // The first weights are requested a few at a time between pieces of the quantizer, the others between the products (all of them in
    // front of the barrier: 15.0 us at 512 tokens, 10 of 20: 14.4).
    constexpr int PRE = KC == 10 || KW < 10 ? KW : OT == 8 && !ROWMAJ ? 12 : OT == 8 ? 8 : 10, EX = 2;
    constexpr int QS = CH % 2 ? 1 : 2, LPS = (PRE + CH / QS - 1) / (CH / QS);
    static_assert(PRE >= EX, "the lanes of row-major weights change EX steps ahead");
    auto load_w = [&](int ks) { wa[ks] = *reinterpret_cast<const int32x4_t*>(rq.wo + wrow + wstep * ks); };
#pragma unroll
    for (int it = 0; it < CH; it += QS) {
#pragma unroll
        for (int ks = it / QS * LPS; ks < (it / QS + 1) * LPS && ks < PRE; ++ks) load_w(ks);
        unsigned pk[QS];
        quant4_group<QS>(pk, [&](int i) { return xv[it + i]; }, [&](int) { return QuantRow{1.f, cq, safe}; });
#pragma unroll
        for (int i = 0; i < QS; ++i) {
            const int c = 16 * (wave + NW * (it + i)) + 4 * q;
            *reinterpret_cast<unsigned*>(tileq + r16 * TILE_RS + c) = pk[i];
            if (tap && a.tap_code) *reinterpret_cast<unsigned*>(a.tap_code + row * C + c) = pk[i];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    if constexpr (ROWMAJ) {
#pragma unroll
        for (int ks = 0; ks < EX; ++ks) wa[ks] = exchange_rows(wa[ks], slot, lane);
    }
    int32x4_t acc = (int32x4_t){0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KW; ++ks) {
        if (ROWMAJ && ks + EX < KW) wa[ks + EX] = exchange_rows(wa[ks + EX], slot, lane);
        const int32x4_t hb = *reinterpret_cast<const int32x4_t*>(tileq + r16 * TILE_RS + 64 * (k0 + ks) + 16 * q);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[ks], hb, acc, 0, 0, 0);
        if (ks + PRE < KW) {
            load_w(ks + PRE);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (KS > 1) {  // integer sums: the same in any order
        int32x4_t* part = reinterpret_cast<int32x4_t*>(smem + 16 * TILE_RS + (ROWMAJ ? NW * 1024 : 0));  // [(KS - 1) OT][64 lanes]
        if (wave >= OT) part[(wave - OT) * 64 + lane] = acc;
        __syncthreads();
        if (wave >= OT) return;
#pragma unroll
        for (int k = 1; k < KS; ++k) acc += part[((k - 1) * OT + wave) * 64 + lane];
    }
    const int c = 16 * gt + 4 * q;
    const float4 w4 = *reinterpret_cast<const float4*>(rq.scales + c);
    const float4 b4 = *reinterpret_cast<const float4*>(rq.scales + C + c);
    const float y0 = (float)acc[0] * (so * w4.x) + b4.x;
    const float y1 = (float)acc[1] * (so * w4.y) + b4.y;
    const float y2 = (float)acc[2] * (so * w4.z) + b4.z;
    const float y3 = (float)acc[3] * (so * w4.w) + b4.w;
    if (n < a.N) {
        const half4_t y = {(_Float16)y0, (_Float16)y1, (_Float16)y2, (_Float16)y3};
        *reinterpret_cast<half4_t*>(rq.out + row * C + c) = y;
    }
}

// What every variant of the block kernel is told about the layer.
static FusedDims fused_dims(const taq_shape& s, int R, const taq_debug* dbg) {
    FusedDims dm = {};
    dm.R = R;
    dm.B = s.B;
    dm.N = s.N;
    dm.T = s.T;
    dm.nt16 = (s.T + 15) / 16;
    dm.w_layout = s.w_layout;
    dm.w_pack_off = (unsigned)weight_pack_offset(s);
    dm.w_bytes = (unsigned)(s.w_layout ? weight_pack_bytes(s) : (size_t)s.C * s.C);
    const float sigma = s.softmax_scale != 0.f ? s.softmax_scale : 1.0f / sqrtf((float)(s.C / s.H));
    dm.sig2 = sigma * 1.4426950408889634f;
    dm.qmaxq = s.bits_q == 4 ? 7.f : 127.f;
    dm.plast = s.bits_prob == 4 ? 15.f : 255.f;
    dm.pmax = s.prob_grid == TAQ_PROB_LOG2 ? 256.f : dm.plast;
    dm.L = kv_layout(s);
    dm.I = kv_image(s);
    if (dbg && R == 1) dm.dbg = *dbg;
    return dm;
}

hipError_t launch_fused_block(const FusedReq* reqs, int R, const taq_shape& s, const taq_debug* dbg, hipStream_t st) {
    if (R < 1 || R > TAQ_MAX_REQ || !fused_supported(s)) return hipErrorInvalidValue;
    FusedTable tab;
    for (int r = 0; r < TAQ_MAX_REQ; ++r) tab.req[r] = reqs[r < R ? r : 0];
    const FusedDims dm = fused_dims(s, R, dbg);
    const int d = s.C / s.H, grid = s.prob_grid;
    // 32-token tiles that would occupy under half of the 256 compute units: 16-token workgroups instead
    // (shape.tok_tile = 32 or 16 forces one variant: for tests and tuning)
    const bool few = s.tok_tile == 16 ? true : s.tok_tile == 32 ? false : ((s.N + 31) / 32) * R * s.B <= 128;
    const int tok = few ? 16 : 32;
    if (d == 40 && s.H == 8) return launch_fused_d40(tab, dm, grid, tok, st);
    if (d == 80 && s.H == 8) return launch_fused_d80(tab, dm, grid, tok, st);
    if (d == 64 && s.H == 10) return launch_fused_d64(tab, dm, grid, tok, st);
    return hipErrorInvalidValue;
}

// Layers too wide for one workgroup (C = 1280), and C = 640 layers of few tokens, two kernels per chunk of tiles: per-token codes of `hidden`, to_q, Q~ and the attention
// per head group, then per-token codes of A^ V~ and to_out.
hipError_t launch_heads(const StageChunk& c, const taq_shape& s, const FusedReq* reqs, int R, size_t ws_step, int tt, const taq_debug* dbg, hipStream_t st) {
    if (!mid_supported(s) || R < 1 || R > TAQ_MAX_REQ) return hipErrorInvalidValue;
    HeadsManyArgs m = {};
    HeadsArgs& a = m.a;
    for (int r = 0; r < R; ++r) m.req[r] = HeadsReq{reqs[r].hidden, reqs[r].packed, reqs[r].wq, reqs[r].scales};
    a.rq = m.req[0];
    m.ws_step = ws_step;
    a.o_op = c.o_op;
    a.o_max = c.o_max;
    const KvLayout L = kv_layout(s);
    a.image = L.image;
    a.image_bytes = L.image_bytes;
    a.k16 = L.k16;
    a.v16t = L.v16t;
    if (L.ntrig != 0) return hipErrorInvalidValue;  // the kernel reads the number of protected tokens at the front of qkv_packed
    a.I = kv_image(s);
    a.w_off = weight_pack_offset(s);
    a.N = s.N; a.NT = c.NT; a.tile0 = c.tile0; a.tile1 = c.tile1; a.T = s.T;
    a.nt16 = (s.T + 15) / 16;
    const int d = s.C / s.H;
    const float sigma = s.softmax_scale != 0.f ? s.softmax_scale : 1.0f / sqrtf((float)d);
    a.sig2 = sigma * 1.4426950408889634f;
    a.qmaxq = s.bits_q == 4 ? 7.f : 127.f;
    a.plast = s.bits_prob == 4 ? 15.f : 255.f;
    a.pmax = s.prob_grid == TAQ_PROB_LOG2 ? 256.f : a.plast;
    a.b0 = c.tile0 / c.NT;
    a.nb = (c.tile1 - 1) / c.NT - a.b0 + 1;
    if (dbg) a.dbg = *dbg;
    const int tiles_b = a.nb == 1 ? c.tile1 - c.tile0 : c.NT;  // tiles of a batch element in the chunk, at most
    const auto launch = s.C == 640 ? (d == 80 ? launch_heads80 : launch_heads64x10) : d == 160 ? launch_heads160 : launch_heads64;
    return launch(m, R, s.prob_grid, tiles_b, tt, s.w_layout == 1, st);
}

template <int C, int OT, int KS, bool ROWMAJ>
static hipError_t launch_tail_some(const TailManyArgs& m, int R, hipStream_t st) {
    const long items = (long)m.a.tiles * (C / 16 / OT);
    if (items > XcdShare::MOST) return hipErrorInvalidValue;
    const unsigned lds = 16 * (C + 16) + (KS - 1) * OT * 1024 + (ROWMAJ ? OT * KS * 1024 : 0);  // (below 64 KiB: needs no attribute)
    const dim3 grid(XcdShare::grid((unsigned)items), R), block(64 * OT * KS);
    if (R > 1) hipLaunchKernelGGL((to_out_tail_kernel<C, OT, KS, ROWMAJ, true>), grid, block, lds, st, m);
    else hipLaunchKernelGGL((to_out_tail_kernel<C, OT, KS, ROWMAJ, false>), grid, block, lds, st, m.a);
    return hipGetLastError();
}
template <int C, int OT, int KS>
static hipError_t launch_tail_cfg(const TailManyArgs& m, int R, bool packed, hipStream_t st) {
    return packed ? launch_tail_some<C, OT, KS, false>(m, R, st) : launch_tail_some<C, OT, KS, true>(m, R, st);
}

hipError_t launch_to_out_tail(const StageChunk& c, const taq_shape& s, const FusedReq* reqs, int R, size_t ws_step, const taq_debug* dbg, hipStream_t st) {
    if (R < 1 || R > TAQ_MAX_REQ) return hipErrorInvalidValue;
    TailManyArgs m = {};
    TailArgs& a = m.a;
    for (int r = 0; r < R; ++r) m.req[r] = TailReq{reqs[r].wo, reqs[r].scales + s.C, reqs[r].out};
    a.rq = m.req[0];
    a.o_op = c.o_op;
    a.o_max = c.o_max;
    a.tap_code = dbg ? dbg->o_code : nullptr;
    a.tap_scale = dbg ? dbg->s_o : nullptr;
    a.w_off = weight_pack_offset(s);
    m.ws_step = ws_step;
    a.N = s.N; a.NT = c.NT; a.tile0 = c.tile0; a.tiles = c.tile1 - c.tile0; a.H = s.H;
    const bool packed = s.w_layout != 0;
    const int ot = tail_ot(s.C, (long)a.tiles * R);
    if (s.C == 1280) {
        if (ot == 2) return launch_tail_cfg<1280, 2, 4>(m, R, packed, st);
        if (ot == 4) return launch_tail_cfg<1280, 4, 2>(m, R, packed, st);
        if (ot == 10) return launch_tail_cfg<1280, 10, 1>(m, R, packed, st);
        return launch_tail_cfg<1280, 8, 1>(m, R, packed, st);
    }
    if (s.C == 640) {
        if (ot == 10) return launch_tail_cfg<640, 10, 1>(m, R, packed, st);
        return launch_tail_cfg<640, 8, 1>(m, R, packed, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace taq
