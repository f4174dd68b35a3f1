// The fused TAQ cross-attention block kernel (PersonalQ, Section III-B) for gfx950: template, configuration
// constants and per-instantiation launchers. Included by one translation unit per (head dimension, heads) family
// (taq_fused_d40.hip, ...), so that the families compile in parallel; taq_fused.hip holds the dispatch.
//
//   hidden --per-token int8--> to_q (int8 MFMA) --Q_a per (token, head): Eq. 2, line 3-->
//   S^T = K~ Q~^T (int8 MFMA, fp16 MFMA for protected rows) --> softmax --> Eq. 3 -->
//   O^T = V~^T A^^T (fp16 MFMA, split operands) --per-token int8--> to_out (int8 MFMA) --> fp16
//
// Nothing between `hidden` and `out` touches HBM: per image token the kernel reads 2C bytes and
// writes 2C bytes; weights and K~/V~ come from L2.
//
// Work split. A workgroup owns 32 image tokens and all heads, one wavefront per head; each wavefront
// carries two column tiles of 16 tokens. Every contraction is computed transposed (output channel or
// text token along the MFMA row axis, image token along the column axis) with 16x16 tiles, so an image
// token stays in lane (token % 16) of its wavefront, in all four quarter-waves, from the first GEMM to
// the last: per-token reductions are register maxima plus two cross-lane swaps, and every intermediate
// (Q~ codes, probabilities, O codes) is handed to the next MFMA as its B operand straight from registers.
// The A operands' contraction order is free, so K~ and V~^T are stored in LDS in the order in which the
// accumulator registers of the previous MFMA come out.
//
// Bit-exact steps (same float32 operation order as the definition): per-token codes of hidden,
// the int32 accumulators, Qf = float(acc) * (s_h * s_wq), Q~ codes and scales.
#pragma once
#include "taq_device.h"

namespace taq {

// Buffer descriptor of a weight matrix: base address, no stride (raw byte offsets), `bytes` addressable, 32-bit data
// format; out-of-range reads return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t weight_rsrc(const int8_t* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(p), 0, (int)bytes, 0x00020000);
}

// A 16 x 64 block of row-major codes, fetched with four neighbouring lanes per row (lane = 4 * row + segment), in MFMA operand
// order (lane = row + 16 * segment): through the KiB at `slot`, which is this wavefront's alone. The segments of a row are
// swizzled, so that neither access has bank conflicts; LDS serves a wavefront in order, so that blocks can follow one another
// without a wait.
__device__ __forceinline__ int32x4_t exchange_rows(int32x4_t w, unsigned char* slot, int lane) {
    const int lr = lane >> 2, ls = lane & 3, r16 = lane & 15, q = lane >> 4;
    *reinterpret_cast<int32x4_t*>(slot + lr * 64 + ((ls ^ ((lr >> 1 ^ lr >> 2) & 3)) << 4)) = w;
    return *reinterpret_cast<const int32x4_t*>(slot + r16 * 64 + ((q ^ ((r16 >> 1 ^ r16 >> 2) & 3)) << 4));
}

// ------------------------------------------------------------------------------------------
// Fused block kernel
// ------------------------------------------------------------------------------------------
struct FusedTable {
    FusedReq req[TAQ_MAX_REQ];
};

struct FusedDims {
    int R, B, N, T;
    int nt16;          // ceil(T/16)
    int w_layout;      // 1: Wq / Wo carry an operand-ordered copy at w_pack_off
    unsigned w_pack_off;
    unsigned w_bytes;  // bytes of each weight buffer (row-major codes, plus the operand-ordered copy if present)
    float sig2;        // softmax scale * log2(e)
    float qmaxq;       // 127 or 7: grid of Q~ (Eq. 2, third line)
    float pmax;        // linear grid: 255 or 15 (Eq. 3); log2 grid: 256, which brings 2^-code * s_V to the linear grid's magnitudes
    float plast;       // log2 grid: the last code, 255 or 15
    KvLayout L;
    KvImage I;
    taq_debug dbg;     // taps (NULL pointers = off); only used when R == 1
};

template <int D, int NH, int NTT, int TOK = 32, bool DENSE = false>
struct FusedCfg {
    static constexpr int G = TOK / (16 * NTT);    // wavefronts per head (token groups of 16*NTT tokens)
    static constexpr int C = D * NH;
    static constexpr int TPH = (D + 15) / 16;     // 16-row tiles per head
    static constexpr int KS = (TPH + 3) / 4;      // K steps of 64 for S^T = K~ Q~^T
    static constexpr int FS = (TPH + 1) / 2;      // K steps of 32 for the protected-row scores
    static constexpr int KC = C / 64;             // K steps of 64 for the projections
    static constexpr int NT = 64 * NH * G;        // threads
    static constexpr int TILE_RS = C + 16;        // bytes per token row of the int8 tile
    // one head's image block at nt tiles of 16 text tokens, and the 1 KiB pieces of the largest (one direct-to-LDS load each)
    static constexpr int head_bytes(int nt) { return (int)kv_image(NH, D, 16 * nt).head_bytes; }
    static constexpr int IMGC = (head_bytes(TAQ_MAX_T / 16) + 1023) / 1024;
    // DENSE: the instantiation meant to run two workgroups per compute unit (layers with more token tiles than compute
    // units): at most 128 registers per lane, so the weights pass through a short ring instead of sitting in registers.
    static constexpr bool PREFETCH_W = TPH * KC <= 16 && NTT == 2 && !DENSE;  // a head's whole weight slice in registers
    // A barrier waits for the last wavefront to have its loads accepted (the texture unit takes one KiB per 16 clocks from all of them),
    // so not all of the slice is requested in front of one. to_q: PQ K steps between the steps of the hidden quantizer, the others behind
    // its barrier (5 of 5 in front 11.87 us at 2 x 4096 tokens, row-major weights 12.84; 4 11.73, 3 11.65 and 12.42, 2 11.69, 1 12.05).
    // to_out: one block of 16 channels in front of the softmax, one in front of each of the two barriers at the quantizer of A^ V~ (all
    // in front of the first 11.65 and 12.42; two, one between them 11.47 and 12.28; so 11.40 and 12.15).
    static constexpr int PQ = KC < 3 ? KC : 3;
    // Otherwise a ring of RING weight loads stays in flight ahead of the projection MFMAs (K step outermost, so that
    // only one step's B operands are live); left to itself the compiler keeps one to ten loads ahead and the loop
    // waits on latency.
    static constexpr int NF = TPH * KC;  // weight loads (16 rows x 64 bytes) of one projection per wavefront
    // As many as the registers take: two wavefronts per SIMD (256 registers each), three at ten heads (168), four DENSE (128);
    // fewer with three or four token tiles, whose accumulators take the rest. (DENSE 6 -> 12: 65.3 -> 63.4 us for 16 requests
    // of 4096 tokens; 24 and 8 -> 32 and 16 with two token tiles: 20.6 -> 19.9 us at eight heads of 80 and 8192 tokens,
    // 21.6 -> 20.9 us at ten of 64; one more step up spills, and at ten heads, whose wavefronts have 168 registers, three token
    // tiles do already: 14 registers in 60 bytes of scratch, 12 in 52 with row-major weights. 39 -> 29.8 us at 12288 tokens of ten
    // heads all the same, for one round instead of two. Row-major weights with four tiles at d = 80 spill 4 in 20 bytes.)
    static constexpr int RING_MAX = DENSE ? 12 : NH > 8 ? (NTT > 2 ? 8 : NTT == 2 ? 16 : 20) : NTT == 4 ? 20 : NTT == 3 ? 28 : 32;
    static constexpr int RING = !PREFETCH_W ? (NF < RING_MAX ? NF : RING_MAX) : 0;
};

// TOK = 32 image tokens per workgroup. NTT = 2: one wavefront per head carrying two column tiles of 16 tokens
// (A operands shared by both tiles). NTT = 1: two wavefronts per head, one tile each (16 wavefronts per CU
// instead of 8: more latency hiding for twice the A-operand traffic). TOK = 16 (with NTT = 1): one wavefront per
// head and half the tokens, for layers whose 32-token tiles would leave most compute units without a workgroup.
// NT16 > 0: the number of 16-token score tiles, ceil(T / 16), is this compile-time constant (5 for the 77 text tokens
// of every configured workload: no run-time guards around the tiles) and the taps on intermediate results are
// compiled out; NT16 = 0: any T up to 96, guards at run time, taps where the caller asks for them.
template <int D, int NH, int NTT, int PG, int TOK = 32, int NT16 = 0, bool DENSE = false, bool ROWMAJ = false>
__global__ __launch_bounds__(64 * NH * (TOK / (16 * NTT)))
__attribute__((amdgpu_waves_per_eu(DENSE ? 4 : 1, DENSE ? 4 : (NH * (TOK / (16 * NTT)) + 3) / 4)))
void fused_block_kernel(FusedTable tab, FusedDims dm) {
    using F = FusedCfg<D, NH, NTT, TOK, DENSE>;
    static_assert(!DENSE || NH * (TOK / (16 * NTT)) == 8, "two 8-wavefront workgroups per compute unit");
    static_assert(TOK == 16 * NTT || TOK == 32, "one wavefront per head, or two of one tile each");
    constexpr int C = F::C, H = NH, TPH = F::TPH, KS = F::KS, FS = F::FS, KC = F::KC, NT = F::NT;
    constexpr bool LEAN = DENSE || (NTT > 2 && NH <= 8);  // no register to spare
    constexpr bool LOGP = PG == TAQ_PROB_LOG2, ROWMAX = PG == TAQ_PROB_ROWMAX;  // grid of the probabilities, Eq. (3)
    constexpr int MT16 = NT16 ? NT16 : 6;  // score tiles the code is unrolled for
    // dwords of codes per test for ties. Whole groups but with row-major weights (4 % slower there at d = 80) and three or four token tiles
    // (registers): the 16 layers of a step of 2 x 64 x 64 249.9 -> 247.2 us, of 8 x 96 x 64 642 -> 640, 16 requests of 4096 x 320 59.1 -> 58.8,
    // 2 x 4096 x 640 20.5 -> 20.4.
    constexpr int QG = ROWMAJ || NTT > 2 ? 1 : TPH;
    // Scores past the protected tokens become minus infinity by selects behind the products instead of starting there, where the four
    // starting values are registers too many: 1 and 8 spilled without, none so. us: 2 x 8192 x 640, eight heads, 33.2 -> 33.0 (0 to 1 % in four
    // runs), ten heads with 50 text tokens, 20 of them protected, log2 grid, 18.45 -> 17.5. Three token tiles at ten heads (14 and 12 spilled or,
    // so, 12 and 11) and row-major weights with four (4 or 3) are no faster so: 29.6 and 31.1 us at 12288 tokens against 29.6 and 31.2, 34.3 at
    // 2 x 8192 against 34.5.
    constexpr bool SELECT = (NTT == 4 && !ROWMAJ) || (NH > 8 && NTT == 1 && NT16 == 0 && LOGP);
    constexpr bool TAPS = NT16 == 0;       // taps of intermediate codes and scales (tests, profiling)
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = wv % NH, lane = tid & 63, r16 = lane & 15, q = LEAN ? opaque(lane >> 4) : lane >> 4;
    // Grid: x = batch element, y = request, z = token tile. Workgroups are dispatched x fastest, so consecutive ones (which round-robin over
    // the 8 XCDs) share a token tile index and differ in the batch element / request: one XCD, few K~/V~ images. The
    // indices come straight from the grid: no integer divisions in front of the first loads.
    const int b = (int)blockIdx.x;
    const int ri = (int)blockIdx.y;
    const int tile = (int)blockIdx.z;
    const int tbase = ((wv / NH) % F::G) * 16 * NTT;  // first tile row of this wavefront's tokens
    const FusedReq rq = tab.req[ri];
    const int N = dm.N, T = dm.T;
    const int nt16 = NT16 ? NT16 : dm.nt16;
    // The image's layout as constants, where the number of score tiles is one: as arguments it cost scalar loads and address arithmetic in every phase.
    // us per layer, as arguments and as constants: 2 x 1024 x 640 (8 heads) 14.0 and 13.8, 2 x 4096 20.9 and 20.8, 8 x 1536 26.8 and 26.7; 2 x 4096 x 320
    // 11.4 and 11.4. With 10 heads of 64 they gain nothing (2 x 4096: 20.95 and 21.07), so there they stay arguments.
    constexpr KvImage CI = kv_image(NH, D, 16 * MT16);
    constexpr bool KNOWN = NT16 > 0 && D != 64;
    auto field = [&](auto m) { return KNOWN ? CI.*m : dm.I.*m; };
    const size_t head_bytes = field(&KvImage::head_bytes);
    const int n0 = tile * TOK;

    // ---- The hidden tile's loads are issued before anything else: they are the head of the kernel's one unavoidable
    // latency chain (HBM), and everything below (scalar loads of layout fields, of the protected-token count from
    // global memory, address arithmetic for the weights) would otherwise sit in front of them.
    // threads per token: 16 with 8-byte loads where there are as many, 8 with 16-byte loads otherwise
    constexpr int TPT = 16 * TOK <= NT ? 16 : 8;
    constexpr int XW = 16 / TPT;                   // 8-byte pieces per load
    const int tok0 = tid / TPT, part0 = tid % TPT;
    const int nq0 = n0 + tok0;
    const size_t row0 = (size_t)b * N + (nq0 < N ? nq0 : N - 1);
    const bool HOLDS = NT == TPT * TOK || tid < TPT * TOK;  // this thread holds a piece of the tile (all do, at 8 heads)
    uint2 xin[KC][XW];
    if (HOLDS) {
        const uint2* xr = reinterpret_cast<const uint2*>(rq.hidden + row0 * C) + part0 * XW;
#pragma unroll
        for (int it = 0; it < KC; ++it) {
            if constexpr (XW == 1) {
                xin[it][0] = xr[it * 16];
            } else {
                const uint4 w = *reinterpret_cast<const uint4*>(xr + it * 16);
                xin[it][0] = make_uint2(w.x, w.y);
                xin[it][XW - 1] = make_uint2(w.z, w.w);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    // This head's block of the K~/V~ image: straight into LDS, 1 KiB per wavefront-wide load (LDS address =
    // base + lane * 16), no registers in between; only this wavefront reads it, so only this wavefront waits for it. The last
    // piece may be fetched more than once.
    auto copy_image = [&]() {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint8_t*>(rq.packed) + dm.L.image + (size_t)b * dm.L.image_bytes + (size_t)h * head_bytes, 0, (int)head_bytes, 0x00020000);
        // the block is a multiple of 256 bytes: the last piece overlaps (a constant where the number of score tiles is fixed)
        constexpr int fixed = NT16 ? F::head_bytes(NT16) : 0;
        const int last = (NT16 ? fixed : (int)head_bytes) - 1024;
#pragma unroll
        for (int k = 0; k < F::IMGC; ++k) {
            if (k == 0 || k * 1024 < last + 1024) {  // (pieces past the block's end at this T are not fetched)
                const int c = k * 1024 < last ? k * 1024 : last;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(smem + (size_t)h * head_bytes + c), 16, lane * 16, c, 0, 0);
            }
        }
    };
    // (row-major weights are exchanged in its place in LDS, and have to be through with it, unless there is a KiB per wavefront besides)
    constexpr bool SLOTS = ROWMAJ && NTT <= 2 && NT16 == 5, EARLY = !ROWMAJ || SLOTS;
    if constexpr (EARLY) {
        copy_image();
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- LDS carve-up
    unsigned char* img = smem;                                  // K~/V~ image blocks of this workgroup's heads
    const size_t img_bytes = (size_t)NH * head_bytes;
    int8_t* tileq = reinterpret_cast<int8_t*>(smem + img_bytes);                 // [TOK][C+16] hidden codes, later O codes
    float* wsc = reinterpret_cast<float*>(smem + img_bytes + TOK * F::TILE_RS);  // s_wq | s_wo | bias_o  [3C]
    float* s_h = wsc + 3 * C;                                    // [TOK]
    unsigned* omax = reinterpret_cast<unsigned*>(s_h + TOK);     // [TOK][NH]
    unsigned char* xslot = SLOTS ? reinterpret_cast<unsigned char*>(omax + TOK * NH) + wv * 1024 : nullptr;  // exchange of row-major weights

    const uint8_t* packed = rq.packed;
    const int ntrig = reinterpret_cast<const int*>(packed + dm.L.ntrig)[b];
    const int nfp = (ntrig + 15) >> 4;  // tiles of 16 protected tokens

    // weight rows of this head: row c = h*D + 16*j + r16 (rows past the head are discarded; clamp keeps reads in bounds)
    // (byte offset of K step ks = wrow[j] + ks * wstep; with the operand-ordered copy a wavefront-wide load is
    // one contiguous KiB, otherwise 16 rows x 64 bytes)
    int wrow[TPH];
    const int wstep = dm.w_layout ? 1024 : 64;
    auto set_wrow = [&](int ln) {
#pragma unroll
        for (int j = 0; j < TPH; ++j) {
            const int row = ln & 15, c = h * D + 16 * j + row;
            wrow[j] = dm.w_layout ? (int)dm.w_pack_off + ((h * TPH + j) * KC) * 1024 + ln * 16 : (c < C ? c : C - 1) * C + 16 * (ln >> 4);
            // Weight rows past the head (the upper lanes of a partly filled last tile) are not fetched: their products are
            // dropped anyway, and at d = 40 they are a sixth of the bytes every CU pulls through its L2. Their lanes carry
            // an offset past the end of the buffer, for which a buffer load returns zero without a memory access.
            if (!((D % 16 == 0) || 16 * j + 16 <= D || row < D - 16 * j)) wrow[j] = 0x7fffffff;
        }
    };
    set_wrow(lane);
    // Buffer loads: the descriptor (base, size) and the step sit in scalar registers and the lane's part is a 32-bit
    // offset, so a load costs no vector address arithmetic (a 64-bit vector add per load otherwise) and the lanes
    // without a row need neither a branch nor registers cleared by hand.
    const __amdgpu_buffer_rsrc_t rs_wq = weight_rsrc(rq.wq, dm.w_bytes), rs_wo = weight_rsrc(rq.wo, dm.w_bytes);
    auto load_w = [&](const __amdgpu_buffer_rsrc_t rs, int j, int off) -> int32x4_t {
        return (int32x4_t)__builtin_amdgcn_raw_buffer_load_b128(rs, wrow[j], off, 0);
    };
    int32x4_t wreg[F::PREFETCH_W ? TPH : 1][F::PREFETCH_W ? KC : 1];
    constexpr int RING = F::RING, NF = F::NF;
    // ROWMAJ: row-major weights through the ring. Fetched as the MFMA wants them (lane = row + 16 * quarter), such a load
    // touches 64 separate 16-byte pieces, which the texture path serves one per clock: 29.4 us at C = 640 and 2048 tokens.
    // Here four neighbouring lanes take the 64 contiguous bytes of a row, the two halves of a 128-byte line one after the
    // other (23.5 -> 19.5 us at 4096 tokens), and the lanes are exchanged through LDS: 18.3 us (operand-ordered weights: 15.0;
    // an exchange by DPP selects in registers: 21.2). The KiB for it lies behind everything else (SLOTS); where it does not fit, it is
    // the start of the head's K~/V~ block: the image is requested when to_q is done with it, and to_out begins when the attention is
    // through with the image.
    static_assert(!ROWMAJ || (D % 16 == 0 && KC % 2 == 0), "whole tiles, whole 128-byte lines");
    const int rm_off = (h * D + (lane >> 2)) * C + 16 * (lane & 3);
    auto ring_load = [&](const __amdgpu_buffer_rsrc_t rs, int f) -> int32x4_t {  // the f-th load of a projection
        if constexpr (ROWMAJ) return (int32x4_t)__builtin_amdgcn_raw_buffer_load_b128(rs, rm_off, 16 * ((f / 2) % TPH) * C + 64 * (f / (2 * TPH) * 2 + f % 2), 0);
        return load_w(rs, f % TPH, wstep * (f / TPH));
    };
    constexpr int RPS = RING ? (RING + KC - 1) / KC : 0;  // ring loads issued per step of the hidden quantizer
    int32x4_t wring[RING ? RING : 1];
    const float* swq = wsc;
    const float* swo = wsc + C;
    const float* bo = wsc + 2 * C;
    unsigned char* imgh = img + (size_t)h * head_bytes;  // this head's block of the K~/V~ image
    const float* img_sk = reinterpret_cast<const float*>(imgh + field(&KvImage::s_k));
    const float* img_bias = reinterpret_cast<const float*>(imgh + field(&KvImage::bias));
    const __half* k16 = reinterpret_cast<const __half*>(packed + dm.L.k16) + (size_t)b * T * C;
    const __half* v16t = reinterpret_cast<const __half*>(packed + dm.L.v16t) + (size_t)b * C * 96;

    // protected (trigger) rows of this head, first tile of 16: fp16 K rows and transposed V rows straight from
    // global memory into MFMA operand registers. Slots past the protected tokens and channels past the head (which would belong to the next
    // head, or lie past the last row of the last head, and a non-finite bit pattern there would survive the multiplication with a zero Q~
    // code) carry an offset past the end: zeros without a memory access. (A load costs by the pieces of memory that it touches, 16 rows of 32
    // bytes if all lanes take part: 15.1 -> 14.7 us at 2048 tokens of 640 channels. Flat loads needed a branch, zeroed registers and 64-bit
    // addresses for each of these.)
    uint2 k16r[FS][2], v16r[TPH];
    auto load_protected = [&]() {
        if (nfp > 0) {
            const __amdgpu_buffer_rsrc_t rs_k = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half*>(k16), 0, T * C * 2, 0x00020000);
            const __amdgpu_buffer_rsrc_t rs_v = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half*>(v16t), 0, C * 96 * 2, 0x00020000);
            constexpr int NONE = 0x7fff0000;
            const int ko = r16 < ntrig ? (r16 * C + h * D + 4 * q) * 2 : NONE, ko_last = D % 16 == 0 || 16 * (TPH - 1) + 4 * q < D ? ko : NONE;
            const int vo = 4 * q < ntrig ? ((h * D + r16) * 96 + 4 * q) * 2 : NONE;
            // (rows past the head repeat its last, as those of V~ do)
            const int vo_last = D % 16 == 0 || r16 < D % 16 ? vo : 4 * q < ntrig ? ((h * D + D % 16 - 1) * 96 + 4 * q) * 2 : NONE;
#pragma unroll
            for (int j = 0; j < 2 * FS; ++j) {
                const uint2_t w = j < TPH ? __builtin_amdgcn_raw_buffer_load_b64(rs_k, (j == TPH - 1 ? ko_last : ko) + 32 * j, 0, 0) : (uint2_t){0u, 0u};
                k16r[j / 2][j % 2] = make_uint2(w[0], w[1]);
            }
#pragma unroll
            for (int k = 0; k < TPH; ++k) {
                const uint2_t w = __builtin_amdgcn_raw_buffer_load_b64(rs_v, k == TPH - 1 ? vo_last : vo, 16 * k * 192, 0);
                v16r[k] = make_uint2(w[0], w[1]);
            }
        }
    };

    // ---- phase 0: the global reads, requested up front (loads return in order): the hidden tile, the K~/V~ image where it is
    // requested early (both above), the weight scales, then between the steps of the quantizer this head's to_q weights
    constexpr int SCV = (3 * C / 4 + NT - 1) / NT;
    float4 scv[SCV];
#pragma unroll
    for (int k = 0; k < SCV; ++k) {
        const int i = tid + k * NT;
        scv[k] = i < 3 * C / 4 ? reinterpret_cast<const float4*>(rq.scales)[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // ---- per-token int8 codes of the hidden tile. The row maximum is taken on the fp16 values themselves, two per
    // instruction (a maximum is exact in any precision); the quantizer's FMAs read the fp16 operands directly.
    float amax = 0.f;
    if (HOLDS) {
        half2_t am2 = {(_Float16)0.f, (_Float16)0.f};
#pragma unroll
        for (int it = 0; it < KC; ++it)
#pragma unroll
            for (int u = 0; u < XW; ++u) {
                const unsigned a0 = xin[it][u].x & 0x7fff7fffu, a1 = xin[it][u].y & 0x7fff7fffu;
                am2 = __builtin_elementwise_max(am2, __builtin_elementwise_max(*reinterpret_cast<const half2_t*>(&a0),
                                                                                 *reinterpret_cast<const half2_t*>(&a1)));
            }
        amax = fmaxf((float)am2[0], (float)am2[1]);
    }
    // The hidden tile has arrived (the unpacking above waited for it). Only now are the 10x larger weight reads
    // issued: the texture path serves requests in arrival order, and the first barrier waits for nothing else.
    __builtin_amdgcn_sched_barrier(0);
    // The weight slice is fetched a few loads at a time between pieces of arithmetic: a wavefront stalls at a
    // vector-memory instruction while the texture unit's queue is full (it coalesces 64 B per clock, and every
    // CU pulls ~300 KB of weights and image per launch), so the requests are spread under the ALU work.
    amax = TPT == 16 ? row16_allmax(amax) : row8_allmax(amax);
    const bool zero0 = amax == 0.f;
    const float sc0 = zero0 ? 1.f : div_grid(amax, 127.f);
    const float safe0 = zero0 ? 1.f : amax;
    const float cq0 = quant_mult(127.f, safe0);
    if (HOLDS && part0 == 0) s_h[tok0] = sc0;
    const QuantRow hrow = {1.f, cq0, safe0};
    const HalfRow half = half_row(cq0, sc0, amax);
    const bool again = TAQ_DOUBT(half.doubt);
    auto hidden4 = [&](int it, int u) {
        const half2_t x01 = *reinterpret_cast<const half2_t*>(&xin[it][u].x), x23 = *reinterpret_cast<const half2_t*>(&xin[it][u].y);
        return make_float4((float)x01[0], (float)x01[1], (float)x23[0], (float)x23[1]);
    };
    auto put_hidden = [&](int it, const unsigned (&pk)[XW]) {
        int8_t* dst = tileq + tok0 * F::TILE_RS + it * 64 + part0 * (4 * XW);
        if constexpr (XW == 1) *reinterpret_cast<unsigned*>(dst) = pk[0];
        else *reinterpret_cast<uint2*>(dst) = make_uint2(pk[0], pk[XW - 1]);
        if (TAPS && dm.dbg.h_code && nq0 < N)
#pragma unroll
            for (int u = 0; u < XW; ++u) *reinterpret_cast<unsigned*>(dm.dbg.h_code + row0 * C + it * 64 + part0 * (4 * XW) + 4 * u) = pk[u];
    };
#pragma unroll
    for (int it = 0; it < KC; ++it) {
        if (F::PREFETCH_W && it < F::PQ) {
#pragma unroll
            for (int j = 0; j < TPH; ++j) wreg[j][it] = load_w(rs_wq, j, wstep * it);
        }
        if constexpr (RING > 0) {  // the first RING loads of to_q, in the order the MFMAs use them
#pragma unroll
            for (int f = it * RPS; f < (it + 1) * RPS && f < RING; ++f) wring[f] = ring_load(rs_wq, f);
        }
        if (HOLDS) {
            unsigned pk[XW];
#pragma unroll
            for (int u = 0; u < XW; ++u) {
                const float4 x = hidden4(it, u);
                pk[u] = quant4_at(x.x, x.y, x.z, x.w, half.m);
            }
            if (RING > 0 && again)  // (step by step, as with QG below)
#pragma unroll
                for (int u = 0; u < XW; ++u) {
                    const float4 x = hidden4(it, u);
                    pk[u] = half_row_settle(pk[u], x.x, x.y, x.z, x.w, hrow);
                }
            put_hidden(it, pk);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if (RING == 0 && again) {  // all of this thread's pieces again
#pragma unroll
        for (int it = 0; it < KC; ++it) {
            unsigned pk[XW];
#pragma unroll
            for (int u = 0; u < XW; ++u) {
                const float4 x = hidden4(it, u);
                pk[u] = half_row_settle(quant4_at(x.x, x.y, x.z, x.w, half.m), x.x, x.y, x.z, x.w, hrow);
            }
            put_hidden(it, pk);
        }
    }
    if (TAPS && HOLDS && dm.dbg.s_h && part0 == 0 && nq0 < N) dm.dbg.s_h[row0] = sc0;
    // ---- weight scales into LDS
#pragma unroll
    for (int k = 0; k < SCV; ++k) {
        const int i = tid + k * NT;
        if (i < 3 * C / 4) reinterpret_cast<float4*>(wsc)[i] = scv[k];
    }
    __syncthreads();

    // this lane's two image tokens: tile rows r16 and 16 + r16
    bool nvalid[NTT];
    size_t tok[NTT];
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        const int n = n0 + tbase + 16 * nt + r16;
        nvalid[nt] = n < N;
        tok[nt] = (size_t)b * N + (n < N ? n : N - 1);
    }

    // A projection whose first RING weight loads are on their way: acc^T[c][n] over the codes in `tileq`; every slot of the
    // ring is refilled as soon as its MFMAs are issued.
    auto ring_project = [&](const __amdgpu_buffer_rsrc_t rs, int32x4_t (&acc)[NTT][TPH], int ln) {
#pragma unroll
        for (int j = 0; j < TPH; ++j)
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) acc[nt][j] = (int32x4_t){0, 0, 0, 0};
        constexpr int RD = RING ? RING : 1;
        const int8_t* xrow = tileq + (tbase + (ln & 15)) * F::TILE_RS + 16 * (ln >> 4);
        constexpr int AHEAD = ROWMAJ ? 4 : 0;  // operands on their way through LDS
        int32x4_t op[AHEAD + 1];
        auto operand = [&](int f) {
            if constexpr (ROWMAJ) op[f % (AHEAD + 1)] = exchange_rows(wring[f % RD], SLOTS ? xslot : imgh, lane);
            else op[0] = wring[f % RD];
        };
#pragma unroll
        for (int f = 0; f < AHEAD; ++f) operand(f);
        constexpr int KG = ROWMAJ ? 2 : 1;  // (the two halves of a 128-byte line of a row one after the other)
#pragma unroll
        for (int ks = 0; ks < KC; ks += KG) {
            int32x4_t hbk[NTT][KG];
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
                for (int k = 0; k < KG; ++k) hbk[nt][k] = *reinterpret_cast<const int32x4_t*>(xrow + 16 * nt * F::TILE_RS + 64 * (ks + k));
#pragma unroll
            for (int jk = 0; jk < TPH * KG; ++jk) {
                const int j = jk / KG, k = jk % KG, f = ks * TPH + jk, g = f + AHEAD;
                if (g < NF) operand(g);
#pragma unroll
                for (int nt = 0; nt < NTT; ++nt) acc[nt][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(op[f % (AHEAD + 1)], hbk[nt][k], acc[nt][j], 0, 0, 0);
                // the slot is free again: the load RING places ahead takes it
                if (ROWMAJ && f == 0) {
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u)
                        if (u + RING < NF) wring[u % RD] = ring_load(rs, u + RING);
                }
                if (g + RING < NF) wring[g % RD] = ring_load(rs, g + RING);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // ================= to_q for this head: Qf^T[c][n]
    int32x4_t hb[NTT][RING == 0 ? KC : 1];
    if constexpr (RING == 0) {
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
            for (int ks = 0; ks < KC; ++ks)
                hb[nt][ks] = *reinterpret_cast<const int32x4_t*>(tileq + (tbase + 16 * nt + r16) * F::TILE_RS + 64 * ks + 16 * q);
    }
    int32x4_t pacc[NTT][TPH];
    if constexpr (F::PREFETCH_W) {
        // K step outermost: the order in which the weight loads were issued, so that the MFMAs follow the weights as they
        // arrive and only one step's worth is left to do after the last load
#pragma unroll
        for (int ks = F::PQ; ks < KC; ++ks)
#pragma unroll
            for (int j = 0; j < TPH; ++j) wreg[j][ks] = load_w(rs_wq, j, wstep * ks);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TPH; ++j)
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) pacc[nt][j] = (int32x4_t){0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KC; ++ks)
#pragma unroll
            for (int j = 0; j < TPH; ++j)
#pragma unroll
                for (int nt = 0; nt < NTT; ++nt)
                    pacc[nt][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wreg[j][ks], hb[nt][ks], pacc[nt][j], 0, 0, 0);
    } else {
        ring_project(rs_wq, pacc, lane);
    }
    // Everything the Q~ step reads from LDS is fetched now: where the image is requested below, no LDS access sits between that and
    // the wait for it (the compiler orders LDS accesses after outstanding direct-to-LDS loads).
    float4 wq4[TPH];
    float shv[NTT];
#pragma unroll
    for (int j = 0; j < TPH; ++j) {
        const int cl = 16 * j + 4 * q;
        wq4[j] = *reinterpret_cast<const float4*>(swq + h * D + (((16 * j + 16 <= D) || cl < D) ? cl : 0));
    }
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) shv[nt] = s_h[tbase + 16 * nt + r16];
    // The image has arrived: it was requested in front of the weights that to_q has consumed (row-major weights, which go through
    // its place in LDS: it is requested now).
    if constexpr (EARLY) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (!EARLY) copy_image();
    load_protected();

    // ---- Eq. (2), third line: Q~ = Q_a(Q) per (token, head)
    unsigned qpk[NTT][TPH];
    float sq2[NTT];
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        const float sh = shv[nt];
        float qf[TPH][4];
        float qmax = 0.f;
#pragma unroll
        for (int j = 0; j < TPH; ++j) {
            const float wv[4] = {wq4[j].x, wq4[j].y, wq4[j].z, wq4[j].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float sc = sh * wv[i];
                qf[j][i] = (float)pacc[nt][j][i] * sc;  // (zero past the head: so are the weights there)
                qmax = fmaxf(qmax, fabsf(qf[j][i]));
            }
        }
        qmax = quad_allmax(qmax);
        const bool qzero = qmax == 0.f;
        const float sQ = qzero ? 1.f : div_grid(qmax, dm.qmaxq);
        const float qsafe = qzero ? 1.f : qmax;
        const float cq = quant_mult(dm.qmaxq, qsafe);
        quant4_group<QG>(qpk[nt], [&](int j) { return make_float4(qf[j][0], qf[j][1], qf[j][2], qf[j][3]); },
                     [&](int) { return QuantRow{1.f, cq, qsafe}; }, dm.qmaxq);
        if (TAPS && dm.dbg.q_code && nvalid[nt]) {
#pragma unroll
            for (int j = 0; j < TPH; ++j)
                if (16 * j + 4 * q < D) *reinterpret_cast<unsigned*>(dm.dbg.q_code + tok[nt] * C + h * D + 16 * j + 4 * q) = qpk[nt][j];
            if (dm.dbg.s_Q && q == 0) dm.dbg.s_Q[tok[nt] * H + h] = sQ;
        }
        sq2[nt] = fmaxf(sQ * dm.sig2, 1e-37f);
    }

    if constexpr (!EARLY) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the head's image block travelled meanwhile
    // One token tile per wavefront: the first RING loads of to_out, a quarter at a time between the phases of the attention (all at
    // once they fill the queue, and the wavefront stands until it has drained)
    auto ring_out = [&](int part) {
        if constexpr (RING > 0 && NTT == 1) {
#pragma unroll
            for (int f = part * RING / 4; f < (part + 1) * RING / 4; ++f) wring[f] = ring_load(rs_wo, f);
        }
    };
    ring_out(0);

    // ================= scores: x[t][n] = (K~ Q~^T)[t][n] * s_K[t]   (times sQ * sigma * log2 e later)
    float S[NTT][MT16][4];
    {
        int32x4_t qop[NTT][KS];  // B operand: dword jj of step ks = codes of tile 4*ks + jj
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) qop[nt][ks][jj] = (4 * ks + jj < TPH) ? (int)qpk[nt][4 * ks + jj] : 0;
        const int8_t* kp = reinterpret_cast<const int8_t*>(imgh + field(&KvImage::kp));
#pragma unroll
        for (int tt = 0; tt < MT16; ++tt) {
            if (tt < nt16) {
                int32x4_t acc[NTT];
#pragma unroll
                for (int nt = 0; nt < NTT; ++nt) acc[nt] = sum_start();
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    int32x4_t ka;
                    if constexpr (TPH % 4 == 0) {  // the lane's 16 bytes of this K step are contiguous
                        ka = *reinterpret_cast<const int32x4_t*>(kp + kp_offset(TPH, 16 * tt + r16, 4 * ks, q));
                    } else {
#pragma unroll
                        for (int jj = 0; jj < 4; ++jj)
                            ka[jj] = (4 * ks + jj < TPH) ? *reinterpret_cast<const int*>(kp + kp_offset(TPH, 16 * tt + r16, 4 * ks + jj, q)) : 0;
                    }
#pragma unroll
                    for (int nt = 0; nt < NTT; ++nt) acc[nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ka, qop[nt][ks], acc[nt], 0, 0, 0);
                }
                const float4 sk = *reinterpret_cast<const float4*>(img_sk + 16 * tt + 4 * q);
                const float4 bi = *reinterpret_cast<const float4*>(img_bias + 16 * tt + 4 * q);
#pragma unroll
                for (int nt = 0; nt < NTT; ++nt) {
                    S[nt][tt][0] = __builtin_fmaf(sum_float(acc[nt][0]), sk.x, bi.x);
                    S[nt][tt][1] = __builtin_fmaf(sum_float(acc[nt][1]), sk.y, bi.y);
                    S[nt][tt][2] = __builtin_fmaf(sum_float(acc[nt][2]), sk.z, bi.z);
                    S[nt][tt][3] = __builtin_fmaf(sum_float(acc[nt][3]), sk.w, bi.w);
                }
            }
        }
    }
    // protected rows: fp16 K rows, the first 16 from registers, further ones (rare) straight from global memory. Scores of
    // protected tile ft (tokens of slots 16*ft .. 16*ft+15) for this lane's image tokens; -inf past ntrig. Only the first
    // tile's scores are held in registers; those of further ones are formed once for the row maximum and once more for the
    // exponentials.
    auto protected_scores = [&](auto first, int ft, const unsigned (&code)[NTT][TPH], floatx4_t (&facc)[NTT]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float none = SELECT || 16 * ft + 4 * q + i < ntrig ? 0.f : TAQ_NEG_INF;
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) facc[nt][i] = none;
        }
        int slot = 16 * ft + r16;
        slot = slot < ntrig ? slot : ntrig - 1;
        const __half* kr = k16 + (size_t)slot * C + h * D + 4 * q;
#pragma unroll
        for (int s = 0; s < FS; ++s) {
            half8_t ka;
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int j = 2 * s + jj;
                uint2 w = k16r[s][jj];
                if constexpr (!decltype(first)::value) w = (j < TPH && 16 * j + 4 * q < D) ? *reinterpret_cast<const uint2*>(kr + 16 * j) : make_uint2(0, 0);
                const half4_t hv = *reinterpret_cast<const half4_t*>(&w);
                ka[4 * jj + 0] = hv[0];
                ka[4 * jj + 1] = hv[1];
                ka[4 * jj + 2] = hv[2];
                ka[4 * jj + 3] = hv[3];
            }
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) {
                half2_t c0, c1, c2 = {(_Float16)0.f, (_Float16)0.f}, c3 = c2;  // Q~ codes of tiles 2s and 2s + 1 as fp16
                biased4_to_half(code[nt][2 * s] ^ 0x80808080u, c0, c1);
                if (2 * s + 1 < TPH) biased4_to_half(code[nt][2 * s + 1 < TPH ? 2 * s + 1 : 0] ^ 0x80808080u, c2, c3);
                const half8_t qh = {c0[0], c0[1], c1[0], c1[1], c2[0], c2[1], c3[0], c3[1]};
                facc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qh, facc[nt], 0, 0, 0);
            }
        }
        if constexpr (SELECT) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool live = 16 * ft + 4 * q + i < ntrig;
#pragma unroll
                for (int nt = 0; nt < NTT; ++nt) facc[nt][i] = live ? facc[nt][i] : TAQ_NEG_INF;
            }
        }
    };
    auto further_scores = [&](int ft, floatx4_t (&facc)[NTT]) {  // (codes as fp16 are not kept for them)
        unsigned code[NTT][TPH];
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
            for (int j = 0; j < TPH; ++j) code[nt][j] = (unsigned)opaque((int)qpk[nt][j]);
        protected_scores(std::false_type{}, ft, code, facc);
    };

    ring_out(1);
    // The LDS operands of O^T = V~^T A^^T (this wavefront's V~ codes and the split V scales) are read now, into
    // registers: issued next to their use, each read's round trip would stand between the softmax and its MFMAs.
    // (Only where registers are plentiful: the instantiation that also holds its weight slices in registers.)
    constexpr bool PRE_V = F::PREFETCH_W;
    auto slice_out = [&](int j0, int j1) {  // to_out's weights of the head's channel blocks j0 .. j1-1
#pragma unroll
        for (int j = 0; j < TPH; ++j)
#pragma unroll
            for (int ks = 0; ks < KC; ++ks)
                if (j >= j0 && j < j1) wreg[j][ks] = load_w(rs_wo, j, wstep * ks);
    };
    if constexpr (F::PREFETCH_W) slice_out(0, 1);
    uint2 vw2[PRE_V ? 3 : 1][PRE_V ? TPH : 1];  // V~^T codes of 32-token step s (s = 0, 1, 2; a single last tile uses .x only)
    uint2 svh[PRE_V ? MT16 : 1], svl[PRE_V ? MT16 : 1];  // fp16 high parts and remainders of s_V * 2^kexp, four text tokens of each tile
    const uint8_t* vt = imgh + field(&KvImage::vt);
    const _Float16* img_sv = reinterpret_cast<const _Float16*>(imgh + field(&KvImage::s_vp));  // [ntok] high parts | [ntok] low parts
    if constexpr (PRE_V) {
#pragma unroll
        for (int tt = 0; tt < MT16; ++tt) {
            svh[tt] = svl[tt] = make_uint2(0u, 0u);
            if (tt < nt16) {
                svh[tt] = *reinterpret_cast<const uint2*>(img_sv + 16 * tt + 4 * q);
                svl[tt] = *reinterpret_cast<const uint2*>(img_sv + field(&KvImage::ntok) + 16 * tt + 4 * q);
            }
        }
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int k = 0; k < TPH; ++k) {
                vw2[s][k] = make_uint2(0u, 0u);
                if (2 * s >= nt16) continue;
                int j = 16 * k + r16;
                j = j < D ? j : D - 1;
                if (2 * s + 1 < nt16) vw2[s][k] = *reinterpret_cast<const uint2*>(vt + (size_t)j * field(&KvImage::cols_v) + 32 * s + 8 * q);
                else vw2[s][k].x = *reinterpret_cast<const unsigned*>(vt + (size_t)j * field(&KvImage::cols_v) + 32 * s + 4 * q);
            }
    }
    __builtin_amdgcn_sched_barrier(0);

    // ================= softmax over the text tokens; Eq. (3); weights of O^T = V~^T A^^T
    float kq[NTT];   // code = rint(E * kq): pmax / Z per image token (row-range grid: pmax / largest unprotected E)
    float lz[NTT];   // log2 Z (log2 grid only)
    float fz[NTT];   // row-range grid only: range / Z
    float mxs[NTT];  // row maximum of the raw scores
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        float mx = TAQ_NEG_INF;
#pragma unroll
        for (int tt = 0; tt < MT16; ++tt)
            if (tt < nt16) mx = fmaxf(mx, fmaxf(fmaxf(S[nt][tt][0], S[nt][tt][1]), fmaxf(S[nt][tt][2], S[nt][tt][3])));
        mxs[nt] = mx;
    }
    floatx4_t fsc[NTT];  // scores of the first protected tile
    if (nfp > 0) {
        protected_scores(std::true_type{}, 0, qpk, fsc);
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt) mxs[nt] = fmaxf(mxs[nt], fmaxf(fmaxf(fsc[nt][0], fsc[nt][1]), fmaxf(fsc[nt][2], fsc[nt][3])));
        for (int ft = 1; ft < nfp; ++ft) {
            floatx4_t facc[NTT];
            further_scores(ft, facc);
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt)
                mxs[nt] = fmaxf(mxs[nt], fmaxf(fmaxf(facc[nt][0], facc[nt][1]), fmaxf(facc[nt][2], facc[nt][3])));
        }
    }
    ring_out(2);
    float Zs[NTT], eus[NTT], offs[NTT];
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        const float mx = quad_allmax(mxs[nt]);
        const float sc = sq2[nt], off = -mx * sc;
        offs[nt] = off;
        float Z = 0.f, eu = 0.f;
#pragma unroll
        for (int tt = 0; tt < MT16; ++tt)
            if (tt < nt16) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float arg = __builtin_fmaf(S[nt][tt][i], sc, off);
                    const float ex = __builtin_amdgcn_exp2f(arg);
                    Z += ex;
                    if (ROWMAX) eu = fmaxf(eu, ex);  // the row's range: its largest unprotected probability (times Z)
                    S[nt][tt][i] = LOGP ? arg : ex;  // the log2 grid rounds the exponent itself
                }
            }
        Zs[nt] = Z;
        eus[nt] = eu;
    }

    // oacc[nt][k]: channel tile k of this head
    floatx4_t oacc[NTT][TPH];
    // protected columns keep A (Eq. 3): E = exp2(score - max), not yet divided by Z, as fp16 high + low parts against the
    // fp16 V rows; the accumulators are brought to the unit of the unprotected columns' weights (pmax * A * 2^kexp) once Z
    // is known.
    auto protected_values = [&](auto first, int ft, const floatx4_t (&facc)[NTT]) {
        half4_t phi[NTT], plo[NTT];
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(facc[nt][i], sq2[nt], offs[nt]));
                const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(facc[nt][i + 1], sq2[nt], offs[nt]));
                Zs[nt] += e0;
                Zs[nt] += e1;
                split_half2(e0, e1, phi[nt], plo[nt], i);
            }
#pragma unroll
        for (int k = 0; k < TPH; ++k) {
            const int j = 16 * k + r16, c = h * D + (j < D ? j : D - 1);
            uint2 w = v16r[k];
            if constexpr (!decltype(first)::value) w = *reinterpret_cast<const uint2*>(v16t + (size_t)c * 96 + 16 * ft + 4 * q);
            const half4_t va = *reinterpret_cast<const half4_t*>(&w);  // slots past ntrig hold zeros
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) {
                oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, phi[nt], decltype(first)::value ? (floatx4_t){0.f, 0.f, 0.f, 0.f} : oacc[nt][k], 0, 0, 0);
                oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, plo[nt], oacc[nt][k], 0, 0, 0);
            }
        }
    };
    if (nfp > 0) {
        protected_values(std::true_type{}, 0, fsc);
        for (int ft = 1; ft < nfp; ++ft) {
            floatx4_t facc[NTT];
            further_scores(ft, facc);
            protected_values(std::false_type{}, ft, facc);
        }
    } else {
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
            for (int k = 0; k < TPH; ++k) oacc[nt][k] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
    }
    ring_out(3);
    const float vpre = nfp > 0 ? reinterpret_cast<const float*>(imgh + field(&KvImage::vpre))[0] : 0.f;
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        const float Z = quad_allsum(Zs[nt]);
        const float kqp = quant_mult(dm.pmax, Z);  // pmax / Z, as the stage path forms it: the same codes from either
        float f = kqp * vpre;                      // protected columns: weight = E * kqp = pmax * A
        kq[nt] = kqp;
        lz[nt] = LOGP ? __builtin_amdgcn_logf(Z) : 0.f;  // log2 Z >= 0: the largest term of Z is 1
        fz[nt] = 1.f;
        if constexpr (ROWMAX) {
            // codes = rint(pmax * E / range), A^ = code * (range / Z) / pmax. Unprotected columns that together weigh
            // less than 2^-40 of the row (or none at all) are dropped: their codes would scale a vanishing range.
            const float eu = quad_allmax(eus[nt]);
            if (eu > Z * 9.094947e-13f) {
                kq[nt] = quant_mult(dm.pmax, eu);
                f = kqp * (vpre * quant_mult(Z, eu));
                fz[nt] = quant_mult(eu, Z);
            }
        }
        if (nfp > 0) {
#pragma unroll
            for (int k = 0; k < TPH; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) oacc[nt][k][i] *= f;
        }
    }
    // unprotected columns: weight = code * s', s' = s_V * 2^kexp, as fp16 high + low parts (V codes are exact in fp16).
    // s' comes from the image already split, s' = sh + sl (two fp16 numbers, |sl| <= 2^-11 |sh|). The code c (an integer
    // below 256) is exact in fp16; in packed fp16 arithmetic, two columns per instruction:
    //   wh = fl(c * sh),  r = fma(c, sh, -wh)  (the rounding error of wh: exact, it needs at most 8 bits),
    //   wl = fma(c, sl, r)                      => wh + wl = c * s' to about 2^-22, relatively.
    // The code itself is formed with one FMA: P * kq + (1.5 * 2^23 + 0x6400) rounds P * kq half-to-even to an integer
    // and leaves 0x6400 + code in the low half of the result: the bit pattern of the fp16 number 1024 + code.
    {
        const half2_t k1024 = {(_Float16)1024.0f, (_Float16)1024.0f};
        // tap: the codes of text tokens t, t + 1 for this lane's image token of tile nt 
        auto tap_pcode = [&](int nt, int t, unsigned c0, unsigned c1) {
            if (nvalid[nt]) {
                uint8_t* row = dm.dbg.p_code + (tok[nt] * H + h) * (size_t)T;
                if (t < T) row[t] = (uint8_t)c0;
                if (t + 1 < T) row[t + 1] = (uint8_t)c1;
            }
        };
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            if (2 * s < nt16) {
                const bool second = 2 * s + 1 < nt16;
                half8_t phi[NTT], plo[NTT];
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    if (a == 0 || second) {
                        uint2 h4, l4;
                        if constexpr (PRE_V) {
                            h4 = svh[2 * s + a < MT16 ? 2 * s + a : 0];
                            l4 = svl[2 * s + a < MT16 ? 2 * s + a : 0];
                        } else {
                            h4 = *reinterpret_cast<const uint2*>(img_sv + 16 * (2 * s + a) + 4 * q);
                            l4 = *reinterpret_cast<const uint2*>(img_sv + field(&KvImage::ntok) + 16 * (2 * s + a) + 4 * q);
                        }
                        const half2_t sh[2] = {*reinterpret_cast<const half2_t*>(&h4.x), *reinterpret_cast<const half2_t*>(&h4.y)};
                        const half2_t sl[2] = {*reinterpret_cast<const half2_t*>(&l4.x), *reinterpret_cast<const half2_t*>(&l4.y)};
#pragma unroll
                        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
                            for (int i2 = 0; i2 < 2; ++i2) {
                                half2_t c;
                                if constexpr (LOGP) {
                                    // -code = clip(rint(log2 A)) = clip(rint(arg - log2 Z)); weight 2^(8 - code) * s': exact
                                    // scalings of sh and sl (a weight below fp16's range is below 2^-30 of the largest)
                                    const float c0 = __builtin_amdgcn_fmed3f(__builtin_rintf(S[nt][2 * s + a][2 * i2] - lz[nt]), -dm.plast, 0.f);
                                    const float c1 = __builtin_amdgcn_fmed3f(__builtin_rintf(S[nt][2 * s + a][2 * i2 + 1] - lz[nt]), -dm.plast, 0.f);
                                    const auto pw = __builtin_amdgcn_cvt_pkrtz(ldexpf(256.0f, (int)c0), ldexpf(256.0f, (int)c1));
                                    c = (half2_t){(_Float16)pw[0], (_Float16)pw[1]};
                                    if (TAPS && dm.dbg.p_code) tap_pcode(nt, 16 * (2 * s + a) + 4 * q + 2 * i2, (unsigned)(int)(-c0), (unsigned)(int)(-c1));
                                } else {
                                    const float m0 = __builtin_fmaf(S[nt][2 * s + a][2 * i2], kq[nt], 12608512.0f);
                                    const float m1 = __builtin_fmaf(S[nt][2 * s + a][2 * i2 + 1], kq[nt], 12608512.0f);
                                    const unsigned u = __builtin_amdgcn_perm(__float_as_uint(m1), __float_as_uint(m0), 0x05040100u);
                                    c = *reinterpret_cast<const half2_t*>(&u) - k1024;
                                    if (TAPS && dm.dbg.p_code) tap_pcode(nt, 16 * (2 * s + a) + 4 * q + 2 * i2, u & 0xFFu, (u >> 16) & 0xFFu);
                                }
                                const half2_t wh = c * sh[i2];
                                const half2_t wl = __builtin_elementwise_fma(c, sl[i2], __builtin_elementwise_fma(c, sh[i2], -wh));
                                phi[nt][4 * a + 2 * i2] = wh[0];
                                phi[nt][4 * a + 2 * i2 + 1] = wh[1];
                                plo[nt][4 * a + 2 * i2] = wl[0];
                                plo[nt][4 * a + 2 * i2 + 1] = wl[1];
                            }
                    } else {
#pragma unroll
                        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                phi[nt][4 * a + i] = (_Float16)0.f;
                                plo[nt][4 * a + i] = (_Float16)0.f;
                            }
                    }
                }
                if (!second && s > 0) sums_settle(oacc);
#pragma unroll
                for (int k = 0; k < TPH; ++k) {
                    int j = 16 * k + r16;
                    j = j < D ? j : D - 1;
                    if (second) {  // two score tiles: 32 tokens deep, a lane's 8 codes are consecutive (vt_pos)
                        const uint2 w = PRE_V ? vw2[PRE_V ? s : 0][PRE_V ? k : 0]
                                              : *reinterpret_cast<const uint2*>(vt + (size_t)j * field(&KvImage::cols_v) + 32 * s + 8 * q);
                        half2_t v0, v1, v2, v3;
                        biased4_to_half(w.x, v0, v1);
                        biased4_to_half(w.y, v2, v3);
                        const half8_t va = {v0[0], v0[1], v1[0], v1[1], v2[0], v2[1], v3[0], v3[1]};
#pragma unroll
                        for (int nt = 0; nt < NTT; ++nt) {
                            oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, phi[nt], oacc[nt][k], 0, 0, 0);
                            oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, plo[nt], oacc[nt][k], 0, 0, 0);
                        }
                    } else {       // a last single tile: 16 tokens deep, in their natural order
                        const unsigned w = PRE_V ? vw2[PRE_V ? s : 0][PRE_V ? k : 0].x
                                                 : *reinterpret_cast<const unsigned*>(vt + (size_t)j * field(&KvImage::cols_v) + 32 * s + 4 * q);
                        half2_t v0, v1;
                        biased4_to_half(w, v0, v1);
                        const half4_t va = {v0[0], v0[1], v1[0], v1[1]};
#pragma unroll
                        for (int nt = 0; nt < NTT; ++nt) {
                            const half4_t ph = {phi[nt][0], phi[nt][1], phi[nt][2], phi[nt][3]};
                            const half4_t pl = {plo[nt][0], plo[nt][1], plo[nt][2], plo[nt][3]};
                            oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, ph, oacc[nt][k], 0, 0, 0);
                            oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, pl, oacc[nt][k], 0, 0, 0);
                        }
                    }
                }
            }
        }
    }

    // LEAN: addresses are formed again instead of kept across the attention (DENSE spilled four registers otherwise, and their
    // reloads wait for the weights on their way: 19.0 us at 16384 tokens, 18.3 without)
    const int lane2 = LEAN ? opaque(lane) : lane;
    if constexpr (LEAN) set_wrow(lane2);
    if constexpr (F::PREFETCH_W) slice_out(1, 2);
    if constexpr (RING > 0 && NTT >= 2) {  // several token tiles per wavefront: the attention needs the registers; the first
#pragma unroll                         // RING loads of to_out travel while A^ V~ is quantized (DENSE: half of them behind the first barrier)
        for (int f = 0; f < RING / (DENSE ? 2 : 1); ++f) wring[f] = ring_load(rs_wo, f);
    }
    // ================= per-token int8 codes of O over all heads
    // O = oacc * of, of = 2^-kexp / pmax (times range / Z on the row-range grid). Where nobody needs O itself (no tap)
    // the products are not formed: the row maximum is max|oacc| * of (a product with a positive
    // constant is monotone, so this IS the maximum of the products), and the quantizer takes oacc and of apart.
    constexpr bool KEEP_O = TAPS;
    const float osc = reinterpret_cast<const float*>(imgh + field(&KvImage::oscale))[0] * inv_pmax(dm.pmax);
    float of[NTT];
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        of[nt] = ROWMAX ? osc * fz[nt] : osc;
        float omx = 0.f;
#pragma unroll
        for (int k = 0; k < TPH; ++k) {
            const bool valid = (16 * k + 16 <= D) || 16 * k + 4 * q < D;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (KEEP_O) oacc[nt][k][i] *= of[nt];
                omx = fmaxf(omx, fabsf(oacc[nt][k][i]));  // (rows past the head repeat its last)
            }
            if (KEEP_O && nvalid[nt] && valid) {
                const float4 o4 = make_float4(oacc[nt][k][0], oacc[nt][k][1], oacc[nt][k][2], oacc[nt][k][3]);
                if (TAPS && dm.dbg.O) *reinterpret_cast<float4*>(dm.dbg.O + tok[nt] * C + h * D + 16 * k + 4 * q) = o4;
            }
        }
        if constexpr (!KEEP_O) omx *= of[nt];
        omx = quad_allmax(omx);
        if (q == 0) omax[(tbase + 16 * nt + r16) * NH + h] = __float_as_uint(omx);
    }
    __syncthreads();  // every wavefront is past its reads of the hidden codes
    if constexpr (F::PREFETCH_W) slice_out(2, TPH);
    if constexpr (RING > 0 && DENSE) {
#pragma unroll
        for (int f = RING / 2; f < RING; ++f) wring[f] = ring_load(rs_wo, f);
    }
    const int r2 = lane2 & 15, q2 = lane2 >> 4;
    float so[NTT];
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        float oamax = 0.f;
#pragma unroll
        for (int w = 0; w < NH; ++w) oamax = fmaxf(oamax, __uint_as_float(omax[(tbase + 16 * nt + r2) * NH + w]));
        const bool ozero = oamax == 0.f;
        so[nt] = ozero ? 1.f : div_grid(oamax, 127.f);
        const float osafe = ozero ? 1.f : oamax;
        const float cq = quant_mult(127.f, osafe);
        unsigned pk[TPH];
        quant4_group<QG>(pk, [&](int jt) { return make_float4(oacc[nt][jt][0], oacc[nt][jt][1], oacc[nt][jt][2], oacc[nt][jt][3]); },
                     [&](int) { return QuantRow{KEEP_O ? 1.f : of[nt], cq, osafe}; });
#pragma unroll
        for (int jt = 0; jt < TPH; ++jt)
            if (16 * jt + 4 * q2 < D) {
                const int c = h * D + 16 * jt + 4 * q2;
                *reinterpret_cast<unsigned*>(tileq + (tbase + 16 * nt + r2) * F::TILE_RS + c) = pk[jt];
                if (TAPS && dm.dbg.o_code && nvalid[nt]) *reinterpret_cast<unsigned*>(dm.dbg.o_code + tok[nt] * C + c) = pk[jt];
            }
        if (TAPS && dm.dbg.s_o && nvalid[nt] && q == 0 && h == 0) dm.dbg.s_o[tok[nt]] = so[nt];
    }
    __syncthreads();

    // ================= to_out: Y^T[c][n] for this head's D output channels
    if constexpr (RING > 0) {
        ring_project(rs_wo, pacc, lane2);
    } else {
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
            for (int ks = 0; ks < KC; ++ks)
                hb[nt][ks] = *reinterpret_cast<const int32x4_t*>(tileq + (tbase + 16 * nt + r16) * F::TILE_RS + 64 * ks + 16 * q);
#pragma unroll
        for (int j = 0; j < TPH; ++j) {
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) pacc[nt][j] = (int32x4_t){0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KC; ++ks) {
                const int32x4_t wa = wreg[j][ks];
#pragma unroll
                for (int nt = 0; nt < NTT; ++nt) pacc[nt][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa, hb[nt][ks], pacc[nt][j], 0, 0, 0);
            }
        }
    }
    // Stores through a buffer descriptor of this batch element's rows of `out`: one 32-bit offset per token instead of a 64-bit
    // address per store, and rows past the last (and channels past the head, whose offset is set past the end) are dropped by
    // the bounds check.
    const __amdgpu_buffer_rsrc_t rs_out = __builtin_amdgcn_make_buffer_rsrc(rq.out + (size_t)b * N * C, 0, N * C * 2, 0x00020000);
#pragma unroll
    for (int j = 0; j < TPH; ++j) {
        const int cl = 16 * j + 4 * q2, c = h * D + cl;
        const float4 w4 = *reinterpret_cast<const float4*>(swo + c);
        const float4 b4 = *reinterpret_cast<const float4*>(bo + c);
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt) {
            const float y0 = (float)pacc[nt][j][0] * (so[nt] * w4.x) + b4.x;
            const float y1 = (float)pacc[nt][j][1] * (so[nt] * w4.y) + b4.y;
            const float y2 = (float)pacc[nt][j][2] * (so[nt] * w4.z) + b4.z;
            const float y3 = (float)pacc[nt][j][3] * (so[nt] * w4.w) + b4.w;
            const half4_t y = {(_Float16)y0, (_Float16)y1, (_Float16)y2, (_Float16)y3};
            int off = ((n0 + tbase + 16 * nt + r2) * C + h * D + 4 * q2) * 2 + 32 * j;
            if (!(16 * j + 16 <= D || cl < D)) off = 0x7fffff00;
            __builtin_amdgcn_raw_buffer_store_b64(*reinterpret_cast<const uint2_t*>(&y), rs_out, off, 0, 0);
        }
    }
}

// Compute units of the current device (asked once per device).
static inline int device_cu_count() {
    static std::atomic<int> cus[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cus[dev].load(std::memory_order_acquire);
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cus[dev].store(n, std::memory_order_release);
    }
    return n;
}

template <int D, int NH, int NTT, int PG, int TOK, int NT16, bool DENSE, bool ROWMAJ>
static hipError_t launch_fused_one(const FusedTable& tab, const FusedDims& dm, size_t bytes, hipStream_t st) {
    static std::atomic<unsigned long long> lds_set{0};
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(&fused_block_kernel<D, NH, NTT, PG, TOK, NT16, DENSE, ROWMAJ>), 160 * 1024, lds_set);
    if (e != hipSuccess) return e;
    const int tiles = (dm.N + TOK - 1) / TOK;
    if (tiles > 65535 || dm.R > 65535) return hipErrorInvalidValue;
    const dim3 grid(dm.B, dm.R, tiles);
    hipLaunchKernelGGL((fused_block_kernel<D, NH, NTT, PG, TOK, NT16, DENSE, ROWMAJ>), grid, dim3(FusedCfg<D, NH, NTT, TOK, DENSE>::NT), bytes, st, tab, dm);
    return hipGetLastError();
}

// The instantiation for the layout of the weights.
template <int D, int NH, int NTT, int PG, int TOK, int NT16>
static hipError_t launch_fused_layout(const FusedTable& tab, const FusedDims& dm, size_t bytes, hipStream_t st) {
    if constexpr (FusedCfg<D, NH, NTT, TOK>::RING > 0 && D % 16 == 0) {
        // (with SLOTS a KiB per wavefront more: at most 156 KiB at 80 text tokens)
        if (!dm.w_layout) return launch_fused_one<D, NH, NTT, PG, TOK, NT16, false, true>(tab, dm, bytes + (NTT <= 2 && NT16 == 5 ? NH * 1024 : 0), st);
    }
    return launch_fused_one<D, NH, NTT, PG, TOK, NT16, false, false>(tab, dm, bytes, st);
}

template <int D, int NH, int NTT, int PG, int TOK, int NT16>
static hipError_t launch_fused_grid(const FusedTable& tab, const FusedDims& dm, hipStream_t st) {
    using F = FusedCfg<D, NH, NTT, TOK>;
    const size_t bytes = dm.I.bytes + TOK * F::TILE_RS + 3 * F::C * 4 + TOK * 4 + TOK * NH * 4;  // = fused_lds_bytes
    if (bytes > 160 * 1024 || dm.I.head_bytes > (size_t)F::IMGC * 1024) return hipErrorInvalidValue;
    if constexpr (NT16 == 5 && D == 40 && NH == 8 && NTT == 2) {
        // More token tiles than compute units and a working set of at most half a compute unit's LDS: the instantiation
        // of which two workgroups share a compute unit (one is in its arithmetic while the other waits for memory).
        if ((dm.N + TOK - 1) / TOK * dm.R * dm.B > device_cu_count() && bytes <= 80 * 1024)
            return launch_fused_one<D, NH, NTT, PG, TOK, NT16, true, false>(tab, dm, bytes, st);
    }
    if constexpr (F::RING > 0 && NT16 == 5 && NTT == 2) {
        // Workgroups that fill a compute unit run in rounds of one per unit; of 48 or 64 tokens each, instead of 32, they take
        // longer (at d = 80 26 and 33 us, against 20; at d = 64 28), but there may be fewer rounds: 12288 tokens
        // 37.2 -> 26.3 us, 16384 tokens 38.2 -> 33.1 us. One round of 32, 48 and 64 tokens with row-major weights: 21.9, 28.6 and
        // 35.1 us at d = 80, 22.6 and 33.1 us at d = 64 (operand-ordered 20.2 and 31.3); the other grids are within 4 % of these.
        const long cu = device_cu_count(), mul = (long)dm.R * dm.B;
        auto rounds = [&](int tok) { return ((dm.N + tok - 1) / tok * mul + cu - 1) / cu; };
        auto fits = [&](int tok) { return bytes + (tok - TOK) * (F::TILE_RS + 4 + NH * 4) <= 160 * 1024; };
        const long cost2 = 20 * rounds(32), cost3 = fits(48) ? (NH <= 8 ? 26 : 28) * rounds(48) : cost2, cost4 = fits(64) ? 33 * rounds(64) : cost2;
        if constexpr (NH <= 8) if (cost4 < cost2 && cost4 < cost3) return launch_fused_layout<D, NH, 4, PG, 64, NT16>(tab, dm, bytes + 32 * (F::TILE_RS + 4 + NH * 4), st);
        if (cost3 < cost2) return launch_fused_layout<D, NH, 3, PG, 48, NT16>(tab, dm, bytes + 16 * (F::TILE_RS + 4 + NH * 4), st);
    }
    return launch_fused_layout<D, NH, NTT, PG, TOK, NT16>(tab, dm, bytes, st);
}

template <int D, int NH, int NTT, int PG, int TOK>
static hipError_t launch_fused_tiles(const FusedTable& tab, const FusedDims& dm, hipStream_t st) {
    // 65 to 80 text tokens: the instantiation without run-time guards around the score tiles
    const bool taps = dm.dbg.h_code || dm.dbg.s_h || dm.dbg.q_code || dm.dbg.s_Q || dm.dbg.O || dm.dbg.o_code || dm.dbg.s_o || dm.dbg.p_code;
    if (dm.nt16 == 5 && !taps) return launch_fused_grid<D, NH, NTT, PG, TOK, 5>(tab, dm, st);
    return launch_fused_grid<D, NH, NTT, PG, TOK, 0>(tab, dm, st);
}

template <int D, int NH, int NTT, int TOK>
static hipError_t launch_fused_cfg(const FusedTable& tab, const FusedDims& dm, int grid, hipStream_t st) {
    if (grid == TAQ_PROB_LOG2) return launch_fused_tiles<D, NH, NTT, TAQ_PROB_LOG2, TOK>(tab, dm, st);
    if (grid == TAQ_PROB_ROWMAX) return launch_fused_tiles<D, NH, NTT, TAQ_PROB_ROWMAX, TOK>(tab, dm, st);
    return launch_fused_tiles<D, NH, NTT, TAQ_PROB_LINEAR, TOK>(tab, dm, st);
}

// Family launchers, one translation unit each. tok = 32 or 16 image tokens per workgroup.
hipError_t launch_fused_d40(const FusedTable& tab, const FusedDims& dm, int grid, int tok, hipStream_t st);   // (d, H) = (40, 8)
hipError_t launch_fused_d80(const FusedTable& tab, const FusedDims& dm, int grid, int tok, hipStream_t st);   // (80, 8)
hipError_t launch_fused_d64(const FusedTable& tab, const FusedDims& dm, int grid, int tok, hipStream_t st);   // (64, 10)

}  // namespace taq
