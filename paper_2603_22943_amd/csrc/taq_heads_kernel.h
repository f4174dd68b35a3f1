// Head-group kernel of the C = 1280 and 640 layers of few tokens (PersonalQ, Section III-B) for gfx950: per-token codes of `hidden`, to_q, Q~ (Eq. 2,
// third line), scores, softmax, Eq. (3) and A^ V~ of a few heads and 16 or 32 image tokens, in one workgroup. Included by one translation
// unit per (head dimension, heads) (taq_heads160.hip, _heads64, _heads80, _heads64x10); A^ V~ leaves it in operand order for to_out_tail_kernel (taq_fused.hip).
//
// The arithmetic is that of the fused block kernel (taq_fused_kernel.h, where each step is derived), everything transposed, an image
// token in lane (token % 16) of its wavefront throughout.
//
// Work split: one wavefront per 16-channel block of the group's heads (NH heads of D: 8 or 10 wavefronts), from the first product to the
// last. In to_q a wavefront multiplies its 16 channels over the whole K range: no partial sums, and the accumulators stay where Q~ is
// quantized from them; what the wavefronts of a head exchange through LDS is the largest |Q| per token and the finished codes. Scores,
// softmax and the weights of Eq. (3) are shared out by tiles of text tokens, A^ V~ by channel blocks. (An earlier form split to_q by K
// range as well, with partial sums through LDS, let four of its eight wavefronts stop there, and the others each form the scores and
// weights of a whole head: 9.3 k clocks behind to_q, against 5.5 k; forming them in all ten wavefronts took 11 k.)
//
// What bounds it: the front half. Hidden rows 41 KB, weights 160 or 205 KB, image 23 or 27 KB pass one compute unit's path at 64 B a clock,
// 4.3 k clocks at 8 heads of 160, 1.8 k until the hidden tile is there in front of them; to_q (every wavefront reads the tile's codes out
// of LDS, 2 k clocks) runs while the weights arrive, and 6 k follow in seven short phases with a barrier each. With the tail kernel of
// its time, us per layer: 512 tokens of 8 heads of 160 18.3 -> 15.95, 64 tokens 14.7 -> 13.0, 496 tokens 21.9 -> 16.0 (whose tiles were not
// dealt to the XCDs in eighths before), 784 tokens of 20 heads of 64 25.5 -> 20.0. C = 640, against the single kernel: 13.6 -> 9.3 us at
// 16 tokens of 8 heads of 80 (6 of them this kernel: the chain of its phases), 14.2 -> 12.1 at 1024, 17.9 -> 16.2 at 1419 with row-major
// weights.
//
// Up to 128 registers with eight wavefronts, 96 with ten, and half of LDS: two workgroups share a compute unit. With TT = 2 a workgroup
// has 32 tokens: more work behind each weight, longer phases; where it saves a round of workgroups it is the faster (heads_plan).
#pragma once
#include "taq_device.h"

namespace taq {

struct HeadsReq {
    const __half* hidden;
    const uint8_t* packed;
    const int8_t* wq;
    const float* s_wq;
};
// (In the order in which they are needed, and without what the instantiation knows: the arguments come from memory line by line, and a
// line that is asked for late stands in the chain.)
struct HeadsArgs {
    HeadsReq rq;
    int N, NT, tile0, tile1, b0, T;
    int groups, nb;              // groups of TT tiles per batch element, batch elements
    unsigned inv_groups;         // inverse32
    float sig2, qmaxq, pmax, plast;  // as in AttnOpArgs; 127 or 7: grid of Q~
    int nt16;
    size_t w_off;  // operand-ordered weights: where they begin
    float* o_op;   // A^ V~ and its largest magnitudes, as the stage path's tiles hold them (StageTile)
    float* o_max;
    size_t image, k16, v16t;     // of KvLayout
    KvImage I;                   // (at other lengths of text than 65 to 80 tokens)
    size_t image_bytes;
    taq_debug dbg;
};
// Several requests (grid y) in a launch, with arguments of their own: a table in HeadsArgs, which the kernel's fields then lie further
// apart with, costs a call of one request 0.25 to 0.5 us.
struct HeadsManyArgs {
    HeadsArgs a;  // (a.rq: not used)
    size_t ws_step;  // bytes from one request's A^ V~ to the next one's
    HeadsReq req[TAQ_MAX_REQ];
};

template <int D, int NH, int NG, int TT, int MT16>
struct HeadsCfg {
    static constexpr int H = NH * NG, C = D * H, TPH = D / 16, NW = NH * TPH, KC = C / 64;
    static constexpr int KS = (TPH + 3) / 4, FS = (TPH + 1) / 2;
    static constexpr int TILE_RS = C + 16;  // bytes per token row of the int8 tile
    // What the attention exchanges, in KiB, in the tile's place (C = 640: a larger one): Q~ codes [NH][TT][KS], with two token tiles overlaid by the weights of the second
    // one; E [NH][MT16 + 1][TT]; protected E as operands [NH][TT]
    static constexpr int X_E = TT > 1 && MT16 > TT * KS ? NH * MT16 : NH * TT * KS, X_P = X_E + NH * TT * (MT16 + 1);
    static constexpr int TILE = 16 * TT * TILE_RS > (X_P + NH * TT) * 1024 ? 16 * TT * TILE_RS : (X_P + NH * TT) * 1024;
    static_assert(TPH >= 4 && TT <= 2, "the weights of the first tile fit the place of the K~ codes");
    // hidden tile: threads per token (whole shares of 8 channels), wavefronts that hold it
    static constexpr int TPT = TT == 1 && C % 256 == 0 ? 32 : 16, HOLD = 16 * TT * TPT / 64;
    static_assert(C % (8 * TPT) == 0 && HOLD <= 8 && NW >= 8, "whole shares, a thread each");
    static size_t lds_bytes(size_t head_bytes) {
        // image | token codes | protected rows (K, V) | scales | maxima
        return NH * head_bytes + TILE + NW * 1024 + 16 * TT * 4 + NW * TT * 16 * 4 + NH * TT * (MT16 + 1) * 16 * 4;
    }
};

template <int D, int NH, int NG, int TT, int PG, int NT16, bool ROWMAJ, bool MANY>
__global__ __launch_bounds__(64 * NH * (D / 16)) __attribute__((amdgpu_waves_per_eu(NH * (D / 16) == 8 ? 4 : 5)))
void heads_kernel(std::conditional_t<MANY, HeadsManyArgs, HeadsArgs> args) {
    const HeadsArgs& a = [&]() -> const HeadsArgs& {
        if constexpr (MANY) return args.a;
        else return args;
    }();
    constexpr int MT16 = NT16 ? NT16 : 6;
    using F = HeadsCfg<D, NH, NG, TT, MT16>;
    static_assert(D % 16 == 0 && F::C % 64 == 0, "whole blocks");
    constexpr int C = F::C, H = F::H, TPH = F::TPH, NW = F::NW, KC = F::KC, KS = F::KS, FS = F::FS;
    constexpr bool LOGP = PG == TAQ_PROB_LOG2, ROWMAX = PG == TAQ_PROB_ROWMAX;
    constexpr bool TAPS = NT16 == 0;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r16 = lane & 15, q = lane >> 4;
    const int hl = wv / TPH, j = wv % TPH;  // head of the group, channel block of the head
    const unsigned ri = MANY ? blockIdx.y : 0u;
    HeadsReq rq = a.rq;
    size_t ws_at = 0;
    if constexpr (MANY) {
        rq = args.req[ri];
        ws_at = ri * args.ws_step;
    }
    asm volatile("" ::"s"(rq.hidden), "s"(rq.packed), "s"(rq.wq), "s"(rq.s_wq), "s"(a.N), "s"(a.NT), "s"(a.groups), "s"(a.inv_groups), "s"(a.nb), "s"(a.w_off), "s"(a.image), "s"(a.k16),
                 "s"(a.v16t), "s"(a.sig2), "s"(a.qmaxq), "s"(a.pmax), "s"(a.o_op));
    constexpr KvImage CI = kv_image(H, D, 16 * MT16);
    auto field = [&](auto m) { return NT16 ? CI.*m : a.I.*m; };
    const size_t head_bytes = field(&KvImage::head_bytes), image_bytes = NT16 ? align_up(CI.bytes, 256) : a.image_bytes;
    // An eighth of the (tile, head group) pairs to an XCD, tile after tile with its groups: the hidden rows come into one L2, and
    // to_out_tail_kernel finds A^ V~ there.
    const int item = XcdShare::item(blockIdx.x, (unsigned)(a.groups * a.nb * NG));
    if (item < 0) return;
    const int tg = item / NG, by = item - tg * NG;  // (NG is a constant)
    const int bi = a.inv_groups ? (int)__umulhi((unsigned)tg, a.inv_groups) : (int)((unsigned)tg / (unsigned)a.groups), gx = tg - bi * a.groups, b = a.b0 + bi;
    const int lo = b * a.NT > a.tile0 ? b * a.NT : a.tile0, hi = (b + 1) * a.NT < a.tile1 ? (b + 1) * a.NT : a.tile1;
    const int tile = lo + gx * TT;
    if (tile >= hi) return;  // (the whole workgroup)
    const int N = a.N, T = a.T, nt16 = NT16 ? NT16 : a.nt16, n0 = (tile - b * a.NT) * 16, h = by * NH + hl;

    // ---- the hidden tiles: 32 or 16 threads per token, 16-byte loads (wavefronts past the eighth, or the fourth: none)
    constexpr int TPT = F::TPT, CH = C / (8 * TPT);
    const int tok0 = tid / TPT, part0 = tid % TPT, nq0 = n0 + tok0;
    const size_t row0 = (size_t)b * N + (nq0 < N ? nq0 : N - 1);
    const bool holds = NW == F::HOLD || wv < F::HOLD;
    uint4 xin[CH];
    if (holds) {
        const uint4* xr = reinterpret_cast<const uint4*>(rq.hidden + row0 * C);
#pragma unroll
        for (int it = 0; it < CH; ++it) xin[it] = xr[it * TPT + part0];
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- LDS
    unsigned char* imgh = smem + (size_t)hl * head_bytes;
    int8_t* tileq = reinterpret_cast<int8_t*>(smem + (size_t)NH * head_bytes);  // [16 TT][C + 16] codes of hidden
    unsigned* qcode = reinterpret_cast<unsigned*>(tileq);                           // later [NH][TT][KS][64 lanes][4] codes of Q~
    unsigned char* prot = reinterpret_cast<unsigned char*>(tileq) + F::TILE;  // K rows [16 slots][NH * D], V columns [NH * D][16 slots]
    float* s_h = reinterpret_cast<float*>(prot + NW * 1024);  // [16 TT]
    float* mx = s_h + 16 * TT;                                // [NW][16 TT] largest |Q|, later largest |A^ V~|, of each block

    // ---- K~/V~ image of the group's heads, straight into LDS, 1 KiB per wavefront-wide load (the last piece may overlap the one before)
    const __amdgpu_buffer_rsrc_t rs_img = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(rq.packed) + a.image + (size_t)b * image_bytes + (size_t)by * NH * head_bytes, 0, (int)(NH * head_bytes), 0x00020000);
    const int img_last = NH * (int)head_bytes - 1024;
    constexpr int IW = NW == F::HOLD ? NW : NW - F::HOLD, IMG_MAX = (NH * (int)kv_image(H, D, TAQ_MAX_T).head_bytes + 1023) / 1024, IPW = (IMG_MAX + IW - 1) / IW;
    auto copy_image = [&](int w) {
#pragma unroll
        for (int k = 0; k < IPW; ++k) {
            const int at = (w + IW * k) * 1024, o = at < img_last ? at : img_last;
            if (at < img_last + 1024)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_img, (__attribute__((address_space(3))) void*)(smem + o), 16, lane * 16, o, 0, 0);
        }
    };
    const int ntrig = reinterpret_cast<const int*>(rq.packed)[b];
    const int nfp = (ntrig + 15) >> 4;
    const __half* k16 = reinterpret_cast<const __half*>(rq.packed + a.k16) + (size_t)b * T * C;
    const __half* v16t = reinterpret_cast<const __half*>(rq.packed + a.v16t) + (size_t)b * C * 96;
    // The first 16 protected K rows and V columns of the group: a KiB of one or the other per wavefront (K rows past the protected tokens
    // carry an offset past the end and are not fetched). Buffer loads all: the compiler counts a direct-to-LDS load of the flat
    // form as one that any later wait has to wait for.
    auto copy_protected = [&]() {
        if (nfp == 0) return;
        const bool isv = wv >= NW / 2;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half*>(isv ? v16t : k16), 0, isv ? C * 96 * 2 : T * C * 2, 0x00020000);
        const int i = (wv - (isv ? NW / 2 : 0)) * 64 + lane;       // 16-byte piece of the rows, of the columns
        const int slot = i / (2 * NW), part = i % (2 * NW);        // (2 NW pieces to a K row of the group, 2 to a V column)
        const int koff = slot < ntrig ? (slot * C + by * NH * D) * 2 + 16 * part : 0x7fffff00, voff = (by * NH * D + (i >> 1)) * 192 + 16 * (i & 1);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(prot + wv * 1024), 16, isv ? voff : koff, 0, 0, 0);
    };

    // ---- this wavefront's weights: 16 rows of Wq, all K steps
    const int woff = !ROWMAJ ? (int)a.w_off + ((h * TPH + j) * KC) * 1024 + lane * 16 : (h * D + 16 * j + (lane >> 2)) * C + 16 * (lane & 3);
    // KPRE weights are requested while the hidden tile is in registers, the others, up to RW on their way at a time, between the products.
    // (All of them and the image requested in front of the barrier: the codes of the tile came 2 k clocks later than the tile, and to_q
    // began when the last weight had arrived; 15.8 -> 15.1 us at 512 tokens of 8 heads of 160, row-major weights 19.5 -> 17.7. 6 to 14 in
    // front and 12 to 16 on their way are within 1 %.) Row-major weights change lanes EX steps ahead of their products.
    constexpr int RW = KC == 10 ? (ROWMAJ ? 8 : 10) : TT == 2 ? 12 : ROWMAJ ? 10 : 14, KPRE = KC == 10 ? 5 : TT == 1 || NW == 8 ? 10 : 0, EX = 2;
    int32x4_t w[KC];
    auto load_w = [&](int ks) { w[ks] = *reinterpret_cast<const int32x4_t*>(rq.wq + woff + (ROWMAJ ? 64 : 1024) * ks); };
    const float4 wq4 = *reinterpret_cast<const float4*>(rq.s_wq + h * D + 16 * j + 4 * q);

    // ---- per-token codes of the hidden tile (every head group of a tile forms the same)
    if (holds) {
        half2_t am2 = {(_Float16)0.f, (_Float16)0.f};
#pragma unroll
        for (int it = 0; it < CH; ++it) {
            const unsigned x[4] = {xin[it].x & 0x7fff7fffu, xin[it].y & 0x7fff7fffu, xin[it].z & 0x7fff7fffu, xin[it].w & 0x7fff7fffu};
#pragma unroll
            for (int e = 0; e < 4; ++e) am2 = __builtin_elementwise_max(am2, *reinterpret_cast<const half2_t*>(&x[e]));
        }
        float amax = fmaxf((float)am2[0], (float)am2[1]);
        // The hidden tile has arrived; the larger reads follow, a few at a time between pieces of the quantizer (a wavefront
        // stands at a load while the texture unit's queue is full).
        __builtin_amdgcn_sched_barrier(0);
        amax = row16_allmax(amax);
        if constexpr (TPT == 32) {
            const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(amax), __float_as_uint(amax), false, false);
            amax = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        }
        const bool zero0 = amax == 0.f;
        const float sc0 = zero0 ? 1.f : div_grid(amax, 127.f), safe0 = zero0 ? 1.f : amax;
        const QuantRow hrow = {1.f, quant_mult(127.f, safe0), safe0};
        const HalfRow half = half_row(hrow.c, sc0, amax);
        const bool again = TAQ_DOUBT(half.doubt);
        const bool tap = TAPS && by == 0 && nq0 < N;
        if (part0 == 0) s_h[tok0] = sc0;
        if (tap && a.dbg.s_h && part0 == 0) a.dbg.s_h[row0] = sc0;
        auto hidden4 = [&](int it, int u) {
            const half2_t* x = reinterpret_cast<const half2_t*>(&xin[it]) + 2 * u;
            return make_float4((float)x[0][0], (float)x[0][1], (float)x[1][0], (float)x[1][1]);
        };
        constexpr int LPI = (KPRE + CH - 1) / CH;
#pragma unroll
        for (int it = 0; it < CH; ++it) {
#pragma unroll
            for (int ks = it * LPI; ks < (it + 1) * LPI && ks < KPRE; ++ks) load_w(ks);
            const float4 x = hidden4(it, 0), y = hidden4(it, 1);
            uint2 pk = make_uint2(quant4_at(x.x, x.y, x.z, x.w, half.m), quant4_at(y.x, y.y, y.z, y.w, half.m));
            if (again) pk = make_uint2(half_row_settle(pk.x, x.x, x.y, x.z, x.w, hrow), half_row_settle(pk.y, y.x, y.y, y.z, y.w, hrow));
            *reinterpret_cast<uint2*>(tileq + tok0 * F::TILE_RS + (it * TPT + part0) * 8) = pk;
            if (tap && a.dbg.h_code) *reinterpret_cast<uint2*>(a.dbg.h_code + row0 * C + (it * TPT + part0) * 8) = pk;
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int ks = 0; ks < KPRE; ++ks) load_w(ks);
    }
#pragma unroll
    for (int ks = KPRE; ks < RW; ++ks) load_w(ks);
    __syncthreads();

    // ---- to_q: this wavefront's 16 channels, two chains of products
    // (row-major weights: the lanes are exchanged through a KiB of LDS, behind everything else)
    auto exchange = [&](int ks) {
        unsigned char* slot = reinterpret_cast<unsigned char*>(mx + (NW + NH * (MT16 + 1)) * TT * 16) + wv * 1024;
        const int lr = lane >> 2, ls = lane & 3;
        *reinterpret_cast<int32x4_t*>(slot + lr * 64 + ((ls ^ ((lr >> 1 ^ lr >> 2) & 3)) << 4)) = w[ks];
        w[ks] = *reinterpret_cast<const int32x4_t*>(slot + r16 * 64 + ((q ^ ((r16 >> 1 ^ r16 >> 2) & 3)) << 4));
    };
    if constexpr (ROWMAJ) {
#pragma unroll
        for (int ks = 0; ks < EX; ++ks) exchange(ks);
    }
    constexpr int CHAINS = TT == 1 ? 2 : 1;
    int32x4_t acc[TT][CHAINS];
#pragma unroll
    for (int nt = 0; nt < TT; ++nt)
#pragma unroll
        for (int c = 0; c < CHAINS; ++c) acc[nt][c] = (int32x4_t){0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KC; ++ks) {
        if (ROWMAJ && ks + EX < KC) exchange(ks + EX);
#pragma unroll
        for (int nt = 0; nt < TT; ++nt) {
            const int32x4_t hb = *reinterpret_cast<const int32x4_t*>(tileq + (16 * nt + r16) * F::TILE_RS + 64 * ks + 16 * q);
            acc[nt][ks % CHAINS] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[ks], hb, acc[nt][ks % CHAINS], 0, 0, 0);
        }
        if (ks + RW < KC) load_w(ks + RW);
        if (ks == (RW < KC ? KC - RW - 1 : 0)) {  // the image and the protected rows behind the weights: they are needed last
            copy_protected();
            if (NW == F::HOLD || !holds) copy_image(NW == F::HOLD ? wv : wv - F::HOLD);
        }
        if (ks + RW < KC || ks == 0) __builtin_amdgcn_sched_barrier(0);
    }
    float qf[TT][4];
#pragma unroll
    for (int nt = 0; nt < TT; ++nt) {
        const float sh = s_h[16 * nt + r16];
        const float wq[4] = {wq4.x, wq4.y, wq4.z, wq4.w};
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            qf[nt][i] = (float)(acc[nt][0][i] + (CHAINS > 1 ? acc[nt][CHAINS - 1][i] : 0)) * (sh * wq[i]);
            m = fmaxf(m, fabsf(qf[nt][i]));
        }
        m = quad_allmax(m);
        if (q == 0) mx[(wv * TT + nt) * 16 + r16] = m;
    }
    // This wavefront's pieces of the image and of the protected rows are in LDS before the barrier: nothing else makes anybody wait
    // for another wavefront's.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();

    // ---- Eq. (2), third line: Q~ = Q_a(Q) per (token, head); codes to the wavefronts of the head (over the codes of hidden)
    float sq2[TT];
    size_t tok[TT];
    bool nvalid[TT];
#pragma unroll
    for (int nt = 0; nt < TT; ++nt) {
        float qmax = 0.f;
#pragma unroll
        for (int k = 0; k < TPH; ++k) qmax = fmaxf(qmax, mx[((hl * TPH + k) * TT + nt) * 16 + r16]);
        const bool qzero = qmax == 0.f;
        const float sQ = qzero ? 1.f : div_grid(qmax, a.qmaxq), qsafe = qzero ? 1.f : qmax;
        const int n = n0 + 16 * nt + r16;
        nvalid[nt] = n < N;
        tok[nt] = (size_t)b * N + (nvalid[nt] ? n : N - 1);
        unsigned pk[1];
        const float cq = quant_mult(a.qmaxq, qsafe);
        quant4_group<1>(pk, [&](int) { return make_float4(qf[nt][0], qf[nt][1], qf[nt][2], qf[nt][3]); }, [&](int) { return QuantRow{1.f, cq, qsafe}; }, a.qmaxq);
        qcode[(((hl * TT + nt) * KS + (j >> 2)) * 64 + lane) * 4 + (j & 3)] = pk[0];
        if (TAPS && a.dbg.q_code && nvalid[nt]) *reinterpret_cast<unsigned*>(a.dbg.q_code + tok[nt] * C + h * D + 16 * j + 4 * q) = pk[0];
        if (TAPS && a.dbg.s_Q && nvalid[nt] && q == 0 && j == 0) a.dbg.s_Q[tok[nt] * H + h] = sQ;
        sq2[nt] = fmaxf(sQ * a.sig2, 1e-37f);
    }
    __syncthreads();
    // Q~ codes of token tile nt, the B operand of the scores
    auto q_operand = [&](int nt, int32x4_t (&qop)[KS]) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qop[ks] = *reinterpret_cast<const int32x4_t*>(qcode + (((hl * TT + nt) * KS + ks) * 64 + lane) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * ks + e >= TPH) qop[ks][e] = 0;
        }
    };

    // ---- scores x[t][n] = (K~ Q~^T)[t][n] * s_K[t] (+ 0 / -inf) and softmax, shared out among the wavefronts of a head: pieces of 16 text
    // tokens by 16 image tokens, and the protected rows of each token tile. What they exchange is the row maximum,
    // E = exp2(score - maximum) and the operands of A^ V~.
    constexpr int NTW = (MT16 * TT + TPH - 1) / TPH;  // pieces of a wavefront: j, j + TPH, ...; piece p: text tile p / TT, token tile p % TT
    const int pt = TPH - 1 - j;                       // token tile of whose protected rows this wavefront takes care, if there is one
    float4* ebuf = reinterpret_cast<float4*>(qcode + F::X_E * 256) + hl * TT * (MT16 + 1) * 64 + lane;  // [MT16 tiles, protected][TT][64 lanes]  E
    uint4* pbuf = reinterpret_cast<uint4*>(qcode + F::X_P * 256) + hl * TT * 64 + lane;   // [TT][64 lanes]  protected E as fp16 high parts, remainders
    // [MT16][64 lanes]  weights likewise: of the first token tile over the K~ codes, of the second over the Q~ codes
    uint4* wbuf0 = reinterpret_cast<uint4*>(imgh + field(&KvImage::kp)) + lane;
    uint4* wbuf1 = reinterpret_cast<uint4*>(qcode) + hl * MT16 * 64 + lane;
    float* mt = mx + (NW + hl * (MT16 + 1)) * TT * 16;                                                        // [MT16 tiles, protected][TT][16]  maxima
    float S[NTW][4];
    const float* img_sk = reinterpret_cast<const float*>(imgh + field(&KvImage::s_k));
    const float* img_bias = reinterpret_cast<const float*>(imgh + field(&KvImage::bias));
#pragma unroll
    for (int u = 0; u < NTW; ++u) {
        const int p = j + TPH * u, tt = p / TT, nt = p % TT;
        if (tt < nt16) {
            int32x4_t sc = sum_start(), qop[KS];
            q_operand(nt, qop);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                int32x4_t ka;
                const int8_t* kp = reinterpret_cast<const int8_t*>(imgh + field(&KvImage::kp));
                if constexpr (TPH % 4 == 0) {
                    ka = *reinterpret_cast<const int32x4_t*>(kp + kp_offset(TPH, 16 * tt + r16, 4 * ks, q));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) ka[e] = 4 * ks + e < TPH ? *reinterpret_cast<const int*>(kp + kp_offset(TPH, 16 * tt + r16, 4 * ks + e, q)) : 0;
                }
                sc = __builtin_amdgcn_mfma_i32_16x16x64_i8(ka, qop[ks], sc, 0, 0, 0);
            }
            const float4 sk = *reinterpret_cast<const float4*>(img_sk + 16 * tt + 4 * q);
            const float4 bi4 = *reinterpret_cast<const float4*>(img_bias + 16 * tt + 4 * q);
            S[u][0] = __builtin_fmaf(sum_float(sc[0]), sk.x, bi4.x);
            S[u][1] = __builtin_fmaf(sum_float(sc[1]), sk.y, bi4.y);
            S[u][2] = __builtin_fmaf(sum_float(sc[2]), sk.z, bi4.z);
            S[u][3] = __builtin_fmaf(sum_float(sc[3]), sk.w, bi4.w);
            const float m = quad_allmax(fmaxf(fmaxf(S[u][0], S[u][1]), fmaxf(S[u][2], S[u][3])));
            if (q == 0) mt[p * 16 + r16] = m;
        }
    }
    // protected rows: scores of tile ft of 16 slots, the first from LDS, further ones (rare) straight from the fp16 K rows;
    // -inf past ntrig. (Slots of LDS that were not fetched hold anything: an operand row reaches no other row of the result.)
    auto protected_scores = [&](auto first, int ft, int nt) {
        floatx4_t f = {0.f, 0.f, 0.f, 0.f};
        int slot = 16 * ft + r16;
        slot = slot < T ? slot : T - 1;
        const __half* kr = k16 + (size_t)slot * C + h * D + 4 * q;
        int32x4_t qop[KS];
        q_operand(nt, qop);
#pragma unroll
        for (int s = 0; s < FS; ++s) {
            half8_t ka;
            half2_t c[4];
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int jt = 2 * s + jj;
                uint2 v = make_uint2(0, 0);
                if (jt < TPH) v = decltype(first)::value ? *reinterpret_cast<const uint2*>(prot + r16 * (32 * NW) + hl * 2 * D + 32 * jt + 8 * q) : *reinterpret_cast<const uint2*>(kr + 16 * jt);
                const half4_t hv = *reinterpret_cast<const half4_t*>(&v);
#pragma unroll
                for (int e = 0; e < 4; ++e) ka[4 * jj + e] = hv[e];
                biased4_to_half((jt < TPH ? (unsigned)qop[jt / 4][jt % 4] : 0u) ^ 0x80808080u, c[2 * jj], c[2 * jj + 1]);
            }
            const half8_t qh = {c[0][0], c[0][1], c[1][0], c[1][1], c[2][0], c[2][1], c[3][0], c[3][1]};
            f = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qh, f, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = 16 * ft + 4 * q + i < ntrig ? f[i] : TAQ_NEG_INF;
        return f;
    };
    floatx4_t fsc;
    if (nfp > 0 && pt < TT) {
        fsc = protected_scores(std::true_type{}, 0, pt);
        float m = fmaxf(fmaxf(fsc[0], fsc[1]), fmaxf(fsc[2], fsc[3]));
        for (int ft = 1; ft < nfp; ++ft) {
            const floatx4_t f = protected_scores(std::false_type{}, ft, pt);
            m = fmaxf(m, fmaxf(fmaxf(f[0], f[1]), fmaxf(f[2], f[3])));
        }
        m = quad_allmax(m);
        if (q == 0) mt[(MT16 * TT + pt) * 16 + r16] = m;
    }
    __syncthreads();

    // ---- E of this wavefront's pieces (log2 grid: the exponent itself is kept)
    float off[TT];
#pragma unroll
    for (int nt = 0; nt < TT; ++nt) {
        float m = nfp > 0 ? mt[(MT16 * TT + nt) * 16 + r16] : TAQ_NEG_INF;
#pragma unroll
        for (int tt = 0; tt < MT16; ++tt)
            if (tt < nt16) m = fmaxf(m, mt[(tt * TT + nt) * 16 + r16]);
        off[nt] = -m * sq2[nt];
    }
    auto of_tile = [](float x0, float x1, int nt) { return TT == 1 || nt == 0 ? x0 : x1; };
#pragma unroll
    for (int u = 0; u < NTW; ++u) {
        const int p = j + TPH * u;
        if (p / TT < nt16) {
            const float sq = of_tile(sq2[0], sq2[TT - 1], p % TT), of = of_tile(off[0], off[TT - 1], p % TT);
            float ex[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float arg = __builtin_fmaf(S[u][i], sq, of);
                ex[i] = __builtin_amdgcn_exp2f(arg);
                S[u][i] = LOGP ? arg : ex[i];
            }
            ebuf[p * 64] = make_float4(ex[0], ex[1], ex[2], ex[3]);
        }
    }
    half4_t phi4, plo4;
    if (nfp > 0 && pt < TT) {
        const float sq = of_tile(sq2[0], sq2[TT - 1], pt), of = of_tile(off[0], off[TT - 1], pt);
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(fsc[i], sq, of));
        split_half2(e[0], e[1], phi4, plo4, 0);
        split_half2(e[2], e[3], phi4, plo4, 2);
        ebuf[(MT16 * TT + pt) * 64] = make_float4(e[0], e[1], e[2], e[3]);
        const uint2 hi2 = *reinterpret_cast<const uint2*>(&phi4), lo2 = *reinterpret_cast<const uint2*>(&plo4);
        pbuf[pt * 64] = make_uint4(hi2.x, hi2.y, lo2.x, lo2.y);
    }
    __syncthreads();

    // ---- Z, in the order of the other kernels: the lane's values one after the other, then the quarters; A^ V~ of this wavefront's 16
    // channels, protected columns first, unnormalised
    floatx4_t osum[1][TT], (&o)[TT] = osum[0];
    float kq[TT], lz[TT], fz[TT];
    const int c0 = hl * D + 16 * j + r16;  // this lane's channel (of the operand) within the group
#pragma unroll
    for (int nt = 0; nt < TT; ++nt) {
        float Z = 0.f, eu = 0.f;
#pragma unroll
        for (int tt = 0; tt < MT16; ++tt)
            if (tt < nt16) {
                const float4 e = ebuf[(tt * TT + nt) * 64];
                Z += e.x;
                Z += e.y;
                Z += e.z;
                Z += e.w;
                if (ROWMAX) eu = fmaxf(eu, fmaxf(fmaxf(e.x, e.y), fmaxf(e.z, e.w)));
            }
        o[nt] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
        auto protected_values = [&](uint2 v, half4_t phi, half4_t plo) {  // slots past ntrig hold zeros
            const half4_t va = *reinterpret_cast<const half4_t*>(&v);
            o[nt] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, phi, o[nt], 0, 0, 0);
            o[nt] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, plo, o[nt], 0, 0, 0);
        };
        if (nfp > 0) {
            const float4 e = ebuf[(MT16 * TT + nt) * 64];
            Z += e.x;
            Z += e.y;
            Z += e.z;
            Z += e.w;
            const uint4 p = pbuf[nt * 64];
            const uint2 ph = make_uint2(p.x, p.y), pl = make_uint2(p.z, p.w);
            protected_values(*reinterpret_cast<const uint2*>(prot + NW * 512 + c0 * 32 + 8 * q), *reinterpret_cast<const half4_t*>(&ph), *reinterpret_cast<const half4_t*>(&pl));
            for (int ft = 1; ft < nfp; ++ft) {
                const floatx4_t f = protected_scores(std::false_type{}, ft, nt);
#pragma unroll
                for (int i = 0; i < 4; i += 2) {
                    const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(f[i], sq2[nt], off[nt])), e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(f[i + 1], sq2[nt], off[nt]));
                    Z += e0;
                    Z += e1;
                    split_half2(e0, e1, phi4, plo4, i);
                }
                protected_values(*reinterpret_cast<const uint2*>(v16t + (size_t)(by * NH * D + c0) * 96 + 16 * ft + 4 * q), phi4, plo4);
            }
        }
        Z = quad_allsum(Z);
        const float kqp = quant_mult(a.pmax, Z);  // pmax / Z
        float rz = 1.f;
        kq[nt] = kqp;
        lz[nt] = LOGP ? __builtin_amdgcn_logf(Z) : 0.f;
        fz[nt] = 1.f;
        if constexpr (ROWMAX) {  // (unprotected columns that together weigh less than 2^-40 of the row are dropped)
            eu = quad_allmax(eu);
            if (eu > Z * 9.094947e-13f) {
                kq[nt] = quant_mult(a.pmax, eu);
                rz = quant_mult(Z, eu);
                fz[nt] = quant_mult(eu, Z);
            }
        }
        if (nfp > 0) {
            const float f = kqp * (reinterpret_cast<const float*>(imgh + field(&KvImage::vpre))[0] * rz);
#pragma unroll
            for (int i = 0; i < 4; ++i) o[nt][i] *= f;
        }
    }
    if (TT > 1 && nfp > 1) __syncthreads();  // (further protected tiles: everybody is through with the Q~ codes)
    // ---- Eq. (3): weights code * s' of this wavefront's pieces
    const _Float16* img_sv = reinterpret_cast<const _Float16*>(imgh + field(&KvImage::s_vp));  // [ntok] high parts | [ntok] low parts
    const half2_t k1024 = {(_Float16)1024.0f, (_Float16)1024.0f};
    auto tap_pcode = [&](int t, unsigned x0, unsigned x1) {  // (one token tile)
        if (nvalid[0]) {
            uint8_t* row = a.dbg.p_code + (tok[0] * H + h) * (size_t)T;
            if (t < T) row[t] = (uint8_t)x0;
            if (t + 1 < T) row[t + 1] = (uint8_t)x1;
        }
    };
#pragma unroll
    for (int u = 0; u < NTW; ++u) {
        const int p = j + TPH * u, tt = p / TT;
        if (tt < nt16) {
            const uint2 h4 = *reinterpret_cast<const uint2*>(img_sv + 16 * tt + 4 * q);
            const uint2 l4 = *reinterpret_cast<const uint2*>(img_sv + field(&KvImage::ntok) + 16 * tt + 4 * q);
            const half2_t vh[2] = {*reinterpret_cast<const half2_t*>(&h4.x), *reinterpret_cast<const half2_t*>(&h4.y)};
            const half2_t vl[2] = {*reinterpret_cast<const half2_t*>(&l4.x), *reinterpret_cast<const half2_t*>(&l4.y)};
            const float kqu = of_tile(kq[0], kq[TT - 1], p % TT), lzu = of_tile(lz[0], lz[TT - 1], p % TT);
            half2_t wh[2], wl[2];
#pragma unroll
            for (int i2 = 0; i2 < 2; ++i2) {
                half2_t c;
                if constexpr (LOGP) {
                    const float x0 = __builtin_amdgcn_fmed3f(__builtin_rintf(S[u][2 * i2] - lzu), -a.plast, 0.f);
                    const float x1 = __builtin_amdgcn_fmed3f(__builtin_rintf(S[u][2 * i2 + 1] - lzu), -a.plast, 0.f);
                    const auto pw = __builtin_amdgcn_cvt_pkrtz(ldexpf(256.0f, (int)x0), ldexpf(256.0f, (int)x1));
                    c = (half2_t){(_Float16)pw[0], (_Float16)pw[1]};
                    if (TAPS && a.dbg.p_code) tap_pcode(16 * tt + 4 * q + 2 * i2, (unsigned)(int)(-x0), (unsigned)(int)(-x1));
                } else {
                    const float m0 = __builtin_fmaf(S[u][2 * i2], kqu, 12608512.0f), m1 = __builtin_fmaf(S[u][2 * i2 + 1], kqu, 12608512.0f);
                    const unsigned u2 = __builtin_amdgcn_perm(__float_as_uint(m1), __float_as_uint(m0), 0x05040100u);
                    c = *reinterpret_cast<const half2_t*>(&u2) - k1024;
                    if (TAPS && a.dbg.p_code) tap_pcode(16 * tt + 4 * q + 2 * i2, u2 & 0xFFu, (u2 >> 16) & 0xFFu);
                }
                wh[i2] = c * vh[i2];
                wl[i2] = __builtin_elementwise_fma(c, vl[i2], __builtin_elementwise_fma(c, vh[i2], -wh[i2]));
            }
            (TT == 1 || p % TT == 0 ? wbuf0 : wbuf1)[tt * 64] = make_uint4(*reinterpret_cast<const unsigned*>(&wh[0]), *reinterpret_cast<const unsigned*>(&wh[1]),
                                      *reinterpret_cast<const unsigned*>(&wl[0]), *reinterpret_cast<const unsigned*>(&wl[1]));
        }
    }
    // (V~ codes on their way across the barrier)
    const uint8_t* vt = imgh + field(&KvImage::vt) + (size_t)(16 * j + r16) * field(&KvImage::cols_v);
    uint2 vw[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        vw[s] = make_uint2(0, 0);
        if (2 * s + 1 < nt16) vw[s] = *reinterpret_cast<const uint2*>(vt + 32 * s + 8 * q);
        else if (2 * s < nt16) vw[s].x = *reinterpret_cast<const unsigned*>(vt + 32 * s + 4 * q);
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        if (2 * s < nt16) {
            half2_t v0, v1, v2, v3;
            biased4_to_half(vw[s].x, v0, v1);
            biased4_to_half(vw[s].y, v2, v3);
#pragma unroll
            for (int nt = 0; nt < TT; ++nt) {
                const uint4* wb = nt == 0 ? wbuf0 : wbuf1;
                const uint4 w0 = wb[2 * s * 64];
                if (2 * s + 1 < nt16) {
                    const uint4 w1 = wb[(2 * s + 1) * 64];
                    const uint4 hi4 = make_uint4(w0.x, w0.y, w1.x, w1.y), lo4 = make_uint4(w0.z, w0.w, w1.z, w1.w);
                    const half8_t va = {v0[0], v0[1], v1[0], v1[1], v2[0], v2[1], v3[0], v3[1]};
                    o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, *reinterpret_cast<const half8_t*>(&hi4), o[nt], 0, 0, 0);
                    o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, *reinterpret_cast<const half8_t*>(&lo4), o[nt], 0, 0, 0);
                } else {
                    const uint2 hi2 = make_uint2(w0.x, w0.y), lo2 = make_uint2(w0.z, w0.w);
                    const half4_t va = {v0[0], v0[1], v1[0], v1[1]};
                    if (nt == 0 && s > 0) sums_settle(osum);
                    o[nt] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, *reinterpret_cast<const half4_t*>(&hi2), o[nt], 0, 0, 0);
                    o[nt] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, *reinterpret_cast<const half4_t*>(&lo2), o[nt], 0, 0, 0);
                }
            }
        }
    }
    // ---- O and its largest magnitude per token of each head
    const float osc = reinterpret_cast<const float*>(imgh + field(&KvImage::oscale))[0] * inv_pmax(a.pmax);
    const size_t th = (size_t)(tile - a.tile0) * H + h;  // (token tile nt: H further on each)
#pragma unroll
    for (int nt = 0; nt < TT; ++nt) {
        const float of = ROWMAX ? osc * fz[nt] : osc;
        const float4 o4 = make_float4(o[nt][0] * of, o[nt][1] * of, o[nt][2] * of, o[nt][3] * of);
        if (TT == 1 || tile + nt < hi) reinterpret_cast<float4*>(reinterpret_cast<char*>(a.o_op) + ws_at)[((th + nt * H) * TPH + j) * 64 + lane] = o4;
        if (TAPS && a.dbg.O && nvalid[nt]) *reinterpret_cast<float4*>(a.dbg.O + tok[nt] * C + h * D + 16 * j + 4 * q) = o4;
        const float omx = quad_allmax(fmaxf(fmaxf(fabsf(o4.x), fabsf(o4.y)), fmaxf(fabsf(o4.z), fabsf(o4.w))));
        if (q == 0) mx[(wv * TT + nt) * 16 + r16] = omx;  // (everybody has read the maxima of Q: barriers ago)
    }
    __syncthreads();
    if (j < TT && q == 0 && tile + j < hi) {
        float om = 0.f;
#pragma unroll
        for (int k = 0; k < TPH; ++k) om = fmaxf(om, mx[((hl * TPH + k) * TT + j) * 16 + r16]);
        reinterpret_cast<float*>(reinterpret_cast<char*>(a.o_max) + ws_at)[(th + j * H) * 16 + r16] = om;
    }
}

template <int D, int NH, int NG, int TT, int PG, int NT16, bool ROWMAJ, bool MANY>
static hipError_t launch_heads_some(HeadsManyArgs m, int R, int tiles_b, hipStream_t st) {
    using F = HeadsCfg<D, NH, NG, TT, NT16 ? NT16 : 6>;
    constexpr auto kernel = &heads_kernel<D, NH, NG, TT, PG, NT16, ROWMAJ, MANY>;
    static std::atomic<unsigned long long> lds_set{0};
    const size_t bytes = F::lds_bytes(m.a.I.head_bytes) + (ROWMAJ ? F::NW * 1024 : 0);
    const hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), 160 * 1024, lds_set);
    if (e != hipSuccess) return e;
    m.a.groups = (tiles_b + TT - 1) / TT;
    if (bytes > 160 * 1024 || (long)m.a.groups * m.a.nb * NG > XcdShare::MOST) return hipErrorInvalidValue;
    const unsigned items = (unsigned)(m.a.groups * m.a.nb * NG);
    m.a.inv_groups = inverse32(m.a.groups, (unsigned long long)m.a.groups * m.a.nb);
    const dim3 grid(XcdShare::grid(items), R), block(64 * F::NW);
    if constexpr (MANY) hipLaunchKernelGGL(kernel, grid, block, bytes, st, m);
    else hipLaunchKernelGGL(kernel, grid, block, bytes, st, m.a);
    return hipGetLastError();
}
template <int D, int NH, int NG, int TT, int PG, int NT16, bool ROWMAJ>
static hipError_t launch_heads_one(const HeadsManyArgs& m, int R, int tiles_b, hipStream_t st) {
    if (R > 1) return launch_heads_some<D, NH, NG, TT, PG, NT16, ROWMAJ, true>(m, R, tiles_b, st);
    return launch_heads_some<D, NH, NG, TT, PG, NT16, ROWMAJ, false>(m, 1, tiles_b, st);
}

template <int D, int NH, int NG, int PG, bool ROWMAJ>
static hipError_t launch_heads_tiles(const HeadsManyArgs& a, int R, int tiles_b, int tt, hipStream_t st) {
    // 65 to 80 text tokens: no run-time guards around the score tiles, no taps
    const bool taps = a.a.dbg.h_code || a.a.dbg.s_h || a.a.dbg.q_code || a.a.dbg.s_Q || a.a.dbg.O || a.a.dbg.p_code;
    if (a.a.nt16 != 5 || taps) return launch_heads_one<D, NH, NG, 1, PG, 0, ROWMAJ>(a, R, tiles_b, st);
    if constexpr (D * NH * NG == 1280)
        if (tt == 2) return launch_heads_one<D, NH, NG, 2, PG, 5, ROWMAJ>(a, R, tiles_b, st);
    return launch_heads_one<D, NH, NG, 1, PG, 5, ROWMAJ>(a, R, tiles_b, st);
}

// tt: token tiles per workgroup, 1 or (C = 1280) 2
template <int D, int NH, int NG>
static hipError_t launch_heads_cfg(const HeadsManyArgs& a, int R, int grid, int tiles_b, int tt, bool packed, hipStream_t st) {
    if (grid == TAQ_PROB_LOG2) return packed ? launch_heads_tiles<D, NH, NG, TAQ_PROB_LOG2, false>(a, R, tiles_b, tt, st) : launch_heads_tiles<D, NH, NG, TAQ_PROB_LOG2, true>(a, R, tiles_b, tt, st);
    if (grid == TAQ_PROB_ROWMAX) return packed ? launch_heads_tiles<D, NH, NG, TAQ_PROB_ROWMAX, false>(a, R, tiles_b, tt, st) : launch_heads_tiles<D, NH, NG, TAQ_PROB_ROWMAX, true>(a, R, tiles_b, tt, st);
    return packed ? launch_heads_tiles<D, NH, NG, TAQ_PROB_LINEAR, false>(a, R, tiles_b, tt, st) : launch_heads_tiles<D, NH, NG, TAQ_PROB_LINEAR, true>(a, R, tiles_b, tt, st);
}

hipError_t launch_heads160(const HeadsManyArgs& a, int R, int grid, int tiles_b, int tt, bool packed, hipStream_t st);  // (d, H) = (160, 8): groups of 1 head
hipError_t launch_heads64(const HeadsManyArgs& a, int R, int grid, int tiles_b, int tt, bool packed, hipStream_t st);   // (64, 20): groups of 2
hipError_t launch_heads80(const HeadsManyArgs& a, int R, int grid, int tiles_b, int tt, bool packed, hipStream_t st);   // (80, 8): groups of 2
hipError_t launch_heads64x10(const HeadsManyArgs& a, int R, int grid, int tiles_b, int tt, bool packed, hipStream_t st);  // (64, 10): groups of 2

}  // namespace taq
