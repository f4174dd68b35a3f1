// The contractions of the kernel-per-stage path (taq_gemm.hip: to_q on operand-ordered weights, taq_gemm_rows.hip: on row-major ones, taq_gemm_out.hip: to_out).
#pragma once
#include "taq_device.h"

namespace taq {

// ------------------------------------------------------------------------------------------
// to_q and to_out of the kernel-per-stage path, on operands in MFMA operand order: a 16 x 64 block is one contiguous KiB, in
// memory and in LDS (conflict-free as it is). Tokens come that way from the quantizer kernels, weights from
// taq_pack_weight; of row-major weights four lanes fetch the 64 bytes of a row, segments swizzled as in
// gemm_i8_lds_kernel. Weight blocks are counted per head (tph = ceil(d/16) blocks each, the last one partly filled), so
// that a wavefront of to_q holds whole heads and quantizes Q~ on its accumulators: what leaves the kernel is one byte per
// channel instead of a float32 for a quantizer kernel to read again, in the registers' own order, which is the order in
// which the attention's score operand wants it.
//
// WM x WN wavefronts of MW token tiles x NW channel blocks each; TPH > 0: to_q with heads of TPH blocks (NW a multiple, or TPH a
// multiple of NW: then TPH / NW wavefronts share a head and exchange its maximum through LDS); TPH = 0: to_out. Blocks go straight
// from global memory into LDS (no registers in between, so that several workgroups share a compute unit), STAGES K steps ahead; the
// operands of the next step are read from LDS while the current one is multiplied; one barrier per step. The LDS reads and the waits
// are written by hand: for reads that it knows of, the compiler waits for every outstanding direct-to-LDS load, which would serialise
// the stages. A wavefront's loads per stage are a constant (blocks past the last are fetched again, K steps past the end carry an
// offset out of range, which fetches nothing), so "stage kc + 1 has arrived" is "at most (STAGES - 2) * NLD loads outstanding".
//
// A step is bound by what the wavefront issues in order: with all reads (10 clocks each) and all loads (each waits its turn at the
// texture unit, 64 bytes a clock) in front of the products, a step took 150 clocks more than its products (16 clocks each). So a
// product goes first, two reads follow each of the first ones and the loads lie evenly behind the others: to_out at 2048 tokens
// of 1280 channels 8.3 -> 7.7 us. A step now takes 360 clocks alone and 405 in sequence there, of which the products are 192 (to_q, two
// wavefronts on a SIMD) and 160: 14 and 13 KiB come through the unit's path from L2 (18 clocks a KiB where nothing else is done) and 40
// and 28 KiB out of LDS. Scales and bias come with the first stage, not at the end. Of the sizes of tile, those that leave no
// compute unit with a second round (tile_cost below). to_q and to_out at C = 1280, us before and after:
//   2048 tokens, heads of 64: 9.3 -> 7.9, 9.9 -> 7.7;  3072, heads of 160: 10.7 -> 9.0, 9.8 -> 8.4;  768, of 160: 8.7 -> 5.5, 6.6 -> 5.9;
//   8192, of 64: 19.8 -> 17.9, 21.3 -> 18.6;  at C = 768 row-major, 4608 tokens: 7.4 -> 6.9, 8.0 -> 7.1.
// (Order of K steps staggered over the workgroups, eight stages instead of four, loads of missing blocks left out by an offset out of
// range: no gain, slower, slower.)
// ------------------------------------------------------------------------------------------
struct GemmOpArgs {
    const int8_t* A;      // token codes in operand order
    const float* sa;      // [tile][16]
    const int8_t* W;      // weight codes
    const float* sw;
    const float* bias;    // to_out
    unsigned* q_op;       // to_q: codes and scales
    float* s_q;
    __half* out;          // to_out
    int8_t* tap_code;     // to_q: row-major taps or NULL
    float* tap_scale;
    float qmax;
    int tiles;            // token tiles of the chunk
    int tile0, NT, N;     // where they are: tile0 + t = b * NT + tile of batch element b
    int KC, C, H, d, tph, MX, NX;
    size_t pack_off;
    unsigned inv_nx, inv_tph;  // inverse32 of NX and tph
};

// The compiler takes the result of this read to be there at once; it knows nothing of the data still on its way into these
// registers. Rule: on every path the destinations pass through `arrived` below (a wait, then an empty asm that takes and gives
// back each of them) before they are used and before the kernel goes on without them. Until then they are alive to the
// compiler, so it places nothing else there; a read whose result nobody takes would leave it free to, with only timing to keep
// the late data from overwriting what it placed. tests/test_waits.py checks the generated code of every kernel.
__device__ __forceinline__ int32x4_t lds_read16(unsigned addr, int off) {
    int32x4_t r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(off));
    return r;
}

// A KiB from memory straight into LDS (lane l: 16 bytes at dst + 16 l).
__device__ __forceinline__ void lds_load1k(const __amdgpu_buffer_rsrc_t rs, unsigned char* dst, int voff, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0, 0);
}

template <int MW, int NW, int WM, int WN, int TPH, int STAGES, bool PACKED>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2)))
void gemm_op_kernel(GemmOpArgs a) {
    constexpr int WAVES = WM * WN, MB = MW * WM, NB = NW * WN, BLK = MB + NB, NLD = (BLK + WAVES - 1) / WAVES;
    constexpr int TP = TPH ? TPH : 1, WPH = TPH > NW ? TPH / NW : 1;  // to_q: wavefronts that share a head
    constexpr int JH = WPH > 1 ? NW : TP, HPW = NW / JH;              // blocks of one head, heads in a wavefront
    static_assert(NLD * (STAGES - 1) < 64, "vmcnt");
    static_assert(TPH == 0 || JH % QPlace<TP>::UNIT == 0, "whole units of Q~");
    static_assert(TPH == 0 || (WPH > 1 ? TPH % NW == 0 && WN % WPH == 0 : NW % TP == 0), "whole heads per workgroup");
    __shared__ __align__(16) unsigned char lds[STAGES * BLK * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int wm = wave % WM, wn = wave / WM;
    // An XCD has an eighth of the workgroups (XcdShare), token block after token block with all their channel blocks, so that its L2
    // fetches those tokens once (the weights, which every XCD reads whole, are the smaller operand). All five stage kernels deal the
    // tokens that way: a stage finds in its own L2 what the one before it wrote. Whole layers, blocks in turn and in eighths: 41.4 -> 39.4
    // us at 8 x 384 tokens of 1280 channels, 34.1 -> 33.4 at 2 x 1024 of 1280 (20 heads), 35.8 -> 34.7 at 2 x 2304 of 768, 38.7 -> 36.9 at
    // 4 x 1000 of 960, 24.6 -> 22.9 at 3 x 711 of 640, 77.3 -> 76.6 at 8 x 1024 of 1280 (where the float32 O no longer fits the L2s). With
    // whole token blocks to an XCD, 25 blocks of 20 workgroups (2 x 784 tokens) were a third round for three XCDs: to_q and to_out 8.6 ->
    // 6.9 and 9.0 -> 6.8 us, 35.6 -> 32 the layer; where the blocks divide by 8 nothing changes.
    // (The arguments that everything waits for are asked for together, not one part behind the branch: 0.1 us.)
    asm volatile("" ::"s"(a.A), "s"(a.W), "s"(a.sa), "s"(a.sw), "s"(a.pack_off), "s"(a.tiles), "s"(a.KC), "s"(a.H), "s"(a.inv_nx));
    const int item = XcdShare::item(blockIdx.x, (unsigned)(a.MX * a.NX));
    if (item < 0) return;
    const int mb = a.inv_nx ? (int)__umulhi((unsigned)item, a.inv_nx) : (int)((unsigned)item / (unsigned)a.NX), nb = item - mb * a.NX;
    const int t0 = mb * MB, g0 = nb * NB, ng = a.H * a.tph;  // first token tile, first weight block, weight blocks
    const int KC = a.KC, C = a.C, d = a.d, tph = TPH ? TPH : a.tph;
    auto head_of = [&](int g) -> int { return TPH ? g / TP : a.inv_tph ? (int)__umulhi((unsigned)g, a.inv_tph) : g; };
    // this wavefront's blocks of a stage: a base in scalar registers, the lane's offset, the bytes of a K step
    const int8_t* base[NLD];
    int size[NLD], step[NLD], voff[NLD], late[NLD];
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
        const int blk = wave + WAVES * u < BLK ? wave + WAVES * u : BLK - 1;
        const bool tok = blk < MB, block = tok || PACKED;  // (a block is 1 KiB per K step)
        const int t = t0 + blk < a.tiles ? t0 + blk : a.tiles - 1, g = g0 + blk - MB < ng ? g0 + blk - MB : ng - 1;
        const int h = head_of(g), row0 = h * d + 16 * (g - h * tph);  // row-major weights: first row (rows past the head: results dropped)
        base[u] = tok ? a.A + (size_t)t * KC * 1024 : PACKED ? a.W + a.pack_off + (size_t)g * KC * 1024 : a.W + (size_t)row0 * C;
        size[u] = block ? KC * 1024 : 16 * C;
        step[u] = block ? 1024 : 64;
        const int lrow = lane >> 2, lseg = (lane & 3) ^ ((lrow >> 1 ^ lrow >> 2) & 3);
        voff[u] = block ? lane * 16 : (row0 + lrow < C ? lrow : C - 1 - row0) * C + 16 * lseg;
        late[u] = !block && (C & 63) && lseg >= 2 ? 32 : 0;  // (C % 64 == 32, last step: codes of the row that meet zero token codes)
    }
    auto load_one = [&](int kc, int s, int u) {
        const int blk = wave + WAVES * u < BLK ? wave + WAVES * u : BLK - 1;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(base[u]), 0, size[u], 0x00020000);
        const int v = WAVES * u + WAVES <= MB ? voff[u] : kc == KC - 1 ? voff[u] - late[u] : voff[u];
        lds_load1k(rs, lds + (s * BLK + blk) * 1024, v | (kc < KC ? 0 : 0x40000000), step[u] * kc);  // (steps past the last: no access)
    };
    int32x4_t acc[NW][MW];
#pragma unroll
    for (int j = 0; j < NW; ++j)
#pragma unroll
        for (int i = 0; i < MW; ++i) acc[j][i] = (int32x4_t){0, 0, 0, 0};
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
    const unsigned ld_a = lds0 + wm * MW * 1024 + lane * 16;
    const unsigned ld_w = lds0 + (MB + wn * NW) * 1024 + (PACKED ? lane * 16 : r16 * 64 + ((q ^ ((r16 >> 1 ^ r16 >> 2) & 3)) << 4));
#pragma unroll
    for (int u = 0; u < NLD; ++u) load_one(0, 0, u);
    __builtin_amdgcn_sched_barrier(0);
    // scales (and the bias) for the end, behind the first stage
    float sam[MW];
    float4 w4[NW], b4[TPH ? 1 : NW];
#pragma unroll
    for (int i = 0; i < MW; ++i) {
        const int t = t0 + MW * wm + i;
        sam[i] = a.sa[(t < a.tiles ? t : a.tiles - 1) * 16 + r16];
    }
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const int g = g0 + wn * NW + j < ng ? g0 + wn * NW + j : ng - 1, h = head_of(g), cl = 16 * (g - h * tph) + 4 * q;
        const int c = h * d + (cl < d ? cl : 0);
        w4[j] = *reinterpret_cast<const float4*>(a.sw + c);
        if constexpr (TPH == 0) b4[j] = *reinterpret_cast<const float4*>(a.bias + c);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 1; s < STAGES; ++s)
#pragma unroll
        for (int u = 0; u < NLD; ++u) load_one(s, s, u);
    __builtin_amdgcn_sched_barrier(0);
    int32x4_t xb[2][MW], wa[2][NW];  // operands of the step being multiplied and of the next
    constexpr int NR = MW + NW, NM = MW * NW;
    auto read_one = [&](int set, int s, int r) {
        if (r < MW) xb[set][r] = lds_read16(ld_a + s * (BLK * 1024), 1024 * r);
        else wa[set][r - MW] = lds_read16(ld_w + s * (BLK * 1024), 1024 * (r - MW));
    };
    // (the builtin: the compiler learns from it that the scales are there, and has no wait of its own in front of the loop)
    constexpr int W0 = (STAGES - 1) * NLD;
    __builtin_amdgcn_s_waitcnt((W0 & 15) | 0x0F70 | (W0 >> 4) << 14);
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int r = 0; r < NR; ++r) read_one(0, 0, r);
    int cur = 0;  // stage of step kc
    auto arrived = [&](int set) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < MW; ++i) asm volatile("" : "+v"(xb[set][i]));
#pragma unroll
        for (int j = 0; j < NW; ++j) asm volatile("" : "+v"(wa[set][j]));
    };
    auto step_k = [&](int kc, int set) {
        // this wavefront has its operands of step kc (so it is done with that stage) and its part of stage kc + 1 has arrived;
        // after the barrier that holds for everybody
        arrived(set);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 2) * NLD) : "memory");
        const int nxt = cur + 1 == STAGES ? 0 : cur + 1;
        int kl = kc + STAGES;
        asm("" : "+s"(kl));  // (a scalar to the compiler: no loop over lanes around the loads)
        // products, two reads behind each of the first ones, then the loads evenly behind the others
        constexpr int RPM = (NR + NM - 1) / NM > 2 ? (NR + NM - 1) / NM : 2, M0 = (NR + RPM - 1) / RPM < NM ? (NR + RPM - 1) / RPM : NM - 1;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            acc[m / MW][m % MW] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[set][m / MW], xb[set][m % MW], acc[m / MW][m % MW], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = m * RPM; r < (m + 1) * RPM && r < NR; ++r) read_one(set ^ 1, nxt, r);
#pragma unroll
            for (int u = 0; u < NLD; ++u)
                if (M0 + u * (NM - M0) / NLD == m) load_one(kl, cur, u);
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = nxt;
    };
    // An odd number of steps: the first by itself, in set 0. It and the loop are entered with the reads waited for, and the loop has one
    // way out: where two ways meet, the compiler may copy registers whose data is still on its way.
    arrived(0);
    int kc = 0;
    if (KC & 1) {
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 2) * NLD) : "memory");
#pragma unroll
        for (int m = 0; m < NM; ++m) acc[m / MW][m % MW] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[0][m / MW], xb[0][m % MW], acc[m / MW][m % MW], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < NR; ++r) read_one(0, 1, r);
#pragma unroll
        for (int u = 0; u < NLD; ++u) load_one(STAGES, 0, u);
        arrived(0);
        cur = 1;
        kc = 1;
    }
    for (; kc < KC; kc += 2) {
        step_k(kc, 0);
        step_k(kc + 1, 1);
    }
    arrived(0);  // the last step's reads, which nobody multiplies
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the steps past the end

    if constexpr (TPH > 0) {
        // Qf = float(acc) * (s_h * s_wq); codes and scale per (token, head), in the defined order
        auto value = [&](int i, int j) {  // four channels of block j of the wavefront (zeros past the head)
            const int32x4_t c = acc[j][i];
            const bool valid = 16 * (WPH > 1 ? (wn % WPH) * NW + j : j % TP) + 4 * q < d;
            const float y0 = (float)c[0] * (sam[i] * w4[j].x), y1 = (float)c[1] * (sam[i] * w4[j].y), y2 = (float)c[2] * (sam[i] * w4[j].z),
                        y3 = (float)c[3] * (sam[i] * w4[j].w);
            return make_float4(valid ? y0 : 0.f, valid ? y1 : 0.f, valid ? y2 : 0.f, valid ? y3 : 0.f);
        };
        float amax[MW][HPW];
#pragma unroll
        for (int i = 0; i < MW; ++i)
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) {
                float m = 0.f;
#pragma unroll
                for (int j = 0; j < JH; ++j) {
                    const float4 y = value(i, hh * JH + j);
                    m = fmaxf(m, fmaxf(fmaxf(fabsf(y.x), fabsf(y.y)), fmaxf(fabsf(y.z), fabsf(y.w))));
                }
                amax[i][hh] = quad_allmax(m);
            }
        if constexpr (WPH > 1) {  // the other wavefronts of the head
            float* xm = reinterpret_cast<float*>(lds);  // [token tile][wn][16]
            __syncthreads();
#pragma unroll
            for (int i = 0; i < MW; ++i)
                if (q == 0) xm[((wm * MW + i) * WN + wn) * 16 + r16] = amax[i][0];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < MW; ++i)
#pragma unroll
                for (int p = 0; p < WPH; ++p) amax[i][0] = fmaxf(amax[i][0], xm[((wm * MW + i) * WN + wn / WPH * WPH + p) * 16 + r16]);
        }
        const int j0 = WPH > 1 ? (wn % WPH) * NW : 0;  // first block within the head
#pragma unroll
        for (int i = 0; i < MW; ++i) {
            const int t = t0 + MW * wm + i;
            if (t >= a.tiles) continue;
#pragma unroll
            for (int hh = 0; hh < HPW; ++hh) {
                const int h = (g0 + wn * NW) / TP + hh;
                if (h >= a.H) continue;
                const bool zero = amax[i][hh] == 0.f;
                const float safe = zero ? 1.f : amax[i][hh], cq = quant_mult(a.qmax, safe), sq = zero ? 1.f : div_grid(amax[i][hh], a.qmax);
                const size_t th = (size_t)t * a.H + h;
                if (q == 0 && j0 == 0) a.s_q[th * 16 + r16] = sq;
                unsigned pk[JH];
                quant4_group<JH>(pk, [&](int j) { return value(i, hh * JH + j); }, [&](int) { return QuantRow{1.f, cq, safe}; }, a.qmax);
                unsigned* qp = a.q_op + (th * TP + j0) * 64;  // (j0: whole units)
#pragma unroll
                for (int j = 0; j < JH; ++j) qp[QPlace<TP>::at(j, lane)] = pk[j];
                if (a.tap_code || a.tap_scale) {
                    const int b = (a.tile0 + t) / a.NT, n = (a.tile0 + t - b * a.NT) * 16 + r16;
                    const size_t tok = (size_t)b * a.N + n;
                    if (a.tap_scale && q == 0 && j0 == 0 && n < a.N) a.tap_scale[tok * a.H + h] = sq;
#pragma unroll
                    for (int j = 0; j < JH; ++j)
                        if (a.tap_code && n < a.N && 16 * (j0 + j) + 4 * q < d) *reinterpret_cast<unsigned*>(a.tap_code + tok * C + h * d + 16 * (j0 + j) + 4 * q) = pk[j];
                }
            }
        }
    } else {
        // fp16(float(acc) * (s_o * s_wo) + bias); four blocks are exchanged between the quarters of the wavefront, which
        // leaves a lane with the 16 channels of one block: 32 contiguous bytes (blocks that do not make four: 8)
#pragma unroll
        for (int i = 0; i < MW; ++i) {
            const int t = t0 + MW * wm + i;
            if (t >= a.tiles) continue;
            const int b = (a.tile0 + t) / a.NT, n = (a.tile0 + t - b * a.NT) * 16 + r16;
            const size_t tok = (size_t)b * a.N + n;
#pragma unroll
            for (int j = 0; j < NW; j += 4) {
                constexpr int U4 = 4;
                const int gw = g0 + wn * NW + j;
                unsigned p0[U4], p1[U4];
#pragma unroll
                for (int u = 0; u < U4; ++u) {
                    const int k = j + u < NW ? j + u : NW - 1;
                    // (converted by the intrinsic: a plain cast may be merged with the addition into one rounding)
                    const __half2 y01 = __floats2half2_rn((float)acc[k][i][0] * (sam[i] * w4[k].x) + b4[k].x, (float)acc[k][i][1] * (sam[i] * w4[k].y) + b4[k].y);
                    const __half2 y23 = __floats2half2_rn((float)acc[k][i][2] * (sam[i] * w4[k].z) + b4[k].z, (float)acc[k][i][3] * (sam[i] * w4[k].w) + b4[k].w);
                    p0[u] = *reinterpret_cast<const unsigned*>(&y01);
                    p1[u] = *reinterpret_cast<const unsigned*>(&y23);
                }
                if (j + 4 <= NW) {
                    quad_transpose(p0);
                    quad_transpose(p1);
                    const int g = gw + q, h = head_of(g), cl = 16 * (g - h * tph);
                    if (g < ng && n < a.N) {
                        uint4* o = reinterpret_cast<uint4*>(a.out + tok * C + h * d + cl);  // (d % 8 == 0: 16-byte aligned)
                        o[0] = make_uint4(p0[0], p1[0], p0[1], p1[1]);
                        if (cl + 16 <= d) o[1] = make_uint4(p0[2], p1[2], p0[3], p1[3]);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < NW - j; ++u) {
                        const int g = gw + u, h = head_of(g), cl = 16 * (g - h * tph) + 4 * q;
                        if (g < ng && n < a.N && cl < d) *reinterpret_cast<uint2*>(a.out + tok * C + h * d + cl) = make_uint2(p0[u], p1[u]);
                    }
                }
            }
        }
    }
}

template <bool PACKED, int MW, int NW, int WM, int WN, int TPH>
static hipError_t launch_gemm_op_cfg(GemmOpArgs a, hipStream_t st) {
    a.NX = (a.H * a.tph + NW * WN - 1) / (NW * WN);
    a.MX = (a.tiles + MW * WM - 1) / (MW * WM);
    if ((long)a.MX * a.NX > XcdShare::MOST) return hipErrorInvalidValue;
    const unsigned items = (unsigned)(a.MX * a.NX), grid = XcdShare::grid(items);
    a.inv_nx = inverse32(a.NX, items);
    a.inv_tph = inverse32(a.tph, (unsigned long long)a.H * a.tph + 64);
    hipLaunchKernelGGL((gemm_op_kernel<MW, NW, WM, WN, TPH, 4, PACKED>), dim3(grid), dim3(64 * WM * WN), 0, st, a);
    return hipGetLastError();
}

// Which tile: per K step a compute unit's matrix cores take 4 clocks for a product of 16 x 16 x 64 (four of them, 16 each) and its path
// from L2 16 for a KiB; a workgroup that has the unit to itself pays about 60 more (barrier, first reads). The tile whose busiest unit is
// through first is taken (XcdShare: an eighth of the workgroups on the 32 units of an XCD). Measured at 2048 tokens of 1280 channels (640, 220, 256 and 160 workgroups of 64 x 64, 96 x 128, 128 x 80 and
// 128 x 128): to_q 8.2, 7.8, -, 8.5 us, to_out 8.6, 7.8, 7.6, 8.3; at 3072, heads of 160: to_q 11.1, 9.5 (96 x 160), 10.5 (128 x 160),
// to_out 10.7, 10.7, 10.6, 8.8; at 768: to_q 6.6 (32 x 160), 9.0, 9.8, to_out 6.4, 7.4, 7.2, 7.9; at 4608 of 768: to_q 8.3, 8.8, -, 7.4.
static inline int tile_cost(const GemmOpArgs& a, int mb, int nb) {
    const long groups = (long)((a.tiles + mb - 1) / mb) * ((a.H * a.tph + nb - 1) / nb), rounds = (groups + 255) / 256;
    const int step = 4 * mb * nb > 16 * (mb + nb) ? 4 * mb * nb : 16 * (mb + nb);
    return rounds > 1 ? (int)(rounds < 100000 ? rounds : 100000) * step : step + 60;
}

// 64 x 64 (tokens x channels) or 128 x 128
template <bool PACKED, int TPH>
static hipError_t launch_gemm_op(const GemmOpArgs& a, hipStream_t st) {
    if (tile_cost(a, 4, 4) <= tile_cost(a, 8, 8)) return launch_gemm_op_cfg<PACKED, 2, 2, 2, 2, TPH>(a, st);
    return launch_gemm_op_cfg<PACKED, 2, 4, 4, 2, TPH>(a, st);
}

// one head of 96, 128 or 160 channels per block, two wavefronts for it: 32 or 128 tokens
template <bool PACKED, int TPH>
static hipError_t launch_gemm_op_wide(const GemmOpArgs& a, hipStream_t st) {
    if (tile_cost(a, 2, TPH) <= tile_cost(a, 8, TPH)) return launch_gemm_op_cfg<PACKED, 1, TPH / 2, 2, 2, TPH>(a, st);
    return launch_gemm_op_cfg<PACKED, 2, TPH / 2, 4, 2, TPH>(a, st);
}

// of 112 or 144 channels: a wavefront for a head, 64 or 128 tokens
template <bool PACKED, int TPH>
static hipError_t launch_gemm_op_odd(const GemmOpArgs& a, hipStream_t st) {
    if (tile_cost(a, 4, TPH) <= tile_cost(a, 8, TPH)) return launch_gemm_op_cfg<PACKED, 1, TPH, 4, 1, TPH>(a, st);
    return launch_gemm_op_cfg<PACKED, 2, TPH, 4, 1, TPH>(a, st);
}

// to_q: heads of tph blocks
template <bool PACKED>
static hipError_t launch_to_q_tiles(const GemmOpArgs& a, hipStream_t st) {
    switch (a.tph) {
        case 1: return launch_gemm_op<PACKED, 1>(a, st);
        case 2: return launch_gemm_op<PACKED, 2>(a, st);
        case 3:  // 64 x 96 or 128 x 96
            if (tile_cost(a, 4, 6) <= tile_cost(a, 8, 6)) return launch_gemm_op_cfg<PACKED, 2, 3, 2, 2, 3>(a, st);
            return launch_gemm_op_cfg<PACKED, 2, 3, 4, 2, 3>(a, st);
        case 4:
            if (tile_cost(a, 6, 8) < tile_cost(a, 4, 4) && tile_cost(a, 6, 8) < tile_cost(a, 8, 8)) return launch_gemm_op_cfg<PACKED, 3, 2, 2, 4, 4>(a, st);
            return launch_gemm_op<PACKED, 4>(a, st);
        case 5:  // 64 x 80 or 128 x 160
            if (tile_cost(a, 4, 5) <= tile_cost(a, 8, 10)) return launch_gemm_op_cfg<PACKED, 1, 5, 4, 1, 5>(a, st);
            return launch_gemm_op_cfg<PACKED, 2, 5, 4, 2, 5>(a, st);
        case 6: return launch_gemm_op_wide<PACKED, 6>(a, st);
        case 7: return launch_gemm_op_odd<PACKED, 7>(a, st);
        case 8: return launch_gemm_op_wide<PACKED, 8>(a, st);
        case 9: return launch_gemm_op_odd<PACKED, 9>(a, st);
        case 10:
            if (tile_cost(a, 6, 10) < tile_cost(a, 2, 10) && tile_cost(a, 6, 10) < tile_cost(a, 8, 10)) return launch_gemm_op_cfg<PACKED, 3, 5, 2, 2, 10>(a, st);
            return launch_gemm_op_wide<PACKED, 10>(a, st);
        default: return hipErrorInvalidValue;
    }
}

// taq_gemm_rows.hip: launch_to_q_tiles of row-major weights; taq_gemm_out.hip: to_out
hipError_t launch_to_q_rows(const GemmOpArgs& a, hipStream_t st);
hipError_t launch_to_out_tiles(const GemmOpArgs& a, bool packed, hipStream_t st);

}  // namespace taq
