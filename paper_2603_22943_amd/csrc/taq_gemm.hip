// int8 x int8 -> int32 GEMM on the gfx950 matrix cores with fused dequantisation.
//
// Serves the W8A8 contractions to_q and to_out of the TAQ block outside the single-kernel and head-group shapes:
// acc[m][n] = sum_k A[m][k] * W[n][k], both operands K-contiguous, result = float(acc) * (sa[m] * sw[n]) (+ bias[n]), in that
// order of float32 operations. gemm_op_kernel is the one of the quantized block; the two in front of it, on row-major operands
// with float32 results, run where a stage beside them is left unquantized (bits_q or bits_prob = 16 with bits_proj = 8).
#include "taq_device.h"

namespace taq {

typedef int int32x16_t __attribute__((ext_vector_type(16)));

// Workgroup = 4 wavefronts in a 2x2 arrangement, each owning one 32x32 accumulator tile
// (V_MFMA_I32_32X32X32_I8: a lane supplies 16 consecutive k of row/column lane%32, the
// upper half-wave the next 16). Operands are read straight from global memory: a lane's
// 16 bytes are contiguous and both operands stay resident in L2 at these sizes.
// K % 32 == 0. Rows beyond M / N are clamped on load and masked on store.
__global__ __launch_bounds__(256) void gemm_i8_kernel(const int8_t* __restrict__ A, const float* __restrict__ sa,
                                                      const int8_t* __restrict__ W, const float* __restrict__ sw,
                                                      const float* __restrict__ bias, int M, int N, int K,
                                                      float* __restrict__ out_f32, __half* __restrict__ out_f16,
                                                      int ldo) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 31, half = lane >> 5;
    const int m0 = blockIdx.x * 64 + (wave & 1) * 32;
    const int n0 = blockIdx.y * 64 + (wave >> 1) * 32;
    if (m0 >= M || n0 >= N) return;
    const int am = min(m0 + r, M - 1);
    const int wn = min(n0 + r, N - 1);
    const int8_t* ap = A + (size_t)am * K + 16 * half;
    const int8_t* wp = W + (size_t)wn * K + 16 * half;
    int32x16_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0;
#pragma unroll 4
    for (int k = 0; k < K; k += 32) {
        int32x4_t a = *reinterpret_cast<const int32x4_t*>(ap + k);
        int32x4_t b = *reinterpret_cast<const int32x4_t*>(wp + k);
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc, 0, 0, 0);
    }
    const int col = n0 + r;
    if (col >= N) return;
    const float swc = sw[col];
    const float bc = bias ? bias[col] : 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = m0 + 8 * (i >> 2) + 4 * half + (i & 3);
        if (row < M) {
            const float sc = sa[row] * swc;
            const float v = (float)acc[i] * sc;
            if (out_f32) out_f32[(size_t)row * ldo + col] = v;
            if (out_f16) out_f16[(size_t)row * ldo + col] = __float2half_rn(v + bc);
        }
    }
}

// ------------------------------------------------------------------------------------------
// LDS-staged kernel for K % 64 == 0: a workgroup of four wavefronts owns 128 rows of A
// (image tokens) x 80 rows of W (output channels: 320, 640 and 1280 are multiples of 80, and 2048 x 1280 outputs are then
// exactly 256 workgroups, one per compute unit). Per K step of 64 the 13 operand blocks (16 rows x 64 codes = 1 KiB
// each) go through LDS, row-major with the 16-byte segments of a row swizzled (below). Software pipeline, one barrier
// per K step, three LDS stages, four register sets for loads in flight: while the ten MFMAs of step k run on one operand
// register set, step k + 1 is read from LDS into the other, steps k + 2 and k + 3 move from registers to LDS and the
// global loads of up to four later steps are outstanding.
// (Direct global->LDS loads are not used here: the compiler waits for every outstanding one before any LDS read that it knows
// of, which would serialise the stages.)
// The product is formed transposed (W rows as the A operand, tokens as the B operand), so that a lane ends up with four
// consecutive output channels of one token: 16-byte float32 / 8-byte fp16 stores.
// ------------------------------------------------------------------------------------------
template <int MB, int NB, int RD>
__global__ __launch_bounds__(256) void gemm_i8_lds_kernel(const int8_t* __restrict__ A, const float* __restrict__ sa,
                                                          const int8_t* __restrict__ W, const float* __restrict__ sw,
                                                          const float* __restrict__ bias, int M, int N, int K,
                                                          float* __restrict__ out_f32, __half* __restrict__ out_f16, int ldo) {
    constexpr int BLK = MB + NB, STAGES = 3, MW = MB / 4;  // blocks per stage; token tiles per wavefront
    constexpr int NLD = (BLK + 3) / 4;                     // loads per wavefront and stage (the last may be idle)
    static_assert(MB % 4 == 0, "four wavefronts share the token tiles");
    __shared__ __align__(16) unsigned char lds[STAGES * BLK * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int m0 = blockIdx.x * (16 * MB), n0 = blockIdx.y * (16 * NB);
    const int KC = K >> 6;
    // global loads: four consecutive lanes fetch the 64 contiguous bytes of one row; MFMA operands: lane (r16, q) holds
    // codes 16q .. 16q+15 of row r16. Segment g of row r sits at r * 64 + (g ^ f(r)) * 16 inside its block, with
    // f(r) = (r >> 1 ^ r >> 2) & 3: the wave-wide 16-byte stores stay contiguous, and the 16-byte operand reads of any
    // eight consecutive lanes fall into eight different 16-byte columns of a 128-byte bank row (of any sixteen lanes:
    // sixteen columns of a 256-byte row).
    const int lrow = lane >> 2, lseg = lane & 3;
    const int st_off = lrow * 64 + ((lseg ^ ((lrow >> 1 ^ lrow >> 2) & 3)) << 4);
    const int ld_off = r16 * 64 + ((q ^ ((r16 >> 1 ^ r16 >> 2) & 3)) << 4);
    // this wavefront's loads of a stage: blocks wave, wave + 4, ... (token blocks first, then weight blocks)
    const int8_t* src[NLD];
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
        const int blk = wave + 4 * u < BLK ? wave + 4 * u : BLK - 1;  // (an idle slot re-reads the last block and drops it)
        const int8_t* base = A;
        int row = 0;
        if (blk < MB) {
            row = m0 + 16 * blk + lrow;
            row = row < M ? row : M - 1;
        } else {
            base = W;
            row = n0 + 16 * (blk - MB) + lrow;
            row = row < N ? row : N - 1;
        }
        src[u] = base + (size_t)row * K + 16 * lseg;
    }
    int32x4_t g[RD][NLD];  // stages on their way from global memory to LDS
    // (No step of the pipeline is conditional: a load past the last stage re-reads the last stage, and what the steps
    // past the end store to and read from LDS is never multiplied. With loads under a condition the compiler's wait
    // counts assume the fewest outstanding loads, which makes every wait a wait for the newest load.)
    auto load_stage = [&](int kc, int slot) {
        const int off = 64 * (kc < KC ? kc : KC - 1);
#pragma unroll
        for (int u = 0; u < NLD; ++u) g[slot][u] = *reinterpret_cast<const int32x4_t*>(src[u] + off);
    };
    auto store_stage = [&](int kc, int slot) {
        unsigned char* dst = lds + (kc % STAGES) * (BLK * 1024) + st_off;
#pragma unroll
        for (int u = 0; u < NLD; ++u)
            if (4 * u + 3 < BLK || wave + 4 * u < BLK) *reinterpret_cast<int32x4_t*>(dst + (wave + 4 * u) * 1024) = g[slot][u];
    };
    int32x4_t acc[NB][MW];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MW; ++i) acc[j][i] = (int32x4_t){0, 0, 0, 0};
    int32x4_t wa[2][NB], xb[2][MW];
    auto read_ops = [&](int kc, int set) {
        const unsigned char* st = lds + (kc % STAGES) * (BLK * 1024) + ld_off;
#pragma unroll
        for (int i = 0; i < MW; ++i) xb[set][i] = *reinterpret_cast<const int32x4_t*>(st + (MW * wave + i) * 1024);
#pragma unroll
        for (int j = 0; j < NB; ++j) wa[set][j] = *reinterpret_cast<const int32x4_t*>(st + (MB + j) * 1024);
    };
    // prologue: stages 0 and 1 in LDS, stages 2 .. 5 in flight, operands of step 0 in registers
    static_assert(RD == 4, "four register sets: the main loop is unrolled four times");
    load_stage(0, 0);
    load_stage(1, 1);
    store_stage(0, 0);
    store_stage(1, 1);
    load_stage(2, 2);
    load_stage(3, 3);
    load_stage(4, 0);
    load_stage(5, 1);
    __syncthreads();
    read_ops(0, 0);
    auto mfmas = [&](int set) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int i = 0; i < MW; ++i) acc[j][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[set][j], xb[set][i], acc[j][i], 0, 0, 0);
    };
    // Steps come in pairs. The even step kc moves stages kc + 2 and kc + 3 from registers to LDS and issues the loads of
    // stages kc + 6 and kc + 7 back to back: the two are the halves of the same 128-byte lines, so the second is served
    // by the line the first brought in. At the barrier of step kc every wavefront is through with reading stage kc
    // (buffer kc % 3, which stage kc + 3 overwrites) and stage kc - 1 (which stage kc + 2 overwrites).
    auto even_step = [&](int kc, int slot) {  // slot = (kc + 2) % 4
        __syncthreads();
        read_ops(kc + 1, 1);
        store_stage(kc + 2, slot);
        store_stage(kc + 3, slot + 1);
        load_stage(kc + 6, slot);
        load_stage(kc + 7, slot + 1);
        mfmas(0);
    };
    auto odd_step = [&](int kc) {
        __syncthreads();
        read_ops(kc + 1, 0);
        mfmas(1);
    };
    int kc = 0;
    for (; kc + 4 <= KC; kc += 4) {
        even_step(kc, 2);
        odd_step(kc + 1);
        even_step(kc + 2, 0);
        odd_step(kc + 3);
    }
    if (kc < KC) even_step(kc, 2);
    if (kc + 1 < KC) odd_step(kc + 1);
    if (kc + 2 < KC) even_step(kc + 2, 0);
    // epilogue: result = float(acc) * (sa[m] * sw[n]) (+ bias[n]). The MFMA leaves lane (r16, q) with channels
    // 16j + 4q .. + 3 of token r16 of its tile; a lane exchange hands lane l the four channels 16j + 4 (l & 3) .. of
    // token l >> 2, so that four consecutive lanes store 64 (fp16: 32) contiguous bytes.
    const int from = ((lane >> 2) + 16 * (lane & 3)) << 2;
#pragma unroll
    for (int i = 0; i < MW; ++i) {
        const int m = m0 + 16 * (MW * wave + i) + lrow;
        const float sam = sa[m < M ? m : M - 1];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            int c[4];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) c[e2] = __builtin_amdgcn_ds_bpermute(from, acc[j][i][e2]);
            const int n = n0 + 16 * j + 4 * lseg;
            if (m >= M || n >= N) continue;  // (N % 4 == 0: a lane's four channels are inside or outside together)
            const float4 w4 = *reinterpret_cast<const float4*>(sw + n);
            const float v0 = (float)c[0] * (sam * w4.x), v1 = (float)c[1] * (sam * w4.y);
            const float v2 = (float)c[2] * (sam * w4.z), v3 = (float)c[3] * (sam * w4.w);
            if (out_f32) *reinterpret_cast<float4*>(out_f32 + (size_t)m * ldo + n) = make_float4(v0, v1, v2, v3);
            if (out_f16) {
                float4 b4 = make_float4(0.f, 0.f, 0.f, 0.f);
                if (bias) b4 = *reinterpret_cast<const float4*>(bias + n);
                __half2 h01 = __floats2half2_rn(v0 + b4.x, v1 + b4.y), h23 = __floats2half2_rn(v2 + b4.z, v3 + b4.w);
                uint2 o;
                o.x = *reinterpret_cast<unsigned*>(&h01);
                o.y = *reinterpret_cast<unsigned*>(&h23);
                *reinterpret_cast<uint2*>(out_f16 + (size_t)m * ldo + n) = o;
            }
        }
    }
}

hipError_t launch_gemm_i8(const int8_t* A, const float* sa, const int8_t* W, const float* sw, const float* bias,
                          int M, int N, int K, float* out_f32, __half* out_f16, int ldo, hipStream_t st) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (K % 64 == 0 && N % 4 == 0 && ldo % 4 == 0) {
        // While 128-token tiles would give every compute unit at most one workgroup, 64-token tiles (two workgroups per
        // unit, each hiding the other's waits) are faster: 7.8 -> 7.0 us at (8192, 320), 11.7 -> 11.2 us at (2048, 1280);
        // with more tiles than that the larger tile's fewer weight reads win (12.1 vs 12.9 us at (8192, 640)).
        const long tiles128 = (long)((M + 127) / 128) * ((N + 79) / 80);
        if (tiles128 <= 256) {
            dim3 grid((M + 63) / 64, (N + 79) / 80);
            hipLaunchKernelGGL((gemm_i8_lds_kernel<4, 5, 4>), grid, dim3(256), 0, st, A, sa, W, sw, bias, M, N, K, out_f32, out_f16, ldo);
        } else {
            dim3 grid((M + 127) / 128, (N + 79) / 80);
            hipLaunchKernelGGL((gemm_i8_lds_kernel<8, 5, 4>), grid, dim3(256), 0, st, A, sa, W, sw, bias, M, N, K, out_f32, out_f16, ldo);
        }
        return hipGetLastError();
    }
    dim3 grid((M + 63) / 64, (N + 63) / 64);  // (M, which may be large, along x)
    hipLaunchKernelGGL(gemm_i8_kernel, grid, dim3(256), 0, st, A, sa, W, sw, bias, M, N, K, out_f32, out_f16, ldo);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// to_q and to_out of the kernel-per-stage path, on operands in MFMA operand order: a 16 x 64 block is one contiguous KiB, in
// memory and in LDS (conflict-free as it is). Tokens come that way from the quantizer kernels, weights from
// taq_pack_weight; of row-major weights four lanes fetch the 64 bytes of a row, segments swizzled as in
// gemm_i8_lds_kernel. Weight blocks are counted per head (tph = ceil(d/16) blocks each, the last one partly filled), so
// that a wavefront of to_q holds whole heads and quantizes Q~ on its accumulators: what leaves the kernel is one byte per
// channel instead of a float32 for a quantizer kernel to read again, in the registers' own order, which is the order in
// which the attention's score operand wants it.
//
// WM x WN wavefronts of MW token tiles x NW channel blocks each; TPH > 0: to_q with heads of TPH blocks (NW a multiple);
// TPH = 0: to_out. Blocks go straight from global memory into LDS (no registers in between, so that several workgroups share
// a compute unit and one's waits are filled by another's MFMAs), STAGES K steps ahead; the operands of the next step are read
// from LDS while the current one is multiplied; one barrier per step. The LDS reads and the waits are written by hand: for
// reads that it knows of, the compiler waits for every outstanding direct-to-LDS load, which would serialise the stages. A
// wavefront's loads per stage are a constant (blocks past the last are fetched again, K steps past the end re-fetch the last
// one into a buffer nobody reads any more), so "stage kc + 1 has arrived" is "at most (STAGES - 2) * NLD loads outstanding".
// Bound by what a compute unit receives per K step, (WM MW + WN NW) KiB. With register staging this took 15.3 us at
// M = 2048, C = 1280 and 41.9 us at M = 8192 (compiler-made register shuffles and one workgroup per unit), 10 and 22 us now.
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
    int KC, C, H, d, tph, packed, MX, NX;
    size_t pack_off;
};

// The compiler takes the result of this read to be there at once; it knows nothing of the data still on its way into these
// registers. Rule: on every path the destinations pass through `arrived` below (a wait, then an empty asm that takes and gives
// back each of them) before they are used and before the kernel goes on without them. Until then they are alive to the
// compiler, so it places nothing else there; a read whose result nobody takes would leave it free to, with only timing to keep
// the late data from overwriting what it placed. tests/test_waits.py checks the generated code of every kernel.
template <int OFF>
__device__ __forceinline__ int32x4_t lds_read16(unsigned addr) {
    int32x4_t r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
    return r;
}
// NR blocks of 1 KiB from addr on, one operand register each.
template <int NR>
__device__ __forceinline__ void lds_read_blocks(int32x4_t (&r)[NR], unsigned addr) {
    static_assert(NR <= 10, "reads are listed one by one");
#define TAQ_RD(J) if constexpr (NR > J) r[NR > J ? J : 0] = lds_read16<1024 * J>(addr);
    TAQ_RD(0) TAQ_RD(1) TAQ_RD(2) TAQ_RD(3) TAQ_RD(4) TAQ_RD(5) TAQ_RD(6) TAQ_RD(7) TAQ_RD(8) TAQ_RD(9)
#undef TAQ_RD
}

template <int MW, int NW, int WM, int WN, int TPH, int STAGES>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2)))
void gemm_op_kernel(GemmOpArgs a) {
    constexpr int WAVES = WM * WN, MB = MW * WM, NB = NW * WN, BLK = MB + NB, NLD = (BLK + WAVES - 1) / WAVES;
    static_assert(NLD * (STAGES - 1) < 64, "vmcnt");
    static_assert(TPH == 0 || NW % (TPH ? TPH : 1) == 0, "whole heads per wavefront");
    __shared__ __align__(16) unsigned char lds[STAGES * BLK * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int wm = wave % WM, wn = wave / WM;
    // Workgroups are dealt to the 8 XCDs in turn. All channel blocks of a token block go to one XCD, one after the other, so
    // that its L2 fetches those tokens once (the weights, which every XCD reads whole, are the smaller operand).
    const int xcd = (int)blockIdx.x & 7, slot = (int)blockIdx.x >> 3;
    const int mb = (slot / a.NX) * 8 + xcd, nb = slot % a.NX;
    if (mb >= a.MX) return;
    const int t0 = mb * MB, g0 = nb * NB, ng = a.H * a.tph;  // first token tile, first weight block, weight blocks
    const int KC = a.KC, C = a.C, d = a.d, tph = TPH ? TPH : a.tph;
    const int8_t* src[NLD];
    int step[NLD], last[NLD];
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
        const int blk = wave + WAVES * u < BLK ? wave + WAVES * u : BLK - 1;
        if (blk < MB) {
            const int t = t0 + blk < a.tiles ? t0 + blk : a.tiles - 1;
            src[u] = a.A + (size_t)t * KC * 1024 + lane * 16;
            step[u] = 1024;
            last[u] = (KC - 1) * 1024;
        } else {
            const int g = g0 + blk - MB < ng ? g0 + blk - MB : ng - 1;
            if (a.packed) {
                src[u] = a.W + a.pack_off + (size_t)g * KC * 1024 + lane * 16;
                step[u] = 1024;
                last[u] = (KC - 1) * 1024;
            } else {
                const int lrow = lane >> 2, lseg = (lane & 3) ^ ((lrow >> 1 ^ lrow >> 2) & 3);
                const int h = g / tph, row = h * d + 16 * (g - h * tph) + lrow;  // (rows past the head: results dropped)
                src[u] = a.W + (size_t)(row < C ? row : C - 1) * C + 16 * lseg;
                step[u] = 64;
                last[u] = C - 16 - 16 * lseg;  // (C % 64 == 32: past the end the row's last codes, which meet zero token codes)
            }
        }
    }
    auto load_stage = [&](int kc, int s) {
#pragma unroll
        for (int u = 0; u < NLD; ++u) {
            const int off = kc * step[u];
            const int blk = wave + WAVES * u < BLK ? wave + WAVES * u : BLK - 1;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[u] + (off < last[u] ? off : last[u])),
                                             (__attribute__((address_space(3))) void*)(lds + (s * BLK + blk) * 1024), 16, 0, 0);
        }
    };
    int32x4_t acc[NW][MW];
#pragma unroll
    for (int j = 0; j < NW; ++j)
#pragma unroll
        for (int i = 0; i < MW; ++i) acc[j][i] = (int32x4_t){0, 0, 0, 0};
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
    const unsigned ld_a = lds0 + wm * MW * 1024 + lane * 16;
    const unsigned ld_w = lds0 + (MB + wn * NW) * 1024 + (a.packed ? lane * 16 : r16 * 64 + ((q ^ ((r16 >> 1 ^ r16 >> 2) & 3)) << 4));
#pragma unroll
    for (int s = 0; s < STAGES; ++s) load_stage(s, s);
    int32x4_t xb[2][MW], wa[2][NW];  // operands of the step being multiplied and of the next
    auto read_ops = [&](int set, int s) {
        lds_read_blocks<MW>(xb[set], ld_a + s * (BLK * 1024));
        lds_read_blocks<NW>(wa[set], ld_w + s * (BLK * 1024));
    };
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 1) * NLD) : "memory");
    read_ops(0, 0);
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
        read_ops(set ^ 1, nxt);
        load_stage(kc + STAGES, cur);
        cur = nxt;
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int i = 0; i < MW; ++i) acc[j][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa[set][j], xb[set][i], acc[j][i], 0, 0, 0);
    };
    // (left from the middle, not by a guarded second half: no path leads from a half whose reads are in flight to its own start)
    for (int kc = 0;;) {
        step_k(kc, 0);
        if (++kc >= KC) break;
        step_k(kc, 1);
        if (++kc >= KC) break;
    }
    arrived(0);  // the last step's reads, which nobody multiplies, are in one set or the other
    arrived(1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the re-fetched steps past the end

#pragma unroll
    for (int i = 0; i < MW; ++i) {
        const int t = t0 + MW * wm + i;
        if (t >= a.tiles) continue;
        const int b = (a.tile0 + t) / a.NT, n = (a.tile0 + t - b * a.NT) * 16 + r16;
        const size_t tok = (size_t)b * a.N + n;
        const float sam = a.sa[t * 16 + r16];
        if constexpr (TPH > 0) {
            // Qf = float(acc) * (s_h * s_wq); codes and scale per (token, head), in the defined order
#pragma unroll
            for (int hh = 0; hh < NW / (TPH ? TPH : 1); ++hh) {
                const int h = (g0 + wn * NW) / TPH + hh;
                if (h >= a.H) continue;
                float v[TPH ? TPH : 1][4];
                float amax = 0.f;
#pragma unroll
                for (int j = 0; j < TPH; ++j) {
                    const int cl = 16 * j + 4 * q;
                    const bool valid = cl < d;
                    const float4 w4 = *reinterpret_cast<const float4*>(a.sw + h * d + (valid ? cl : 0));
                    const float wv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float y = (float)acc[hh * TPH + j][i][e] * (sam * wv[e]);
                        v[j][e] = valid ? y : 0.f;
                        amax = fmaxf(amax, fabsf(v[j][e]));
                    }
                }
                amax = quad_allmax(amax);
                const bool zero = amax == 0.f;
                const float safe = zero ? 1.f : amax, cq = quant_mult(a.qmax, safe), sq = zero ? 1.f : amax / a.qmax;
                const size_t th = (size_t)t * a.H + h;
                if (q == 0) a.s_q[th * 16 + r16] = sq;
                if (a.tap_scale && q == 0 && n < a.N) a.tap_scale[tok * a.H + h] = sq;
                unsigned pk[TPH ? TPH : 1];
                quant4_group<TPH ? TPH : 1>(pk, [&](int j) { return make_float4(v[j][0], v[j][1], v[j][2], v[j][3]); }, [&](int) { return QuantRow{1.f, cq, safe}; }, a.qmax);
#pragma unroll
                for (int j = 0; j < TPH; ++j) {
                    a.q_op[(th * TPH + j) * 64 + lane] = pk[j];
                    if (a.tap_code && n < a.N && 16 * j + 4 * q < d) *reinterpret_cast<unsigned*>(a.tap_code + tok * C + h * d + 16 * j + 4 * q) = pk[j];
                }
            }
        } else {
            // fp16(float(acc) * (s_o * s_wo) + bias); four blocks are exchanged between the quarters of the wavefront, which
            // leaves a lane with the 16 channels of one block: 32 contiguous bytes
#pragma unroll
            for (int j = 0; j < NW; j += 4) {
                const int gw = g0 + wn * NW + j;
                unsigned p0[4], p1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int g = gw + u < ng ? gw + u : ng - 1, h = g / tph, cl = 16 * (g - h * tph) + 4 * q;
                    const int c = h * d + (cl < d ? cl : 0);
                    const float4 w4 = *reinterpret_cast<const float4*>(a.sw + c);
                    const float4 b4 = *reinterpret_cast<const float4*>(a.bias + c);
                    // (converted by the intrinsic: a plain cast may be merged with the addition into one rounding)
                    const __half2 y01 = __floats2half2_rn((float)acc[j + u][i][0] * (sam * w4.x) + b4.x, (float)acc[j + u][i][1] * (sam * w4.y) + b4.y);
                    const __half2 y23 = __floats2half2_rn((float)acc[j + u][i][2] * (sam * w4.z) + b4.z, (float)acc[j + u][i][3] * (sam * w4.w) + b4.w);
                    p0[u] = *reinterpret_cast<const unsigned*>(&y01);
                    p1[u] = *reinterpret_cast<const unsigned*>(&y23);
                }
                quad_transpose(p0);
                quad_transpose(p1);
                const int g = gw + q, h = g / tph, cl = 16 * (g - h * tph);
                if (g < ng && n < a.N) {
                    uint4* o = reinterpret_cast<uint4*>(a.out + tok * C + h * d + cl);  // (d % 8 == 0: 16-byte aligned)
                    o[0] = make_uint4(p0[0], p1[0], p0[1], p1[1]);
                    if (cl + 16 <= d) o[1] = make_uint4(p0[2], p1[2], p0[3], p1[3]);
                }
            }
        }
    }
}

template <int MW, int NW, int WM, int WN, int TPH>
static hipError_t launch_gemm_op_cfg(GemmOpArgs a, hipStream_t st) {
    a.NX = (a.H * a.tph + NW * WN - 1) / (NW * WN);
    a.MX = (a.tiles + MW * WM - 1) / (MW * WM);
    hipLaunchKernelGGL((gemm_op_kernel<MW, NW, WM, WN, TPH, 4>), dim3(8 * ((a.MX + 7) / 8) * a.NX), dim3(64 * WM * WN), 0, st, a);
    return hipGetLastError();
}

// Blocks of 64 tokens x 64 channels (four wavefronts over the tokens) while there are at most three per compute unit: the more
// units fetch the weights, the sooner they are there. Above, 128 x 128 with eight wavefronts: half the bytes per product. At
// C = 1280 5.4 and 8.4 us at 64 tokens, 7.1 and 8.9 us at 1024, 9.4 and 9.3 us at 2048, 24.8 and 20.6 us at 8192; at C = 768 the
// lines cross between 3072 and 4608 tokens (576 and 864 blocks), at 640 above 4608 (720), at 320 above 8192 (640). Blocks of
// 64 x 128 lie between the two at most sizes and win nowhere by more than 3 %; 256 tokens or channels are slower everywhere.
template <int NW, int TPH>
static hipError_t launch_gemm_op(const GemmOpArgs& a, hipStream_t st) {
    if ((long)((a.tiles + 3) / 4) * ((a.H * a.tph + NW - 1) / NW) <= 768) return launch_gemm_op_cfg<1, NW, 4, 1, TPH>(a, st);
    return launch_gemm_op_cfg<2, NW, 4, 2, TPH>(a, st);
}

// Heads of 96 channels and more fill a wavefront: one head per block, and 128 tokens take twice the accumulators instead.
template <int TPH>
static hipError_t launch_gemm_op_wide(const GemmOpArgs& a, hipStream_t st) {
    if ((long)((a.tiles + 7) / 8) * a.H <= 256) return launch_gemm_op_cfg<1, TPH, 4, 1, TPH>(a, st);
    return launch_gemm_op_cfg<2, TPH, 4, 1, TPH>(a, st);
}

static GemmOpArgs gemm_op_args(const StageChunk& c, const taq_shape& s, const int8_t* W, const float* sw) {
    GemmOpArgs a = {};
    a.A = c.code;
    a.sa = c.s;
    a.W = W;
    a.sw = sw;
    a.tiles = c.tile1 - c.tile0;
    a.tile0 = c.tile0;
    a.NT = c.NT;
    a.N = s.N;
    a.KC = (s.C + 63) / 64;
    a.C = s.C;
    a.H = s.H;
    a.d = s.C / s.H;
    a.tph = (a.d + 15) / 16;
    a.packed = s.w_layout == 1 && s.C % 64 == 0;
    a.pack_off = weight_pack_offset(s);
    return a;
}

hipError_t launch_to_q_op(const StageChunk& c, const taq_shape& s, const int8_t* Wq, const float* s_wq, const taq_debug* dbg, hipStream_t st) {
    GemmOpArgs a = gemm_op_args(c, s, Wq, s_wq);
    a.q_op = c.q_op;
    a.s_q = c.s_q;
    a.qmax = s.bits_q == 4 ? 7.f : 127.f;
    a.tap_code = dbg ? dbg->q_code : nullptr;
    a.tap_scale = dbg ? dbg->s_Q : nullptr;
    switch (a.tph) {
        case 1: return launch_gemm_op<4, 1>(a, st);
        case 2: return launch_gemm_op<4, 2>(a, st);
        case 3: return launch_gemm_op<3, 3>(a, st);
        case 4: return launch_gemm_op<4, 4>(a, st);
        case 5: return launch_gemm_op<5, 5>(a, st);
        case 6: return launch_gemm_op_wide<6>(a, st);
        case 7: return launch_gemm_op_wide<7>(a, st);
        case 8: return launch_gemm_op_wide<8>(a, st);
        case 9: return launch_gemm_op_wide<9>(a, st);
        case 10: return launch_gemm_op_wide<10>(a, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_to_out_op(const StageChunk& c, const taq_shape& s, const int8_t* Wo, const float* s_wo, const float* bias, __half* out,
                            hipStream_t st) {
    GemmOpArgs a = gemm_op_args(c, s, Wo, s_wo);
    a.bias = bias;
    a.out = out;
    return launch_gemm_op<4, 0>(a, st);
}

}  // namespace taq
