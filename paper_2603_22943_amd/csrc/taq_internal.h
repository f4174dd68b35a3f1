// Internal declarations shared by the libtaq translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "taq.h"

#define TAQ_MAX_T 96        // text tokens the attention core holds in LDS (3 tiles of 32)
#define TAQ_MAX_D 160       // largest head dimension (5 steps of 32)
#define TAQ_MAX_H 64
#define TAQ_MAX_REQ 16       // requests of one grouped launch

namespace taq {

static constexpr size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ceil(2^32 / n), whose product with x has x / n as its high word while x * n < 2^32; 0 (divide) for n = 1 or a larger x
static inline unsigned inverse32(unsigned n, unsigned long long x) {
    return n == 1 || x * n >> 32 ? 0u : (unsigned)(((1ull << 32) + n - 1) / n);
}

// Which of n items of a launch a workgroup has. Workgroups go to the 8 XCDs in turn; every XCD gets an eighth of the items, one after
// the other, and no two XCDs differ by more than one item (whole rows of items to an XCD would leave its 32 compute units up to a round
// of workgroups more than those of the others). tests/test_xcd_share.py counts.
struct XcdShare {
    static constexpr long MOST = 1l << 28;
    static unsigned grid(unsigned n) { return 8 * ((n + 7) / 8); }
    __host__ __device__ static int item(unsigned block, unsigned n) {  // or -1
        const unsigned xcd = block & 7, i = (xcd * n >> 3) + (block >> 3);
        return i < ((xcd + 1) * n >> 3) ? (int)i : -1;
    }
};

// Layout of qkv_packed: fixed by the shape alone, every section 256-byte aligned.
struct KvLayout {
    size_t ntrig;     // i32 [B]        number of protected tokens
    size_t trig_idx;  // i32 [B][T]     token index of protected slot s (first ntrig valid)
    size_t slot_of;   // i32 [B][T]     slot of token t, or -1 if unprotected
    size_t s_k;       // f32 [B][H][T]  0 on protected tokens
    size_t s_v;       // f32 [B][H][T]
    size_t k_code;    // u8  [B][T][Cb] Cb = C (8 bit) | C/2 (4 bit) | 0 (16 bit)
    size_t v_code;
    size_t k16;       // f16 [B][T][C]  protected rows, compacted by slot
    size_t v16;
    size_t v16t;      // f16 [B][C][96] protected V rows transposed (slot along the last axis)
    size_t image;     // [B][image_bytes] operand-ordered K~/V~ image of the attention kernels
    size_t image_bytes;
    size_t total;
    int Cb;
};

// LDS-ready image of the integer part of K~/V~ for one batch element (with bits_kv = 16: no integer rows at all): one
// self-contained block per head, so that the wavefront that owns a head copies and waits for its own
// block only. Offsets are relative to the head block.
struct KvImage {
    int tph;        // 16-channel tiles per head = ceil(d/16)
    int nt16;       // ceil(T/16): score tiles of 16 text tokens
    int ntok;       // 16*nt16: text tokens with padding; length of the per-token arrays below
    int rows_k;     // = ntok: text-token rows of the K part
    int cols_v;     // = ntok: token positions per V^T row (see vt_pos)
    size_t kp;      // i8  [rows_k][tph][4 quarter-lanes][4]  K codes in MFMA operand order (see kp_offset)
    size_t vt;      // u8  [d][cols_v]   V codes (+128) transposed, tokens in accumulator-register order
    size_t s_k;     // f32 [ntok]  per-token K scale of this head, 0 on protected / padding tokens
    size_t s_vp;    // f16 [2][ntok]  s_V * 2^kexp as an fp16 high part [0][t] and the fp16 remainder [1][t]
    size_t bias;    // f32 [ntok]  0 for unprotected tokens, -inf for protected / padding (same in every head)
    size_t oscale;  // f32       2^-kexp / 255
    size_t vpre;    // f32       2^kexp
    size_t head_bytes;  // one head's block, a multiple of 256 bytes
    size_t bytes;   // H * head_bytes
};

// Byte offset, within the K part of a head block, of the 4 codes of text token t, 16-channel tile j, quarter q
// (channels 16*j + 4*q .. +3 of the head). A lane of the score MFMA holds row t, quarter q and needs tiles
// 4*ks .. 4*ks+3 for K step ks. When the head has a multiple of 4 tiles those 16 bytes are laid out contiguously,
// [t][ks][q][tile%4][4], so that the lane reads them with one 16-byte LDS load and the 64 lanes of a wavefront hit
// consecutive 16-byte slots (no bank conflicts; a 64-byte row of [t][tile][q][4] would put 16 rows on 2 bank
// groups). Otherwise [t][tile][q][4].
__host__ __device__ static inline size_t kp_offset(int tph, int t, int j, int q) {
    if ((tph & 3) == 0) return ((((size_t)t * (tph >> 2) + (j >> 2)) * 4 + q) * 4 + (j & 3)) * 4;
    return (((size_t)t * tph + j) * 4 + q) * 4;
}

// Place of text token t in a V^T row of the image. Tokens come in steps of 32 (two score tiles of 16), permuted within
// a step to the accumulator-register order of the score MFMA: token 32*s + 16*a + 4*q + e sits at 32*s + 8*q + 4*a + e,
// so that a lane's 8 probabilities of the step meet 8 consecutive V codes. A last single tile (nt16 odd) keeps its
// natural order 4*q + e: it is contracted with a 16-deep MFMA.
__host__ __device__ static inline int vt_pos(int t, int nt16) {
    if ((nt16 & 1) && (t >> 4) == nt16 - 1) return t;
    return (t & ~31) + 8 * ((t >> 2) & 3) + 4 * ((t >> 4) & 1) + (t & 3);
}

// (a constant expression: the fused kernels, which are compiled for a head size, take theirs from here)
static constexpr KvImage kv_image(int H, int d, int T) {
    KvImage I = {};
    I.tph = (d + 15) / 16;
    I.nt16 = (T + 15) / 16;
    I.ntok = 16 * I.nt16;
    I.rows_k = I.ntok;
    I.cols_v = I.ntok;
    size_t off = 0;
    auto take = [&off](size_t bytes) { size_t o = off; off = align_up(off + bytes, 16); return o; };
    I.kp = take(I.rows_k * (size_t)I.tph * 16);
    I.vt = take(d * (size_t)I.cols_v);
    I.s_k = take(I.ntok * 4);
    I.s_vp = take(I.ntok * 4);
    I.bias = take(I.ntok * 4);
    I.oscale = take(4);
    I.vpre = take(4);
    I.head_bytes = align_up(off, 256);  // (at least 1 KiB: the kernels copy it in 1 KiB pieces, the last one overlapping)
    I.bytes = H * I.head_bytes;
    return I;
}
static inline KvImage kv_image(const taq_shape& s) { return kv_image(s.H, s.C / s.H, s.T); }

// Operand-ordered copy of a [C, C] weight matrix: for head h, 16-row tile j of the head, K step ks (64 codes),
// lane l = r + 16*q: the 16 codes W[min(h*d + 16*j + r, C-1)][64*ks + 16*q ...]; 1 KiB per (h, j, ks).
// It sits behind the row-major codes, 256-byte aligned.
static inline size_t weight_pack_offset(const taq_shape& s) { return align_up((size_t)s.C * s.C, 256); }
static inline size_t weight_pack_bytes(const taq_shape& s) {
    const size_t d = s.C / s.H;
    return weight_pack_offset(s) + (size_t)s.H * ((d + 15) / 16) * (s.C / 64) * 1024;
}

// LDS bytes of the fused block kernel: K~/V~ image, int8 token tile, weight scales, per-token scratch.
static inline size_t fused_lds_bytes(const taq_shape& s, int tok = 32) {
    return kv_image(s).bytes + tok * ((size_t)s.C + 16) + 3 * (size_t)s.C * 4 + tok * 4 + tok * (size_t)s.H * 4;
}

// Shapes the fused block kernel is instantiated for: (d, H) = (40, 8), (80, 8), (64, 10), as long as
// its working set fits the 160 KiB of LDS of a compute unit.
// Any of the full-precision modes (an unquantized projection, Q~ or probabilities): the float32 kernel-per-stage path.
static inline bool fp_mode(const taq_shape& s) { return s.bits_proj == 16 || s.bits_q == 16 || s.bits_prob == 16; }

static inline bool fused_supported(const taq_shape& s) {
    if (fp_mode(s)) return false;
    if (s.bits_kv != 4 && s.bits_kv != 8) return false;
    if (s.C % s.H) return false;
    const int d = s.C / s.H;
    if (!((d == 40 && s.H == 8) || (d == 80 && s.H == 8) || (d == 64 && s.H == 10))) return false;
    if (s.N > 16 * 65535) return false;  // token tiles are a y / z dimension of the grid
    return fused_lds_bytes(s) <= 160 * 1024;
}

// Shapes of the head-group kernels (to_q + Q~ + attention per head group, then to_out): (d, H) = (160, 8) with one head per workgroup,
// (64, 20), (80, 8) and (64, 10) with two.
static inline bool mid_supported(const taq_shape& s) {
    if (fp_mode(s)) return false;
    if (s.bits_kv != 4 && s.bits_kv != 8) return false;
    if (s.C % s.H) return false;
    const int d = s.C / s.H;
    if (!((d == 160 && s.H == 8) || (d == 64 && s.H == 20) || (d == 80 && s.H == 8) || (d == 64 && s.H == 10))) return false;
    return s.N <= 16 * 65535;
}
// Which kernels take such a layer. In front: the head-group kernel (taq_heads_kernel.h), with one or two tiles of 16 tokens to a workgroup,
// or three kernels of the stage path. Behind: to_out_tail_kernel, or two kernels of the stage path. us per layer by tiles of 16 tokens, six
// layers with weights, inputs and outputs of their own in turn, 77 text tokens; "1t", "2t", "1", "2": head groups of one and two tiles, with and
// without the tail kernel; "s": stages.
//   d = 160: 4 1t 11.7, s 24.3; 32 1t 14.5, 2t 18.3, s 26.2; 33 1t 21.1, 2t 19.5, s 26.7; 51 2t 20.6, 2 22.9, s 27.8; 52 2t 22.8, 2 22.8, 1 24.1, s 27.8;
//     64 2t 23.0, 2 22.7, 1 24.8, s 28.1; 65 1 28.3, 2 31.5, s 30.7; 80 1 29.1, 2 29.5, s 31.1; 88 1 30.7, s 31.6; 96 1 32.5, 2 33.1, s 31.7;
//     row-major weights 32 1t 17.4, s 27.2; 33 1t 25.2, 2t 22.4; 52 2t 25.2, 2 24.9; 64 2 24.7, 1 27.8, s 29.4; 65 1 32.9, s 32.7; 80 2 33.1, s 32.9;
//     64 tokens of text 51 1t 23.0, 1 25.3, s 29.2; 64 1 25.9, s 29.7; 88 1 32.2, s 33.1; 96 1 34.1, s 32.9;
//   d = 64: 25 1t 14.5, s 24.7; 51 1t 19.3, 2t 22.1, s 27.0; 52 1t 26.1, 1 26.1, s 27.0; 80 1 28.1, 2 27.2, s 28.9; 102 1 30.7, 2 28.9, s 31.9;
//     103 1 32.1, 2 34.6, s 31.9; row-major weights 25 1t 16.5, s 24.9; 51 1t 22.1, 1 23.7, s 27.4; 52 1 28.5, s 27.6; 80 1 31.9, s 30.6.
// The lines are rounds of workgroups: two of the head-group kernel share a compute unit (512 of them: 32 and 64 groups of 8 heads, 51 of
// 10; two tiles of d = 64 with row-major weights leave no LDS for that), and two of the tail kernel (10 to a tile). From 89 tiles of
// d = 160 on, stages are the faster by up to 3 % when the same call is repeated, but in the 16 layers of a UNet step head groups are: 96 tiles
// (4 elements of 24) 460 and 470 us a step of five such layers, 8 of 12 461 and 471. The line follows the step.
// shape.tok_tile = 16 or 32 forces head groups (of one tile, with the tail kernel) or stages (tests and tuning).
//
// C = 640: the single kernel ("f") takes 14 us however few tokens there are, as every workgroup pulls both weight matrices (820 KB) through
// one compute unit; a head group pulls a quarter or a fifth of one of them.
//   d = 80: 1 1t 9.3, f 13.5; 32 1t 10.5, f 14.2; 64 1t 11.9, f 13.9; 72 1t 13.3, f 13.9; 74 1t 14.2, f 13.9; 80 1t 14.1, f 13.9;
//     row-major weights 32 1t 11.7, f 17.5; 64 1t 13.4, 2t 15.5, f 17.3; 65 1t 15.2, 2t 16.3; 96 1t 16.6, 2t 16.8, f 17.4; 100 1t 17.0, f 17.3; 104 1t 17.8,
//     2t 18.0, f 17.3; 128 1t 18.4, 2t 18.2, f 17.5;
//   d = 64: 1 1t 9.7, f 14.4; 51 1t 11.8, f 14.7; 64 1t 12.1, f 14.6; 102 1t 14.4, f 14.6; 103 1t 15.9, f 14.6;
//     row-major weights 51 1t 12.8, 2t 14.9, f 17.2; 52 1t 14.1, 2t 15.2; 102 1t 16.2, 2t 16.7, f 17.1; 103 2t 19.4, f 17.1.
// (One round of workgroups, one to a compute unit or two: 64 groups of 4, 51 and 102 of 5; behind it the second round grows from unit to unit.
// From 73 tiles of d = 80 on the single kernel is the faster by up to 5 % when the same call is repeated; in the 16 layers of a UNet step 4 elements
// of 20 take 226 us with head groups and 233 with it, 2 of 40 226 and 224.5. 100 tiles with row-major weights, which cost the single kernel
// 3.5 us.) Two tiles to a workgroup are the faster form at no size where head groups are the
// faster kernels. Other lengths of text: the same lines, but for row-major weights at d = 80 (64). At d = 64 and more than 80 tokens of text the
// single kernel does not fit and stages are what is compared with: 51 13.1, s 21.5; 102 16.0, s 23.6.
// shape.tok_tile = 16 or 32 forces the single kernel of as many tokens, or stages.
// Workgroups of two tiles (per head group): both tiles of one are of the same batch element, so one element's last workgroup may have one only.
// The lines of the two-tile forms count these. us, two tiles per workgroup and one: d = 160, 64 elements of 16 tokens 31.2 and 25.4 (stages
// 30.1), 12 of 80 tokens 31.0 and 24.7 (stages 28.5), row-major 34.7 and 28.2; d = 64, 100 of 16 39.9 and 33.5, 34 of 48 35.2 and 30.6.
static inline long tile_pairs(const taq_shape& s) { return (long)s.B * (((s.N + 15) / 16 + 1) / 2); }
struct HeadsPlan {
    int tiles;  // tiles of 16 tokens per workgroup of the head-group kernel; 0: stages in front
    bool tail;  // to_out_tail_kernel behind it
};
static inline HeadsPlan heads_plan(const taq_shape& s) {
    if (s.tok_tile) return {s.tok_tile == 16 && s.C == 1280 ? 1 : 0, true};
    const long tiles = (long)s.B * ((s.N + 15) / 16), pairs = tile_pairs(s);
    const bool wide = s.C / s.H == 160, packed = s.w_layout == 1, two = (s.T + 15) / 16 == 5;  // (two tiles: C = 1280, 65 to 80 text tokens)
    if (s.C == 640 && s.H == 8) return {tiles <= (packed ? 80 : two ? 100 : 64) ? 1 : 0, true};
    if (s.C == 640) return {tiles <= 102 ? 1 : 0, true};
    if (wide) return {tiles <= 32 ? 1 : tiles <= 64 ? (two && pairs <= 32 ? 2 : 1) : packed && tiles <= 96 ? 1 : 0, tiles <= 51};
    if (!packed || !two) return {tiles <= 51 ? 1 : 0, true};
    return {tiles < 80 ? 1 : tiles <= 102 ? (pairs <= 51 ? 2 : 1) : 0, tiles <= 51};
}
// R requests in grouped launches of the head-group kernels: tiles of 16 tokens per workgroup, or 0 (the single kernel, or request after
// request). n: tiles of a request, t: of all, e: of a request as workgroups of two count them. us per call, "1" and "2" grouped with one and
// two tiles, "r" request after request, "f" the single kernel's grouped launch; 77 text tokens, operand-ordered weights where nothing else
// is said.
//   C = 1280, d = 160: R x n = 2 x 2 1 12.9, r 24.2; 2 x 16 1 17.6, 2 19.9, r 27.3; 16 x 2 1 25.8, 2 24.3, r 187; 4 x 10 1 29.4, 2 24.8, r 52; 16 x 32 2 148,
//     r 254; 2 x 100 2 62.5, r 65.6; 4 x 128 2 124, r 135; 6 x 144 2 217, r 217; 6 x 160 2 241, r 231; 8 x 160 2 322, r 332; 2 x 160 2 81, r 76;
//     row-major 2 x 16 1 19.2, 2 21.7; 6 x 6 1 32.0, 2 26.7; 2 x 64 2 43.7, r 48.5; 2 x 128 2 78, r 74; 4 x 128 2 141, r 147; 90 tokens of text 2 x 64 1 47.9, r 54.4; 2 x 100 1 72, r 71; 6 x 100 1 186, r 228;
//   d = 64: 2 x 8 1 17.5, 2 18.4; 3 x 8 1 21.3, 2 20.6, r 40; 16 x 8 2 61.6, r 210; 2 x 100 2 53.1, r 57; 2 x 160 2 84, r 75; 6 x 144 2 211, r 210; 6 x 160 2 232, r 225; 8 x 160 2 309, r 324;
//     row-major 6 x 8 1 34.8, 2 30.0, r 89; 2 x 64 1 49.4, 2 51.4, r 57.8; 2 x 100 1 69, r 65; 6 x 100 1 186, r 214; 6 x 160 1 284, r 267;
//   C = 640, d = 80: 2 x 24 1 12.7, f 13.2; 3 x 16 1 13.2, f 16.2; 6 x 10 1 16.5, f 16.2; row-major 6 x 10 1 17.4, f 19.6; 16 x 6 1 24.9, f 19.2; d = 64: 3 x 16 1 13.0,
//     f 16.5; 2 x 32 1 14.3, f 14.2; row-major 6 x 10 1 19.0, f 19.1; more text than the single kernel takes: 16 x 16 1 40, r 189; 2 x 160 1 44, r 53.
// Requests of several elements (elements x tiles): d = 160, 16 x (3 x 1) 1 36.3, 2 40.9; 16 x (2 x 3) 1 62.8, 2 56.6; 2 x (20 x 5) 2 61.5, r 67.1; 2 x (34 x 3)
//     2 70.5, r 68.9; 6 x (40 x 3) 2 216, r 222; 6 x (50 x 3) 2 273, r 255; 6 x (160 x 1) 2 396, r 308; d = 64, row-major, 2 x (21 x 3) 1 46.2, 2 59.4, r 57.1.
static inline int grouped_heads(const taq_shape& s, int R) {
    if (!mid_supported(s) || s.tok_tile || R < 2) return 0;
    const long n = (long)s.B * ((s.N + 15) / 16), t = R * n, e = 2 * tile_pairs(s);
    const bool packed = s.w_layout == 1, two = (s.T + 15) / 16 == 5 && s.N > 16;
    if (s.C == 640) return fused_supported(s) ? t <= (s.H == 8 ? (packed ? 48 : 64) : 51) : n <= 160;
    if (n > (packed && two ? (R < 6 ? 100 : R < 8 ? 144 : 160) : R < 4 ? 64 : 100) || (packed && two && e > (R < 6 ? 120 : 160))) return 0;
    if (!two) return 1;
    if (s.C / s.H == 160) return t <= 32 ? 1 : 2;
    return t <= 20 || (!packed && e >= 64) ? 1 : 2;
}

// to_out_tail_kernel: output tiles of 16 channels per workgroup, each by 8 / ot wavefronts at ot = 2 and 4 and by one otherwise. The fewest
// output tiles with which all workgroups run at once, one to a compute unit; where 10 leave some units a second one, 8. us per layer, d = 160:
// 64 tokens ot 2 11.7, 4 11.9, 8 12.6; 128 tokens 2 13.3, 4 12.7, 8 13.0; 256 tokens 4 13.5, 8 13.0; 512 tokens 8 14.4 (64 units have two
// workgroups), 10 13.5; 700 tokens (two rounds with 10) 8 17.85, 10 19.8.
static inline int tail_ot(int C, long tiles) {
    const long per = C / 16;  // output tiles of a token tile
    if (C == 1280 && tiles * (per / 2) <= 256) return 2;
    if (C == 1280 && tiles * (per / 4) <= 256) return 4;
    return tiles * (per / 8) > 256 && tiles * (per / 10) <= 256 ? 10 : 8;
}

// The next launch of a batched call with `left` requests to go: how many of them it takes, and their head groups' tiles of 16 tokens per workgroup
// (0: the single kernel, or request after request). Asked for each launch of up to 16: of 17 requests the last goes out as a call of one does.
struct GroupedLaunch {
    int n, heads;
};
static inline GroupedLaunch grouped_launch(const taq_shape& s, int left) {
    const int n = left < TAQ_MAX_REQ ? left : TAQ_MAX_REQ, heads = grouped_heads(s, n);
    return {heads || fused_supported(s) ? n : 1, heads};
}

static inline KvLayout kv_layout(const taq_shape& s) {
    KvLayout L;
    size_t off = 0;
    const size_t B = s.B, T = s.T, C = s.C, H = s.H;
    L.Cb = s.bits_kv == 8 ? s.C : (s.bits_kv == 4 ? s.C / 2 : 0);
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    L.ntrig = take(B * 4);
    L.trig_idx = take(B * T * 4);
    L.slot_of = take(B * T * 4);
    L.s_k = take(B * H * T * 4);
    L.s_v = take(B * H * T * 4);
    L.k_code = take(B * T * (size_t)L.Cb);
    L.v_code = take(B * T * (size_t)L.Cb);
    L.k16 = take(B * T * C * 2);
    L.v16 = take(B * T * C * 2);
    L.v16t = take(B * C * 96 * 2);
    L.image_bytes = align_up(kv_image(s).bytes, 256);
    L.image = take(B * L.image_bytes);
    L.total = off;
    return L;
}

// Workspace of taq_quantize_kv.
struct KvWorkspace {
    size_t w_code;  // i8  [2C][Cc]   Wk rows then Wv rows
    size_t s_w;     // f32 [2C]
    size_t x_code;  // i8  [B*T][Cc], or (Cc % 64 == 0) tiles of 16 tokens in operand order
    size_t s_x;     // f32 [B*T]
    size_t rows_f;  // f32 [B*T][2C]  dequantised projection rows (K then V channels)
    size_t total;
};

static inline KvWorkspace kv_workspace(const taq_shape& s) {
    KvWorkspace W;
    size_t off = 0;
    const size_t M = (size_t)s.B * s.T, C2 = 2 * (size_t)s.C, Cc = s.Cc;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    W.w_code = take(C2 * Cc);
    W.s_w = take(C2 * 4);
    W.x_code = take((size_t)s.B * align_up(s.T, 16) * Cc);
    W.s_x = take(M * 4);
    W.rows_f = take(M * C2 * 4);
    W.total = off;
    return W;
}

// Kernel-per-stage path: its buffers hold tiles of 16 image tokens (NT = ceil(N/16) per batch element) in the order in
// which the next kernel's matrix operands are read, so that every access is a contiguous KiB or 256 bytes. One tile:
struct StageTile {
    size_t code;   // i8  [ceil(C/64)][64 lanes][16]  codes of hidden, later of A^ V~ (lane = token + 16 * quarter of the K step)
    size_t s;      // f32 [16]                        their scales
    size_t q;      // u32 [H][tph][64 lanes]          Q~ codes as the to_q accumulators leave them, zero past the head
    size_t s_q;    // f32 [H][16]
    size_t o;      // f32 [H][tph][64 lanes][4]       A^ V~
    size_t o_max;  // f32 [H][16]                     largest |A^ V~| of each (head, token)
    size_t total;
};
static inline StageTile stage_tile(const taq_shape& s) {
    StageTile t;
    const size_t H = s.H, tph = (s.C / s.H + 15) / 16, kc = (s.C + 63) / 64;
    t.code = kc * 1024;
    t.s = 64;
    t.q = H * tph * 256;
    t.s_q = H * 64;
    t.o = H * tph * 1024;
    t.o_max = H * 64;
    t.total = t.code + t.s + t.q + t.s_q + t.o + t.o_max;
    return t;
}
static inline size_t stage_tiles(const taq_shape& s) { return (size_t)s.B * ((s.N + 15) / 16); }

// Tiles [tile0, tile1) of the call (tile = b * NT + tile within the batch element) and their buffers.
struct StageChunk {
    int NT, tile0, tile1;
    int8_t* code;
    float* s;
    unsigned* q_op;
    float* s_q;
    float* o_op;
    float* o_max;
};
// How many tiles fit `bytes` of workspace (sections 256-byte aligned), and the buffers of a chunk of `n` tiles in it.
static inline size_t stage_chunk_bytes(const taq_shape& s, size_t n) {
    const StageTile t = stage_tile(s);
    return align_up(n * t.code, 256) + align_up(n * t.s, 256) + align_up(n * t.q, 256) + align_up(n * t.s_q, 256) + align_up(n * t.o, 256) +
           align_up(n * t.o_max, 256);
}
static inline StageChunk stage_chunk(const taq_shape& s, uint8_t* ws, size_t tile0, size_t tile1) {
    const StageTile t = stage_tile(s);
    const size_t n = tile1 - tile0;
    StageChunk c;
    c.NT = (s.N + 15) / 16;
    c.tile0 = (int)tile0;
    c.tile1 = (int)tile1;
    auto take = [&](size_t bytes) { uint8_t* p = ws; ws += align_up(bytes, 256); return p; };
    c.code = reinterpret_cast<int8_t*>(take(n * t.code));
    c.s = reinterpret_cast<float*>(take(n * t.s));
    c.q_op = reinterpret_cast<unsigned*>(take(n * t.q));
    c.s_q = reinterpret_cast<float*>(take(n * t.s_q));
    c.o_op = reinterpret_cast<float*>(take(n * t.o));
    c.o_max = reinterpret_cast<float*>(take(n * t.o_max));
    return c;
}

// Workspace of taq_cross_attn (per request): the full-precision modes use these sections; head groups and stages lay their tiles (StageChunk) out in
// the same memory.
struct AttnWorkspace {
    size_t h_code;  // i8  [B*N][C]
    size_t s_h;     // f32 [B*N]
    size_t q_f;     // f32 [B*N][C]
    size_t q_code;  // i8  [B*N][C]
    size_t s_q;     // f32 [B*N][H]
    size_t o_f;     // f32 [B*N][C]
    size_t o_code;  // i8  [B*N][C]
    size_t s_o;     // f32 [B*N]
    size_t least;   // what taq_cross_attn_static asks for: all sections, also of shapes whose tiles could go through less, a few at a time
    size_t total;   // with all tiles of the stage path at once
};

static inline AttnWorkspace attn_workspace(const taq_shape& s) {
    AttnWorkspace W;
    size_t off = 0;
    const size_t M = (size_t)s.B * s.N, C = s.C, H = s.H;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    W.h_code = take(M * C);
    W.s_h = take(M * 4);
    W.q_f = take(M * C * 4);
    W.q_code = take(M * C);
    W.s_q = take(M * H * 4);
    W.o_f = take(M * C * 4);
    W.o_code = take(M * C);
    W.s_o = take(M * 4);
    const size_t one = stage_chunk_bytes(s, 1), all = stage_chunk_bytes(s, stage_tiles(s));
    W.least = off > one ? off : one;
    W.total = W.least > all ? W.least : all;
    return W;
}

// Kernels that use more than 64 KiB of dynamic LDS need that attribute set once per kernel and device. `done` is the
// kernel's bit mask of devices that have it (one static per kernel instantiation, the library's only state); setting
// the attribute twice from two host threads that race here is harmless.
static inline hipError_t ensure_dynamic_lds(const void* kernel, int bytes, std::atomic<unsigned long long>& done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    done.fetch_or(bit, std::memory_order_release);
    return hipSuccess;
}

// ---- kernel launchers (each returns a hipError_t from the launch) ----------------

// Per-row symmetric int8 codes of fp16 rows: x [M][K] -> code [M][K], scale [M].
hipError_t launch_rowquant_f16(const __half* x, int M, int K, int8_t* code, float* scale, hipStream_t st);
// Same for float32 rows.
hipError_t launch_rowquant_f32(const float* x, int M, int K, int8_t* code, float* scale, hipStream_t st);
// Per-(row, head) symmetric codes (8 or 4 bit, one per byte) of float32 rows: x [M][C] -> code [M][C], scale [M][H].
hipError_t launch_headquant_f32(const float* x, int M, int C, int H, int bits, int8_t* code, float* scale, hipStream_t st);

// First launch of taq_quantize_kv: per-row int8 codes of the context rows (context == NULL: skipped) and of the rows of
// Wk / Wv (NULL: codes given by the caller), plus the protected-token bookkeeping, in one kernel.
hipError_t launch_kv_prep(const __half* context, int M, int8_t* x_code, float* s_x, const __half* Wk, const __half* Wv,
                          int C, int8_t* w_code, float* s_w, int K, const uint8_t* mask, int B, int T, int bits,
                          int* ntrig, int* trig_idx, int* slot_of, hipStream_t st);
// Second launch of taq_quantize_kv (bits_kv 4 or 8): per (head, batch element) the integer K/V projection, Eq. (2)
// codes and scales into qkv_packed, and the head's block of the operand-ordered image where the shape has one.
// The same launch computes the protected fp16 rows (K16, V16, V16T) from the unquantized context rows.
hipError_t launch_kv_head(const int8_t* x_code, const float* s_x, const int8_t* w_code, const float* s_w, uint8_t* packed,
                          const __half* context, const taq_shape& s, hipStream_t st);
// Per-(head, token) codes and scales of unprotected K/V rows, written into qkv_packed.
hipError_t launch_kv_pack(const float* rows_f, const int* slot_of, int B, int T, int C, int H, int bits,
                          uint8_t* k_code, uint8_t* v_code, float* s_k, float* s_v, hipStream_t st);
// Protected K/V rows: fp16 context row x int8 weight codes, fp32 accumulate, fp16 store.
hipError_t launch_kv_trigger_rows(const __half* context, const int8_t* w_code, const float* s_w,
                                  const int* ntrig, const int* trig_idx, int B, int T, int C, int Cc,
                                  __half* k16, __half* v16, __half* v16t, hipStream_t st);
// Expansion of qkv_packed for tests.
hipError_t launch_kv_unpack(const uint8_t* packed, const taq_shape& s, int8_t* k_codes, int8_t* v_codes,
                            float* k_scales, float* v_scales, __half* k_trig, __half* v_trig, hipStream_t st);

// int8 GEMM  acc[m][n] = sum_k A[m][k]*W[n][k]  with dequantisation acc*(sa[m]*sw[n]):
//   out_f32 != NULL: float32 result [M][ldo];  out_f16 != NULL: fp16(result + bias[n]).
hipError_t launch_gemm_i8(const int8_t* A, const float* sa, const int8_t* W, const float* sw,
                          const float* bias, int M, int N, int K, float* out_f32, __half* out_f16,
                          int ldo, hipStream_t st);

// Full-precision stages (shape.bits_proj / bits_q / bits_prob = 16), float32 arithmetic:
//   out[m][n] = sum_k A[m][k] * W[n][k] (+ bias[n]); A f16 or f32 [M][K], W f16 [N][K]; float32 and / or fp16 result;
//   with fp16 rows one float32 FMA chain per output in K order
hipError_t launch_gemm_fp(const void* A, bool a_is_f32, const __half* W, const float* bias, int M, int N, int K,
                          float* out_f32, __half* out_f16, int ldo, hipStream_t st);
//   rows of A to a workgroup of that chain's kernel, z matrices W: 16 up to 20 workgroups to each of 256 compute units, 32 beyond, where reading less
//   from LDS counts for more than rounds that end evenly (tests/host/fullprec_rule.cpp has the timings)
inline int gemm_seq_rows(int M, int N, int z) { return (size_t)((M + 15) / 16) * ((N + 63) / 64) * z < 5120 ? 16 : 32; }
//   K and V rows of a context in one launch: rows_f [M][2C], the same sums as two calls of launch_gemm_fp
hipError_t launch_gemm_kv_rows(const __half* context, const __half* Wk, const __half* Wv, int M, int C, int K, float* rows_f, hipStream_t st);
//   fp16 rows on the matrix cores (any order of summation: for sums that no quantizer reads), out f32 [M][N]; tiles of 32 x 32 outputs, or of
//   64 x 64 where that would be more than 1152 small workgroups: four to each of 256 compute units are at work at once, all that
//   their LDS takes, and an eighth more cost no more than the large tiles do; from 1400 on they do (tests/host/fullprec_rule.cpp has the timings)
inline bool gemm_f16_small(int M, int N) { return (size_t)((M + 31) / 32) * ((N + 31) / 32) <= 1152; }
hipError_t launch_gemm_f16(const __half* A, const __half* W, int M, int N, int K, float* out, hipStream_t st);
//   the same as launch_gemm_fp for every head's slice of the contraction by itself: out[m][h][n] = sum over k in head h (A f32 [M][K], K = H*d)
hipError_t launch_gemm_f32_heads(const float* A, const __half* W, int M, int N, int K, int H, float* out, hipStream_t st);
//   protected K / V rows (fp16, compacted by slot, plus the transposed V copy) from float32 projection rows [B*T][2C]
hipError_t launch_kv_rows_from_f32(const float* rows_f, const int* ntrig, const int* trig_idx, int B, int T, int C,
                                   __half* k16, __half* v16, __half* v16t, hipStream_t st);
//   scores, softmax, Eq. (3), A^ V~ with Q unquantized (q_f) or as codes and scales, probabilities at shape.bits_prob
hipError_t launch_attn_fp(const float* q_f, const int8_t* q_code, const float* s_q, const uint8_t* packed, const taq_shape& s,
                          float* o_f, uint8_t* p_code, hipStream_t st);
//   mean squared difference of two fp16 arrays into a device double
hipError_t launch_mse_f16(const __half* x, const __half* y, size_t n, double* out, hipStream_t st);

// Token-sensitivity sweep of Eq. (1) in full precision (taq_sens.hip): workspace sections and the launch sequence.
#define TAQ_SENS_MAX_H 32
// Wavefronts to each workgroup of the attention (16 image tokens, head): up to 1024 workgroups four are never slower, from 1536 on one is as fast
// (1 %) or faster; between the two it depends on the text's length (tests/host/fullprec_rule.cpp has the timings).
inline int sens_wavefronts(int workgroups) { return workgroups <= 1024 ? 4 : 1; }
struct SensWorkspace {
    size_t rows_f;  // f32 [B*T][2C]             projection rows of the text tokens
    size_t kx, vx;  // f32, 1+nb planes of [B*T][C]: fp16 rows as float32, then the change each width makes (K in operand order)
    size_t va;      // f32 [1+nb][B*T][H][C]     the V planes through each head's slice of to_out
    size_t q_f;     // f32 [B*N][C]
    size_t o;       // f32 [chunk][C]            reference attention output
    size_t p;       // f32 [chunk][H][C]         ... through each head's slice of to_out
    size_t ab;      // f32 [chunk][ntok][nb][H][2]
    size_t dom;     // i32 [chunk][H]            swept token whose change is taken from md, or -1
    size_t dcoef;   // f32 [chunk][H][nb]        its factors
    size_t md;      // f32 [chunk][C]            mean of the other tokens' V rows minus its own
    size_t part;    // f64 [nb][ntok][npart]     partial sums of squares
    size_t total;
    int np, chunk, npart;
};
SensWorkspace sens_workspace(const taq_shape& s, int ntok, int nbits);
hipError_t launch_token_sensitivity(const void* hidden, const void* context, const __half* Wk, const __half* Wv, const __half* Wq,
                                    const __half* Wo, const float* bias, const int* tokens, int ntok, const int* bits, int nbits,
                                    const taq_shape& s, double* out, uint8_t* ws, hipStream_t st);

// K~/V~ image for the fused kernel, from the codes and scales already in qkv_packed.
hipError_t launch_kv_image(uint8_t* packed, const taq_shape& s, hipStream_t st);
// Row-major weight codes -> row-major codes + operand-ordered copy (weight_pack_bytes).
hipError_t launch_pack_weight(const int8_t* codes, const taq_shape& s, int8_t* out, hipStream_t st);

// One request of the fused block kernel.
struct FusedReq {
    const __half* hidden;
    const uint8_t* packed;
    const int8_t* wq;
    const int8_t* wo;
    const float* scales;
    __half* out;
};
// Whole block in one kernel (shapes of fused_supported only). dbg may be NULL.
hipError_t launch_fused_block(const FusedReq* reqs, int R, const taq_shape& s, const taq_debug* dbg, hipStream_t st);
// ---- kernel-per-stage path, on a chunk of tiles (StageChunk); taps in `dbg` are written by the kernel that computes them
// per-token codes of hidden
hipError_t launch_rowquant_op(const StageChunk& c, const taq_shape& s, const __half* hidden, const taq_debug* dbg, hipStream_t st);
// to_q with the per-(token, head) quantizer of Eq. (2), third line
hipError_t launch_to_q_op(const StageChunk& c, const taq_shape& s, const int8_t* Wq, const float* s_wq, const taq_debug* dbg, hipStream_t st);
// scores, softmax, Eq. (3), A^ V~
struct AttnOpArgs {
    const unsigned* q_op;
    const float* s_q;
    const uint8_t* packed;
    float* o_op;
    float* o_max;
    uint8_t* p_code;  // taps or NULL
    float* O;
    KvLayout L;
    KvImage I;
    int N, NT, tile0, tile1, b0, C, H, d, T, nt16;
    int groups, nb;              // groups of tiles per batch element, batch elements
    unsigned inv_groups, inv_h;  // inverse32 of groups and H
    float sig2;   // softmax scale * log2(e)
    float pmax;   // linear grid: 255 or 15; log2 grid: 256 (brings 2^-code * s_V to the linear grid's magnitudes)
    float plast;  // log2 grid: the last code, 255 or 15
};
hipError_t launch_attn_op(const StageChunk& c, const taq_shape& s, const uint8_t* packed, const taq_debug* dbg, hipStream_t st);
// per-token codes of A^ V~ (over the codes of hidden, which are done with)
hipError_t launch_oquant_op(const StageChunk& c, const taq_shape& s, const taq_debug* dbg, hipStream_t st);
// to_out, bias, fp16
hipError_t launch_to_out_op(const StageChunk& c, const taq_shape& s, const int8_t* Wo, const float* s_wo, const float* bias, __half* out,
                            hipStream_t st);

// Head-group path (shapes of mid_supported) on a chunk of tiles, two kernels: (1) per-token codes of `hidden`, to_q, Q~ and the
// attention per head group; (2) per-token codes of A^ V~ and to_out. Taps in `dbg` are written by the kernel that computes them.
// Up to 16 requests of one shape: `c` is the first one's chunk, the others' buffers lie ws_step bytes further on each (taps: one request).
hipError_t launch_heads(const StageChunk& c, const taq_shape& s, const FusedReq* reqs, int R, size_t ws_step, int tt, const taq_debug* dbg, hipStream_t st);
hipError_t launch_to_out_tail(const StageChunk& c, const taq_shape& s, const FusedReq* reqs, int R, size_t ws_step, const taq_debug* dbg, hipStream_t st);

}  // namespace taq
