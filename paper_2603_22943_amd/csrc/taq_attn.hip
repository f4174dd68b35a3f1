// Attention of the kernel-per-stage path (PersonalQ, Section III-B) on gfx950 matrix cores, for any head dimension:
//   A  = softmax(Q~ K~^T / sqrt(d))            over the T text tokens of one head
//   A^ = M_A*A + (1-M_A)*Q_a(A)                Eq. (3)
//   O  = A^ V~
// from Q~ codes in operand order (taq_gemm.hip) and the operand-ordered K~/V~ image of qkv_packed to float32 O in operand
// order and its largest magnitude per (token, head).
//
// The arithmetic is that of the fused block kernel's attention phases (taq_fused_kernel.h, where each step is derived):
// everything transposed, an image token in lane (token % 16) of its wavefront from the scores to O; integer scores; the
// probability code formed in one FMA; weights code * s_V as exact packed-fp16 products split in high and low parts;
// protected columns in two run-time loops over the handful of protected rows.
//
// Work split: a workgroup of four wavefronts owns one head of one batch element and 4 * NTT tiles of 16 image tokens, so
// that the head's image block (8 to 27 KiB, fetched once into LDS) serves them all and several workgroups share a
// compute unit. Bound by vector issue (softmax and Eq. 3, about 12 instructions per probability). The kernel that stood
// here before staged and split K~/V~ itself in every workgroup, whatever the number of tokens: 31 us at B = 2, N = 2304,
// 12 heads of 64. Half of a wavefront's clocks go before the first score, on loads that wait their turn at the texture unit: Q~ codes
// in the widest pieces, protected rows once per workgroup and taps compiled out took it from 8.6 to 8.2 us there, 7.4 to 6.9 at 2048
// tokens of 20 heads of 64, 18.1 to 17.7 at 8192, 9.4 to 8.8 at 4000 tokens of 12 heads of 80.
#include "taq_device.h"

namespace taq {

template <int TPH, int NTT, int PG, int NT16>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TPH <= 3 ? 3 : 2)))
void attn_op_kernel(AttnOpArgs a) {
    constexpr bool LOGP = PG == TAQ_PROB_LOG2, ROWMAX = PG == TAQ_PROB_ROWMAX;
    constexpr bool TAPS = NT16 == 0;  // (of probability codes and O)
    constexpr bool PLDS = TPH <= 5;   // the first protected rows through LDS
    constexpr int MT16 = NT16 ? NT16 : 6, KS = (TPH + 3) / 4, FS = (TPH + 1) / 2;
    extern __shared__ __align__(16) unsigned char img[];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, r16 = lane & 15, q = lane >> 4;
    const int T = a.T, C = a.C, H = a.H, d = a.d, nt16 = NT16 ? NT16 : a.nt16;
    // tiles of the chunk: tile index t (of the whole call) = b * NT + tile within the batch element. The groups of 4 NTT tiles of all batch
    // elements, counted from the chunk's first, each with all its heads, are dealt to the XCDs in eighths. (With whole
    // groups to an XCD, 17 groups of 12 heads were 36 workgroups on five XCDs and none on two: 5.2 -> 4.4 us at 1088 tokens; the image of a
    // head is small beside what the groups read. The arguments that everything waits for are asked for together, not behind the branch.)
    asm volatile("" ::"s"(a.q_op), "s"(a.s_q), "s"(a.packed), "s"(a.L.image), "s"(a.L.image_bytes), "s"(a.I.head_bytes), "s"(a.NT), "s"(a.inv_groups), "s"(a.inv_h));
    const int item = XcdShare::item(blockIdx.x, (unsigned)(a.groups * a.nb * H));
    if (item < 0) return;
    const int group = a.inv_h ? (int)__umulhi((unsigned)item, a.inv_h) : (int)((unsigned)item / (unsigned)H), h = item - group * H;
    const int bi = a.inv_groups ? (int)__umulhi((unsigned)group, a.inv_groups) : (int)((unsigned)group / (unsigned)a.groups), gx = group - bi * a.groups, b = a.b0 + bi;
    const int lo = b * a.NT > a.tile0 ? b * a.NT : a.tile0, hi = (b + 1) * a.NT < a.tile1 ? (b + 1) * a.NT : a.tile1;
    const int first = lo + (gx * 4 + wave) * NTT;  // this wavefront's first tile
    if (lo + gx * 4 * NTT >= hi) return;           // (the whole workgroup)
    const unsigned char* gimg = a.packed + a.L.image + (size_t)b * a.L.image_bytes + (size_t)h * a.I.head_bytes;
    // straight into LDS in pieces of 1 KiB, all under way at once (of the last one the lanes inside the block)
    for (int o = wave * 1024; o < (int)a.I.head_bytes; o += 4096)
        if (o + lane * 16 < (int)a.I.head_bytes)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(gimg + o + lane * 16),
                                             (__attribute__((address_space(3))) void*)(img + o), 16, 0, 0);
    const int ntrig = reinterpret_cast<const int*>(a.packed + a.L.ntrig)[b];
    const int nfp = (ntrig + 15) >> 4;
    const __half* k16 = reinterpret_cast<const __half*>(a.packed + a.L.k16) + (size_t)b * T * C + h * d;
    const __half* v16t = reinterpret_cast<const __half*>(a.packed + a.L.v16t) + ((size_t)b * C + h * d) * 96;

    // Q~ codes of this head, the B operand as it is (zero past the head), and their scales
    int tile[NTT];
    bool live[NTT];
    unsigned qpk[NTT][TPH];
    float sq2[NTT];
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        live[nt] = first + nt < hi;
        tile[nt] = live[nt] ? first + nt : hi - 1;
        const size_t th = (size_t)(tile[nt] - a.tile0) * H + h;
        const unsigned* qp = a.q_op + th * TPH * 64;
#pragma unroll
        for (int j = 0; j < TPH; ++j) qpk[nt][j] = qp[QPlace<TPH>::at(j, lane)];
        sq2[nt] = fmaxf(a.s_q[th * 16 + r16] * a.sig2, 1e-37f);
    }
    // The first 16 protected K rows [slot][16 TPH channels] and V columns [channel][16 slots] of this head. A load costs by the pieces of
    // memory that it touches, one a clock at the texture unit. Heads of up to 80 channels put them into LDS behind the image, once for the
    // workgroup (as operands of every wavefront, up to 10 loads of 16 pieces, they took 1 to 2 of 11 k clocks); of K only the rows that
    // there are. Wide heads, whose workgroups are few and wait for all of LDS, load operands, without slots past the protected tokens:
    // for the layer 40.6 us against 41.3 through LDS at 3072 tokens of 8 heads of 160 (75.9 against 74.4 at 8192).
    unsigned char* prot = img + a.I.head_bytes;
    if (PLDS && nfp > 0) {
        constexpr int PPS = 2 * TPH, KIB = 512 * TPH;  // 16-byte pieces of a slot; bytes of the K rows, of the V columns
        const int slots = ntrig < T ? ntrig : T;
        for (int o = wave * 1024; o < 2 * KIB; o += 4096) {
            // (K rows and V columns are taken together as one list of pieces; a KiB holds some of each where TPH is odd)
            const int i = (o >> 4) + lane, slot = i / PPS, part = i % PPS, v = i - 16 * PPS, c = v >> 1;
            const bool isv = v >= 0;
            const __half* src = isv ? v16t + (size_t)(c < d ? c : d - 1) * 96 + 8 * (v & 1) : k16 + (size_t)slot * C + 8 * part;
            if (o + lane * 16 < 2 * KIB && (isv || (slot < slots && 8 * part < d)))
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)(prot + o), 16, 0, 0);
        }
    }
    // This wavefront's pieces are in LDS before the barrier: nothing else makes anybody wait for another wavefront's.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    uint2 k16r[PLDS ? 1 : FS][2], v16r[PLDS ? 1 : TPH];
    if constexpr (!PLDS) {
#pragma unroll
        for (int s = 0; s < FS; ++s)
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) k16r[s][jj] = make_uint2(0, 0);
#pragma unroll
        for (int k = 0; k < TPH; ++k) v16r[k] = make_uint2(0, 0);
        if (r16 < ntrig) {
            const __half* kr = k16 + (size_t)(r16 < T ? r16 : T - 1) * C + 4 * q;
#pragma unroll
            for (int s = 0; s < FS; ++s)
#pragma unroll
                for (int jj = 0; jj < 2; ++jj)
                    if (2 * s + jj < TPH && 16 * (2 * s + jj) + 4 * q < d) k16r[s][jj] = *reinterpret_cast<const uint2*>(kr + 16 * (2 * s + jj));
        }
        if (4 * q < ntrig) {
#pragma unroll
            for (int k = 0; k < TPH; ++k) {
                const int c = 16 * k + r16 < d ? 16 * k + r16 : d - 1;
                v16r[k] = *reinterpret_cast<const uint2*>(v16t + (size_t)c * 96 + 4 * q);
            }
        }
    }
    __syncthreads();
    if (first >= hi) return;  // (no barrier follows)

    // ---- scores x[t][n] = (K~ Q~^T)[t][n] * s_K[t] (+ 0 / -inf)
    const float* img_sk = reinterpret_cast<const float*>(img + a.I.s_k);
    const float* img_bias = reinterpret_cast<const float*>(img + a.I.bias);
    float S[NTT][MT16][4];
    {
        int32x4_t qop[NTT][KS];
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) qop[nt][ks][jj] = (4 * ks + jj < TPH) ? (int)qpk[nt][4 * ks + jj < TPH ? 4 * ks + jj : 0] : 0;
        const unsigned char* kp = img + a.I.kp;
#pragma unroll
        for (int tt = 0; tt < MT16; ++tt) {
            if (tt < nt16) {
                int32x4_t acc[NTT];
#pragma unroll
                for (int nt = 0; nt < NTT; ++nt) acc[nt] = sum_start();
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    int32x4_t ka;
                    if constexpr (TPH % 4 == 0) {
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
    // ---- protected rows: scores of tile ft of 16 slots, the first from LDS, further ones (rare) straight from the fp16
    // K rows; -inf past ntrig
    auto protected_scores = [&](auto head, int ft, floatx4_t (&facc)[NTT]) {
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt) facc[nt] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
        int slot = 16 * ft + r16;
        slot = slot < T ? slot : T - 1;
        const __half* kr = k16 + (size_t)slot * C + 4 * q;
#pragma unroll
        for (int s = 0; s < FS; ++s) {
            half8_t ka;
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int j = 2 * s + jj;
                uint2 w = make_uint2(0, 0);
                if (j < TPH && 16 * j + 4 * q < d)
                    w = !decltype(head)::value ? *reinterpret_cast<const uint2*>(kr + 16 * j)
                        : PLDS ? *reinterpret_cast<const uint2*>(prot + r16 * (32 * TPH) + 32 * j + 8 * q) : k16r[PLDS ? 0 : s][jj];
                const half4_t hv = *reinterpret_cast<const half4_t*>(&w);
#pragma unroll
                for (int e = 0; e < 4; ++e) ka[4 * jj + e] = hv[e];
            }
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) {
                unsigned c01 = qpk[nt][2 * s], c23 = qpk[nt][2 * s + 1 < TPH ? 2 * s + 1 : 0];
                if constexpr (!decltype(head)::value) {  // (codes as fp16 are not kept for them)
                    c01 = (unsigned)opaque((int)c01);
                    c23 = (unsigned)opaque((int)c23);
                }
                half2_t c0, c1, c2 = {(_Float16)0.f, (_Float16)0.f}, c3 = c2;
                biased4_to_half(c01 ^ 0x80808080u, c0, c1);
                if (2 * s + 1 < TPH) biased4_to_half(c23 ^ 0x80808080u, c2, c3);
                const half8_t qh = {c0[0], c0[1], c1[0], c1[1], c2[0], c2[1], c3[0], c3[1]};
                facc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ka, qh, facc[nt], 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = 16 * ft + 4 * q + i < ntrig;
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) facc[nt][i] = in ? facc[nt][i] : TAQ_NEG_INF;
        }
    };

    // ---- softmax
    float mxs[NTT];
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        float mx = TAQ_NEG_INF;
#pragma unroll
        for (int tt = 0; tt < MT16; ++tt)
            if (tt < nt16) mx = fmaxf(mx, fmaxf(fmaxf(S[nt][tt][0], S[nt][tt][1]), fmaxf(S[nt][tt][2], S[nt][tt][3])));
        mxs[nt] = mx;
    }
    floatx4_t fsc[NTT];  // scores of the first protected tile; those of further ones are formed again for the exponentials
    if (nfp > 0) {
        protected_scores(std::true_type{}, 0, fsc);
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt) mxs[nt] = fmaxf(mxs[nt], fmaxf(fmaxf(fsc[nt][0], fsc[nt][1]), fmaxf(fsc[nt][2], fsc[nt][3])));
        for (int ft = 1; ft < nfp; ++ft) {
            floatx4_t facc[NTT];
            protected_scores(std::false_type{}, ft, facc);
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt)
                mxs[nt] = fmaxf(mxs[nt], fmaxf(fmaxf(facc[nt][0], facc[nt][1]), fmaxf(facc[nt][2], facc[nt][3])));
        }
    }
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
                    if (ROWMAX) eu = fmaxf(eu, ex);
                    S[nt][tt][i] = LOGP ? arg : ex;
                }
            }
        Zs[nt] = Z;
        eus[nt] = eu;
    }
    floatx4_t oacc[NTT][TPH];
    auto protected_values = [&](auto head, int ft, const floatx4_t (&facc)[NTT]) {  // protected columns keep A, unnormalised here
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
            const int c = 16 * k + r16 < d ? 16 * k + r16 : d - 1;
            const uint2 w = !decltype(head)::value ? *reinterpret_cast<const uint2*>(v16t + (size_t)c * 96 + 16 * ft + 4 * q)
                            : PLDS ? *reinterpret_cast<const uint2*>(prot + 512 * TPH + c * 32 + 8 * q) : v16r[PLDS ? 0 : k];
            const half4_t va = *reinterpret_cast<const half4_t*>(&w);  // slots past ntrig hold zeros
#pragma unroll
            for (int nt = 0; nt < NTT; ++nt) {
                oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, phi[nt], decltype(head)::value ? (floatx4_t){0.f, 0.f, 0.f, 0.f} : oacc[nt][k], 0, 0, 0);
                oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x16f16(va, plo[nt], oacc[nt][k], 0, 0, 0);
            }
        }
    };
    if (nfp > 0) {
        protected_values(std::true_type{}, 0, fsc);
        for (int ft = 1; ft < nfp; ++ft) {
            floatx4_t facc[NTT];
            protected_scores(std::false_type{}, ft, facc);
            protected_values(std::false_type{}, ft, facc);
        }
    } else {
#pragma unroll
        for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
            for (int k = 0; k < TPH; ++k) oacc[nt][k] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
    }
    float kq[NTT], lz[NTT], fz[NTT];
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        const float Z = quad_allsum(Zs[nt]);
        const float kqp = quant_mult(a.pmax, Z);  // pmax / Z
        float rz = 1.f;
        kq[nt] = kqp;
        lz[nt] = LOGP ? __builtin_amdgcn_logf(Z) : 0.f;
        fz[nt] = 1.f;
        if constexpr (ROWMAX) {  // (unprotected columns that together weigh less than 2^-40 of the row are dropped)
            const float eu = quad_allmax(eus[nt]);
            if (eu > Z * 9.094947e-13f) {
                kq[nt] = quant_mult(a.pmax, eu);
                rz = quant_mult(Z, eu);
                fz[nt] = quant_mult(eu, Z);
            }
        }
        if (nfp > 0) {
            const float f = kqp * (reinterpret_cast<const float*>(img + a.I.vpre)[0] * rz);
#pragma unroll
            for (int k = 0; k < TPH; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) oacc[nt][k][i] *= f;
        }
    }

    // ---- Eq. (3) and O^T = V~^T A^^T over the unprotected columns
    const uint8_t* vt = img + a.I.vt;
    const _Float16* img_sv = reinterpret_cast<const _Float16*>(img + a.I.s_vp);  // [ntok] high parts | [ntok] low parts
    const half2_t k1024 = {(_Float16)1024.0f, (_Float16)1024.0f};
    auto tap_pcode = [&](int nt, int t, unsigned c0, unsigned c1) {
        const int n = (tile[nt] - b * a.NT) * 16 + r16;
        if (live[nt] && n < a.N) {
            uint8_t* row = a.p_code + (((size_t)b * a.N + n) * H + h) * (size_t)T;
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
            for (int u = 0; u < 2; ++u) {
                constexpr int LAST = MT16 - 1;
                const int tt = 2 * s + u < MT16 ? 2 * s + u : LAST;
                if (u == 0 || second) {
                    const uint2 h4 = *reinterpret_cast<const uint2*>(img_sv + 16 * tt + 4 * q);
                    const uint2 l4 = *reinterpret_cast<const uint2*>(img_sv + a.I.ntok + 16 * tt + 4 * q);
                    const half2_t sh[2] = {*reinterpret_cast<const half2_t*>(&h4.x), *reinterpret_cast<const half2_t*>(&h4.y)};
                    const half2_t sl[2] = {*reinterpret_cast<const half2_t*>(&l4.x), *reinterpret_cast<const half2_t*>(&l4.y)};
#pragma unroll
                    for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
                        for (int i2 = 0; i2 < 2; ++i2) {
                            half2_t c;
                            if constexpr (LOGP) {
                                const float c0 = __builtin_amdgcn_fmed3f(__builtin_rintf(S[nt][tt][2 * i2] - lz[nt]), -a.plast, 0.f);
                                const float c1 = __builtin_amdgcn_fmed3f(__builtin_rintf(S[nt][tt][2 * i2 + 1] - lz[nt]), -a.plast, 0.f);
                                const auto pw = __builtin_amdgcn_cvt_pkrtz(ldexpf(256.0f, (int)c0), ldexpf(256.0f, (int)c1));
                                c = (half2_t){(_Float16)pw[0], (_Float16)pw[1]};
                                if (TAPS && a.p_code) tap_pcode(nt, 16 * tt + 4 * q + 2 * i2, (unsigned)(int)(-c0), (unsigned)(int)(-c1));
                            } else {
                                const float m0 = __builtin_fmaf(S[nt][tt][2 * i2], kq[nt], 12608512.0f);
                                const float m1 = __builtin_fmaf(S[nt][tt][2 * i2 + 1], kq[nt], 12608512.0f);
                                const unsigned w = __builtin_amdgcn_perm(__float_as_uint(m1), __float_as_uint(m0), 0x05040100u);
                                c = *reinterpret_cast<const half2_t*>(&w) - k1024;
                                if (TAPS && a.p_code) tap_pcode(nt, 16 * tt + 4 * q + 2 * i2, w & 0xFFu, (w >> 16) & 0xFFu);
                            }
                            const half2_t wh = c * sh[i2];
                            const half2_t wl = __builtin_elementwise_fma(c, sl[i2], __builtin_elementwise_fma(c, sh[i2], -wh));
                            phi[nt][4 * u + 2 * i2] = wh[0];
                            phi[nt][4 * u + 2 * i2 + 1] = wh[1];
                            plo[nt][4 * u + 2 * i2] = wl[0];
                            plo[nt][4 * u + 2 * i2 + 1] = wl[1];
                        }
                } else {
#pragma unroll
                    for (int nt = 0; nt < NTT; ++nt)
#pragma unroll
                        for (int i = 0; i < 4; ++i) phi[nt][4 * u + i] = plo[nt][4 * u + i] = (_Float16)0.f;
                }
            }
            if (!second && s > 0) sums_settle(oacc);
#pragma unroll
            for (int k = 0; k < TPH; ++k) {
                const int j = 16 * k + r16 < d ? 16 * k + r16 : d - 1;
                if (second) {
                    const uint2 w = *reinterpret_cast<const uint2*>(vt + (size_t)j * a.I.cols_v + 32 * s + 8 * q);
                    half2_t v0, v1, v2, v3;
                    biased4_to_half(w.x, v0, v1);
                    biased4_to_half(w.y, v2, v3);
                    const half8_t va = {v0[0], v0[1], v1[0], v1[1], v2[0], v2[1], v3[0], v3[1]};
#pragma unroll
                    for (int nt = 0; nt < NTT; ++nt) {
                        oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, phi[nt], oacc[nt][k], 0, 0, 0);
                        oacc[nt][k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, plo[nt], oacc[nt][k], 0, 0, 0);
                    }
                } else {
                    const unsigned w = *reinterpret_cast<const unsigned*>(vt + (size_t)j * a.I.cols_v + 32 * s + 4 * q);
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
    // ---- O and its largest magnitude per token of this head
    const float osc = reinterpret_cast<const float*>(img + a.I.oscale)[0] * inv_pmax(a.pmax);
#pragma unroll
    for (int nt = 0; nt < NTT; ++nt) {
        const float of = ROWMAX ? osc * fz[nt] : osc;
        const size_t th = (size_t)(tile[nt] - a.tile0) * H + h;
        const int n = (tile[nt] - b * a.NT) * 16 + r16;
        float omx = 0.f;
#pragma unroll
        for (int k = 0; k < TPH; ++k) {
            const bool valid = 16 * k + 4 * q < d;
            const float4 o4 = make_float4(oacc[nt][k][0] * of, oacc[nt][k][1] * of, oacc[nt][k][2] * of, oacc[nt][k][3] * of);
            if (valid) omx = fmaxf(omx, fmaxf(fmaxf(fabsf(o4.x), fabsf(o4.y)), fmaxf(fabsf(o4.z), fabsf(o4.w))));
            if (live[nt] && valid) {
                reinterpret_cast<float4*>(a.o_op)[(th * TPH + k) * 64 + lane] = o4;
                if (TAPS && a.O && n < a.N) *reinterpret_cast<float4*>(a.O + ((size_t)b * a.N + n) * C + h * d + 16 * k + 4 * q) = o4;
            }
        }
        omx = quad_allmax(omx);
        if (live[nt] && q == 0) a.o_max[th * 16 + r16] = omx;
    }
}

template <int TPH, int NTT, int PG, int NT16>
static hipError_t launch_attn_cfg(AttnOpArgs a, int tiles_b, int nb, hipStream_t st) {
    a.groups = (tiles_b + 4 * NTT - 1) / (4 * NTT);
    a.nb = nb;
    if ((long)a.groups * nb * a.H > XcdShare::MOST) return hipErrorInvalidValue;
    const unsigned items = (unsigned)(a.groups * nb * a.H);
    a.inv_h = inverse32(a.H, items);
    a.inv_groups = inverse32(a.groups, (unsigned)(a.groups * nb));
    hipLaunchKernelGGL((attn_op_kernel<TPH, NTT, PG, NT16>), dim3(XcdShare::grid(items)), dim3(256), a.I.head_bytes + (TPH <= 5 ? 1024 * TPH : 0), st, a);
    return hipGetLastError();
}

template <int TPH, int PG, int NTT>
static hipError_t launch_attn_text(const AttnOpArgs& a, int tiles_b, int nb, hipStream_t st) {
    // 65 to 80 text tokens (the 77-token prompts): no run-time guards around the score tiles, and no taps, whose branches keep the
    // compiler from reading V~ ahead of the products
    if (a.nt16 == 5 && !a.p_code && !a.O) return launch_attn_cfg<TPH, NTT, PG, 5>(a, tiles_b, nb, st);
    return launch_attn_cfg<TPH, NTT, PG, 0>(a, tiles_b, nb, st);
}

// Two tiles per wavefront share the operand conversions, one is done sooner. One and two, us, by workgroups of two: heads of 64, 320
// workgroups (2048 tokens of 20 heads) 6.9 and 7.5, 432 8.3 and 8.2, 600 9.9 and 10.4, 640 10.5 and 10.7, 768 11.8 and 11.1 (the layer
// 46.5 and 46.1), 780 11.8 and 13.0, 960 14.0 and 13.8, 1280 16.9 and 16.0, 2048 24.0 and 22.1; of 32, 1128 11.6 and 11.6, 1536 13.9 and
// 13.0; of 80, 384 8.7 and 9.2, 852 14.7 and 15.4; of 40, 1024 11.7 and 11.0. Wide heads have no registers for two.
template <int TPH, int PG>
static hipError_t launch_attn_grid(const AttnOpArgs& a, int tiles_b, int nb, hipStream_t st) {
    if constexpr (TPH <= 5) {
        if ((long)((tiles_b + 7) / 8) * a.H * nb > 640) return launch_attn_text<TPH, PG, 2>(a, tiles_b, nb, st);
    }
    return launch_attn_text<TPH, PG, 1>(a, tiles_b, nb, st);
}

template <int TPH>
static hipError_t launch_attn_tph(const AttnOpArgs& a, int grid, int tiles_b, int nb, hipStream_t st) {
    if (grid == TAQ_PROB_LOG2) return launch_attn_grid<TPH, TAQ_PROB_LOG2>(a, tiles_b, nb, st);
    if (grid == TAQ_PROB_ROWMAX) return launch_attn_grid<TPH, TAQ_PROB_ROWMAX>(a, tiles_b, nb, st);
    return launch_attn_grid<TPH, TAQ_PROB_LINEAR>(a, tiles_b, nb, st);
}

hipError_t launch_attn_op(const StageChunk& c, const taq_shape& s, const uint8_t* packed, const taq_debug* dbg, hipStream_t st) {
    AttnOpArgs a;
    a.q_op = c.q_op;
    a.s_q = c.s_q;
    a.packed = packed;
    a.o_op = c.o_op;
    a.o_max = c.o_max;
    a.p_code = dbg ? dbg->p_code : nullptr;
    a.O = dbg ? dbg->O : nullptr;
    a.L = kv_layout(s);
    a.I = kv_image(s);
    a.N = s.N; a.NT = c.NT; a.tile0 = c.tile0; a.tile1 = c.tile1;
    a.C = s.C; a.H = s.H; a.d = s.C / s.H; a.T = s.T;
    a.nt16 = (s.T + 15) / 16;
    const float sigma = s.softmax_scale != 0.f ? s.softmax_scale : 1.0f / sqrtf((float)a.d);
    a.sig2 = sigma * 1.4426950408889634f;
    a.plast = s.bits_prob == 4 ? 15.f : 255.f;
    a.pmax = s.prob_grid == TAQ_PROB_LOG2 ? 256.f : a.plast;
    a.b0 = c.tile0 / c.NT;
    const int nb = (c.tile1 - 1) / c.NT - a.b0 + 1;
    const int tiles_b = nb == 1 ? c.tile1 - c.tile0 : c.NT;  // tiles of a batch element in the chunk, at most
    if (nb > 65535) return hipErrorInvalidValue;  // (nobody has K~/V~ of more: batch elements are a y dimension in taq_quantize_kv)
    switch ((a.d + 15) / 16) {
#define TAQ_ATT(N) case N: return launch_attn_tph<N>(a, s.prob_grid, tiles_b, nb, st);
        TAQ_ATT(1) TAQ_ATT(2) TAQ_ATT(3) TAQ_ATT(4) TAQ_ATT(5) TAQ_ATT(6) TAQ_ATT(7) TAQ_ATT(8) TAQ_ATT(9) TAQ_ATT(10)
#undef TAQ_ATT
        default: return hipErrorInvalidValue;
    }
}

}  // namespace taq
