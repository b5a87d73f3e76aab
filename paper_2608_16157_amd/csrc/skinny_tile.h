// Expert tiles of few token rows: at most 64 rows x 128 weight rows, the weights streaming once
// through LDS.  A part of the grouped GEMM kernel (gemm.hip); internal.
//
// Most groups of a decode batch or a short prompt chunk have few rows (of the 69 groups of a
// DeepSeek-V3-shaped layer with 300 tokens and Zipf routing, 48 have at most 16), so these tiles
// are bound by HBM: what counts is the weight bytes a CU keeps in flight, how long it has none in
// flight between tiles, and how few other bytes move.  Hence
//  - each weight row moves in 128-byte pieces (bf16, fp8; 64-byte pieces for MXFP4), 128 rows a
//    stage, with the tiles of a group on one XCD: a pure stream of such stages reaches 6.3 TB/s
//    here, of the large tiles' 256 rows x 64 bytes 4.6-5.6, of 256 x 32 bytes (MXFP4) 2.9-4.6; and
//    with 4096-byte rows dealt round-robin over the XCDs 5.5;
//  - only 16, 32 or 64 activation rows are staged, and the ring takes the LDS that this leaves;
//  - a tile's first weight requests wait for one dependent look-up, its slot: the rows' tokens are
//    looked up behind them, by scalar loads, and the tables come by DMA (a vector load's wait would
//    drain the requests made before it).  This order alone took 4-6 % off the whole layer
//    (DeepSeek-V3 64 tokens 397 -> 380 us, Qwen3 300 tokens 212 -> 203 us).
// Against the streaming GEMV kernels, whose waves each read the activations again from L2 and stop
// streaming while a batch is multiplied (layer times): Qwen3 160 tokens 200 -> 133 us, DeepSeek-V3
// 64 tokens 434 -> 380 us, 200 tokens 909 -> 622 us, DeepSeek-V4-Flash 7 tokens 71.4 -> 70.0 us, 200
// tokens 349 -> 221 us; against 128 x 256 tiles with padding: DeepSeek-V3 300 tokens 837 -> 729 us,
// DeepSeek-V4-Flash 400 tokens 419 -> 293 us.
#pragma once

#include "ftmoe_device.h"
#include "ftmoe_internal.h"
#include "gemm_tile.h"

namespace ftmoe {

constexpr int kSkinnyBN = 128;   // weight rows per tile

// K values per stage (BK) and weight row bytes per stage (BRB)
template <int WT> struct STr;
template <> struct STr<FT_DT_BF16> { static constexpr int BK = 64, BRB = 2 * BK; };
template <> struct STr<FT_DT_FP8E4M3FN_B128> { static constexpr int BK = 128, BRB = BK; };
template <> struct STr<FT_DT_MXFP4> { static constexpr int BK = 128, BRB = BK / 2; };

// One tile of a group of `len` <= kSkinnyRows rows (rows beg ..), weight tile nt, by the four waves
// of the workgroup.  ring: kRing bytes of LDS; s_scale: fp8 block scales of the tile's weight rows
// (2 x 64); s_tok, s_gate: kSkinnyRows = 64 entries.
template <int WT, int EPI, int kRing>
__device__ __forceinline__ void skinny_tile(const ExpertArgs &a, int slot, int beg, int len, int nt, uint8_t *ring,
                                            float *s_scale, int32_t *s_tok, float *s_gate) {
    constexpr bool kFp8 = WT == FT_DT_FP8E4M3FN_B128, kFp4 = WT == FT_DT_MXFP4;
    constexpr int NW = 4, BN = kSkinnyBN, kThreads = NW * kWave;
    constexpr int BK = STr<WT>::BK, BRB = STr<WT>::BRB, ARB = 2 * BK;
    constexpr int BSTAGE = BN * BRB, XSTAGE = kFp4 ? 256 * NW : 0;
    constexpr int B_INSTR = 32 * BRB / 1024;        // 1 KB DMA instructions per wave
    constexpr int A_ROWS = 1024 / ARB, B_ROWS = 1024 / BRB, A_CHUNKS = ARB / 16, B_CHUNKS = BRB / 16;
    static_assert(BK == 128 || BK == 64, "stages of whole or half K blocks");
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t / kWave), lane = lane_id();
    const int H = a.H, I = a.I;
    const int K = EPI == GEMM_GATEUP ? H : I;
    const int nrows = EPI == GEMM_GATEUP ? 2 * I : H;
    const int nk = K / BK, nkb = K / 128;

    // B tile: wave w's 32 rows; gate/up: the 16 gate rows of h columns [hc0, hc0 + 16), hc0 = 64 nt
    // + 16 w, then the 16 matching up rows
    const size_t brow_bytes = static_cast<size_t>(nk) * BRB;
    const uint8_t *bexp = static_cast<const uint8_t *>(EPI == GEMM_GATEUP ? a.w13 : a.w2) +
                          static_cast<size_t>(slot) * nrows * brow_bytes;
    uint32_t boff[B_INSTR];
#pragma unroll
    for (int ii = 0; ii < B_INSTR; ++ii) {
        const int q = ii * B_ROWS + lane / B_CHUNKS;
        int wrow;
        if constexpr (EPI == GEMM_GATEUP) {
            const int hc0 = nt * (BN / 2) + 16 * wave;
            wrow = q < 16 ? hc0 + q : I + hc0 + q - 16;
        } else {
            wrow = nt * BN + 32 * wave + q;
        }
        boff[ii] = static_cast<uint32_t>(wrow * brow_bytes) + (swz<BRB>(q, lane % B_CHUNKS) << 4);
    }
    // MXFP4 scales of a stage: wave w moves run w of the tile's 128 weight rows (128 bytes; lanes 32
    // .. 63 fetch them again into the next 128 bytes, so that every lane is active)
    const uint8_t *xexp = nullptr;
    uint32_t xoff = 0;
    if constexpr (kFp4) {
        const int l = lane & 31;
        const int row = EPI == GEMM_GATEUP ? (l < 16 ? nt * 64 + 4 * l : I + nt * 64 + 4 * (l - 16)) : nt * BN + 4 * l;
        xexp = static_cast<const uint8_t *>(EPI == GEMM_GATEUP ? a.s13 : a.s2) + static_cast<size_t>(slot) * (K / 32) * nrows;
        xoff = static_cast<uint32_t>(wave * nrows + row);
    }
    // Tables, moved into LDS ahead of the stages (every wave moves all of them: equal counts)
    if constexpr (kFp8) {
        const float *sp = static_cast<const float *>(EPI == GEMM_GATEUP ? a.s13 : a.s2) +
                          static_cast<size_t>(slot) * (nrows / 128) * nkb;
#pragma unroll
        for (int which = 0; which < (EPI == GEMM_GATEUP ? 2 : 1); ++which) {
            const int r = EPI == GEMM_GATEUP ? (nt * (BN / 2) + (which ? I : 0)) / 128 : nt;
            dma4(reinterpret_cast<const uint8_t *>(sp + static_cast<size_t>(r) * nkb), 4 * min(lane, nkb - 1),
                 lds_address(reinterpret_cast<uint8_t *>(s_scale)) + which * 256);
        }
    }
    if constexpr (EPI == GEMM_DOWN) {
        const uint32_t r = 4 * min(lane, len - 1);
        dma4(reinterpret_cast<const uint8_t *>((a.wv.ypart ? a.wv.row_pair : a.wv.row_tok) + beg), r,
             lds_address(reinterpret_cast<uint8_t *>(s_tok)));
        dma4(reinterpret_cast<const uint8_t *>(a.wv.row_gate + beg), r, lds_address(reinterpret_cast<uint8_t *>(s_gate)));
    }
    const uint32_t lring = lds_address(ring);

    // ML 16-row MFMA tiles (16x16x32) by two 16-column ones per wave (gate/up: its gate rows and its up
    // rows, so SiLU(gate) * up is formed in registers)
    auto body = [&](auto ml) {
        constexpr int ML = decltype(ml)::value, NT = 2;
        constexpr int ASZ = ML * 16 * ARB, STG = ASZ + BSTAGE + XSTAGE;
        constexpr int NSR = kRing / STG, NS = NSR < 8 ? NSR : 8;
        constexpr int A_TOT = ASZ / 1024, A_PW = (A_TOT + NW - 1) / NW;
        constexpr int PER_STAGE = A_PW + B_INSTR + (kFp4 ? 1 : 0);
        static_assert(NS >= 2 && NS * PER_STAGE < 64, "ring depth, vmcnt range");
        auto issue_b = [&](int kt, uint32_t l) {
            const uint8_t *bs = bexp + static_cast<size_t>(kt) * BRB;
#pragma unroll
            for (int ii = 0; ii < B_INSTR; ++ii) dma16(bs, boff[ii], l + ASZ + (wave * B_INSTR + ii) * 1024);
            if constexpr (kFp4)
                dma4(xexp + static_cast<size_t>(kt) * (BK / 32) * nrows, xoff, l + ASZ + BSTAGE + wave * 256);
        };
        // The weights of the first stages are requested as soon as the slot is known; their latency
        // covers the look-up of the rows' tokens, which takes scalar loads only: a vector load's
        // wait would cover the requests made before it.
#pragma unroll
        for (int st = 0; st < NS - 1; ++st)
            if (st < nk) issue_b(st, lring + st * STG);
        const uint8_t *asrc[A_PW];
        uint32_t alds[A_PW];
#pragma unroll
        for (int ii = 0; ii < A_PW; ++ii) {
            const int idx = (wave + NW * ii) % A_TOT, row0 = idx * A_ROWS, j = lane / A_CHUNKS;
            const uint8_t *rowp;
            // padding rows repeat the last row; never stored
            if constexpr (EPI == GEMM_GATEUP) {
                int tok[A_ROWS];
#pragma unroll
                for (int q = 0; q < A_ROWS; ++q) tok[q] = scalar_load(a.wv.row_tok + beg + min(len - 1, row0 + q));
                int mine = tok[0];
#pragma unroll
                for (int q = 1; q < A_ROWS; ++q) mine = j == q ? tok[q] : mine;
                rowp = static_cast<const uint8_t *>(a.x) + static_cast<size_t>(mine) * H * 2;
            } else {
                rowp = static_cast<const uint8_t *>(a.wv.h) + static_cast<size_t>(beg + min(len - 1, row0 + j)) * I * 2;
            }
            asrc[ii] = rowp + (swz<ARB>(row0 + j, lane % A_CHUNKS) << 4);
            alds[ii] = idx * 1024;
        }
        auto issue_a = [&](int kt, uint32_t l) {
#pragma unroll
            for (int ii = 0; ii < A_PW; ++ii) dma16(asrc[ii] + static_cast<size_t>(kt) * ARB, l + alds[ii]);
        };
#pragma unroll
        for (int st = 0; st < NS - 1; ++st)
            if (st < nk) issue_a(st, lring + st * STG);
        // The sums are formed as the GEMV kernels form them, so that results do not depend on which of
        // the two evaluates a call: part is the running 128-wide K block, acc the blocks of the
        // running K range (a quarter of the blocks, or a half where they only split two ways), tot
        // the ranges before it.  One chain over K would be cheaper still, but its rounding doubles the
        // share of h elements that fall on a neighbouring bf16 value (error of the layer output
        // against 64 bits, Qwen3 160 tokens, rms of 16 inputs: 3.5e-5 against 1.6e-5).
        const int ksp = nkb % 4 != 0 && nkb % 2 == 0 ? 2 : 4, per = (nkb + ksp - 1) / ksp;
        const int fn = lane & 15, fq = lane >> 4;   // row or column, K part of the MFMA operands
        floatx4_t tot[ML][NT], acc[ML][NT], part[ML][NT];
#pragma unroll
        for (int i = 0; i < ML; ++i)
#pragma unroll
            for (int n = 0; n < NT; ++n) tot[i][n] = acc[i][n] = part[i][n] = floatx4_t{};
        auto mma = [&](u32x4_t av, u32x4_t bv, floatx4_t c) {
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(av), as_bf16x8(bv), c, 0, 0, 0);
        };
        auto flush = [&](int kb) {
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const float sc = kFp8 ? s_scale[(EPI == GEMM_GATEUP ? 64 * n : 0) + kb] : 1.0f;
#pragma unroll
                for (int i = 0; i < ML; ++i) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        // a block with scale 0 adds nothing
                        const float sum = kFp8 ? fmaf(sc, part[i][n][e], acc[i][n][e]) : acc[i][n][e] + part[i][n][e];
                        acc[i][n][e] = kFp8 && sc == 0.0f ? acc[i][n][e] : sum;
                    }
                    part[i][n] = floatx4_t{};
                }
            }
            if ((kb + 1) % per == 0 || kb + 1 == nkb) {
#pragma unroll
                for (int i = 0; i < ML; ++i)
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) tot[i][n][e] += acc[i][n][e];
                        acc[i][n] = floatx4_t{};
                    }
            }
        };
        uint32_t so = 0, sp = (NS - 1) * STG;   // slots of stage kt and of stage kt - 1
        for (int kt = 0; kt < nk; ++kt) {
            // stage kt has landed; what was requested after its last part may be outstanding (the
            // first NS - 1 stages' activations were requested after all of their weights)
            if (kt + NS - 1 > nk) {
                wait_vmcnt<0>();
            } else if (kt >= NS - 2) {
                wait_vmcnt<(NS - 2) * PER_STAGE>();
            } else {
                static_for<0, NS - 2>([&](auto j) {
                    constexpr int J = decltype(j)::value;
                    if (kt == J) wait_vmcnt<(NS - 2 - J) * A_PW + J * PER_STAGE>();
                });
            }
            wait_lgkmcnt0();   // this wave's reads of stage kt - 1, whose slot is refilled next
            stage_barrier();
            if (kt + NS - 1 < nk) {
                issue_b(kt + NS - 1, lring + sp);
                issue_a(kt + NS - 1, lring + sp);
            }
            const uint8_t *A = ring + so, *B = A + ASZ + wave * 32 * BRB, *X = A + ASZ + BSTAGE;
            auto ard = [&](int i, int c) {
                return *reinterpret_cast<const u32x4_t *>(A + (i * 16 + fn) * ARB + (swz<ARB>(fn, c) << 4));
            };
            auto brd = [&](int n, int c) {
                return *reinterpret_cast<const u32x4_t *>(B + (n * 16 + fn) * BRB + (swz<BRB>(n * 16 + fn, c) << 4));
            };
            // weight chunk c = 4 p + fq of a lane's row (8, 16 or 32 K values) against the activation
            // chunks of the same K values
#pragma unroll
            for (int p = 0; p < B_CHUNKS / 4; ++p) {
                const int c = 4 * p + fq;
                u32x4_t b[NT];
#pragma unroll
                for (int n = 0; n < NT; ++n) b[n] = brd(n, c);
                if constexpr (WT == FT_DT_BF16) {
#pragma unroll
                    for (int i = 0; i < ML; ++i) {
                        const u32x4_t av = ard(i, c);
#pragma unroll
                        for (int n = 0; n < NT; ++n) part[i][n] = mma(av, b[n], part[i][n]);
                    }
                } else if constexpr (kFp8) {
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        u32x4_t w[NT];
#pragma unroll
                        for (int n = 0; n < NT; ++n) w[n] = fp8x8_to_bf16x8(b[n][2 * s], b[n][2 * s + 1]);
#pragma unroll
                        for (int i = 0; i < ML; ++i) {
                            const u32x4_t av = ard(i, 2 * c + s);
#pragma unroll
                            for (int n = 0; n < NT; ++n) part[i][n] = mma(av, w[n], part[i][n]);
                        }
                    }
                } else {
                    float xs[NT];
#pragma unroll
                    for (int n = 0; n < NT; ++n)   // tile row of the column: gate half, then up half
                        xs[n] = fp4_scale_operand(X[c * 256 + (EPI == GEMM_GATEUP ? 64 * n + 16 * wave : 32 * wave + 16 * n) + fn]);
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        u32x4_t w[NT];
#pragma unroll
                        for (int n = 0; n < NT; ++n) w[n] = fp4x8_scaled_to_bf16x8(b[n][s], xs[n]);
#pragma unroll
                        for (int i = 0; i < ML; ++i) {
                            const u32x4_t av = ard(i, 4 * c + s);
#pragma unroll
                            for (int n = 0; n < NT; ++n) part[i][n] = mma(av, w[n], part[i][n]);
                        }
                    }
                }
            }
            if (BK == 128 || (kt & 1)) flush(kt * BK / 128);
            sp = so;
            so = so + STG == NS * STG ? 0 : so + STG;
        }
        // element e of a 16 x 16 tile in lane (fn, fq): row 4 fq + e, column fn
        if constexpr (EPI == GEMM_GATEUP) {
            uint16_t *hout = static_cast<uint16_t *>(a.wv.h) + nt * (BN / 2) + 16 * wave + fn;
#pragma unroll
            for (int i = 0; i < ML; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = 16 * i + 4 * fq + e;
                    if (row < len)
                        hout[static_cast<size_t>(beg + row) * I] = f32_to_bf16(silu_f32(tot[i][0][e]) * tot[i][1][e]);
                }
        } else {
#pragma unroll
            for (int i = 0; i < ML; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = 16 * i + 4 * fq + e;
                    if (row < len) {
                        const size_t o = static_cast<size_t>(s_tok[row]) * H + nt * BN + 32 * wave + fn;
                        const float gw = s_gate[row];
#pragma unroll
                        for (int n = 0; n < NT; ++n) {
                            const float y = gw * tot[i][n][e];
                            if (a.wv.ypart) a.wv.ypart[o + 16 * n] = y;
                            else unsafeAtomicAdd(a.out + o + 16 * n, y);
                        }
                    }
                }
        }
    };
    static_for<1, kSkinnyRows / 16 + 1>([&](auto ml) {
        constexpr int ML = decltype(ml)::value;
        if ((len + 15) / 16 == ML) body(ml);
    });
}

}  // namespace ftmoe
