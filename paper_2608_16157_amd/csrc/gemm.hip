// Grouped expert GEMM on MFMA tiles for many-token chunks (prefill): bf16, fp8 or MXFP4 weights,
// bf16 activations (fp8 ones in the optional FT_ACT_FP8_1x128_POW2 mode), float32 accumulation.
//
// The same two projections as the streaming path (Section 3.2, grouped evaluation of the GPU
// execution set; weights addressed through the slot, Section 4.2), shaped for matrix-core reuse:
//   gate/up: h[rows of g] = silu(X_g W1^T) * (X_g W3^T)       tile = BM rows x BN/2 h columns
//   down   : out[tok] += gate * (h_g W2^T)                    tile = BM rows x BN out columns
//
// Work decomposition.  Groups of more than kSkinnyRows rows: one workgroup per (group, BM-row M tile,
// BN-row N tile).  Each wave computes 128 rows of the tile for its own 64 columns, as 4 x 2 MFMA
// 32x32x16 tiles (the bf16 MFMA shape with the highest measured throughput on gfx950), so every
// weight element is read from LDS (and, for fp8 or MXFP4, widened) by exactly one wave.  The tile is
// 128 x 256 with 4 waves and two workgroups per CU, so one multiplies while the other waits at a
// stage barrier or runs its prologue or epilogue.  (256 x 256 tiles of 8 waves, one workgroup per
// CU, move a third fewer bytes per flop; measured faster on dense shapes but slower on routed prefill
// batches, whose expert groups of about 256 rows leave nearly empty tail tiles that still stream a
// whole weight tile.)  Groups of up to kSkinnyRows rows: skinny tiles (skinny_tile.h) in the same
// launch.
// These tiles are bound by how fast global memory fills LDS (measured: 17 TB/s for L2-resident
// 64-byte row pieces, 7-11 TB/s once the data comes from the Infinity Cache or HBM), so the tile
// is as large as LDS and the occupancy allow: a 128 x 256 tile moves 768 bytes per K step for
// 65536 flops, a third less per flop than 128 x 128, while the 128-row M tile keeps the padding
// of the small expert groups in check.
// Tiles are enumerated per group, in bands of up to kBandM M tiles, each band N-tile-major with
// the M tile fastest, through the per-M-tile group map the router writes, so the tiles that
// share a weight tile and those that share activation rows run at the same time; the block ->
// tile map keeps consecutive tiles on one XCD (workgroups are dealt to the 8 XCDs round-robin)
// to share its L2.  The router numbers the groups in cost classes (the shared expert, groups of
// several M tiles, then one-tile groups by their live 32-row sub-tiles), and tiles neither stage nor
// multiply sub-tiles that hold only padding rows.  All tiles of a projection go out in one launch,
// dealt to the XCDs by the number of tiles the routing produced.  (Before the deal went by that number
// the idle blocks of the grid were dealt too, and the grid had to be cut into launches of about one
// round of the chip; cut so, the current kernel takes 0.478 ms for the Qwen3 4096-token layer against
// 0.458, 3.52 against 3.11 ms for the DeepSeek-V3 8192-token layer with fp8 activations.)
//
// Data movement.  A (activation rows, gathered through row_tok for gate/up) and B (weight rows,
// kept in their storage format) go straight from global memory into LDS with global_load_lds
// (16 bytes per lane), through a ring of NS stages of BK K-values.  Every LDS row keeps its
// 16-byte chunks XOR-swizzled by the row index, so MFMA operand reads of consecutive rows hit
// distinct banks.  The main loop is software-pipelined: each MFMA sub-step's operands are read
// from LDS while the previous sub-step's MFMAs run, and the stage hand-off (an explicit vmcnt
// wait plus s_barrier; a __syncthreads would drain every stage in flight) sits in the last
// sub-step of a stage, so the first reads of the next stage overlap its last MFMAs.
//
// fp8 weights carry one float32 scale per 128 x 128 block, and the product is formed exactly as
// weight-only dequantisation defines it: the codes are widened to bf16 unscaled (exact), the
// MFMAs sum each 128-wide K block's products in float32, and the block's scale multiplies that
// partial sum.  A wave's 64 columns lie in at most two scale blocks (the gate and the up half of
// a gate/up tile, one block for down), so one scale per column half and K block applies to all
// of the wave's accumulators of that half.  Rather than keeping a second accumulator set for the
// running block, the accumulators carry the sum in units of the current block's scale: at the
// start of block k they are multiplied by s(k-1) / s(k), the MFMAs then add block k's unscaled
// partial sum, and after the last block one multiply by its scale gives sum_k s(k) P(k).  A block
// with scale 0 contributes nothing: its ratio is 1 (the previous scale is carried on) and, in the
// tiles that hold such a block, its widened codes are masked to zero.  The gate/up B tile puts
// each wave's 32 gate rows next to the 32 matching up rows, so SiLU(gate) * up is formed in
// registers.
#include "ftmoe_device.h"
#include "ftmoe_internal.h"
#include "gemm_tile.h"
#include "skinny_tile.h"

#include <algorithm>

namespace ftmoe {

constexpr int kWaveCols = 64;                           // weight rows of the tile per wave
constexpr int kGemmWaves = kGemmBN / kWaveCols;
constexpr int kGemmThreads = kGemmWaves * kWave;
constexpr int kGemmOcc = 2;                             // workgroups per CU
constexpr int kMI = kGemmBM / 32, kNJ = kWaveCols / 32; // 32 x 32 MFMA tiles per wave
constexpr int kBM = kGemmBM;                            // token rows per tile
constexpr int kBN = kGemmBN;                            // weight rows per tile
static_assert(kGemmWaves == 4 && kMI == 4, "128 x 256 tiles of four waves");
#ifndef FT_GEMM_BAND
#define FT_GEMM_BAND 8
#endif
constexpr int kBandM = FT_GEMM_BAND;  // M tiles that run together on each weight tile

// Per weight format: K values per stage (BK) and weight row bytes per stage (BRB).
// Internal weight-format code of fp8 weights with fp8 activations (FT_ACT_FP8_1x128_POW2): fp8 x
// fp8 products on the scaled 32x32x64 MFMA.
constexpr int kWtFp8Act = 16;
template <int WT> struct GTr;
template <> struct GTr<FT_DT_BF16> {
    static constexpr int BK = 32, BRB = 2 * BK;
};
template <> struct GTr<FT_DT_FP8E4M3FN_B128> {
    static constexpr int BK = 64, BRB = BK;
};
// fp8 weights and fp8 activations: 64 K values per stage (one 32x32x64 MFMA step).
template <> struct GTr<kWtFp8Act> {
    static constexpr int BK = 64, BRB = BK;
};
// MXFP4: 64 K values (32 code bytes) per weight row and stage, so that one lane's 16-byte chunk
// of a row is a whole 32-value scale run
template <> struct GTr<FT_DT_MXFP4> {
    static constexpr int BK = 64, BRB = BK / 2;
};

typedef int i32x8_t __attribute__((ext_vector_type(8)));
__device__ __forceinline__ i32x8_t cat_u32x8(u32x4_t lo, u32x4_t hi) {
    return i32x8_t{static_cast<int>(lo[0]), static_cast<int>(lo[1]), static_cast<int>(lo[2]), static_cast<int>(lo[3]),
                   static_cast<int>(hi[0]), static_cast<int>(hi[1]), static_cast<int>(hi[2]), static_cast<int>(hi[3])};
}

// Block b of nl + ns -> large tile t (returned as t) or skinny tile t (as ~t).  Each XCD (blocks are
// dealt to them round-robin, b mod 8) takes a contiguous run of both kinds, the large tiles first:
// they run longest, and the short skinny tiles fill the last round.  Measured against taking both
// kinds alternately, so that matrix-bound and HBM-bound tiles share a CU: DeepSeek-V3 at 1200 tokens
// 1.39 against 1.52 ms, 8192 tokens 3.89 against 4.10 ms, DeepSeek-V4-Flash at 200 tokens 178 against
// 196 us; and against the skinny tiles first: 1.43 and 3.93 ms, 227 us.
__device__ __forceinline__ int mixed_tile(int b, int nl, int ns) {
    const int x = b & 7, i = b >> 3;
    const int ql = nl >> 3, rl = nl & 7, qs = ns >> 3, rs = ns & 7;
    // XCDs 0 .. rl - 1 have one more large tile, the next rs (mod 8) one more skinny tile, as the
    // nl + ns blocks are dealt
    const uint32_t m = ((1u << rs) - 1u) << rl, more = (m | (m >> 8)) & 0xFFu;
    const int cl = ql + (x < rl);
    return i < cl ? ql * x + min(x, rl) + i : ~(qs * x + __popc(more & ((1u << x) - 1u)) + i - cl);
}

// The grid's first dimension is at most this many blocks: one dimension holds fewer than 2^32 threads,
// and the largest call (1048576 tokens of 65 experts, H = 8192) has 17 million down tiles.
constexpr int kGridXLog = 22;

template <int WT, int EPI>
__global__ __launch_bounds__(kGemmThreads, kGemmOcc) void grouped_gemm(ExpertArgs a, int ntn) {
    constexpr bool kAq = WT == kWtFp8Act;                          // fp8 activations (fp8 x fp8 MFMA)
    constexpr bool kFp8 = WT == FT_DT_FP8E4M3FN_B128 || kAq;        // fp8 weights with block scales
    constexpr bool kWiden8 = WT == FT_DT_FP8E4M3FN_B128;            // fp8 weights widened to bf16
    constexpr bool kFp4 = WT == FT_DT_MXFP4;
    constexpr int BK = GTr<WT>::BK;
    constexpr int ARB = kAq ? BK : BK * 2;           // A row bytes per stage (bf16, or fp8 codes)
    constexpr int BRB = GTr<WT>::BRB;                // B row bytes per stage
    constexpr int ASUB = 32 * ARB;                   // A bytes of one 32-row sub-tile and stage
    constexpr int BSTAGE = kBN * BRB;
    constexpr int B_INSTR = BSTAGE / 1024 / kGemmWaves;   // 1 KB DMA instructions per wave
    // MXFP4: one more DMA per wave and stage brings a quarter of the stage's e8m0 scales
    constexpr int XSTAGE = kFp4 ? 1024 : 0;          // LDS per scale stage: 4 waves x 256 bytes
    static_assert(!kFp8 || 128 % BK == 0, "an fp8 K stage lies in one scale block");
    constexpr int kStagesPerKb = kFp8 ? 128 / BK : 1;
    constexpr int kMaxKb = 64;                       // K <= 8192
    constexpr int kMaxStages = 6;                    // of the ring
    // The ring: as many stages as fit the LDS left by the tables, two workgroups to a CU.  A tile
    // with ML live 32-row sub-tiles stages only those rows, so thin tiles get a deeper ring.
    constexpr int kTables = (kFp8 ? 16 * kGemmWaves * kMaxKb : 0) + (kAq ? kBM * kMaxKb + 4 * kGemmWaves * kBM + 4 * kBM : 0) +
                            8 * kBM + 256;
    constexpr int kRing = (81920 - kTables) / 1024 * 1024;
    __shared__ __attribute__((aligned(1024))) uint8_t s_ring[kRing];
    // fp8: per wave and column half, the factor applied to the accumulators at the start of each
    // 128-wide K block, a mask that zeroes the widened codes of blocks with scale 0, and the scale
    // of the last block (applied after the K loop)
    __shared__ float s_ratio[kFp8 ? kGemmWaves : 1][2][kFp8 ? kMaxKb : 1];
    __shared__ uint32_t s_keep[kFp8 ? kGemmWaves : 1][2][kFp8 ? kMaxKb : 1];
    __shared__ float s_last[kGemmWaves][2];
    __shared__ int32_t s_zeroblk[kGemmWaves];   // fp8: a column group's scales hold a 0
    __shared__ int32_t s_tok[kBM];
    __shared__ float s_gate[kBM];
    // fp8 activations: e8m0 scale byte of each tile row and K block, and (gate/up epilogue) the
    // per-wave largest |h| of each row and the rows' h exponents
    __shared__ __attribute__((aligned(256))) uint8_t s_ascale[kAq ? kBM * kMaxKb : 1];
    __shared__ float s_hmax[kAq ? kGemmWaves : 1][kAq ? kBM : 1];
    __shared__ int32_t s_hexp[kAq ? kBM : 1];

    const int t = threadIdx.x, blk = static_cast<int>(blockIdx.y << kGridXLog | blockIdx.x);
    if constexpr (EPI == GEMM_GATEUP) {
        // zero the output that the down projection accumulates into
        const size_t n4 = static_cast<size_t>(a.T) * a.H / 4;
        float4 *o4 = reinterpret_cast<float4 *>(a.out);
        for (size_t i = static_cast<size_t>(blk) * kGemmThreads + t; i < n4;
             i += static_cast<size_t>(gridDim.x) * gridDim.y * kGemmThreads)
            o4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // tile of this block: L among the large tiles, or ~L among the skinny ones
    const int nlarge = scalar_load(a.wv.grp_meta + 4) * ntn;
    int L;
    if constexpr (kAq) {
        if (blk >= nlarge) return;
        L = xcd_remap(blk, nlarge);
    } else {
        const int nskinny = (scalar_load(a.wv.grp_meta) - scalar_load(a.wv.grp_meta + 5)) * (kBN / kSkinnyBN) * ntn;
        if (blk >= nlarge + nskinny) return;
        L = mixed_tile(blk, nlarge, nskinny);
    }
    L = __builtin_amdgcn_readfirstlane(L);
    if constexpr (!kAq) {
        if (L < 0) {
            const int gs = scalar_load(a.wv.grp_meta + 5) + ~L / (kBN / kSkinnyBN * ntn);
            skinny_tile<WT, EPI, kRing>(a, scalar_load(a.wv.grp_slot + gs), scalar_load(a.wv.grp_beg + gs),
                                        scalar_load(a.wv.grp_len + gs), ~L % (kBN / kSkinnyBN * ntn), s_ring,
                                        &s_ratio[0][0][0], s_tok, s_gate);
            return;
        }
    }
    // group g owns logical tiles [off_g * ntn, off_{g+1} * ntn), so L / ntn is one of its M tiles;
    // inside the group, bands of up to kBandM M tiles, each band N-tile-major with the M tile
    // fastest
    const int g = scalar_load(a.wv.mt_group + L / ntn);
    const int off = scalar_load(a.wv.grp_mt_off + g), mtc = scalar_load(a.wv.grp_mt_off + g + 1) - off;
    const int local = L - off * ntn;
    const int band = local / (kBandM * ntn), rem = local - band * (kBandM * ntn);
    const int bm = min(kBandM, mtc - band * kBandM);
    const int nt = rem / bm, mt = band * kBandM + rem % bm;
    const int slot = scalar_load(a.wv.grp_slot + g);
    const int beg = scalar_load(a.wv.grp_beg + g);
    const int len = scalar_load(a.wv.grp_len + g);
    const int H = a.H, I = a.I;
    const int K = EPI == GEMM_GATEUP ? H : I;
    const int nrows = EPI == GEMM_GATEUP ? 2 * I : H;
    const int m0 = mt * kBM;
    const int wave = __builtin_amdgcn_readfirstlane(t / kWave), lane = lane_id();

    // ---- DMA sources: this lane's 16 bytes in each of its 1 KB DMA instructions.  Lane i of
    // an instruction writes LDS bytes [16 i, 16 i + 16) of its 1 KB block, i.e. row i / CHUNKS of
    // the block at chunk position i % CHUNKS, so it fetches the chunk that belongs there.
    constexpr int A_ROWS = 1024 / ARB, B_ROWS = 1024 / BRB;   // rows per DMA instruction
    constexpr int A_CHUNKS = ARB / 16, B_CHUNKS = BRB / 16;
    // B tile row -> weight row.  gate/up: wave n's 64 rows are the 32 gate rows of h columns
    // [hc0, hc0 + 32), hc0 = nt * BN/2 + 32 n, followed by the 32 matching up rows (I + hc0 ...).
    // Each wave moves the rows it multiplies.
    const size_t brow_bytes = static_cast<size_t>(K / BK) * BRB;
    const uint8_t *bexp = static_cast<const uint8_t *>(EPI == GEMM_GATEUP ? a.w13 : a.w2) +
                          static_cast<size_t>(slot) * nrows * brow_bytes;
    uint32_t boff[B_INSTR];   // one expert's matrix is at most 256 MB (H, I <= 8192)
#pragma unroll
    for (int ii = 0; ii < B_INSTR; ++ii) {
        const int row = (wave * B_INSTR + ii) * B_ROWS + lane / B_CHUNKS;
        int wrow;
        if constexpr (EPI == GEMM_GATEUP) {
            const int q = row % kWaveCols;
            const int hc0 = nt * (kBN / 2) + wave * (kWaveCols / 2);
            wrow = q < kWaveCols / 2 ? hc0 + q : I + hc0 + q - kWaveCols / 2;
        } else {
            wrow = nt * kBN + row;
        }
        boff[ii] = static_cast<uint32_t>(wrow * brow_bytes) + (swz<BRB>(row, lane % B_CHUNKS) << 4);
    }
    const int wn = wave;
    const int fn = lane & 31, fq = lane >> 5;
    // MXFP4 scales (run-major in memory: the scales of one 32-wide K run of consecutive weight
    // rows are contiguous).  A stage covers runs 2 kt and 2 kt + 1 of the tile's 256 weight rows,
    // which are 4 segments of 128 contiguous bytes (gate/up: the 128 gate rows and the 128 up
    // rows of the tile; down: two halves of its 256 rows).  Wave w = 2 run + half (mod 4) moves
    // segment (run, half) with one 4-byte-per-lane DMA into bytes [256 w, 256 w + 128) of the
    // stage; lanes 32..63 fetch the same segment again into the next 128 bytes, so the instruction
    // has every lane active and stays in bounds.
    const uint8_t *xexp = nullptr;
    uint32_t xoff = 0;
    int xcol[kNJ] = {};
    if constexpr (kFp4) {
        const int xr = (wave >> 1) & 1, xh = wave & 1;
        const int row0 = EPI == GEMM_GATEUP ? (xh ? I : 0) + nt * (kBN / 2) : nt * kBN + xh * (kBN / 2);
        xexp = static_cast<const uint8_t *>(EPI == GEMM_GATEUP ? a.s13 : a.s2) +
               static_cast<size_t>(slot) * (K / 32) * nrows;
        xoff = static_cast<uint32_t>(xr * nrows + row0 + 4 * (lane & 31));
        // this lane's scale byte for column tile j, run fq: segment (fq, half) at 256 (2 fq + half)
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
            const int half = EPI == GEMM_GATEUP ? j : (wn * kWaveCols + j * 32) / (kBN / 2);
            const int r = EPI == GEMM_GATEUP ? wn * (kWaveCols / 2) + fn : (wn * kWaveCols + j * 32 + fn) % (kBN / 2);
            xcol[j] = 256 * (2 * fq + half) + r;
        }
    }
    const int nk = K / BK, nkb = K / 128;
    // ---- gate/up: the first stages are requested before the tables below are looked up, so that the
    // two latencies overlap.  (The tables' waits then cover all of these stages: little beside gate/up's
    // long K loop, but on the down projection waiting for the first stage alone is better.)  Together
    // with the exponents by DMA, DeepSeek-V3 with fp8 activations: gate/up 2048 tokens 920 -> 880 us,
    // 8192 tokens 1.92 -> 1.80 ms; down with the early request 502 -> 523 us.
    const int mlive = __builtin_amdgcn_readfirstlane((min(len - m0, kBM) + 31) / 32);   // live 32-row sub-tiles
    constexpr int A_MAX = ASUB * kMI / 1024 / kGemmWaves;   // A DMA instructions per wave and stage, at most
    const int a_tot = mlive * (ASUB / 1024);                // and of the tile
    // A instruction ii of this wave: where the instructions do not split evenly, some are done
    // twice (the same bytes to the same place), which keeps every wave's count equal
    const uint8_t *asrc[A_MAX];
    uint32_t alds[A_MAX];
#pragma unroll
    for (int ii = 0; ii < A_MAX; ++ii) {
        const int idx = (wave + kGemmWaves * ii) % a_tot;
        const int row = idx * A_ROWS + lane / A_CHUNKS;
        const int r = min(len - 1, m0 + row);      // padding rows repeat the last row; never stored
        constexpr size_t EB = kAq ? 1 : 2;   // bytes per activation element
        const uint8_t *rowp;
        if constexpr (EPI == GEMM_GATEUP)
            rowp = (kAq ? a.wv.xq : static_cast<const uint8_t *>(a.x)) + static_cast<size_t>(a.wv.row_tok[beg + r]) * H * EB;
        else
            rowp = (kAq ? a.wv.hq : static_cast<const uint8_t *>(a.wv.h)) + static_cast<size_t>(beg + r) * I * EB;
        asrc[ii] = rowp + (swz<ARB>(row, lane % A_CHUNKS) << 4);
        alds[ii] = idx * 1024;
    }
    // fp8 activations: each tile row's exponent byte of every K block (rows of x by token, rows of h by
    // position), 64 bytes a row; where a row's bytes are whole words they come by DMA, 4 rows at a time
    constexpr int X_MAX = kAq ? kBM / 4 / kGemmWaves : 1;
    const uint8_t *esrc[X_MAX];
    const bool ewords = nkb % 4 == 0;
    if constexpr (kAq) {
#pragma unroll
        for (int ii = 0; ii < X_MAX; ++ii) {
            const int r = min(len - 1, m0 + (wave + kGemmWaves * ii) * 4 + lane / 16);
            const size_t srow = EPI == GEMM_GATEUP ? static_cast<size_t>(a.wv.row_tok[beg + r]) : static_cast<size_t>(beg + r);
            esrc[ii] = (EPI == GEMM_GATEUP ? a.wv.xs : a.wv.hs) + srow * nkb + 4 * min(lane % 16, nkb / 4 - 1);
        }
    }
    const uint32_t lring = lds_address(s_ring);
    auto issue = [&](auto apw, int kt, uint32_t so, uint32_t asz) {
        const uint32_t l = lring + so;
#pragma unroll
        for (int ii = 0; ii < A_MAX; ++ii)
            if (ii < apw) dma16(asrc[ii] + static_cast<size_t>(kt) * ARB, l + alds[ii]);
        const uint8_t *bs = bexp + static_cast<size_t>(kt) * BRB;
#pragma unroll
        for (int ii = 0; ii < B_INSTR; ++ii) dma16(bs, boff[ii], l + asz + (wave * B_INSTR + ii) * 1024);
        if constexpr (kFp4)
            dma4(xexp + static_cast<size_t>(kt) * (BK / 32) * nrows, xoff, l + asz + BSTAGE + wave * 256);
    };
    constexpr bool kEarly = EPI == GEMM_GATEUP;
    if constexpr (kEarly) {
        const int asz = mlive * ASUB, stg = asz + BSTAGE + XSTAGE, ns = min(kMaxStages, kRing / stg);
        for (int st = 0; st < ns; ++st) issue((a_tot + kGemmWaves - 1) / kGemmWaves, min(st, nk - 1), st * stg, asz);
    }
    if constexpr (kAq) {
        if (ewords) {
            const uint32_t le = lds_address(s_ascale);
#pragma unroll
            for (int ii = 0; ii < X_MAX; ++ii)
                if (ii < 2 * mlive) dma4(esrc[ii], le + (wave + kGemmWaves * ii) * 256);
        } else {
            const uint8_t *src = EPI == GEMM_GATEUP ? a.wv.xs : a.wv.hs;
            for (int idx = t; idx < 32 * mlive * nkb; idx += kGemmThreads) {
                const int r = idx / nkb, kb = idx - r * nkb, rr = min(len - 1, m0 + r);
                const size_t srow = EPI == GEMM_GATEUP ? static_cast<size_t>(a.wv.row_tok[beg + rr]) : static_cast<size_t>(beg + rr);
                s_ascale[r * kMaxKb + kb] = src[srow * nkb + kb];
            }
        }
    }
    // fp8 block-scale tables of each wave's columns (gate half and up half of a gate/up tile; one
    // block for down), staged in LDS before the pipeline starts: a vector load inside the loop
    // would make the compiler drain the DMA stages.  Lane kb of each wave holds
    // K block kb: s'(kb) = the scale of the last block at or before kb whose scale is not 0 (1
    // before the first), found with a wave max-scan of the indices of such blocks; the ratio of
    // block kb is s'(kb-1) / s'(kb) (1 for block 0).  One load per lane instead of a walk over
    // the K blocks, whose dependent loads held every tile's start back by several microseconds.
    if constexpr (kFp8) {
        const float *sp = static_cast<const float *>(EPI == GEMM_GATEUP ? a.s13 : a.s2);
        uint64_t zero = 0;
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            int r;
            if constexpr (EPI == GEMM_GATEUP) {
                const int hc0 = nt * (kBN / 2) + wn * (kWaveCols / 2);
                r = which == 0 ? hc0 / 128 : (I + hc0) / 128;
            } else {
                r = (nt * kBN + wn * kWaveCols) / 128;
            }
            const float *row = sp + (static_cast<size_t>(slot) * (nrows / 128) + r) * nkb;
            const float sc = lane < nkb ? row[lane] : 1.0f;
            const bool nz = sc != 0.0f;
            zero |= __ballot(lane < nkb && !nz);
            const uint32_t last = wave_incl_max_u32(nz ? static_cast<uint32_t>(lane) + 1u : 0u);
            const float cur = last ? __shfl(sc, static_cast<int>(last) - 1) : 1.0f;
            const float prev = __shfl(cur, max(lane - 1, 0));
            if (lane < nkb) {
                s_ratio[wn][which][lane] = lane == 0 ? 1.0f : prev / cur;
                s_keep[wn][which][lane] = nz ? 0xFFFFFFFFu : 0u;
            }
            if (lane == nkb - 1) s_last[wn][which] = cur;
        }
        if (lane == 0) s_zeroblk[wn] = zero != 0;
    }
    // token and gate of each row of the tile (down projection epilogue)
    if constexpr (EPI == GEMM_DOWN) {
        for (int i = t; i < kBM; i += kGemmThreads) {
            const int r = min(len - 1, m0 + i);
            s_tok[i] = a.wv.row_tok[beg + r];
            s_gate[i] = a.wv.row_gate[beg + r];
        }
    }

    constexpr int KS = kAq ? BK / 64 : BK / 16;   // MFMA sub-steps per K stage
    // Operands of one 32x32x16 MFMA sub-step.  The lane (r = lane % 32, kg = lane / 32) holds 8 K
    // values of row r for each operand; which 8 is free as long as A and B agree.  bf16 weights:
    // sub-step ks takes K [16 ks + 8 kg, +8), i.e. 16-byte chunk 2 ks + kg of both rows.  fp8
    // weights: a lane reads one 16-byte chunk of its weight row, 16 K values, for two sub-steps,
    // so sub-step ks = 2 p + s takes K [32 p + 16 kg + 8 s, +8): weight chunk 2 p + kg (bytes
    // 8 s ..), activation chunk 4 p + 2 kg + s.  MXFP4 weights: a lane reads weight chunk kg, 32
    // K values under one scale, for all four sub-steps, so sub-step ks takes K [32 kg + 8 ks, +8):
    // word ks of the chunk, activation chunk 4 kg + ks.  Weight chunks and scales are carried
    // over from the sub-step that read them.
    // fp8 activations: lane (r, kg) holds bytes [32 kg, 32 kg + 32) of the stage's 64-byte row r
    // for both operands (chunks 2 kg and 2 kg + 1; the MFMA pairs the same byte slots of A and
    // B), and its row's exponent byte for the K block.
    struct Frag {
        u32x4_t a[kMI];
        u32x4_t b[kNJ];
        u32x4_t a2[kAq ? kMI : 1];   // fp8 activations: second 16 bytes of each operand
        u32x4_t b2[kAq ? kNJ : 1];
        uint32_t as[kAq ? kMI : 1];  // fp8 activations: e8m0 scale byte of the lane's row
        uint32_t xb[kNJ];   // MXFP4 e8m0 scale byte of each column tile
        float sc[2];        // fp8: accumulator factor of this K block, gate (or down) and up half
        uint32_t keep[2];   // fp8: code mask of this K block (0 for a block with scale 0)
    };
    // zs: the tile holds an fp8 K block with scale 0 (codes of such blocks are masked)
    // A, B, X: the stage's areas in the ring
    auto load_frag = [&](const uint8_t *A, const uint8_t *B, const uint8_t *X, auto ks, auto ml, auto zs, Frag &f,
                         const Frag &prev, int kt) {
        constexpr int KSI = decltype(ks)::value, ML = decltype(ml)::value;
        constexpr bool ZS = decltype(zs)::value;
        const int ca = kWiden8 ? 4 * (KSI / 2) + 2 * fq + (KSI % 2) : (kFp4 ? 4 * fq + KSI : 2 * KSI + fq);
        if constexpr (kFp8) {
            if constexpr (KSI == 0) {
                const int kb = (kt * BK) / 128;
                f.sc[0] = s_ratio[wn][0][kb];
                f.sc[1] = s_ratio[wn][1][kb];
                if constexpr (ZS) {
                    f.keep[0] = s_keep[wn][0][kb];
                    f.keep[1] = s_keep[wn][1][kb];
                }
            } else {
                f.sc[0] = prev.sc[0];
                f.sc[1] = prev.sc[1];
                if constexpr (ZS) {
                    f.keep[0] = prev.keep[0];
                    f.keep[1] = prev.keep[1];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < ML; ++i) {
            const int ra = i * 32 + fn;
            if constexpr (kAq) {
                f.a[i] = *reinterpret_cast<const u32x4_t *>(A + ra * ARB + (swz<ARB>(ra, 4 * KSI + 2 * fq) << 4));
                f.a2[i] = *reinterpret_cast<const u32x4_t *>(A + ra * ARB + (swz<ARB>(ra, 4 * KSI + 2 * fq + 1) << 4));
                if constexpr (KSI == 0) f.as[i] = s_ascale[ra * kMaxKb + (kt * BK) / 128];
                else f.as[i] = prev.as[i];
            } else {
                f.a[i] = *reinterpret_cast<const u32x4_t *>(A + ra * ARB + (swz<ARB>(ra, ca) << 4));
            }
        }
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
            const int rb = wn * kWaveCols + j * 32 + fn;
            if constexpr (kFp4) {
                if constexpr (KSI == 0) {
                    f.b[j] = *reinterpret_cast<const u32x4_t *>(B + rb * BRB + (swz<BRB>(rb, fq) << 4));
                    f.xb[j] = X[xcol[j]];
                } else {
                    f.b[j] = prev.b[j];
                    f.xb[j] = prev.xb[j];
                }
            } else if constexpr (kAq) {
                f.b[j] = *reinterpret_cast<const u32x4_t *>(B + rb * BRB + (swz<BRB>(rb, 4 * KSI + 2 * fq) << 4));
                f.b2[j] = *reinterpret_cast<const u32x4_t *>(B + rb * BRB + (swz<BRB>(rb, 4 * KSI + 2 * fq + 1) << 4));
                if constexpr (ZS) {
                    const uint32_t keep = (EPI == GEMM_GATEUP && j >= kNJ / 2) ? f.keep[1] : f.keep[0];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        f.b[j][q] &= keep;
                        f.b2[j][q] &= keep;
                    }
                }
            } else if constexpr (kFp8) {
                if constexpr (KSI % 2 == 0) {
                    f.b[j] = *reinterpret_cast<const u32x4_t *>(B + rb * BRB + (swz<BRB>(rb, 2 * (KSI / 2) + fq) << 4));
                    if constexpr (ZS) {
                        // codes of a block with scale 0 become +0
                        const uint32_t keep = (EPI == GEMM_GATEUP && j >= kNJ / 2) ? f.keep[1] : f.keep[0];
#pragma unroll
                        for (int q = 0; q < 4; ++q) f.b[j][q] &= keep;
                    }
                } else {
                    f.b[j] = prev.b[j];
                }
            } else {
                f.b[j] = *reinterpret_cast<const u32x4_t *>(B + rb * BRB + (swz<BRB>(rb, ca) << 4));
            }
        }
    };
    // rs: this sub-step opens a 128-wide K block (fp8: the accumulators take the block's factor)
    auto mma = [&](auto &acc, const Frag &f, auto ks, auto ml, auto zs, auto rs) {
        constexpr int KSI = decltype(ks)::value, ML = decltype(ml)::value;
        constexpr bool ZS = decltype(zs)::value, RS = decltype(rs)::value;
        u32x4_t bf[kNJ];
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
            if constexpr (kFp4) {
                bf[j] = fp4x8_scaled_to_bf16x8(f.b[j][KSI], fp4_scale_operand(f.xb[j]));
            } else if constexpr (kWiden8) {
                bf[j] = KSI % 2 == 0 ? fp8x8_to_bf16x8(f.b[j][0], f.b[j][1]) : fp8x8_to_bf16x8(f.b[j][2], f.b[j][3]);
            } else {
                bf[j] = f.b[j];
            }
        }
        // a tile's accumulators take the block factor just before its MFMA, so the multiplies of one
        // tile can run while the previous tile's MFMA executes (see interleave)
#pragma unroll
        for (int i = 0; i < ML; ++i)
#pragma unroll
            for (int j = 0; j < kNJ; ++j) {
                if constexpr (kFp8 && RS) acc[i][j] *= (EPI == GEMM_GATEUP && j >= kNJ / 2) ? f.sc[1] : f.sc[0];
                if constexpr (kAq)   // formats 0 (fp8 e4m3) for both; B's scale byte 127 (1.0)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        cat_u32x8(f.a[i], f.a2[i]), cat_u32x8(f.b[j], f.b2[j]), acc[i][j], 0, 0, 0,
                        static_cast<int>(f.as[i]), 0, 127);
                else
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f.a[i]), as_bf16x8(bf[j]),
                                                                         acc[i][j], 0, 0, 0);
            }
    };

    // Software pipeline.  The ring holds NS stages; the DMA of stage kt + NS goes into the slot of
    // stage kt once every wave has read all of stage kt.  Each sub-step's operands are read from
    // LDS while the previous sub-step's MFMAs run, and the hand-off sits in the last sub-step of
    // a stage: wait for this wave's share of stage kt + 1 (stages kt + 2 .. kt + NS - 1 may stay
    // outstanding) and for its LDS reads of stage kt, barrier, refill the slot of stage kt, read
    // the first operands of stage kt + 1, then run the last MFMAs of stage kt.  Past the end the
    // DMA re-reads the last stage: with a branch around it the loop lost 6-9 % in the fp8 x fp8 kernels
    // (DeepSeek-V3, 2048 tokens: gate/up 1053 against 997 us, down 654 against 590).
    // ML: the 32-row MFMA sub-tiles of the M tile that hold at least one real row; the others
    // hold padding only, so they are neither staged nor multiplied.
    // Order of one sub-step's instructions: its MFMAs with the next sub-step's operand reads
    // (sub-step ks2 of the same or the next stage) threaded between them, one read after each
    // MFMA.  Measured 2-4 % faster than issuing all the reads first behind an explicit wait.
    // In a sub-step that opens an fp8 K block (rsv) each MFMA is preceded by the 16 multiplies of
    // its tile's block factor (the first also by the widening of the sub-step's weight operands).
    auto interleave = [&](auto ks2, auto ml, auto zs, auto rsv) {
        constexpr int K2 = decltype(ks2)::value, ML = decltype(ml)::value;
        constexpr bool ZS = decltype(zs)::value, RSV = decltype(rsv)::value;
        constexpr bool kReadsB = kFp4 ? K2 == 0 : (kWiden8 ? K2 % 2 == 0 : true);
        constexpr int kReads = (kAq ? (K2 == 0 ? 3 : 2) * ML : ML) + (kReadsB ? (kAq ? 2 : 1) * kNJ : 0) +
                               (kFp4 && K2 == 0 ? kNJ : 0) + (kFp8 && K2 == 0 ? (ZS ? 4 : 2) : 0);
        constexpr int kMfma = ML * kNJ;
        constexpr int kPairs = kReads < kMfma ? kReads : kMfma;
        if constexpr (RSV) {
            static_for<0, kMfma>([&](auto q) {
                constexpr int Q = decltype(q)::value;
                __builtin_amdgcn_sched_group_barrier(0x002, Q == 0 && kWiden8 ? 16 + 4 * kNJ : 16, 0);   // VALU
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                           // one MFMA
                if constexpr (Q < kReads) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
            });
            if constexpr (kReads > kMfma) __builtin_amdgcn_sched_group_barrier(0x100, kReads - kMfma, 0);
        } else {
            static_for<0, kPairs>([&](auto) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
            });
            if constexpr (kMfma > kPairs) __builtin_amdgcn_sched_group_barrier(0x008, kMfma - kPairs, 0);
            if constexpr (kReads > kPairs) __builtin_amdgcn_sched_group_barrier(0x100, kReads - kPairs, 0);
        }
    };
    // One tile with ML live sub-tiles: the K loop and the epilogue, instantiated together (a common
    // epilogue would merge the accumulators of all instances, whose copies then spilled).
    auto tile = [&](auto ml, auto zs) {
        constexpr int ML = decltype(ml)::value;
        // ML x kNJ tiles of 32 x 32 per wave; for a gate/up tile, column tiles [0, kNJ/2) are the
        // wave's gate columns and [kNJ/2, kNJ) the matching up columns
        floatx16_t acc[ML][kNJ];
#pragma unroll
        for (int i = 0; i < ML; ++i)
#pragma unroll
            for (int j = 0; j < kNJ; ++j) acc[i][j] = floatx16_t{};
        constexpr int ASZ = ML * ASUB, STG = ASZ + BSTAGE + XSTAGE;
        constexpr int NSR = kRing / STG, NS = NSR < kMaxStages ? NSR : kMaxStages;   // ring depth
        constexpr int A_TOT = ASZ / 1024;                             // A DMA instructions per stage
        constexpr int A_PW = (A_TOT + kGemmWaves - 1) / kGemmWaves;   // and per wave
        constexpr int PER_STAGE = A_PW + B_INSTR + (kFp4 ? 1 : 0);
        static_assert(NS >= 2 && NS * PER_STAGE < 64, "ring depth, vmcnt range");
        Frag cur, nxt;
        uint32_t so = 0, sn = STG;   // ring offsets of stage kt and of the next one
        // stage kt, the I-th of an unrolled turn; fp8 K blocks open at the stages with I * BK = 0
        // mod 128
        auto stage = [&](auto i, int kt) {
            constexpr int I = decltype(i)::value;
            constexpr bool kOpens = kFp8 && (I * BK) % 128 == 0;
            static_for<0, KS>([&](auto ks) {
                constexpr int KSI = decltype(ks)::value;
                if constexpr (KSI + 1 == KS) {
                    wait_vmcnt<(NS - 2) * PER_STAGE>();
                    wait_lgkmcnt0();
                    stage_barrier();
                    issue(ic<A_PW>{}, min(kt + NS, nk - 1), so, ASZ);
                }
                // The sub-steps before the hand-off outrank the CU's other workgroup, whose loads and
                // hand-offs then fall into this one's MFMAs: gate/up at 8192 tokens DeepSeek-V3 2.34 ->
                // 2.30 ms, DeepSeek-V4-Flash 812 -> 787 us; the other kernels lost or kept their time.
                constexpr bool kPrio = EPI == GEMM_GATEUP && (kWiden8 || kFp4);
                if constexpr (kPrio && KSI == 0) __builtin_amdgcn_s_setprio(1);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int kRescale = (kOpens && KSI == 0) ? 1 : 0;
                mma(acc, cur, ks, ml, zs, ic<kRescale>{});
                const uint8_t *st = s_ring + (KSI + 1 < KS ? so : sn);
                load_frag(st, st + ASZ, st + ASZ + BSTAGE, ic<(KSI + 1) % KS>{}, ml, zs, nxt, cur,
                          KSI + 1 < KS ? kt : min(kt + 1, nk - 1));
                interleave(ic<(KSI + 1) % KS>{}, ml, zs, ic<kRescale>{});
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (kPrio && KSI + 2 == KS) __builtin_amdgcn_s_setprio(0);
                cur = nxt;
            });
            so = sn;
            sn = sn + STG == NS * STG ? 0 : sn + STG;
        };
        if constexpr (!kEarly) {
#pragma unroll
            for (int st = 0; st < NS; ++st) issue(ic<A_PW>{}, min(st, nk - 1), st * STG, ASZ);
            wait_vmcnt<(NS - 1) * PER_STAGE>();
            wait_lgkmcnt0();
            stage_barrier();
        }
        load_frag(s_ring, s_ring + ASZ, s_ring + ASZ + BSTAGE, ic<0>{}, ml, zs, cur, cur, 0);
        for (int kt0 = 0; kt0 < nk; kt0 += kStagesPerKb)
            static_for<0, kStagesPerKb>([&](auto i) { stage(i, kt0 + decltype(i)::value); });
        wait_vmcnt<0>();   // the redundant tail stages
        if constexpr (kFp8) {
            // the accumulators hold the sum in units of the last block's scale
            const float sg = s_last[wn][0], su = s_last[wn][1];
#pragma unroll
            for (int i = 0; i < ML; ++i)
#pragma unroll
                for (int j = 0; j < kNJ; ++j) acc[i][j] *= (EPI == GEMM_GATEUP && j >= kNJ / 2) ? su : sg;
        }

        // ---- epilogue: element e of a 32 x 32 tile in lane (fn, fq) is row 8 (e / 4) + 4 fq + e % 4,
        // column fn
        if constexpr (EPI == GEMM_GATEUP && kAq) {
            // fp8 activations: h = silu(gate) * up rounded to bf16, then quantised per row over the
            // tile's 128 h columns (one 128-channel block): the row's largest |h| over the 4 waves'
            // 32 columns each, its exponent, e4m3fn codes into hq and the exponent byte into hs.
            // A lane holds column fn of rows 8 (e / 4) + 4 fq + e % 4 of each 32-row sub-tile i.
            const int nbh = I / 128;
#pragma unroll
            for (int i = 0; i < ML; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float hv = bf16_to_f32(f32_to_bf16(silu_f32(acc[i][0][e]) * acc[i][1][e]));
                    acc[i][0][e] = hv;
                    // largest |h| of the row over the 32 lanes of this half-wave
                    uint32_t m = __float_as_uint(fabsf(hv));
                    m = max(m, dpp_u32<kDppRowRor1>(m));
                    m = max(m, dpp_u32<kDppRowRor2>(m));
                    m = max(m, dpp_u32<kDppRowRor4>(m));
                    m = max(m, dpp_u32<kDppRowRor8>(m));
                    m = max(m, static_cast<uint32_t>(__shfl_xor(static_cast<int>(m), 16)));
                    if (fn == 0) s_hmax[wn][i * 32 + (e >> 2) * 8 + 4 * fq + (e & 3)] = __uint_as_float(m);
                }
            __syncthreads();
            if (t < kBM) {
                float m = s_hmax[0][t];
#pragma unroll
                for (int w = 1; w < kGemmWaves; ++w) m = fmaxf(m, s_hmax[w][t]);
                const int ex = act_scale_exp(m);
                s_hexp[t] = ex;
                if (m0 + t < len) a.wv.hs[static_cast<size_t>(beg + m0 + t) * nbh + nt] = static_cast<uint8_t>(ex + 127);
            }
            __syncthreads();
            const int col0 = nt * (kBN / 2) + wn * (kWaveCols / 2) + fn;
#pragma unroll
            for (int i = 0; i < ML; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int rl = i * 32 + (e >> 2) * 8 + 4 * fq + (e & 3);
                    if (m0 + rl < len)
                        a.wv.hq[static_cast<size_t>(beg + m0 + rl) * I + col0] =
                            static_cast<uint8_t>(e4m3_rne(ldexpf(acc[i][0][e], -s_hexp[rl])));
                }
        } else if constexpr (EPI == GEMM_GATEUP) {
            uint16_t *hout = static_cast<uint16_t *>(a.wv.h);
            const int col0 = nt * (kBN / 2) + wn * (kWaveCols / 2) + fn;
#pragma unroll
            for (int i = 0; i < ML; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = m0 + i * 32 + (e >> 2) * 8 + 4 * fq + (e & 3);
                    if (row < len) {
                        uint16_t *hrow = hout + static_cast<size_t>(beg + row) * I + col0;
#pragma unroll
                        for (int j = 0; j < kNJ / 2; ++j)
                            hrow[j * 32] = f32_to_bf16(silu_f32(acc[i][j][e]) * acc[i][j + kNJ / 2][e]);
                    }
                }
        } else {
#pragma unroll
            for (int i = 0; i < ML; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int rl = i * 32 + (e >> 2) * 8 + 4 * fq + (e & 3);
                    if (m0 + rl < len) {
                        const size_t o = static_cast<size_t>(s_tok[rl]) * H + nt * kBN + wn * kWaveCols + fn;
                        const float gw = s_gate[rl];
#pragma unroll
                        for (int j = 0; j < kNJ; ++j) unsafeAtomicAdd(a.out + o + j * 32, gw * acc[i][j][e]);
                    }
                }
        }
    };

    // the tables (gate/up: and the first stages) have landed, and the stores of the zeroing loop, which
    // must not count against the DMA waits of the main loop
    wait_vmcnt<0>();
    __syncthreads();
    bool any_zero_scale = false;
    if constexpr (kFp8)
        for (int w = 0; w < kGemmWaves; ++w) any_zero_scale |= s_zeroblk[w] != 0;
    // one instance per live sub-tile count
    static_for<1, kMI + 1>([&](auto q) {
        constexpr int ML = decltype(q)::value;
        if (mlive == ML) {
            if constexpr (kFp8) {
                if (any_zero_scale) tile(ic<ML>{}, ic<1>{});
                else tile(ic<ML>{}, ic<0>{});
            } else {
                tile(ic<ML>{}, ic<0>{});
            }
        }
    });
}

template <int WT, int EPI>
static void launch_tiles(const ExpertArgs &a, hipStream_t s) {
    const int ntn = EPI == GEMM_GATEUP ? a.I / (kBN / 2) : a.H / kBN;
    const long rows = static_cast<long>(a.T) * a.k + (a.shared ? a.T : 0);
    // upper bounds of the tiles any routing of the call can produce: large ones (full M tiles plus
    // one ragged tile per group of more than skinny_rows rows) and skinny ones
    const long large = (rows / kBM + std::min<long>(a.max_groups, rows / (a.skinny_rows + 1))) * ntn;
    const long skinny = a.skinny_rows > 0 ? static_cast<long>(a.max_groups) * (kBN / kSkinnyBN) * ntn : 0;
    const long n = large + skinny, gx = std::min(n, 1L << kGridXLog);
    const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>((n + gx - 1) / gx));
    hipLaunchKernelGGL((grouped_gemm<WT, EPI>), grid, dim3(kGemmThreads), 0, s, a, ntn);
}

template <int WT>
static hipError_t launch_gemm_wt(const ExpertArgs &a, hipStream_t s, const Prof &prof) {
    if (!prof.mark(1)) return hipErrorUnknown;
    if constexpr (WT == kWtFp8Act)   // x into e4m3fn codes and exponents
        if (hipError_t e = launch_act_quant_x(a, s); e != hipSuccess) return e;
    launch_tiles<WT, GEMM_GATEUP>(a, s);
    if (!prof.mark(2)) return hipErrorUnknown;
    launch_tiles<WT, GEMM_DOWN>(a, s);
    if (!prof.mark(3)) return hipErrorUnknown;
    return hipGetLastError();
}

hipError_t launch_gemm(const ExpertArgs &a, hipStream_t s, const Prof &prof) {
    if (a.act_quant) return launch_gemm_wt<kWtFp8Act>(a, s, prof);
    if (a.w_dtype == FT_DT_BF16) return launch_gemm_wt<FT_DT_BF16>(a, s, prof);
    if (a.w_dtype == FT_DT_MXFP4) return launch_gemm_wt<FT_DT_MXFP4>(a, s, prof);
    return launch_gemm_wt<FT_DT_FP8E4M3FN_B128>(a, s, prof);
}

// A streaming call (below kGemmMinTokens): skinny tiles for every group.  A group of more than
// kSkinnyRows rows takes one per kSkinnyRows rows, the M tiles of a weight tile next to each other
// (ceil(T / kSkinnyRows) <= 4 of them are dealt for each such group; those past its rows end at once).
// Large tiles are faster on such groups (DeepSeek-V3 200 tokens 548 against 622 us, 64 tokens 380
// either way), but their one chain of sums over K loses precision against the GEMV kernels' blocked
// sums, which calls of this size have had (error of the layer output against 64 bits at 200 tokens, rms
// of 16 inputs: 5.2e-5 against 2.1e-5).
template <int WT, int EPI>
__global__ __launch_bounds__(kGemmThreads, kGemmOcc) void skinny_gemm(ExpertArgs a, int ntn) {
    constexpr int kRing = (81920 - 8 * kSkinnyRows - 512) / 1024 * 1024;
    __shared__ __attribute__((aligned(1024))) uint8_t s_ring[kRing];
    __shared__ float s_scale[2 * 64];
    __shared__ int32_t s_tok[kSkinnyRows];
    __shared__ float s_gate[kSkinnyRows];
    if (EPI == GEMM_GATEUP && !a.wv.ypart) {
        // zero the output that the down projection accumulates into
        const size_t n4 = static_cast<size_t>(a.T) * a.H / 4;
        float4 *o4 = reinterpret_cast<float4 *>(a.out);
        for (size_t i = static_cast<size_t>(blockIdx.x) * kGemmThreads + threadIdx.x; i < n4;
             i += static_cast<size_t>(gridDim.x) * kGemmThreads)
            o4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const int mtm = (a.T + kSkinnyRows - 1) / kSkinnyRows;
    const int G = scalar_load(a.wv.grp_meta), GL = scalar_load(a.wv.grp_meta + 5);
    const int nlarge = GL * mtm * ntn, nskinny = (G - GL) * ntn;
    if (static_cast<int>(blockIdx.x) >= nlarge + nskinny) return;
    const int L = __builtin_amdgcn_readfirstlane(mixed_tile(blockIdx.x, nlarge, nskinny));
    const int g = L < 0 ? GL + ~L / ntn : L / (mtm * ntn);
    const int nt = L < 0 ? ~L % ntn : L / mtm % ntn, m0 = L < 0 ? 0 : L % mtm * kSkinnyRows;
    const int slot = scalar_load(a.wv.grp_slot + g), beg = scalar_load(a.wv.grp_beg + g);
    const int len = scalar_load(a.wv.grp_len + g) - m0;
    if (len <= 0) return;
    skinny_tile<WT, EPI, kRing>(a, slot, beg + m0, min(len, kSkinnyRows), nt, s_ring, s_scale, s_tok, s_gate);
}

hipError_t launch_skinny(const ExpertArgs &a, hipStream_t s, bool down) {
    // upper bound of the tiles: every group (max_groups), or every row beyond kSkinnyRows a group
    const long rows = static_cast<long>(a.T) * a.k + (a.shared ? a.T : 0);
    const long mtm = (a.T + kSkinnyRows - 1) / kSkinnyRows;
    const long large = std::min<long>(a.max_groups, rows / (kSkinnyRows + 1));
    const int ntn = down ? a.H / kSkinnyBN : 2 * a.I / kSkinnyBN;
    const dim3 grid(static_cast<unsigned>((large * mtm + a.max_groups) * ntn)), blk(kGemmThreads);
    auto go = [&](auto wt) {
        constexpr int WT = decltype(wt)::value;
        if (down) hipLaunchKernelGGL((skinny_gemm<WT, GEMM_DOWN>), grid, blk, 0, s, a, ntn);
        else hipLaunchKernelGGL((skinny_gemm<WT, GEMM_GATEUP>), grid, blk, 0, s, a, ntn);
    };
    if (a.w_dtype == FT_DT_BF16) go(ic<FT_DT_BF16>{});
    else if (a.w_dtype == FT_DT_MXFP4) go(ic<FT_DT_MXFP4>{});
    else go(ic<FT_DT_FP8E4M3FN_B128>{});
    return hipGetLastError();
}

}  // namespace ftmoe
