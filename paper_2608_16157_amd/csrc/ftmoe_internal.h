// Internal host/device interface of libftmoe: argument bundles, workspace layout, launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <condition_variable>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

#include "ftmoe.h"

namespace ftmoe {

constexpr int kMaxExperts = 1024;
constexpr int kMaxTopK = 64;
constexpr int kTokPerBlk = 16;          // tokens per workgroup in the multi-block router
constexpr int kBlkPerPart = 16;         // router blocks per part of its scan (the part table)
constexpr int kMaxPlaceBlks = 256;      // router blocks up to which route_place takes the scan and the scatter
constexpr int kFusedMaxPairs = 2048;    // T*k handled by the single-workgroup router
constexpr int kFusedMaxLds = 64 * 1024;
constexpr int kGemmBM = 128;            // token rows per MFMA GEMM tile
constexpr int kGemmBN = 256;            // weight rows per MFMA GEMM tile
constexpr int kSkinnyRows = 64;         // most token rows of a skinny tile (skinny_tile.h)
constexpr int kSkinnyMinTokens = 4;     // fewest tokens of a call that takes skinny tiles (skinny_path)
constexpr int kGemmMinTokens = 256;     // token count from which the matrix-core path's workspace and combine are used

struct HostMailbox;   // a worker pool's device <-> host mailbox (defined with CpuPool)

// Routing outputs (the caller's ft_route_t, flattened).
struct RouteOut {
    int32_t *topk_ids;
    float *topk_w;
    int32_t *topk_slot;
    int32_t *hit_pairs;
    int32_t *miss_pairs;
    int32_t *hit_off;
    int32_t *miss_off;
    int32_t *counts;
};

// Views into the caller's workspace.
//  rows: the hit list positions 0..n_hit-1 followed by T rows of the shared expert; row r
//  evaluates token row_tok[r] with gate row_gate[r].  Groups: one per hit expert and one of the shared
//  expert; group g covers rows [grp_beg[g], +grp_len[g]) and reads the weights of bank row grp_slot[g].
//  Rows are in expert order, groups are not: those of more than skinny_rows rows come first (the shared
//  expert's ahead of them), then the skinny ones (the shared expert's last).  Inside either kind the
//  order is that of the experts, or of cost classes (scan_experts).  The one-wave router of one or two
//  tokens keeps expert order with the shared expert last, and writes neither the M tile map (grp_mt_off,
//  mt_group) nor grp_meta[4] and [5]: no call that small runs a kernel that reads them.
struct WsView {
    int32_t *eff_slot;   // [E] (written and read by the four-launch router only)
    int32_t *blk_hist;   // [nblk][E] per-block expert counts, then [ceil(nblk / kBlkPerPart)][E] part sums
    int32_t *grp_meta;   // [8]: G (groups incl. shared), U (hit groups), n_hit, T, M tiles, first skinny group
    int32_t *grp_slot;   // [E+1]
    int32_t *grp_beg;    // [E+1]
    int32_t *grp_len;    // [E+1]
    int32_t *grp_mt_off; // [E+2] exclusive prefix of ceil(len / kGemmBM) over the groups that are not skinny
    int32_t *mt_group;   // [max M tiles] group of each GEMM M tile
    int32_t *row_tok;    // [T*k + T]
    float *row_gate;     // [T*k + T]
    int32_t *row_pair;   // [T*k + T] pair index p = t*k + j of the row (T*k + t for the shared rows)
    void *h;             // [T*k + T][I] SwiGLU activations (bf16, or f32 for f32 weights)
    float *ypart;        // streaming path: [T*k + T][H] gate-weighted expert outputs by pair
                         // index, summed per token in a fixed order by the combine (else null)
    // fp8 activations (FT_ACT_FP8_1x128_POW2), else null.  Matrix-core path: x and h as e4m3fn
    // codes with one e8m0 exponent byte (e + 127) per token (row) and 128-channel block.
    // Streaming path: x quantised and widened back to bf16 (h is quantised in place).
    uint8_t *xq;         // [T][H]
    uint8_t *xs;         // [T][H/128]
    uint8_t *hq;         // [T*k + T][I]
    uint8_t *hs;         // [T*k + T][I/128]
    uint16_t *xd;        // [T][H] bf16
};

struct RouteArgs {
    const float *logits;
    const int32_t *slot_table;
    int T, E, k, gating, n_slots, shared_slot, nbits, scan_parts;
    int skinny_rows;   // groups of up to this many rows are skinny: numbered last, without M tiles
    RouteOut ro;
    WsView wv;
};

struct ExpertArgs {
    const void *w13;
    const void *w2;
    const void *s13;   // float32 block scales (fp8) or uint8 e8m0 scales (MXFP4)
    const void *s2;
    const void *x;
    float *out;
    int T, H, I, k, w_dtype, n_slots, shared;
    int act_quant;    // FT_ACT_*
    int max_groups;   // upper bound on groups, known on the host
    int skinny_rows;  // matrix-core path: groups of up to this many rows go to the skinny tiles
    // routing of a one- or two-token call done by the gate/up kernel itself (logits != nullptr;
    // otherwise the router ran before and the workspace holds its groups)
    const float *logits;
    const int32_t *slot_table;
    int E, gating, shared_slot, nbits;
    RouteOut ro;
    WsView wv;
};

struct WsLayout {
    size_t eff_slot, blk_hist, grp_meta, grp_slot, grp_beg, grp_len, grp_mt_off, mt_group, row_tok,
        row_gate, row_pair, h, ypart, ypart_bytes, xq, xs, hq, hs, xd, total;
};

// Whether a call of T tokens runs the matrix-core GEMM path (many tokens, shapes that tile);
// the launcher additionally needs at least one evaluation group.
inline bool gemm_shape(int T, int H, int I, int w_dtype) {
    if (w_dtype == FT_DT_F32) return false;
    return T >= kGemmMinTokens && H % kGemmBN == 0 && I % (kGemmBN / 2) == 0 && H <= 8192 && I <= 8192;
}

// Whether a projection of a streaming call of T tokens runs the skinny tiles (gemm.hip) instead of the
// GEMV kernels; the two form the same sums in the same order.  The tiles win where groups hold enough
// rows, or (MXFP4) the activations are large beside the weights, for their activations are read once
// per 128 weight rows.  Measured per projection, GEMV against tiles in us: bf16 (Qwen3) gate/up 32
// tokens 45 against 52, 64: 64.1 / 63.7, 72: 69.6 / 67.1, 160: 111 / 83, down 32: 27.8 / 27.5, 40:
// 32.1 / 29.0, 160: 81 / 41; fp8 (DeepSeek-V3) gate/up 16: 152 / 156, 18: 163 / 162, 64: 265 / 239, down
// 16: 81 / 82, 20: 91 / 86; MXFP4 (DeepSeek-V4-Flash) layer 3: 55.5 / 55.7, 5: 64.3 / 58.3, 32: 117 / 101;
// its down projection alone at 4 and 6 tokens -2 and -4 % of the layer, at 7 +1 % (4096 x 7168, 8 experts: 4
// tokens -13 %, 7: +1 %).  Over 15 more layer shapes (8 to 1024 experts, uniform and Zipf 1.2 routing) the
// limits hold to within 5 % of the layer, but for weight rows a multiple of 4096 bytes apart: the 128 row
// pieces of a stage then begin in the same few memory channels.  There, in % of the layer, uniform /
// Zipf routing: fp8 H = 4096 (3968, 4224: 0 to +6) gate/up 24 tokens -11 / -14, 64: -8 / -2, 96: -8 / +4, 128:
// -7 / +7; bf16 H = 2048 (1920, 2176: +2 to +13) 65: -5 / -5, 96: -5 / +4, 192: -3 / +15; MXFP4 I = 8192 down 10:
// -15 / -18, 64: -7 / 0, 128: -7 / +32.  The bf16 down projection keeps its limit (I = 2048, 33: -2 / +2, 65: 0 / +5).
// Below, K is the projection's (H, or I of the down projection); it is bounded by the tiles' table of
// fp8 scales and their 32-bit weight offsets.
inline bool skinny_path(int T, int H, int I, int w_dtype, bool down) {
    if (w_dtype == FT_DT_F32 || T >= kGemmMinTokens || H > 8192 || I > 8192) return false;
    const bool bf16 = w_dtype == FT_DT_BF16, fp4 = w_dtype == FT_DT_MXFP4;
    const int K = down ? I : H, row_bytes = bf16 ? 2 * K : fp4 ? K / 2 : K;
    if (row_bytes % 4096 == 0 && !(bf16 && down)) return T >= 96;
    return T >= (bf16 ? (down ? 33 : 65) : fp4 ? (down ? 7 : kSkinnyMinTokens) : 17);
}
// Group rows up to which a group goes to the skinny tiles (the fp8 x fp8 kernels have none).
inline int skinny_rows_of(int T, int act_quant) {
    return act_quant != FT_ACT_EXACT && T >= kGemmMinTokens ? 0 : kSkinnyRows;
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Upper bound of the GEMM M tiles any routing of T tokens can produce: every row in full tiles
// plus one ragged tile per group (E routed groups and the shared expert).
inline size_t gemm_max_mtiles(int T, int k, int E) {
    const size_t rows = static_cast<size_t>(T) * k + T;
    return (rows + kGemmBM - 1) / kGemmBM + E + 1;
}

inline WsLayout ws_layout(int E, int H, int I, int k, int w_dtype, int combine, int act_quant, int T) {
    WsLayout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + bytes, 256);
        return at;
    };
    const size_t nblk = (static_cast<size_t>(T) + kTokPerBlk - 1) / kTokPerBlk;
    const size_t rows = static_cast<size_t>(T) * k + T;
    L.eff_slot = take(4u * E);
    const size_t nparts = (nblk + kBlkPerPart - 1) / kBlkPerPart;
    L.blk_hist = take(4u * (nblk + nparts) * E);
    L.grp_meta = take(32);
    L.grp_slot = take(4u * (E + 1));
    L.grp_beg = take(4u * (E + 1));
    L.grp_len = take(4u * (E + 1));
    L.grp_mt_off = take(4u * (E + 2));
    L.mt_group = take(4u * gemm_max_mtiles(T, k, E));
    L.row_tok = take(4u * rows);
    L.row_gate = take(4u * rows);
    L.row_pair = take(4u * rows);
    const bool aq = act_quant == FT_ACT_FP8_1x128_POW2, gemm = gemm_shape(T, H, I, w_dtype);
    // the fp8-activation matrix-core path keeps h only as codes (hq, hs)
    L.h = take(aq && gemm ? 0 : rows * I * (w_dtype == FT_DT_F32 ? 4u : 2u));
    L.ypart_bytes = (gemm || combine != FT_COMBINE_ORDERED) ? 0 : rows * H * 4u;
    L.ypart = take(L.ypart_bytes);
    L.xq = take(aq && gemm ? static_cast<size_t>(T) * H : 0);
    L.xs = take(aq && gemm ? static_cast<size_t>(T) * (H / 128) : 0);
    L.hq = take(aq && gemm ? rows * I : 0);
    L.hs = take(aq && gemm ? rows * (I / 128) : 0);
    L.xd = take(aq && !gemm ? static_cast<size_t>(T) * H * 2 : 0);

    L.total = o;
    return L;
}


// Optional stage events of ft_moe_forward_profiled (recorded only when given).
struct Prof {
    const ft_prof_events_t *ev;
    hipStream_t s;
    Prof(const ft_prof_events_t *e, hipStream_t st) : ev(e), s(st) {}
    bool mark(int i) const {
        if (!ev || !ev->ev[i]) return true;
        return hipEventRecord(static_cast<hipEvent_t>(ev->ev[i]), s) == hipSuccess;
    }
};

// Device-side cache control of one layer step (cache.hip).
constexpr int kPlanMaxFill = 64;      // most LRU candidates (K) per step
constexpr int kPlanMaxSlots = 4096;   // most cache slots the planner handles

struct PlanArgs {
    int E, k, n_slots, shared_slot, K;
    double b_pcie, b_host;
    uint32_t step;
    uint32_t *clock;   // device step counter, or null (then `step` is the stamp)
    const int32_t *hit_off, *miss_off, *miss_pairs, *route_counts;
    int32_t *topk_slot;
    int32_t *slot_table, *slot_expert;
    uint32_t *slot_stamp;
    int32_t *fill_expert, *fill_slot, *evict_expert, *cpu_expert, *counts;
};

// Cache fills and the exact merge (fill.hip).
constexpr size_t kFillChunk = 64 * 1024;   // bytes of one bank row a fill block copies
struct FillArgs {
    int E, n_slots;
    const int32_t *plan_counts, *fill_expert, *fill_slot;
    const uint8_t *host[4];   // pinned host pool (device-visible addresses): w13, w2, s13, s2
    uint8_t *dev[4];          // device banks
    size_t row_bytes[4];      // bytes of one expert's row in each bank (0 = bank absent)
};
hipError_t launch_cache_fill(const FillArgs &a, int max_fill, hipStream_t s);
hipError_t launch_add_partial(float *out, const float *other, size_t n, hipStream_t s);
// Host staging of a hybrid step (device-visible addresses of pinned host buffers).
struct StageArgs {
    const int32_t *counts, *cpu_expert, *topk_ids;
    const float *topk_w;
    const void *x;
    int32_t *h_counts, *h_cpu, *h_ids;
    float *h_w;
    void *h_x;
    int E;
    size_t pk, x16;   // routed pairs; 16-byte chunks of x (x rows are 16-byte multiples)
};
hipError_t launch_stage_host(const StageArgs &a, hipStream_t s);
// Post a task to a pool's mailbox (device side), and wait until the pool reports it done.
hipError_t launch_mailbox_post(HostMailbox *mbox_dev, uint64_t task, hipStream_t s);
hipError_t launch_mailbox_wait(HostMailbox *mbox_dev, hipStream_t s);

// Bytes of one expert in each bank (w13, w2, s13, s2) for a weight dtype; H, I multiples of 128.
struct ExpertBytes {
    size_t w13, w2, s13, s2;
};
inline ExpertBytes expert_bytes(int w_dtype, size_t H, size_t I) {
    switch (w_dtype) {
        case FT_DT_F32: return {2 * I * H * 4, H * I * 4, 0, 0};
        case FT_DT_BF16: return {2 * I * H * 2, H * I * 2, 0, 0};
        case FT_DT_FP8E4M3FN_B128: return {2 * I * H, H * I, (2 * I / 128) * (H / 128) * 4, (H / 128) * (I / 128) * 4};
        default: return {I * H, H * I / 2, 2 * I * (H / 32), H * (I / 32)};   // MXFP4
    }
}
inline bool has_scales(int w_dtype) { return w_dtype == FT_DT_FP8E4M3FN_B128 || w_dtype == FT_DT_MXFP4; }

// Every host-checkable condition of ft_moe_forward (FT_OK when the call would be enqueued).
ft_status_t check_forward(const ft_moe_desc_t *desc, const ft_banks_t *banks, const float *logits,
                          const int32_t *slot_table, const void *x, int32_t T, const float *out_partial,
                          const ft_route_t *route, const void *ws, size_t ws_bytes);

// Mailbox of a worker pool in pinned host memory, written by the device and the pool's listener
// thread: the device posts a step (task pointer, then a new sequence number), the listener runs
// the task and echoes the number into `done`, which a device kernel waits for.
struct alignas(64) HostMailbox {
    uint64_t posted;     // last posted sequence number (device writes)
    uint64_t task;       // host address of the posted step's task (device writes)
    uint64_t done;       // last finished sequence number (listener writes)
    uint64_t timeouts;   // device waits that gave up (device writes)
};

// The CPU branch's persistent worker pool (host_experts.cpp), behind the opaque ft_cpu_pool_t.
struct CpuPool {
    struct Job {
        int n;
        const std::function<void(int, std::vector<float> &)> &fn;
    };
    std::vector<std::thread> workers;
    std::vector<int> cpus;        // CPU each worker is pinned to, -1 if not pinned
    std::mutex mu, run_mu;
    std::condition_variable cv_work, cv_done;
    const Job *current = nullptr;
    uint64_t gen = 0;             // job generation
    std::atomic<int> next{0};     // next work item of the current job
    int busy = 0;                 // workers not yet done with the current job
    bool stop = false;
    // the listener thread polls the mailbox and runs each posted task (through run())
    std::thread listener;
    std::atomic<bool> quit{false};
    HostMailbox *mbox = nullptr;       // pinned host memory
    HostMailbox *mbox_dev = nullptr;   // its device-visible address
    void (*task_fn)(void *) = nullptr; // what a posted task runs
    static CpuPool *create(int n_threads, bool pin, void (*task_fn)(void *));
    ~CpuPool();
    void run(int n_items, const std::function<void(int, std::vector<float> &)> &fn);
    void worker_loop();
    void listen_loop();
};

// CPU branch of a layer step (host_experts.cpp).
struct CpuBank {
    const void *w;       // one expert's matrix, row-major
    const void *s;       // its fp8 block scales (float32) or MXFP4 scales (uint8), or null
};
struct CpuExpertArgs {
    int E, H, I, k, T, w_dtype, x_dtype, n_list;
    CpuPool *pool;                   // workers, or null: the calling thread alone
    const void *w13, *w2;            // host expert pool, [E][2I][H] and [E][H][I]
    const void *s13, *s2;            // fp8 / MXFP4 scales per expert, or null
    const void *x;                   // [T][H]
    const int32_t *topk_ids;         // [T][k]
    const float *topk_w;             // [T][k]
    const int32_t *list;             // experts to evaluate (distinct ids)
    float *out;                      // [T][H], overwritten
};
void cpu_experts(const CpuExpertArgs &a);

// Evaluation groups of a hybrid step from its routing after the cache plan (route.hip).
struct RegroupArgs {
    int E, T, k, shared_slot, skinny_rows;
    const int32_t *hit_off, *miss_off, *hit_pairs, *miss_pairs, *topk_slot;
    const float *topk_w;
    WsView wv;
};
hipError_t launch_regroup(const RegroupArgs &a, hipStream_t s);

hipError_t launch_route(const RouteArgs &a, hipStream_t s);
hipError_t launch_cache_plan(const PlanArgs &a, hipStream_t s);
hipError_t launch_experts(const ExpertArgs &a, hipStream_t s, const Prof &prof);
hipError_t launch_gemm(const ExpertArgs &a, hipStream_t s, const Prof &prof);
hipError_t launch_skinny(const ExpertArgs &a, hipStream_t s, bool down);
// fp8 activations (quant.hip): x into codes and exponents (matrix-core path) or into quantised
// bf16 (streaming path); h quantised in place (streaming path)
hipError_t launch_act_quant_x(const ExpertArgs &a, hipStream_t s);
hipError_t launch_act_quant_h(const ExpertArgs &a, hipStream_t s);

}  // namespace ftmoe
