// cmoe_internal.h - device layout and kernel launchers shared by the HIP
// translation units of libcmoe.so.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cmoe {

constexpr int kNctr = 5;          // per (stream, layer) counters: A, hits, D, P, T
constexpr int kCtrA = 0, kCtrHits = 1, kCtrD = 2, kCtrP = 3, kCtrT = 4;
constexpr int kMaxN = 256;        // experts per layer handled by the kernels
constexpr int kMaxK = 64;         // Top-K handled by the kernels (one lane per selected expert)
constexpr int kMaxSplit = 4;         // router split-K partials per logit, at most
constexpr int kRouterWaves = 4;      // router: wavefronts per workgroup, one k sub-range each
constexpr int kMaxBatch = 64;        // layers of one batch (one launch of each phase), at most
// workgroups of a copy launch: out of an HBM pool (measured with the copy
// kernel's pieces), and over the host link, which many readers slow down:
// pieces of 32 KB with 128, 96, 64, 48 and 40 workgroups take 284, 281, 277, 276
// and 275 us (one layer of the 128-expert shape at one stream, about one expert
// of 9.4 MB, 280 with one 16-byte load per thread in source order before), 12.00,
// -, 11.90, 11.88 and 11.94 ms (16 experts of 37.7 MB, 11.98 before); pieces of
// 16 or 64 KB 11.84 or 12.11 ms and 313 or 297 us
constexpr int kCopyBlocksDevice = 512, kCopyBlocksHost = 48;
// FFN work unit: up to this many of an expert's tokens: 64 with one wavefront
// per workgroup, 128 in the grouped launch (whose workgroups stage the
// activations in LDS for the four row tiles).  In bf16 a unit is one pass over
// the expert's weights; in fp32 one for every 32 of its tokens
constexpr int kUnitTokens = 64, kUnitTokensGrouped = 128;
// grouped bf16 shape: units of more than this many tokens have launches of
// their own, whose wavefronts take two row tiles
constexpr int kLightTokens = 32;

// Every pointer the kernels use, carved out of the caller's buffers.
struct Layout {
    int32_t L, N, K, d, F, C, S, mode, dtype, NW, n_slots, n_r, nsplit, rdk, warmup;
    int32_t G;             // layers per batch: the per-batch buffers below hold G layers
    int32_t iT, iS;        // router slot of the Temporal / Spatio Router, -1 if not used
    int32_t max_units;     // entries of units per layer step: max_heavy, then min(N, S K); without
                           // max_heavy min(N, S K) + S K / unit_tokens
    int32_t max_heavy;     // units of more than kLightTokens tokens per layer step, at most
                           // S K / (kLightTokens + 1) (grouped bf16 shape with many tokens per
                           // expert; else 0): the first max_heavy entries of units
    int32_t unit_tokens;   // tokens per work unit: kUnitTokens, or kUnitTokensGrouped (grouped launch)
    int32_t ffn_waves;     // wavefronts per bf16 FFN workgroup: 1, or 4 (grouped: units of more
                           // than 16 tokens share their activations through LDS)
    int32_t xcd_units;     // 1: the bf16 FFN grids put each work unit's workgroups on one XCD,
                           // 0: on all XCDs in turn
    int32_t policy;        // retention priority (cmoe_policy)
    float lrfu_w;          // LRFU decay per token, fl32(2^-lambda)
    int64_t expert_elems;  // 3 d F
    // weights: router slot r (0 native, then temporal, then spatio, as used)
    const void* rw[3];
    const float* bias;
    const void* pool;
    int32_t pool_host;     // 1: the pool is pinned host memory read over the host link
    // arena: [L][n_slots] experts
    void* arena;
    // state
    unsigned long long* cache;  // [S][L][NW]  cache membership bits
    float* aT;                  // [S][L][N]   previous token's a-score: s^T (full mode),
                                //             p^R (Spatio-only mode)
    float* pol;                 // [S][L][N]   classical retention priority
    float* pS;                  // [2][S][N]   Spatio Router distribution of the last layer of the
                                //             latest two batches (by batch parity)
    unsigned long long* mid;    // [L][S][NW]  cache membership after the token's refinement
    int64_t* ctr;               // [S][L][kNctr]
    int64_t* phys;              // [L][2]      physical fills: demand, proactive
    unsigned long long* active_sum;  // [L]    distinct experts executed (counted tokens)
    unsigned long long* selcount;    // [L][N] native selections per expert (counted tokens)
    int32_t* slot_of;           // [L][N]      slot of each expert, -1 absent
    int32_t* slot_exp;          // [L][n_slots] expert in each slot, -1 free
    int32_t* slot_stamp;        // [L][n_slots] arena clock at the last use of each slot's expert
    int32_t* snap_of;           // [N]         slot_of and slot_exp of the layer that a fill launch
    int32_t* snap_exp;          // [n_slots]   handles, as the cache step before it found them
    int32_t* copy_list;         // [L][2][N]   the last residency launch's copies, demand and proactive:
                                //             (slot << 8) | expert
    int32_t* copy_n;            // [L][2]      their numbers
    // workspace
    double* zpart;              // [G][S][n_r][nsplit][N] router partial sums
    float* logits;              // [L][S][n_r][N]
    int32_t* sel;               // [L][S][K]
    float* gates;               // [L][S][K]
    int32_t* events;            // [L][S][4]   hits, D, P, 0 of the last token
    int32_t* step_fills;        // [L][2]      physical fills of the last token
    int32_t* bcount;            // [G][N]      tokens per expert; zero between batches
    int32_t* pairs;             // [G][N][S]   (stream << 8) | k of each token of an expert
    void* act;                  // [G][S][K][F] SwiGLU intermediate (dtype)
    void* yp;                   // [G][S][K][d] gated expert outputs (dtype)
    int32_t* units;             // [G][max_units][4] FFN work units of the current round:
                                //             {(pass << 8) | expert, slot, tokens, 0}, the big ones
                                //             from entry 0, the others from entry max_heavy, each list
                                //             heaviest first if some bucket takes several passes;
                                //             {-1, -1, 0, 0} past the end of a list
    int32_t* round_of;          // [G][N]      FFN round of each expert executed by the layer
                                //             step, -1 if not executed
};

// cache-step kernel flags
constexpr uint32_t kFlagInject = 1u;  // logits come from the caller
constexpr uint32_t kFlagRefine = 2u;  // refine each layer before its access (modes with a Spatio Router)
constexpr uint32_t kFlagCount = 4u;   // this token is counted

// The cache step of layers l0 .. l0 + nl - 1 (one batch).
struct StepArgs {
    int32_t l0, nl;
    int32_t R;          // refinement budget
    int32_t psw;        // pS buffer this batch writes (it reads the other one)
    uint32_t flags;
    int32_t t;          // token index (LRU clock)
    int32_t snap;       // copy layer l0's slot maps for the fill launch that follows
    const float* z[3];  // injected logits [S][L][N] per router slot (kFlagInject)
};

// The residency events of layers l0 .. l0 + nl - 1 (one batch), or one round
// of them: each layer's arena must hold the union of the streams' caches, or,
// when the union does not fit, the experts of this FFN round.
struct ResidencyArgs {
    int32_t l0, nl;
    int32_t refined;  // round 0: the proactive event (caches after the refinement) comes first
    int32_t round;    // FFN round of the layer step (0 plans the rounds)
    int32_t counted;
    int32_t units;    // lay out the FFN work units of this round
    int32_t last;     // last round: the bucket counts are zeroed for the next batch
    int32_t clk;      // arena clock: the last use the first event stamps (the demand event after it: clk + 1)
};

// Optional timing of one launch: with events, they take the kernel's own
// start and end timestamps (hipExtLaunchKernel), not those of markers
// recorded on the stream around the launch.
struct Timing {
    hipEvent_t start = nullptr, stop = nullptr;
};

template <typename... KArgs, typename... Args>
inline void launch_kernel(void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t st, const Timing& tm,
                          Args... args) {
    if (tm.start)
        hipExtLaunchKernelGGL(kernel, grid, block, 0, st, tm.start, tm.stop, 0, args...);
    else
        hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
}

hipError_t launch_init(const Layout& lo, hipStream_t st);  // state, and the workspace if bound
// router logits of layers l0 .. l0 + nl - 1; dirty: also zeroes the batch's bucket counts
hipError_t launch_router(const Layout& lo, int l0, int nl, const void* h, bool dirty, hipStream_t st,
                         const Timing& tm = {});
hipError_t launch_cache_step(const Layout& lo, const StepArgs& a, hipStream_t st, const Timing& tm = {});
hipError_t launch_residency(const Layout& lo, const ResidencyArgs& f, hipStream_t st, const Timing& tm = {});
// the demand event of layer f.l0 (nl 1, not refined, n_slots enough for the union
// of the caches) and its copies in one launch
hipError_t launch_fill(const Layout& lo, const ResidencyArgs& f, hipStream_t st, const Timing& tm = {});
// the copies the last residency launch listed for layers l0 .. l0 + nl - 1;
// kind: 0 demand, 1 proactive
hipError_t launch_copies(const Layout& lo, int l0, int nl, int kind, hipStream_t st, const Timing& tm = {});
// the FFN round of layers l0 .. l0 + nl - 1, numbers b0 .. of their batch; with
// max_heavy > 0 a launch of its own (heavy) for the big units comes first
hipError_t launch_ffn_up(const Layout& lo, int l0, int b0, int nl, const void* h, hipStream_t st, const Timing& tm = {},
                         const Timing& heavy = {});
hipError_t launch_ffn_down(const Layout& lo, int l0, int b0, int nl, hipStream_t st, const Timing& tm = {},
                           const Timing& heavy = {});
// the combine of layers l0 .. l0 + nl - 1
hipError_t launch_combine(const Layout& lo, int l0, int nl, float* y, hipStream_t st, const Timing& tm = {});
// streaming read of the read_probe_bytes(bytes) bytes at src: the largest
// multiple of the probe's block size within `bytes`
int64_t read_probe_bytes(int64_t bytes);
hipError_t launch_read_probe(const void* src, int64_t bytes, hipStream_t st, const Timing& tm);

}  // namespace cmoe
