// ffn.hip - the SwiGLU expert FFN over the resident expert weights
// ("execute the MoE layer", Algorithm 2), grouped by expert:
//   a_e = silu(W_gate,e x) * (W_up,e x),  y_(s,k) = g_(s,k) W_down,e a_e,
//   y_s = sum_k y_(s,k)  (k in ascending order).
// Each expert's weights are read from its HBM slot once per work unit (a
// pass over up to 64 or 128 of its tokens; nearly every expert needs one; in
// fp32 a unit of more than 32 tokens takes several passes), so the layer step
// streams about |union of selected experts| x expert_bytes: the kernels are
// HBM-bound.
//
// bf16: one wavefront per 16 rows of W_gate and of W_up (gate/up kernel) or
// per 32 rows of W_down (down kernel), one wavefront per workgroup or four
// (grouped: consecutive row tiles of one unit, units of more than 16 tokens
// sharing their activations through LDS; with many tokens per expert the big
// units run in launches of their own, two row tiles per wavefront), on the
// bf16 matrix core
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation).  The expert's tokens form the
// 16 columns of the B operand (groups of 16 tokens; several groups reuse the
// loaded weights).  Per 64-wide k chunk, lane (r, g) of the A operand holds
// W[row r][kc + 8 g .. + 8] and W[row r][kc + 32 + 8 g .. + 8]; the two MFMAs
// of a chunk take k-slots kc + 8 g + {0..7} and kc + 32 + 8 g + {0..7}, the
// same for both operands.  Each activation load of a wavefront on its own
// (units of up to 16 tokens) thus reads one contiguous 64-byte half of a
// token's 128-byte k chunk; shared activations are loaded in whole chunks.
// The weights come from the expert's HBM slot in packed order (the copy
// kernel writes it so): each A operand load of a wavefront reads one
// contiguous kilobyte and each wavefront streams one contiguous block.  The
// SwiGLU intermediate is stored in bf16 (the input type of the down kernel's
// matrix core).
//
// fp32: the same units on the fp32 matrix core, in passes of up to 32 tokens
// one after another, over transposed weights (the copy kernel writes them so).
#include "cmoe_internal.h"

namespace cmoe {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kNG = 4;          // token groups (of 16) per pass when a unit holds more than 16
static_assert(kUnitTokens == 16 * kNG, "one work unit is one pass over the weights");
constexpr int kUnroll = 4;      // k chunks per load block, one token group
constexpr int kUnrollSolo = 1;  // k chunks per load block, kNG token groups in one wavefront: this
                                // path is rare in the launches that use it, and a deeper block would
                                // set the register budget (and so the occupancy) of the whole kernel
constexpr int kWaves = 4;       // wavefronts per grouped or heavy workgroup, on consecutive row tiles of one unit
static_assert(kUnitTokensGrouped == 128, "the widest heavy pass takes eight token groups");

__device__ inline bf16x8 as_bf16x8(uint4 v) {
    bf16x8 r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}

// Expert weights are read once per layer step and never again from cache:
// stream them with nontemporal loads (measured on MI355X for this access
// pattern, one contiguous block per wavefront: 7.0 TB/s against 6.1 TB/s
// for ordinary loads).
__device__ inline uint4 load_stream(const uint4* p) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return uint4{v.x, v.y, v.z, v.w};
}

__device__ inline f32x4 mfma_bf16(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}

__device__ inline float silu_mul(float g, float u) { return g / (1.0f + __expf(-g)) * u; }

__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
    // round to nearest even
    uint32_t a = __float_as_uint(lo), b = __float_as_uint(hi);
    a += 0x7FFFu + ((a >> 16) & 1u);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return (a >> 16) | (b & 0xFFFF0000u);
}

// Gated output of (stream s, slot k) at d-rows j .. j + 3 (c0) and
// j + 16 .. j + 19 (c1), rounded to bf16 like the SwiGLU intermediate: the
// combine adds them in fp32.
__device__ inline void store_gated(const Layout& lo, int bl, int s, int k, int j, float gk, const f32x4& c0, const f32x4& c1) {
    uint16_t* dst = reinterpret_cast<uint16_t*>(lo.yp) + (((int64_t)bl * lo.S + s) * lo.K + k) * lo.d + j;
    *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(gk * c0[0], gk * c0[1]), pack_bf16x2(gk * c0[2], gk * c0[3]));
    *reinterpret_cast<uint2*>(dst + 16) =
        make_uint2(pack_bf16x2(gk * c1[0], gk * c1[1]), pack_bf16x2(gk * c1[2], gk * c1[3]));
}

// The FFN grids take a batch of layers (y), so that the next layer's first
// workgroups run beside this layer's last ones.  Per layer they hold wgn
// workgroups per work unit; consecutive workgroups go
// to the eight XCDs in turn.  With xcd_units, workgroup b takes unit
// u = 8 (q / wgn) + b % 8 and part q % wgn of it, q = b / 8, so that all the
// workgroups of a unit have the same b % 8: a unit runs on one XCD and its
// tokens' activations are fetched into one L2 instead of eight.  Each XCD
// takes every eighth unit of the list (heaviest first if some bucket takes
// several units, else in expert order).  That grid is rounded
// up to whole groups of eight units; u may exceed the last unit.  Without
// it, workgroup b takes unit b / wgn, part b % wgn, and every unit is spread
// over all XCDs: with few tokens per expert there is little to share, and
// whole units per XCD were measured to stream the weights more slowly (up to
// 15% at one token per expert).
__device__ inline void unit_of_block(int b, int wgn, bool xcd, int& u, int& j) {
    if (xcd) {
        const int q = b >> 3, g = q / wgn;
        u = g * 8 + (b & 7);
        j = q - g * wgn;
    } else {
        u = b / wgn;
        j = b - u * wgn;
    }
}

inline int unit_groups(const Layout& lo, int units) { return lo.xcd_units ? (units + 7) / 8 * 8 : units; }

__device__ inline const uint16_t* slot_base(const Layout& lo, int l, int slot) {
    return reinterpret_cast<const uint16_t*>(lo.arena) + ((int64_t)l * lo.n_slots + slot) * lo.expert_elems;
}

// The SwiGLU intermediate [S][K][F] of layer bl of the batch.
template <typename T>
__device__ inline T* act_base(const Layout& lo, int bl) {
    return static_cast<T*>(lo.act) + (int64_t)bl * lo.S * lo.K * lo.F;
}

// U consecutive 64-wide k chunks of one 16-row (gate/up) or 2 x 16-row (down)
// weight tile against NG groups of 16 token columns.  All weight and
// activation loads of the block are issued before the first matrix-core
// instruction, so a wavefront waits once per block.  Token columns past the
// bucket (also whole groups past it in the last pass) repeat the bucket's last
// token and their output columns are discarded: column j of the product
// depends on column j of B only.
template <int NG, int U>
__device__ inline void mfma_block(const uint4* __restrict__ tile, int c, const uint16_t* const* xb, f32x4* acc0,
                                  f32x4* acc1) {
    uint4 A[U][4], X[NG][U][2];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const uint4* ch = tile + (int64_t)(c + i) * 256;
        A[i][0] = load_stream(ch);
        A[i][1] = load_stream(ch + 64);
        A[i][2] = load_stream(ch + 128);
        A[i][3] = load_stream(ch + 192);
    }
#pragma unroll
    for (int q = 0; q < NG; ++q) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int kc = (c + i) * 64;
            X[q][i][0] = *reinterpret_cast<const uint4*>(xb[q] + kc);
            X[q][i][1] = *reinterpret_cast<const uint4*>(xb[q] + kc + 32);
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // keep every load of the block ahead of the matrix-core work
#pragma unroll
    for (int q = 0; q < NG; ++q) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            acc0[q] = mfma_bf16(A[i][0], X[q][i][0], acc0[q]);
            acc0[q] = mfma_bf16(A[i][1], X[q][i][1], acc0[q]);
            acc1[q] = mfma_bf16(A[i][2], X[q][i][0], acc1[q]);
            acc1[q] = mfma_bf16(A[i][3], X[q][i][1], acc1[q]);
        }
    }
}

// The k loop of one pass: blocks of U chunks, then single chunks.
template <int NG, int U>
__device__ inline void mfma_pass(const uint4* __restrict__ tile, int nchunk, const uint16_t* const* xb, f32x4* acc0,
                                 f32x4* acc1) {
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        acc0[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        acc1[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    int c = 0;
    for (; c + U <= nchunk; c += U) mfma_block<NG, U>(tile, c, xb, acc0, acc1);
    for (; c < nchunk; ++c) mfma_block<NG, 1>(tile, c, xb, acc0, acc1);
}

// Grouped shape, units of more than 16 tokens: the kWaves wavefronts of a
// workgroup take consecutive row tiles of one unit, T each, load the
// activations of each block of U k-chunks from global memory once, into LDS,
// and read their B fragments from there.  NG token groups of 16, columns past
// the bucket repeating its last token.
//
// What bounds it: the L1 caches, whose misses in flight are all in use 66% of
// the time (128 experts d = 2048, F = 768, 64 tokens each, T = 1; a third of the
// lines are activations; with T = 2 71%, a fifth): more loads in flight per
// wavefront only made each take longer, a second block of weights in flight
// included.  So fewer lines:
// a staging load takes whole 128-byte lines (8 tokens x one chunk; 16 tokens x
// half a line fetched each line twice), and with many tokens per expert the
// big units run in a launch of their own with T = 2, which halves the
// activation lines and the LDS reads per byte of weights at two wavefronts per
// SIMD.  Measured, gate/up and down of a layer with 64 tokens per expert:
// 158 + 92 us with half lines, 150 + 88 us with whole lines, 146 + 85 us with
// T = 2; with 128 tokens per expert of d = F = 2880: 370 + 200, 320 + 175 and
// 275 + 146 us.  T = 2 for units of 17 to 32 tokens is slower than T = 1 at
// four wavefronts per SIMD (16 tokens per expert on average, d = 4096,
// F = 1536: 2151 + 1176 us against 1980 + 1089 us for four layers).
//
// Slot (group q, chunk i, half hh) of the buffer holds, for lane (r, g), token
// column r's 8 values at k = 64 (c + i) + 32 hh + 8 g.  A staging load of a
// wavefront covers 8 token rows: lane 8 t + j loads unit j (half j / 4,
// g = j % 4) of token t, which goes to lane place (r, g) of its half's slot
// with r xored with 2 j, so that the eight units of a row, 256 bytes or more
// apart, fall into different banks.
constexpr int kHeavyTiles = 2;   // row tiles per wavefront of the big units' launch
constexpr int kHeavySlots = 16;  // slots of one buffer (16 KB), two buffers: NG U <= 8

__device__ inline int lds_place(int r, int j) { return 16 * (j & 3) + (r ^ (2 * j)); }

// The staging loads of a block: load n = kPer w + i of wavefront w takes token
// half th of group q and one chunk.
template <int NG, int U>
struct Staging {
    static constexpr int kPer = NG * U * 2 / kWaves;
    static_assert(NG * U * 2 <= kHeavySlots && NG * U * 2 % kWaves == 0, "the loads fill the wavefronts evenly");
    // token row (of the unit) whose values this lane loads in its load i
    __device__ static __forceinline__ int row(int tid, int i) {
        const int n = kPer * (tid >> 6) + i, q = n / (2 * U), th = n % (2 * U) / U;
        return 16 * q + 8 * th + ((tid >> 3) & 7);
    }
    __device__ static __forceinline__ void load(u32x4 (&v)[kPer], const uint16_t* const (&xs)[kPer], int c, int nchunk,
                                                int wv) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int ch = (kPer * wv + i) % U;
            v[i] = *reinterpret_cast<const u32x4*>(xs[i] + min(c + ch, nchunk - 1) * 64);
        }
    }
    __device__ static __forceinline__ void store(const u32x4 (&v)[kPer], u32x4 (*x)[64], int tid, int wv) {
        const int t = (tid >> 3) & 7, j = tid & 7;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int n = kPer * wv + i, q = n / (2 * U), th = n % (2 * U) / U, ch = n % U;
            x[(q * U + ch) * 2 + (j >> 2)][lds_place(8 * th + t, j)] = v[i];
        }
    }
};

__device__ inline u32x4 load_stream4(const uint4* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ inline f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// One pass of NG token groups over T weight tiles (16-row gate/up or
// 2 x 16-row down), `next` 16-byte units apart.  Every wavefront of the
// workgroup runs the loop and its barriers; a wavefront that is not `active` (no
// tile left for it) re-reads the first tile's first chunk (cached), and its
// products are dropped.  Every global load is unconditional, so that the waits
// before the LDS stores cover the staging loads only.  No branch in the loop:
// one around the matrix-core work made the compiler copy the accumulators.
template <int T, int NG, int U>
__device__ __forceinline__ void mfma_pass_heavy(const uint4* __restrict__ tile, int64_t next, int nchunk,
                                                const uint16_t* const (&xs)[Staging<NG, U>::kPer], bool active,
                                                u32x4 (*x)[kHeavySlots][64], int tid, f32x4 (&acc0)[T][NG],
                                                f32x4 (&acc1)[T][NG]) {
    using St = Staging<NG, U>;
    const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p0 = lds_place(lane & 15, lane >> 4), p1 = lds_place(lane & 15, 4 + (lane >> 4));
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            acc0[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
            acc1[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    // The activations of block c + U are loaded while block c computes;
    // their LDS stores then wait only for them, not for the weight loads
    // issued after them.  Two buffers: one barrier per block.
    u32x4 st[St::kPer];
    St::load(st, xs, 0, nchunk, wv);
    int b = 0;
    for (int c = 0; c < nchunk; c += U, b ^= 1) {
        u32x4 A[U][T][4];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint4* ch = tile + (int64_t)(active ? min(c + i, nchunk - 1) : 0) * 256;
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int j = 0; j < 4; ++j) A[i][t][j] = load_stream4(ch + t * next + 64 * j);
        }
        St::store(st, x[b], tid, wv);
        __syncthreads();
        St::load(st, xs, c + U, nchunk, wv);
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (U == 1 || c + i < nchunk) {
#pragma unroll
                for (int q = 0; q < NG; ++q) {
                    if (q % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // bounds the B fragments held at once
                    const u32x4 X0 = x[b][(q * U + i) * 2][p0], X1 = x[b][(q * U + i) * 2 + 1][p1];
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        acc0[t][q] = mfma_bf16(A[i][t][0], X0, acc0[t][q]);
                        acc1[t][q] = mfma_bf16(A[i][t][2], X0, acc1[t][q]);
                    }
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        acc0[t][q] = mfma_bf16(A[i][t][1], X1, acc0[t][q]);
                        acc1[t][q] = mfma_bf16(A[i][t][3], X1, acc1[t][q]);
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------- bf16
// Token groups of one pass over the weights: one group (up to 16 tokens, the
// common case) with a deep k block, or kNG groups with a shallower one.
template <int NG, int U>
__device__ inline void up_passes(const Layout& lo, int l, int bl, int ft, const int32_t* __restrict__ bk, int m,
                                 const uint4* __restrict__ tileA, const uint16_t* __restrict__ h, int lane) {
    const int r = lane & 15, g = lane >> 4;
    const int d = lo.d;
    uint16_t* act = act_base<uint16_t>(lo, bl);
    for (int t0 = 0; t0 < m; t0 += 16 * NG) {
        const int ng = min(NG, (m - t0 + 15) / 16);
        int pr[NG];
        const uint16_t* xb[NG];
#pragma unroll
        for (int q = 0; q < NG; ++q) pr[q] = bk[min(t0 + 16 * q + r, m - 1)];
#pragma unroll
        for (int q = 0; q < NG; ++q) xb[q] = h + ((int64_t)(pr[q] >> 8) * lo.L + l) * d + 8 * g;
        f32x4 cg[NG], cu[NG];
        mfma_pass<NG, U>(tileA, d / 64, xb, cg, cu);
        // D[i][j]: row i = 4 g + rr of this 16-row tile, token column j = r
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            if (q >= ng) break;
            const int tok = t0 + 16 * q + r;
            if (tok < m) {
                uint2 o;
                o.x = pack_bf16x2(silu_mul(cg[q][0], cu[q][0]), silu_mul(cg[q][1], cu[q][1]));
                o.y = pack_bf16x2(silu_mul(cg[q][2], cu[q][2]), silu_mul(cg[q][3], cu[q][3]));
                const int pair = pr[q];
                const int64_t row = (int64_t)(pair >> 8) * lo.K + (pair & 255);  // token (s, k)
                *reinterpret_cast<uint2*>(act + row * lo.F + ft * 16 + 4 * g) = o;
            }
        }
    }
}

// Work unit u (the residency kernel lays them out) = tokens [ut p, ut (p + 1))
// of expert e's bucket, ut = lo.unit_tokens: {(p << 8) | e, slot, tokens, 0}.
struct Unit {
    int slot, m;         // m = 0: no work
    const int32_t* bk;   // the unit's tokens
};

template <bool HEAVY>
__device__ inline Unit unit_at(const Layout& lo, int bl, int u) {
    const int n = HEAVY ? lo.max_heavy : lo.max_units - lo.max_heavy;
    const int4 ui = reinterpret_cast<const int4*>(lo.units)[(int64_t)bl * lo.max_units + (HEAVY ? 0 : lo.max_heavy) +
                                                            min(u, n - 1)];
    const int e = ui.x & 255, t0 = lo.unit_tokens * (ui.x >> 8);
    const bool none = u >= n || ui.x < 0 || ui.y < 0 || ui.y >= lo.n_slots || ui.z <= 0;
    return Unit{ui.y, none ? 0 : ui.z, lo.pairs + ((int64_t)bl * lo.N + e) * lo.S + t0};
}

// A unit of up to 16 NG tokens: F-tiles ft .. ft + T - 1 of each wavefront.
template <int T, int NG, int U>
__device__ __forceinline__ void up_heavy(const Layout& lo, int l, int bl, int ft, const Unit& un,
                                         const uint16_t* __restrict__ h, int tid, u32x4 (*x)[kHeavySlots][64]) {
    const int lane = tid & 63, r = lane & 15, g = lane >> 4, nchunk = lo.d / 64;
    const bool active = ft < lo.F / 16;  // F / 16 is even: both tiles or none
    const uint16_t* xs[Staging<NG, U>::kPer];
#pragma unroll
    for (int i = 0; i < Staging<NG, U>::kPer; ++i) {
        const int p = un.bk[min(Staging<NG, U>::row(tid, i), un.m - 1)];
        xs[i] = h + ((int64_t)(p >> 8) * lo.L + l) * lo.d + 8 * (tid & 7);
    }
    const uint4* tile = reinterpret_cast<const uint4*>(slot_base(lo, l, un.slot)) +
                        (int64_t)(active ? ft : 0) * nchunk * 256 + lane;
    f32x4 cg[T][NG], cu[T][NG];
    mfma_pass_heavy<T, NG, U>(tile, (int64_t)nchunk * 256, nchunk, xs, active, x, tid, cg, cu);
    if (!active) return;
    uint16_t* act = act_base<uint16_t>(lo, bl);
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int tok = 16 * q + r;
        if (tok < un.m) {
            const int pair = un.bk[tok];
            uint16_t* o = act + ((int64_t)(pair >> 8) * lo.K + (pair & 255)) * lo.F + 16 * ft + 4 * g;
#pragma unroll
            for (int t = 0; t < T; ++t)
                *reinterpret_cast<uint2*>(o + 16 * t) =
                    make_uint2(pack_bf16x2(silu_mul(cg[t][q][0], cu[t][q][0]), silu_mul(cg[t][q][1], cu[t][q][1])),
                               pack_bf16x2(silu_mul(cg[t][q][2], cu[t][q][2]), silu_mul(cg[t][q][3], cu[t][q][3])));
        }
    }
}

// Workgroup (u, j): the W 16-row F-tiles W j + wavefront of unit u (F is a
// multiple of 64, so every wavefront has a tile).  W = kWaves: units of up to
// 16 GROUPS tokens, those of more than 16 sharing their activations through
// LDS; W = 1: a wavefront on its own.
template <int W, int GROUPS>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(3))) void ffn_up_bf16(
    Layout lo, int l0, int b0, const uint16_t* __restrict__ h) {
    const int l = l0 + blockIdx.y, bl = b0 + blockIdx.y;
    int u, j;
    unit_of_block(blockIdx.x, lo.F / (16 * W), lo.xcd_units != 0, u, j);
    const Unit un = unit_at<false>(lo, bl, u);
    if (un.m == 0) return;
    const int lane = threadIdx.x & 63, ft = j * W + (threadIdx.x >> 6);
    // packed slot layout: chunk c of this row tile is 256 units of 16 bytes,
    // gate half 0, gate half 1, up half 0, up half 1, each 64 units
    const uint4* tileA =
        reinterpret_cast<const uint4*>(slot_base(lo, l, un.slot)) + (int64_t)ft * (lo.d / 64) * 256 + lane;
    if (un.m <= 16) {  // workgroup-uniform
        up_passes<1, kUnroll>(lo, l, bl, ft, un.bk, un.m, tileA, h, lane);
    } else if constexpr (GROUPS > 0) {
        __shared__ u32x4 x[2][kHeavySlots][64];
        if (GROUPS == 2 || un.m <= 32)
            up_heavy<1, 2, 4>(lo, l, bl, ft, un, h, threadIdx.x, x);
        else if (un.m <= 64)
            up_heavy<1, 4, 2>(lo, l, bl, ft, un, h, threadIdx.x, x);
        else
            up_heavy<1, 8, 1>(lo, l, bl, ft, un, h, threadIdx.x, x);
    } else {
        up_passes<kNG, kUnrollSolo>(lo, l, bl, ft, un.bk, un.m, tileA, h, lane);
    }
}

constexpr int kHeavyRows = kHeavyTiles * kWaves;  // row tiles per heavy workgroup

// Workgroup (u, j): F-tiles 8 j .. 8 j + 7 of a big unit.
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2))) void ffn_up_heavy(
    Layout lo, int l0, int b0, const uint16_t* __restrict__ h) {
    __shared__ u32x4 x[2][kHeavySlots][64];
    const int l = l0 + blockIdx.y, bl = b0 + blockIdx.y, tid = threadIdx.x;
    int u, j;
    unit_of_block(blockIdx.x, (lo.F / 16 + kHeavyRows - 1) / kHeavyRows, lo.xcd_units != 0, u, j);
    const Unit un = unit_at<true>(lo, bl, u);
    if (un.m == 0) return;  // workgroup-uniform
    const int ft = j * kHeavyRows + kHeavyTiles * (tid >> 6);
    if (un.m <= 64)
        up_heavy<kHeavyTiles, 4, 2>(lo, l, bl, ft, un, h, tid, x);
    else if (un.m <= 96)
        up_heavy<kHeavyTiles, 6, 1>(lo, l, bl, ft, un, h, tid, x);
    else
        up_heavy<kHeavyTiles, 8, 1>(lo, l, bl, ft, un, h, tid, x);
}

template <int NG, int U>
__device__ inline void down_passes(const Layout& lo, int l, int bl, int dt, const int32_t* __restrict__ bk, int m,
                                   const uint4* __restrict__ tileB, int lane) {
    const int r = lane & 15, g = lane >> 4;
    const int F = lo.F;
    const uint16_t* act = act_base<uint16_t>(lo, bl);
    for (int t0 = 0; t0 < m; t0 += 16 * NG) {
        const int ng = min(NG, (m - t0 + 15) / 16);
        int pr[NG];
        const uint16_t* xb[NG];
#pragma unroll
        for (int q = 0; q < NG; ++q) pr[q] = bk[min(t0 + 16 * q + r, m - 1)];
#pragma unroll
        for (int q = 0; q < NG; ++q) xb[q] = act + ((int64_t)(pr[q] >> 8) * lo.K + (pr[q] & 255)) * F + 8 * g;
        f32x4 c0[NG], c1[NG];
        mfma_pass<NG, U>(tileB, F / 64, xb, c0, c1);
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            if (q >= ng) break;
            const int tok = t0 + 16 * q + r;
            if (tok < m) {
                const int s = pr[q] >> 8, k = pr[q] & 255;
                const float gk = lo.gates[((int64_t)l * lo.S + s) * lo.K + k];
                store_gated(lo, bl, s, k, dt * 32 + 4 * g, gk, c0[q], c1[q]);
            }
        }
    }
}

// A unit of up to 16 NG tokens: d-tiles dt .. dt + T - 1 of each wavefront (d / 32
// is even: all or none).
template <int T, int NG, int U>
__device__ __forceinline__ void down_heavy(const Layout& lo, int l, int bl, int dt, const Unit& un, int tid,
                                           u32x4 (*x)[kHeavySlots][64]) {
    const int lane = tid & 63, r = lane & 15, g = lane >> 4, nchunk = lo.F / 64;
    const bool active = dt < lo.d / 32;
    const uint16_t* act = act_base<uint16_t>(lo, bl);
    const uint16_t* xs[Staging<NG, U>::kPer];
#pragma unroll
    for (int i = 0; i < Staging<NG, U>::kPer; ++i) {
        const int p = un.bk[min(Staging<NG, U>::row(tid, i), un.m - 1)];
        xs[i] = act + ((int64_t)(p >> 8) * lo.K + (p & 255)) * lo.F + 8 * (tid & 7);
    }
    const uint4* tile = reinterpret_cast<const uint4*>(slot_base(lo, l, un.slot)) + (int64_t)lo.F * lo.d / 4 +
                        (int64_t)(active ? dt : 0) * nchunk * 256 + lane;
    f32x4 c0[T][NG], c1[T][NG];
    mfma_pass_heavy<T, NG, U>(tile, (int64_t)nchunk * 256, nchunk, xs, active, x, tid, c0, c1);
    if (!active) return;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int tok = 16 * q + r;
        if (tok < un.m) {
            const int pair = un.bk[tok];
            const int s = pair >> 8, k = pair & 255;
            const float gk = lo.gates[((int64_t)l * lo.S + s) * lo.K + k];
#pragma unroll
            for (int t = 0; t < T; ++t) store_gated(lo, bl, s, k, (dt + t) * 32 + 4 * g, gk, c0[t][q], c1[t][q]);
        }
    }
}

// Workgroup (u, j): the W 32-row d-tiles W j + wavefront of unit u.
template <int W, int GROUPS>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(3))) void ffn_down_bf16(Layout lo, int l0, int b0) {
    const int l = l0 + blockIdx.y, bl = b0 + blockIdx.y;
    const int dtn = lo.d / 32;
    int u, j;
    unit_of_block(blockIdx.x, (dtn + W - 1) / W, lo.xcd_units != 0, u, j);
    const Unit un = unit_at<false>(lo, bl, u);
    if (un.m == 0) return;
    const int lane = threadIdx.x & 63, dt = j * W + (threadIdx.x >> 6);
    if (dt >= dtn && !(GROUPS > 0 && un.m > 16)) return;  // wavefront-uniform; the path of bigger units has barriers
    // packed slot layout: after the gate/up part (F d / 4 units), chunk c of
    // this 32-row tile is 256 units: rows 0-15 half 0, half 1, rows 16-31
    // half 0, half 1, each 64 units
    const uint4* tileB = reinterpret_cast<const uint4*>(slot_base(lo, l, un.slot)) + (int64_t)lo.F * lo.d / 4 +
                         (int64_t)dt * (lo.F / 64) * 256 + lane;
    if (un.m <= 16) {
        down_passes<1, kUnroll>(lo, l, bl, dt, un.bk, un.m, tileB, lane);
    } else if constexpr (GROUPS > 0) {
        __shared__ u32x4 x[2][kHeavySlots][64];
        if (GROUPS == 2 || un.m <= 32)
            down_heavy<1, 2, 4>(lo, l, bl, dt, un, threadIdx.x, x);
        else if (un.m <= 64)
            down_heavy<1, 4, 2>(lo, l, bl, dt, un, threadIdx.x, x);
        else
            down_heavy<1, 8, 1>(lo, l, bl, dt, un, threadIdx.x, x);
    } else {
        down_passes<kNG, kUnrollSolo>(lo, l, bl, dt, un.bk, un.m, tileB, lane);
    }
}

// Workgroup (u, j): d-tiles 8 j .. 8 j + 7 of a big unit.
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2))) void ffn_down_heavy(Layout lo, int l0,
                                                                                                     int b0) {
    __shared__ u32x4 x[2][kHeavySlots][64];
    const int l = l0 + blockIdx.y, bl = b0 + blockIdx.y, tid = threadIdx.x;
    int u, j;
    unit_of_block(blockIdx.x, (lo.d / 32 + kHeavyRows - 1) / kHeavyRows, lo.xcd_units != 0, u, j);
    const Unit un = unit_at<true>(lo, bl, u);
    if (un.m == 0) return;  // workgroup-uniform
    const int dt = j * kHeavyRows + kHeavyTiles * (tid >> 6);
    if (un.m <= 64)
        down_heavy<kHeavyTiles, 4, 2>(lo, l, bl, dt, un, tid, x);
    else if (un.m <= 96)
        down_heavy<kHeavyTiles, 6, 1>(lo, l, bl, dt, un, tid, x);
    else
        down_heavy<kHeavyTiles, 8, 1>(lo, l, bl, dt, un, tid, x);
}

// ---------------------------------------------------------------- fp32
// On the fp32 matrix core (v_mfma_f32_16x16x4_f32), over transposed weights
// W^T [k][row] (the copy kernel writes them so).  A workgroup takes 64 rows of
// one work unit and cuts k into four ranges, one per wavefront (whole blocks of
// 16), whose partial products are added in LDS in wavefront order.  In a block
// of 16 k, lane (r, g) loads W^T[k0 + 4 g + j][4 r .. 4 r + 3] for j = 0 .. 3:
// 256 contiguous bytes per row and 1 KB per instruction; its value i is the A
// operand (row r, k-slot g) of the product that gives rows 4 r' + i, r' = 0 ..
// 15, and step j takes k = k0 + 4 g + j on both sides, so that the B operand is
// value j of the 16-byte load x[k0 + 4 g ..] of token column r.
// HBM-bound: a pass of up to 16 kNG32 tokens streams the expert once, where
// one lane per row walked k once for each token.  Measured (6 layers of 60
// experts, d = 704, F = 448, 13 streams, gate/up and down of a token step):
// 237 + 119 us before, 123 + 61 us now (5.5 TB/s); the error against fp64
// falls from 8.2e-7 to 4.2e-7 (four chains instead of one).  kNG32 = 4 holds
// 362 registers and one wave per SIMD: 139 + 71 us; a budget of four waves per
// SIMD spills: 130 + 63.
constexpr int kNG32 = 2;  // token groups (of 16) per pass
constexpr int kWaves32 = 4;

typedef float f32x4v __attribute__((ext_vector_type(4)));

__device__ inline f32x4 load_stream_f32(const float* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(p));
}

// acc[m][q][i] += the products of one block of 16 k, M matrices `stride`
// floats apart, ld floats between their rows.
template <int M, int NG, int U>
__device__ inline void block_f32(const float* __restrict__ w, int64_t stride, int64_t ld, const float* const* xb, int k0,
                                 f32x4 (&acc)[M][NG][4]) {
    f32x4 a[U][M][4], x[U][NG];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j) a[u][m][j] = load_stream_f32(w + m * stride + (int64_t)(k0 + 16 * u + j) * ld);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < NG; ++q) x[u][q] = *reinterpret_cast<const f32x4*>(xb[q] + k0 + 16 * u);
    __builtin_amdgcn_sched_barrier(0);  // keep every load of the block ahead of the matrix-core work
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int q = 0; q < NG; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[m][q][i] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][m][j][i], x[u][q][j], acc[m][q][i], 0, 0, 0);
}

// The products of 64 rows with up to 16 NG token columns over k in [0, kn),
// kn a multiple of 16: returned in wavefront 0's acc, summed over the
// workgroup.  w points at the workgroup's first row of k = 4 g, column 4 r;
// xb at each token column's value at k = 4 g.
template <int M, int NG, int U>
__device__ inline void pass_f32(const float* __restrict__ w, int64_t stride, int64_t ld, const float* const* xb, int kn,
                                f32x4 (&acc)[M][NG][4], f32x4 (*red)[M * 4][64]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int q = 0; q < NG; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[m][q][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nb = kn / 16, b1 = __builtin_amdgcn_readfirstlane(nb * (wv + 1) / kWaves32);
    int b = __builtin_amdgcn_readfirstlane(nb * wv / kWaves32);
    for (; b + U <= b1; b += U) block_f32<M, NG, U>(w, stride, ld, xb, 16 * b, acc);
    for (; b < b1; ++b) block_f32<M, NG, 1>(w, stride, ld, xb, 16 * b, acc);
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        if (wv > 0) {
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) red[wv - 1][m * 4 + i][lane] = acc[m][q][i];
        }
        __syncthreads();
        if (wv == 0) {
#pragma unroll
            for (int v = 0; v < kWaves32 - 1; ++v)
#pragma unroll
                for (int m = 0; m < M; ++m)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[m][q][i] = acc[m][q][i] + red[v][m * 4 + i][lane];
        }
        __syncthreads();  // the buffer is free for the next group
    }
}

// Gate/up of tokens [t0, t0 + 16 NG) of a unit of m tokens: rows 64 ft .. of F.
template <int NG, int U>
__device__ inline void up_f32(const Layout& lo, int l, int bl, int ft, const int32_t* __restrict__ bk, int t0, int m,
                              const float* __restrict__ slot, const float* __restrict__ h, f32x4 (*red)[8][64]) {
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, F = lo.F;
    int pr[NG];
    const float* xb[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) pr[q] = bk[min(t0 + 16 * q + r, m - 1)];
#pragma unroll
    for (int q = 0; q < NG; ++q) xb[q] = h + ((int64_t)(pr[q] >> 8) * lo.L + l) * lo.d + 4 * g;
    f32x4 acc[2][NG][4];
    pass_f32<2, NG, U>(slot + (int64_t)4 * g * F + 64 * ft + 4 * r, (int64_t)F * lo.d, F, xb, lo.d, acc, red);
    if (threadIdx.x >= 64) return;
    float* act = act_base<float>(lo, bl);
    // product i, value v: row 4 (4 g + v) + i, token column r
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        if (t0 + 16 * q + r < m) {
            float* o = act + ((int64_t)(pr[q] >> 8) * lo.K + (pr[q] & 255)) * F + 64 * ft + 16 * g;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                f32x4 y;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float a = acc[0][q][i][v];
                    y[i] = a / (1.0f + expf(-a)) * acc[1][q][i][v];
                }
                *reinterpret_cast<f32x4*>(o + 4 * v) = y;
            }
        }
    }
}

template <int NG, int U>
__device__ inline void down_f32(const Layout& lo, int l, int bl, int dt, const int32_t* __restrict__ bk, int t0, int m,
                                const float* __restrict__ slot, f32x4 (*red)[4][64]) {
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4, d = lo.d;
    const float* act = act_base<float>(lo, bl);
    int pr[NG];
    const float* xb[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) pr[q] = bk[min(t0 + 16 * q + r, m - 1)];
#pragma unroll
    for (int q = 0; q < NG; ++q) xb[q] = act + ((int64_t)(pr[q] >> 8) * lo.K + (pr[q] & 255)) * lo.F + 4 * g;
    f32x4 acc[1][NG][4];
    pass_f32<1, NG, U>(slot + (int64_t)2 * lo.F * d + (int64_t)4 * g * d + 64 * dt + 4 * r, 0, d, xb, lo.F, acc, red);
    if (threadIdx.x >= 64) return;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        if (t0 + 16 * q + r < m) {
            const int s = pr[q] >> 8, k = pr[q] & 255;
            const float gk = lo.gates[((int64_t)l * lo.S + s) * lo.K + k];
            float* o = static_cast<float*>(lo.yp) + (((int64_t)bl * lo.S + s) * lo.K + k) * d + 64 * dt + 16 * g;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                f32x4 y;
#pragma unroll
                for (int i = 0; i < 4; ++i) y[i] = gk * acc[0][q][i][v];
                *reinterpret_cast<f32x4*>(o + 4 * v) = y;
            }
        }
    }
}

// Workgroup (u, ft): rows 64 ft .. of work unit u.
template <bool UP>
__global__ __launch_bounds__(64 * kWaves32) __attribute__((amdgpu_waves_per_eu(3))) void ffn_f32(Layout lo, int l0, int b0, const float* __restrict__ h) {
    __shared__ f32x4 red[kWaves32 - 1][UP ? 8 : 4][64];
    const int l = l0 + blockIdx.y, bl = b0 + blockIdx.y;
    int u, ft;
    unit_of_block(blockIdx.x, (UP ? lo.F : lo.d) / 64, lo.xcd_units != 0, u, ft);
    const Unit un = unit_at<false>(lo, bl, u);  // max_heavy is 0: the whole list
    if (un.m == 0) return;
    const int m = un.m;
    const int32_t* bk = un.bk;
    const float* w = static_cast<const float*>(lo.arena) + ((int64_t)l * lo.n_slots + un.slot) * lo.expert_elems;
    if (m <= 16) {  // workgroup-uniform
        if constexpr (UP)
            up_f32<1, 2>(lo, l, bl, ft, bk, 0, m, w, h, red);
        else
            down_f32<1, 4>(lo, l, bl, ft, bk, 0, m, w, red);
    } else {
        for (int t = 0; t < m; t += 16 * kNG32) {
            if constexpr (UP)
                up_f32<kNG32, 1>(lo, l, bl, ft, bk, t, m, w, h, red);
            else
                down_f32<kNG32, 1>(lo, l, bl, ft, bk, t, m, w, red);
        }
    }
}

}  // namespace

hipError_t launch_ffn_up(const Layout& lo, int l0, int b0, int nl, const void* h, hipStream_t st,
                         const Timing& tm, const Timing& heavy) {
    const int units = unit_groups(lo, lo.max_units - lo.max_heavy), big = unit_groups(lo, lo.max_heavy);
    if (lo.dtype == 1) {
        const uint16_t* hb = static_cast<const uint16_t*>(h);
        const dim3 grid(units * (lo.F / (16 * kWaves)), nl), block(64 * kWaves);
        if (lo.ffn_waves == kWaves && big > 0) {
            launch_kernel(ffn_up_heavy, dim3(big * ((lo.F / 16 + kHeavyRows - 1) / kHeavyRows), nl), block, st, heavy, lo,
                          l0, b0, hb);
            launch_kernel(ffn_up_bf16<kWaves, 2>, grid, block, st, tm, lo, l0, b0, hb);
        } else if (lo.ffn_waves == kWaves) {
            launch_kernel(ffn_up_bf16<kWaves, 8>, grid, block, st, tm, lo, l0, b0, hb);
        } else {
            launch_kernel(ffn_up_bf16<1, 0>, dim3(units * (lo.F / 16), nl), dim3(64), st, tm, lo, l0, b0, hb);
        }
    } else {
        launch_kernel(ffn_f32<true>, dim3(units * (lo.F / 64), nl), dim3(64 * kWaves32), st, tm, lo, l0, b0,
                      static_cast<const float*>(h));
    }
    return hipGetLastError();
}

hipError_t launch_ffn_down(const Layout& lo, int l0, int b0, int nl, hipStream_t st, const Timing& tm,
                           const Timing& heavy) {
    const int units = unit_groups(lo, lo.max_units - lo.max_heavy), big = unit_groups(lo, lo.max_heavy);
    if (lo.dtype == 1) {
        const int dtn = lo.d / 32;
        const dim3 grid(units * ((dtn + kWaves - 1) / kWaves), nl), block(64 * kWaves);
        if (lo.ffn_waves == kWaves && big > 0) {
            launch_kernel(ffn_down_heavy, dim3(big * ((dtn + kHeavyRows - 1) / kHeavyRows), nl), block, st, heavy, lo, l0,
                          b0);
            launch_kernel(ffn_down_bf16<kWaves, 2>, grid, block, st, tm, lo, l0, b0);
        } else if (lo.ffn_waves == kWaves) {
            launch_kernel(ffn_down_bf16<kWaves, 8>, grid, block, st, tm, lo, l0, b0);
        } else {
            launch_kernel(ffn_down_bf16<1, 0>, dim3(units * dtn, nl), dim3(64), st, tm, lo, l0, b0);
        }
    } else {
        launch_kernel(ffn_f32<false>, dim3(units * (lo.d / 64), nl), dim3(64 * kWaves32), st, tm, lo, l0, b0,
                      static_cast<const float*>(nullptr));
    }
    return hipGetLastError();
}

}  // namespace cmoe
