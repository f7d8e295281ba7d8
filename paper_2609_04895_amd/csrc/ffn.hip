// ffn.hip - the SwiGLU expert FFN over the resident expert weights
// ("execute the MoE layer", Algorithm 2), grouped by expert:
//   a_e = silu(W_gate,e x) * (W_up,e x),  y_(s,k) = g_(s,k) W_down,e a_e,
//   y_s = sum_k y_(s,k)  (k in ascending order).
// Each expert's weights are read from its HBM slot once per work unit (a
// pass over up to 64 of its tokens; nearly every expert needs one), so the
// layer step streams about |union of selected experts| x expert_bytes: the
// kernels are HBM-bound.
//
// bf16: one wavefront per 16 rows of W_gate and of W_up (gate/up kernel) or
// per 32 rows of W_down (down kernel), one wavefront per workgroup or four
// (grouped: consecutive row tiles of one unit, big units sharing their
// activations through LDS), on the bf16 matrix core
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation).  The expert's tokens form the
// 16 columns of the B operand (groups of 16 tokens; several groups reuse the
// loaded weights).  Per 64-wide k chunk, lane (r, g) of the A operand holds
// W[row r][kc + 8 g .. + 8] and W[row r][kc + 32 + 8 g .. + 8]; the two MFMAs
// of a chunk take k-slots kc + 8 g + {0..7} and kc + 32 + 8 g + {0..7}, the
// same for both operands.  Each activation load thus reads one contiguous
// 64-byte half of a token's 128-byte k chunk.
// The weights come from the expert's HBM slot in packed order (the fill
// kernel writes it so): each A operand load of a wavefront reads one
// contiguous kilobyte and each wavefront streams one contiguous block.  The
// SwiGLU intermediate is stored in bf16 (the input type of the down kernel's
// matrix core).
//
// fp32: the same units on the fp32 matrix core, over transposed weights (the
// copy kernel writes them so).
#include "cmoe_internal.h"

namespace cmoe {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kNG = 4;          // token groups (of 16) per pass when a unit holds more than 16
static_assert(kUnitTokens == 16 * kNG, "one work unit is one pass over the weights");
constexpr int kUnroll = 4;      // k chunks per load block, one token group
constexpr int kUnrollWide = 2;  // k chunks per load block, kNG token groups sharing LDS (grouped launch)
constexpr int kUnrollSolo = 1;  // k chunks per load block, kNG token groups in one wavefront: this
                                // path is rare in the launches that use it, and a deeper block would
                                // set the register budget (and so the occupancy) of the whole kernel
constexpr int kWaves = 4;       // wavefronts per grouped workgroup: consecutive row tiles of one work unit
constexpr int kNGWide = kUnitTokensGrouped / 16;  // token groups of the widest pass (grouped launch)
static_assert(kNGWide == 8, "the wide staging split gives each thread four of the eight groups");

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
// tokens' activations are fetched into one L2 instead of eight.  Units come
// heaviest first, and each XCD takes every eighth one.  That grid is rounded
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

inline int unit_groups(const Layout& lo) { return lo.xcd_units ? (lo.max_units + 7) / 8 * 8 : lo.max_units; }

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

// Grouped launch, units of more than 16 tokens: the kWaves wavefronts of a
// workgroup (row tiles of the same unit) load the activations of each block
// of U k-chunks from global memory once, into LDS, and read their B
// fragments from there.
// Slot (group q, chunk i, half hh) of a buffer holds, for lane (r, g), token
// column r's 8 values at k = 64 (c + i) + 32 hh + 8 g.  Two buffers: one
// barrier per block.
template <int U>
struct HeavyLds {
    uint4 x[2][kNG * U * 2][64];
};
static_assert(kWaves == 4, "the staging split below assumes 4 wavefronts");

// Staging loads of thread tid (U = 2): group q, chunk tid / 128, half
// (tid / 64) % 2, lane tid % 64 for every q, whose token row and k offset are
// the thread's own xb[q] (a chunk past the end is clamped; it is never used).
struct Staged {
    uint4 v[kNG];
};

template <int U>
__device__ inline Staged stage_load(const uint16_t* const* xb, int c, int nchunk, int tid) {
    static_assert(U == 2, "the staging split assumes two chunks per block");
    const int i = tid >> 7, hh = (tid >> 6) & 1;
    const int off = min(c + i, nchunk - 1) * 64 + 32 * hh;
    Staged st;
#pragma unroll
    for (int q = 0; q < kNG; ++q) st.v[q] = *reinterpret_cast<const uint4*>(xb[q] + off);
    return st;
}

// LDS stores of the ng groups in use (wavefront-uniform).
template <int U>
__device__ inline void stage_store(uint4 (*xs)[64], int tid, int ng, const Staged& st) {
    const int i = tid >> 7, hh = (tid >> 6) & 1;
#pragma unroll
    for (int q = 0; q < kNG; ++q)
        if (q < ng) xs[(q * U + i) * 2 + hh][tid & 63] = st.v[q];
}

// One pass of ng (up to kNG) token groups over a 16-row (gate/up) or
// 2 x 16-row (down) weight tile with the activations shared through LDS.
// Every wavefront of the workgroup runs the loop (and its barriers); only
// `active` wavefronts run the matrix-core work.  Every global load is
// unconditional, so that the waits before the LDS stores cover the staging
// loads only: the weight loads of an inactive wavefront re-read its tile's
// first chunk (cached), and staging loads of unused groups repeat the last
// token.
template <int U>
__device__ inline void mfma_pass_shared(const uint4* __restrict__ tile, int nchunk, const uint16_t* const* xb, int ng,
                                        bool active, HeavyLds<U>& sm, int tid, f32x4* acc0, f32x4* acc1) {
    const int lane = tid & 63;
    ng = __builtin_amdgcn_readfirstlane(ng);
#pragma unroll
    for (int q = 0; q < kNG; ++q) {
        acc0[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        acc1[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // The activations of block c + U are loaded while block c computes;
    // their LDS stores then wait only for them, not for the weight loads
    // issued after them.
    Staged st = stage_load<U>(xb, 0, nchunk, tid);
    int b = 0;
    for (int c = 0; c < nchunk; c += U, b ^= 1) {
        uint4 A[U][4];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint4* ch = tile + (int64_t)(active ? min(c + i, nchunk - 1) : 0) * 256;
            A[i][0] = load_stream(ch);
            A[i][1] = load_stream(ch + 64);
            A[i][2] = load_stream(ch + 128);
            A[i][3] = load_stream(ch + 192);
        }
        stage_store<U>(sm.x[b], tid, ng, st);
        __syncthreads();
        st = stage_load<U>(xb, c + U, nchunk, tid);
        if (!active) continue;
#pragma unroll
        for (int q = 0; q < kNG; ++q) {
            if (q >= ng) break;
            uint4 X[U][2];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                X[i][0] = sm.x[b][(q * U + i) * 2][lane];
                X[i][1] = sm.x[b][(q * U + i) * 2 + 1][lane];
            }
#pragma unroll
            for (int i = 0; i < U; ++i) {
                if (c + i < nchunk) {
                    acc0[q] = mfma_bf16(A[i][0], X[i][0], acc0[q]);
                    acc0[q] = mfma_bf16(A[i][1], X[i][1], acc0[q]);
                    acc1[q] = mfma_bf16(A[i][2], X[i][0], acc1[q]);
                    acc1[q] = mfma_bf16(A[i][3], X[i][1], acc1[q]);
                }
            }
        }
    }
}

// Grouped launch, units of 65 to kUnitTokensGrouped tokens (a hot expert's
// tokens in one pass, so its weights are streamed once): the activations of
// one k chunk for all eight token groups (16 KB) are staged in LDS once per
// workgroup, two buffers, one barrier per chunk.  Slot (group q, half hh)
// holds, for lane (r, g), token column r's 8 values at k = 64 c + 32 hh + 8 g.
// Its 32 KB share the workgroup's LDS with HeavyLds.
struct WideLds {
    uint4 x[2][kNGWide * 2][64];
};
union GroupedLds {
    HeavyLds<kUnrollWide> narrow;
    WideLds wide;
};

// Staging of thread tid: groups 4 (tid / 128) .. + 3 at half (tid / 64) % 2
// of chunk c (clamped; a chunk past the end is never used), from the token
// rows xs of those four groups.
__device__ __forceinline__ Staged wide_stage_load(const uint16_t* const* xs, int c, int nchunk, int tid) {
    const int off = min(c, nchunk - 1) * 64 + 32 * ((tid >> 6) & 1);
    Staged st;
#pragma unroll
    for (int q = 0; q < 4; ++q) st.v[q] = *reinterpret_cast<const uint4*>(xs[q] + off);
    return st;
}

__device__ __forceinline__ void wide_stage_store(uint4 (*xb)[64], int tid, int ng, const Staged& st) {
    const int q0 = 4 * (tid >> 7), hh = (tid >> 6) & 1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (q0 + q < ng) xb[(q0 + q) * 2 + hh][tid & 63] = st.v[q];
}

// One pass of ng (up to 8) token groups over a 16-row (gate/up) or 2 x 16-row
// (down) weight tile, the activations shared through LDS, one k chunk per
// block: the next chunk's weights are loaded while the current one computes.
// As in the four-group pass, every wavefront runs the loop and its barriers
// and every global load is unconditional; only `active` wavefronts compute.
__device__ __forceinline__ void mfma_pass_wide(const uint4* __restrict__ tile, int nchunk, const uint16_t* const* xs, int ng,
                                      bool active, WideLds& sm, int tid, f32x4* acc0, f32x4* acc1) {
    const int lane = tid & 63;
    ng = __builtin_amdgcn_readfirstlane(ng);
#pragma unroll
    for (int q = 0; q < kNGWide; ++q) {
        acc0[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        acc1[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    Staged st = wide_stage_load(xs, 0, nchunk, tid);
    int b = 0;
    for (int c = 0; c < nchunk; ++c, b ^= 1) {
        uint4 A[4];
        const uint4* ch = tile + (int64_t)(active ? c : 0) * 256;
#pragma unroll
        for (int j = 0; j < 4; ++j) A[j] = load_stream(ch + 64 * j);
        wide_stage_store(sm.x[b], tid, ng, st);
        __syncthreads();
        st = wide_stage_load(xs, c + 1, nchunk, tid);
        if (active) {
#pragma unroll
            for (int q = 0; q < kNGWide; ++q) {
                if (q >= ng) break;
                const uint4 X0 = sm.x[b][q * 2][lane], X1 = sm.x[b][q * 2 + 1][lane];
                acc0[q] = mfma_bf16(A[0], X0, acc0[q]);
                acc0[q] = mfma_bf16(A[1], X1, acc0[q]);
                acc1[q] = mfma_bf16(A[2], X0, acc1[q]);
                acc1[q] = mfma_bf16(A[3], X1, acc1[q]);
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

// A unit of 17 to 16 kNG tokens: one pass with the activations shared by the
// workgroup.
__device__ inline void up_heavy(const Layout& lo, int l, int bl, int ft, const int32_t* __restrict__ bk, int m,
                                const uint4* __restrict__ tileA, const uint16_t* __restrict__ h, int tid,
                                HeavyLds<kUnrollWide>& sm) {
    const int lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int d = lo.d;
    uint16_t* act = act_base<uint16_t>(lo, bl);
    int pr[kNG];
    const uint16_t* xb[kNG];
#pragma unroll
    for (int q = 0; q < kNG; ++q) pr[q] = bk[min(16 * q + r, m - 1)];
#pragma unroll
    for (int q = 0; q < kNG; ++q) xb[q] = h + ((int64_t)(pr[q] >> 8) * lo.L + l) * d + 8 * g;
    f32x4 cg[kNG], cu[kNG];
    mfma_pass_shared<kUnrollWide>(tileA, d / 64, xb, (m + 15) / 16, true, sm, tid, cg, cu);
#pragma unroll
    for (int q = 0; q < kNG; ++q) {
        const int tok = 16 * q + r;
        if (tok < m) {
            uint2 o;
            o.x = pack_bf16x2(silu_mul(cg[q][0], cu[q][0]), silu_mul(cg[q][1], cu[q][1]));
            o.y = pack_bf16x2(silu_mul(cg[q][2], cu[q][2]), silu_mul(cg[q][3], cu[q][3]));
            const int pair = pr[q];
            const int64_t row = (int64_t)(pair >> 8) * lo.K + (pair & 255);
            *reinterpret_cast<uint2*>(act + row * lo.F + ft * 16 + 4 * g) = o;
        }
    }
}

// A unit of 65 to kUnitTokensGrouped tokens: one pass, eight token groups,
// the activations shared by the workgroup.
__device__ __forceinline__ void up_heavy_wide(const Layout& lo, int l, int bl, int ft, const int32_t* __restrict__ bk, int m,
                                     const uint4* __restrict__ tileA, const uint16_t* __restrict__ h, int tid,
                                     WideLds& sm) {
    const int lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int d = lo.d, q0 = 4 * (tid >> 7);
    uint16_t* act = act_base<uint16_t>(lo, bl);
    const uint16_t* xs[4];  // token rows of this thread's staging groups
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int p = bk[min(16 * (q0 + q) + r, m - 1)];
        xs[q] = h + ((int64_t)(p >> 8) * lo.L + l) * d + 8 * g;
    }
    f32x4 cg[kNGWide], cu[kNGWide];
    mfma_pass_wide(tileA, d / 64, xs, (m + 15) / 16, true, sm, tid, cg, cu);
#pragma unroll
    for (int q = 0; q < kNGWide; ++q) {
        const int tok = 16 * q + r;
        if (tok < m) {
            uint2 o;
            o.x = pack_bf16x2(silu_mul(cg[q][0], cu[q][0]), silu_mul(cg[q][1], cu[q][1]));
            o.y = pack_bf16x2(silu_mul(cg[q][2], cu[q][2]), silu_mul(cg[q][3], cu[q][3]));
            const int pair = bk[tok];
            const int64_t row = (int64_t)(pair >> 8) * lo.K + (pair & 255);
            *reinterpret_cast<uint2*>(act + row * lo.F + ft * 16 + 4 * g) = o;
        }
    }
}

// Work unit u (the fill kernel lays them out, heaviest first) = tokens
// [ut p, ut (p + 1)) of expert e's bucket, ut = lo.unit_tokens; workgroup
// (u, j) runs that pass for the W 16-row F-tiles W j + wavefront (F is a
// multiple of 64, so every wavefront has a tile).  W = 1: every wavefront
// on its own; W = kWaves: grouped.
template <int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(3))) void ffn_up_bf16(Layout lo, int l0, int b0,
                                                                                                  const uint16_t* __restrict__ h) {
    const int l = l0 + blockIdx.y, bl = b0 + blockIdx.y;
    const int wgn = lo.F / (16 * W);
    int u, j;
    unit_of_block(blockIdx.x, wgn, lo.xcd_units != 0, u, j);
    if (u >= lo.max_units) return;
    const int lane = threadIdx.x & 63;
    const int ft = j * W + (threadIdx.x >> 6);
    const int4 ui = reinterpret_cast<const int4*>(lo.units)[(int64_t)bl * lo.max_units + u];  // expert, pass, slot, tokens in one load
    if (ui.x < 0) return;
    const int e = ui.x & 255, t0 = lo.unit_tokens * (ui.x >> 8), slot = ui.y, m = ui.z;
    if (m <= 0 || slot < 0 || slot >= lo.n_slots) return;
    const int32_t* bk = lo.pairs + ((int64_t)bl * lo.N + e) * lo.S + t0;
    // packed slot layout: chunk c of this row tile is 256 units of 16 bytes,
    // gate half 0, gate half 1, up half 0, up half 1, each 64 units
    const uint4* tileA =
        reinterpret_cast<const uint4*>(slot_base(lo, l, slot)) + (int64_t)ft * (lo.d / 64) * 256 + lane;
    if (m <= 16) {  // workgroup-uniform
        up_passes<1, kUnroll>(lo, l, bl, ft, bk, m, tileA, h, lane);
    } else if constexpr (W == 1) {
        up_passes<kNG, kUnrollSolo>(lo, l, bl, ft, bk, m, tileA, h, lane);
    } else {
        __shared__ GroupedLds sm;
        if (m <= 16 * kNG)
            up_heavy(lo, l, bl, ft, bk, m, tileA, h, threadIdx.x, sm.narrow);
        else
            up_heavy_wide(lo, l, bl, ft, bk, m, tileA, h, threadIdx.x, sm.wide);
    }
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

// A unit of 17 to 16 kNG tokens in the grouped launch: one pass with
// the SwiGLU intermediate shared by the workgroup.  Wavefronts past the last
// d-tile (d not a multiple of 32 W) take part in the staging and barriers
// only.
__device__ inline void down_heavy(const Layout& lo, int l, int bl, int dt, bool active, const int32_t* __restrict__ bk, int m,
                                  const uint4* __restrict__ tileB, int tid, HeavyLds<kUnrollWide>& sm) {
    const int lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int F = lo.F;
    const uint16_t* act = act_base<uint16_t>(lo, bl);
    int pr[kNG];
    const uint16_t* xb[kNG];
#pragma unroll
    for (int q = 0; q < kNG; ++q) pr[q] = bk[min(16 * q + r, m - 1)];
#pragma unroll
    for (int q = 0; q < kNG; ++q) xb[q] = act + ((int64_t)(pr[q] >> 8) * lo.K + (pr[q] & 255)) * F + 8 * g;
    f32x4 c0[kNG], c1[kNG];
    mfma_pass_shared<kUnrollWide>(tileB, F / 64, xb, (m + 15) / 16, active, sm, tid, c0, c1);
    if (!active) return;
#pragma unroll
    for (int q = 0; q < kNG; ++q) {
        const int tok = 16 * q + r;
        if (tok < m) {
            const int s = pr[q] >> 8, k = pr[q] & 255;
            const float gk = lo.gates[((int64_t)l * lo.S + s) * lo.K + k];
            store_gated(lo, bl, s, k, dt * 32 + 4 * g, gk, c0[q], c1[q]);
        }
    }
}

// A unit of 65 to kUnitTokensGrouped tokens in the grouped launch: one pass,
// eight token groups, the SwiGLU intermediate shared by the workgroup.
__device__ __forceinline__ void down_heavy_wide(const Layout& lo, int l, int bl, int dt, bool active, const int32_t* __restrict__ bk,
                                       int m, const uint4* __restrict__ tileB, int tid, WideLds& sm) {
    const int lane = tid & 63, r = lane & 15, g = lane >> 4;
    const int F = lo.F, q0 = 4 * (tid >> 7);
    const uint16_t* act = act_base<uint16_t>(lo, bl);
    const uint16_t* xs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int p = bk[min(16 * (q0 + q) + r, m - 1)];
        xs[q] = act + ((int64_t)(p >> 8) * lo.K + (p & 255)) * F + 8 * g;
    }
    f32x4 c0[kNGWide], c1[kNGWide];
    mfma_pass_wide(tileB, F / 64, xs, (m + 15) / 16, active, sm, tid, c0, c1);
    if (!active) return;
#pragma unroll
    for (int q = 0; q < kNGWide; ++q) {
        const int tok = 16 * q + r;
        if (tok < m) {
            const int pair = bk[tok];
            const int s = pair >> 8, k = pair & 255;
            const float gk = lo.gates[((int64_t)l * lo.S + s) * lo.K + k];
            store_gated(lo, bl, s, k, dt * 32 + 4 * g, gk, c0[q], c1[q]);
        }
    }
}

// Workgroup (u, j): the W 32-row d-tiles W j + wavefront of unit u.
template <int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(3))) void ffn_down_bf16(Layout lo, int l0, int b0) {
    const int l = l0 + blockIdx.y, bl = b0 + blockIdx.y;
    const int dtn = lo.d / 32;
    const int wgn = (dtn + W - 1) / W;
    int u, j;
    unit_of_block(blockIdx.x, wgn, lo.xcd_units != 0, u, j);
    if (u >= lo.max_units) return;
    const int lane = threadIdx.x & 63;
    const int dt = j * W + (threadIdx.x >> 6);
    const bool active = dt < dtn;
    const int4 ui = reinterpret_cast<const int4*>(lo.units)[(int64_t)bl * lo.max_units + u];  // expert, pass, slot, tokens in one load
    if (ui.x < 0) return;
    const int e = ui.x & 255, t0 = lo.unit_tokens * (ui.x >> 8), slot = ui.y, m = ui.z;
    if (m <= 0 || slot < 0 || slot >= lo.n_slots) return;
    const int32_t* bk = lo.pairs + ((int64_t)bl * lo.N + e) * lo.S + t0;
    // packed slot layout: after the gate/up part (F d / 4 units), chunk c of
    // this 32-row tile is 256 units: rows 0-15 half 0, half 1, rows 16-31
    // half 0, half 1, each 64 units
    const uint4* tileB = reinterpret_cast<const uint4*>(slot_base(lo, l, slot)) + (int64_t)lo.F * lo.d / 4 +
                         (int64_t)(active ? dt : 0) * (lo.F / 64) * 256 + lane;
    if (m <= 16) {  // workgroup-uniform; this path has no barriers
        if (active) down_passes<1, kUnroll>(lo, l, bl, dt, bk, m, tileB, lane);
    } else if constexpr (W == 1) {
        down_passes<kNG, kUnrollSolo>(lo, l, bl, dt, bk, m, tileB, lane);
    } else {
        __shared__ GroupedLds sm;
        if (m <= 16 * kNG)
            down_heavy(lo, l, bl, dt, active, bk, m, tileB, threadIdx.x, sm.narrow);
        else
            down_heavy_wide(lo, l, bl, dt, active, bk, m, tileB, threadIdx.x, sm.wide);
    }
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
    if (u >= lo.max_units) return;
    const int4 ui = reinterpret_cast<const int4*>(lo.units)[(int64_t)bl * lo.max_units + u];
    if (ui.x < 0) return;
    const int e = ui.x & 255, t0 = lo.unit_tokens * (ui.x >> 8), slot = ui.y, m = ui.z;
    if (m <= 0 || slot < 0 || slot >= lo.n_slots) return;
    const int32_t* bk = lo.pairs + ((int64_t)bl * lo.N + e) * lo.S + t0;
    const float* w = static_cast<const float*>(lo.arena) + ((int64_t)l * lo.n_slots + slot) * lo.expert_elems;
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
                         const Timing& tm) {
    if (lo.dtype == 1) {
        const uint16_t* hb = static_cast<const uint16_t*>(h);
        if (lo.ffn_waves == kWaves)
            launch_kernel(ffn_up_bf16<kWaves>, dim3(unit_groups(lo) * (lo.F / (16 * kWaves)), nl), dim3(64 * kWaves), st,
                          tm, lo, l0, b0, hb);
        else
            launch_kernel(ffn_up_bf16<1>, dim3(unit_groups(lo) * (lo.F / 16), nl), dim3(64), st, tm, lo, l0, b0, hb);
    } else {
        launch_kernel(ffn_f32<true>, dim3(unit_groups(lo) * (lo.F / 64), nl), dim3(64 * kWaves32), st, tm, lo, l0, b0,
                      static_cast<const float*>(h));
    }
    return hipGetLastError();
}

hipError_t launch_ffn_down(const Layout& lo, int l0, int b0, int nl, hipStream_t st, const Timing& tm) {
    if (lo.dtype == 1) {
        const int dtn = lo.d / 32;
        if (lo.ffn_waves == kWaves)
            launch_kernel(ffn_down_bf16<kWaves>, dim3(unit_groups(lo) * ((dtn + kWaves - 1) / kWaves), nl),
                          dim3(64 * kWaves), st, tm, lo, l0, b0);
        else
            launch_kernel(ffn_down_bf16<1>, dim3(unit_groups(lo) * dtn, nl), dim3(64), st, tm, lo, l0, b0);
    } else {
        launch_kernel(ffn_f32<false>, dim3(unit_groups(lo) * (lo.d / 64), nl), dim3(64 * kWaves32), st, tm, lo, l0, b0,
                      static_cast<const float*>(nullptr));
    }
    return hipGetLastError();
}

}  // namespace cmoe
