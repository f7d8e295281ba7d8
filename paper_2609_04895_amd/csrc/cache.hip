// cache.hip - the per-(stream, layer) cache state machine of the decode step.
//
// cache_step_kernel: one wavefront per (stream, layer) of a batch of layers;
// expert e of the layer lives in lane e % 64, register e / 64.  For layer l it
//   - finishes the router logits (adds the split-K partials in ascending
//     order, adds the native bias, rounds once to fp32),
//   - computes p^R, p^T (router policy) and p^S (modes with a Spatio
//     Router) with the fixed fp32 softmax described below (Section 2,
//     Section 3.2, Section 3.3),
//   - selects S = TopK by native logit (ties: lower index) and the gate
//     weights p^R_S / sum p^R_S,
//   - counts hits and demand misses against the resident set (Section 2),
//   - applies the post-access retention update (Algorithm 1: each
//     demand-loaded expert in ascending order fills free room or replaces
//     the lowest-priority resident that is not selected now; ties evict the
//     lower index), with priority s^T = p^R + p^T or, for the classical
//     cache-update baselines (Section 4.1, Table 1), the LRU time, LFU count
//     or LRFU value, updated first,
//   - stores the next token's a-score (Section 3.3: s^T in the full mode;
//     p^R in the Spatio-only ablation of Section 5 / Appendix B.4) and p^S
//     as the prediction for the causal successor.
// In the modes with a Spatio Router each layer is refined before its access
// (Algorithm 2): candidates Top_R(s^ST), s^ST = a + p^S of the causal
// predecessor, examined in descending order; a non-resident candidate fills
// free room, else replaces the lowest-s^ST resident when its score is strictly
// higher (an inserted expert takes the LRU time of the refinement).  The first
// layer of a token takes the previous token's last-layer p^S (the wrap-around
// of the causal predecessor).
//
// The same kernel groups the layer's (stream, k) selections by expert for the
// FFN (fixed-capacity buckets filled with integer atomics).  Physical
// residency, and the counts of selections and of distinct experts, are the
// residency kernel's.
//
// Fixed fp32 softmax: m = max z; u_e = exp(z_e - m) with the exponential
// below; the sum is a strided halving over the next power of two P >= N
// (v[i] += v[i + w] for w = P/2 .. 1, missing entries +0), which maps onto
// in-lane adds for w >= 64 and shuffle-down adds for w < 64; p_e = u_e / sum
// (IEEE division).  exp(x), x <= 0: +0 below -80; else k = rint(x / ln 2),
// r = x - k ln2_hi - k ln2_lo (Cody & Waite; ln2_hi is fl32(ln 2) with the low
// 8 fraction bits cleared, ln2_lo = fl32(ln 2 - ln2_hi)), a degree-7 Taylor
// polynomial in Horner form with coefficients fl32(1/n!), scaled by 2^k.
// Build with -ffp-contract=off: every operation here is rounded separately.
#include <math.h>

#include "cmoe_internal.h"

namespace cmoe {

namespace {

constexpr int kPolicyRouter = 0, kPolicyLRU = 1, kPolicyLFU = 2;  // cmoe_policy; 3 = LRFU

constexpr float kLn2Hi = 0x1.62e4p-1f;       // 0x3f317200
constexpr float kLn2Lo = 0x1.7f7d1cp-20f;    // 0x35bfbe8e
constexpr float kInvLn2 = 0x1.715476p+0f;    // fl32(1 / ln 2)
constexpr float kC0 = 1.0f, kC1 = 1.0f, kC2 = 0.5f;
constexpr float kC3 = 0x1.555556p-3f;        // fl32(1/6)
constexpr float kC4 = 0x1.555556p-5f;        // fl32(1/24)
constexpr float kC5 = 0x1.111112p-7f;        // fl32(1/120)
constexpr float kC6 = 0x1.6c16c2p-10f;       // fl32(1/720)
constexpr float kC7 = 0x1.a01a02p-13f;       // fl32(1/5040)

__device__ inline float canon_exp(float x) {
    if (x < -80.0f) return 0.0f;
    const float k = __builtin_rintf(x * kInvLn2);
    float r = __builtin_fmaf(-k, kLn2Hi, x);
    r = __builtin_fmaf(-k, kLn2Lo, r);
    float p = kC7;
    p = __builtin_fmaf(p, r, kC6);
    p = __builtin_fmaf(p, r, kC5);
    p = __builtin_fmaf(p, r, kC4);
    p = __builtin_fmaf(p, r, kC3);
    p = __builtin_fmaf(p, r, kC2);
    p = __builtin_fmaf(p, r, kC1);
    p = __builtin_fmaf(p, r, kC0);
    return __builtin_ldexpf(p, (int)k);
}

// Order-preserving map of fp32 onto uint32 (larger float -> larger key);
// -0 and +0 map to the same key.
__device__ inline uint32_t ord32(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7FFFFFFFu) == 0) u = 0;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Cross-lane steps without the LDS crossbar (all 64 lanes active):
// DPP quad permutations and mirrors inside 16-lane rows, and the gfx950
// permlane swaps across rows.  permlane16_swap(x, x) returns, in every lane,
// the pair {own value, value of lane ^ 16} in some order (permlane32_swap:
// lane ^ 32), so an order-free combine of the pair is the combine with that
// partner.
// Lanes whose source is outside their row read 0 (bound_ctrl); no step
// below uses such a lane's result.  The move folds into the consuming
// max or add as one DPP instruction.
template <int CTRL>
__device__ inline unsigned dpp(unsigned v) {
    return (unsigned)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
constexpr int kQuadXor1 = 0xB1;     // quad_perm 1,0,3,2
constexpr int kQuadXor2 = 0x4E;     // quad_perm 2,3,0,1
constexpr int kRowHalfMirror = 0x141;
constexpr int kRowMirror = 0x140;
constexpr int kRowShl1 = 0x101;     // lane i reads lane i + n of its row

// maximum (MAX) or minimum of a 32-bit unsigned value over the wavefront,
// wave-uniform
template <bool MAX>
__device__ inline uint32_t wave_reduce_u32(uint32_t v) {
    auto op = [](uint32_t a, uint32_t b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); };
    v = op(v, dpp<kQuadXor1>(v));
    v = op(v, dpp<kQuadXor2>(v));
    v = op(v, dpp<kRowHalfMirror>(v));
    v = op(v, dpp<kRowMirror>(v));
    const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = op(p[0], p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = op(q[0], q[1]);
    return __builtin_amdgcn_readfirstlane(v);
}

// The largest key (wave-uniform) and the lowest expert index e = 64 j + lane
// holding it: a 32-bit reduction, then one ballot per register.
template <int NPL>
__device__ inline int argmax_lowest(const uint32_t (&key)[NPL], uint32_t& kmax) {
    uint32_t b = key[0];
#pragma unroll
    for (int j = 1; j < NPL; ++j) b = key[j] > b ? key[j] : b;
    kmax = wave_reduce_u32<true>(b);
    int e = -1;
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        const unsigned long long bal = __ballot(key[j] == kmax);
        if (e < 0 && bal) e = j * 64 + __builtin_ctzll(bal);
    }
    return e;
}

// The fixed softmax (described at the top of this file) of R independent
// logit vectors, step by step for all of them at once so that the latencies
// of their cross-lane reductions overlap.  Wavefront maximum: DPP and
// permlane-swap max steps; sum: strided halving over the next power of two
// P >= N, in-lane adds for w >= 64, then for w = 32 .. 1 lane i < w adds lane
// i + w (the tree of lane 0 is exactly that order), lane 0's total taken.
template <int NPL, int R>
__device__ inline void softmax_fixed(const float (&z)[3][NPL], int N, int lane, float (&p)[3][NPL]) {
    unsigned u[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float m = -INFINITY;
#pragma unroll
        for (int j = 0; j < NPL; ++j)
            if (j * 64 + lane < N) m = fmaxf(m, z[r][j]);
        u[r] = __float_as_uint(m);
    }
    // wavefront maxima
#pragma unroll
    for (int r = 0; r < R; ++r) u[r] = __float_as_uint(fmaxf(__uint_as_float(u[r]), __uint_as_float(dpp<kQuadXor1>(u[r]))));
#pragma unroll
    for (int r = 0; r < R; ++r) u[r] = __float_as_uint(fmaxf(__uint_as_float(u[r]), __uint_as_float(dpp<kQuadXor2>(u[r]))));
#pragma unroll
    for (int r = 0; r < R; ++r)
        u[r] = __float_as_uint(fmaxf(__uint_as_float(u[r]), __uint_as_float(dpp<kRowHalfMirror>(u[r]))));
#pragma unroll
    for (int r = 0; r < R; ++r) u[r] = __float_as_uint(fmaxf(__uint_as_float(u[r]), __uint_as_float(dpp<kRowMirror>(u[r]))));
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const auto q = __builtin_amdgcn_permlane16_swap(u[r], u[r], false, false);
        u[r] = __float_as_uint(fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1])));
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const auto q = __builtin_amdgcn_permlane32_swap(u[r], u[r], false, false);
        u[r] = __float_as_uint(fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1])));
    }
    float v[R][NPL];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float m = __uint_as_float(__builtin_amdgcn_readfirstlane(u[r]));
#pragma unroll
        for (int j = 0; j < NPL; ++j) {
            const bool in = j * 64 + lane < N;
            p[r][j] = in ? canon_exp(z[r][j] - m) : 0.0f;
            v[r][j] = p[r][j];
        }
    }
    int P = 1;
    while (P < N) P <<= 1;
#pragma unroll
    for (int jw = NPL / 2; jw >= 1; jw >>= 1) {
        if (jw * 64 * 2 <= P) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int j = 0; j < jw; ++j) v[r][j] = v[r][j] + v[r][j + jw];
        }
    }
    // cross-lane halving steps (w < 64)
    const int Pw = P < 64 ? P : 64;
    float x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = v[r][0];
    if (Pw >= 64) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned w = __float_as_uint(x[r]);
            const auto q = __builtin_amdgcn_permlane32_swap(w, w, false, false);
            x[r] = x[r] + __uint_as_float(q[1]);
        }
    }
    if (Pw >= 32) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned w = __float_as_uint(x[r]);
            const auto q = __builtin_amdgcn_permlane16_swap(w, w, false, false);
            x[r] = x[r] + __uint_as_float(q[1]);
        }
    }
    if (Pw >= 16) {
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = x[r] + __uint_as_float(dpp<kRowShl1 + 7>(__float_as_uint(x[r])));
    }
    if (Pw >= 8) {
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = x[r] + __uint_as_float(dpp<kRowShl1 + 3>(__float_as_uint(x[r])));
    }
    if (Pw >= 4) {
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = x[r] + __uint_as_float(dpp<kRowShl1 + 1>(__float_as_uint(x[r])));
    }
    if (Pw >= 2) {
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = x[r] + __uint_as_float(dpp<kRowShl1>(__float_as_uint(x[r])));
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float sum = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x[r]), 0));
#pragma unroll
        for (int j = 0; j < NPL; ++j) p[r][j] = p[r][j] / sum;
    }
}

template <int NPL>
__device__ inline bool bit_of(const unsigned long long (&w)[NPL], int e) {
    bool b = false;
#pragma unroll
    for (int j = 0; j < NPL; ++j)
        if (j == (e >> 6)) b = (w[j] >> (e & 63)) & 1ull;
    return b;
}

// Lowest-scoring member (bit set in member words) with the lowest index on
// ties; returns (ord(score) << 32) | e, or ~0 if there is no member.
template <int NPL>
__device__ inline unsigned long long argmin_member(const float (&sc)[NPL], const unsigned long long (&member)[NPL],
                                                   int N, int lane) {
    uint32_t key[NPL];
    bool in[NPL];
    uint32_t b = 0xFFFFFFFFu;
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        const int e = j * 64 + lane;
        in[j] = e < N && ((member[j] >> lane) & 1ull);
        key[j] = in[j] ? ord32(sc[j]) : 0xFFFFFFFFu;
        b = key[j] < b ? key[j] : b;
    }
    const uint32_t kmin = wave_reduce_u32<false>(b);
    int e = -1;
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        const unsigned long long bal = __ballot(in[j] && key[j] == kmin);
        if (e < 0 && bal) e = j * 64 + __builtin_ctzll(bal);
    }
    return e < 0 ? ~0ull : (((unsigned long long)kmin << 32) | (unsigned)e);
}

template <int NPL>
__device__ inline void set_bit(unsigned long long (&w)[NPL], int e) {
#pragma unroll
    for (int j = 0; j < NPL; ++j)
        if (j == (e >> 6)) w[j] |= 1ull << (e & 63);
}

template <int NPL>
__device__ inline void clear_bit(unsigned long long (&w)[NPL], int e) {
#pragma unroll
    for (int j = 0; j < NPL; ++j)
        if (j == (e >> 6)) w[j] &= ~(1ull << (e & 63));
}

// Pre-access refinement of one (stream, layer) cache (Algorithm 2), in
// registers: cw is updated, ins gets the experts inserted here; returns their
// number (an expert inserted and replaced again counts).
template <int NPL>
__device__ int refine_one(const Layout& lo, int R, const float (&pred)[NPL], const float (&aTv)[NPL],
                          unsigned long long (&cw)[NPL], unsigned long long (&ins)[NPL], int lane) {
    const int N = lo.N;
    float sST[NPL];
    uint32_t cand[NPL];  // ordered scores; 0 = not a candidate (no real score maps to 0)
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        const int e = j * 64 + lane;
        if (e < N) {
            sST[j] = aTv[j] + pred[j];
            cand[j] = ord32(sST[j]);
        } else {
            sST[j] = 0.0f;
            cand[j] = 0u;
        }
    }
    int count = 0, nP = 0;
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        count += __popcll(cw[j]);
        ins[j] = 0ull;
    }
    const int Rn = R < N ? R : N;
    for (int i = 0; i < Rn; ++i) {
        uint32_t ord_e;
        const int e = argmax_lowest(cand, ord_e);  // highest s^ST, lower index on ties
#pragma unroll
        for (int j = 0; j < NPL; ++j)
            if (j == (e >> 6) && lane == (e & 63)) cand[j] = 0u;
        if (bit_of(cw, e)) continue;              // already resident
        if (count < lo.C) {
            set_bit(cw, e);
            set_bit(ins, e);
            ++count;
            ++nP;
        } else {
            const unsigned long long mn = argmin_member(sST, cw, N, lane);
            const int v = (int)(mn & 0xFFFFFFFFull);
            const uint32_t ord_v = (uint32_t)(mn >> 32);
            if (ord_e > ord_v) {  // strictly higher priority
                clear_bit(cw, v);
                clear_bit(ins, v);
                set_bit(cw, e);
                set_bit(ins, e);
                ++nP;
            }
        }
    }
    return nP;
}

// One (stream, layer) of a batch: refinement (REF) and access.  bl is the
// layer's index in its batch.
template <int NPL, int NR, bool INJECT, int ZS, bool REF>
__device__ void stream_step(const Layout& lo, const StepArgs& a, int s, int bl, int lane) {
    const int N = lo.N, L = lo.L, K = lo.K, l = a.l0 + bl;
    const bool spatio = lo.iS > 0;           // a Spatio Router (always the last slot)
    const bool classical = lo.policy != kPolicyRouter;
    const bool counted = (a.flags & kFlagCount) != 0;
    const int64_t sl = (int64_t)s * L + l;

    // Every load is issued before the first use, so that their latencies
    // overlap: the a-scores, cache words, classical priorities and counters
    // of this (stream, layer), the native bias, and the logits (router split
    // partials, up to ZS per logit, or the injected logits).  Rows and splits
    // are clamped into range and words, experts and splits past the end masked
    // where they are used: a load under a branch of its own makes the compiler
    // wait for it where the branches join.
    float aTv[NPL], polv[NPL], pS_st[NPL], bz[NPL];
    unsigned long long cw[NPL];
    const float* brow = lo.bias ? lo.bias + (int64_t)l * N : lo.pol;  // without a bias: any N readable floats
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        const int ec = min(j * 64 + lane, N - 1), jw = min(j, lo.NW - 1);
        cw[j] = lo.cache[sl * lo.NW + jw];
        polv[j] = lo.pol[sl * N + ec];
        bz[j] = brow[ec];
        if (REF) {
            pS_st[j] = lo.pS[((int64_t)(a.psw ^ 1) * lo.S + s) * N + ec];
            aTv[j] = lo.aT[sl * N + ec];
        }
    }
    int64_t ctr_a[kNctr];  // counters this wavefront updates (lane 0 owns them)
#pragma unroll
    for (int c = 0; c < kNctr; ++c) ctr_a[c] = lo.ctr[sl * kNctr + c];
    // slot r < NR: this layer's logits; slot NR (REF): the Spatio logits of
    // the causal predecessor, when that layer is in this batch
    constexpr int NZ = NR + (REF ? 1 : 0);
    double pv[NZ][NPL][ZS];
    float zin[NZ][NPL];
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        const int ec = min(j * 64 + lane, N - 1);  // lanes past N read a valid address and discard it
#pragma unroll
        for (int r = 0; r < NZ; ++r) {
            const int rr = r < NR ? r : NR - 1, lb = r < NR ? bl : max(bl - 1, 0);
            if (INJECT) {
                zin[r][j] = a.z[rr][((int64_t)s * L + a.l0 + lb) * N + ec];
            } else {
                const double* zp = lo.zpart + (((int64_t)lb * lo.S + s) * NR + rr) * lo.nsplit * N + ec;
#pragma unroll
                for (int u = 0; u < ZS; ++u) pv[r][j][u] = zp[(int64_t)min(u, lo.nsplit - 1) * N];
            }
        }
    }

    // logits: the splits added in ascending order, the native bias, rounded once
    float z[3][NPL], zp[NPL];
#pragma unroll
    for (int r = NR; r < 3; ++r)
#pragma unroll
        for (int j = 0; j < NPL; ++j) z[r][j] = 0.0f;
#pragma unroll
    for (int r = 0; r < NZ; ++r) {
#pragma unroll
        for (int j = 0; j < NPL; ++j) {
            float v;
            if (INJECT) {
                v = zin[r][j];
            } else {
                double acc = 0.0;
#pragma unroll
                for (int p = 0; p < ZS; ++p)
                    if (p < lo.nsplit) acc += pv[r][j][p];
                if (r == 0 && lo.bias) acc += (double)bz[j];
                v = (float)acc;
            }
            const int e = j * 64 + lane;
            if (r < NR) {
                if (e < N) lo.logits[(((int64_t)l * lo.S + s) * NR + r) * N + e] = v;
                z[r][j] = e < N ? v : 0.0f;
            } else {
                zp[j] = e < N ? v : 0.0f;
            }
        }
    }
    // router slots: 0 native, then temporal (router policy), then spatio.  The
    // NR softmaxes run together; with refinement the Spatio slot holds the
    // predecessor's logits, the prediction for this layer.
    float zz[3][NPL], pz[3][NPL], pR[NPL], pT[NPL], pred[NPL];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int j = 0; j < NPL; ++j) zz[r][j] = (REF && r == NR - 1) ? zp[j] : z[r][j];
    softmax_fixed<NPL, NR>(zz, N, lane, pz);
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        pR[j] = pz[0][j];
        pT[j] = (NR >= 2 && !classical) ? pz[1][j] : 0.0f;
        // the first layer of a batch is predicted by the previous batch's last
        // layer (for layer 0: the previous token's)
        if (REF) pred[j] = bl > 0 ? pz[NR - 1][j] : (j * 64 + lane < N ? pS_st[j] : 0.0f);
    }

    // Top-K by native logit, lower index first on ties
    uint32_t key[NPL];  // ordered native logits; 0 = taken or past N (no real logit maps to 0)
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        const int e = j * 64 + lane;
        key[j] = e < N ? ord32(z[0][j]) : 0u;
    }
    unsigned long long sw[NPL];
#pragma unroll
    for (int j = 0; j < NPL; ++j) sw[j] = 0ull;
    float gsum = 0.0f, my_p = 0.0f;
    int my_sel = 0;
    for (int k = 0; k < K; ++k) {
        uint32_t kmax;
        const int e = argmax_lowest(key, kmax);  // highest logit, lower index on ties
        float pv = 0.0f;
#pragma unroll
        for (int j = 0; j < NPL; ++j) {
            if (j == (e >> 6) && lane == (e & 63)) {
                key[j] = 0u;
                pv = pR[j];
            }
        }
        pv = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(pv), e & 63));
        gsum = gsum + pv;
        set_bit(sw, e);
        if (lane == k) {
            my_p = pv;
            my_sel = e;
        }
    }
    // the priorities, loaded with the logits, are waited for here: a first use
    // behind the branch below would wait for the atomic in it as well
#pragma unroll
    for (int j = 0; j < NPL; ++j) asm volatile("" : "+v"(polv[j]));
    int64_t bucket = 0;  // lane k < K: bucket of its selection and position in it
    uint32_t bucket_pos = 0;
    if (lane < K) {
        const int64_t o = ((int64_t)l * lo.S + s) * K + lane;
        lo.sel[o] = my_sel;
        lo.gates[o] = my_p / gsum;
        // token (s, k) joins the bucket of its expert; the position inside
        // the bucket does not affect any result (each token is its own
        // column of the expert's matrix products).  The position is used
        // at the end of the step, so the atomic's round trip overlaps the
        // rest of it; unsigned, since the sign extension of an address offset
        // was placed here, with a wait for the atomic (256 streams, one layer:
        // 9.1 us with the wait, 8.5 without).
        bucket = (int64_t)bl * N + my_sel;
        bucket_pos = (uint32_t)atomicAdd(&lo.bcount[bucket], 1);
    }

#pragma unroll
    for (int j = 0; j < NPL; ++j)
        if (j >= lo.NW) cw[j] = 0ull;
    int nP = 0;
    if (REF) {
        unsigned long long ins[NPL];
        nP = refine_one<NPL>(lo, a.R, pred, aTv, cw, ins, lane);
        if (lane == 0)  // what the proactive residency event of this layer sees
            for (int j = 0; j < lo.NW; ++j) lo.mid[((int64_t)l * lo.S + s) * lo.NW + j] = cw[j];
        if (lo.policy == kPolicyLRU) {  // inserted as the most recently used, at 2t + 1
#pragma unroll
            for (int j = 0; j < NPL; ++j)
                if ((ins[j] >> lane) & 1ull) polv[j] = (float)(2 * a.t + 1);
        }
    }

    // retention priority of Algorithm 1
    float sT[NPL];
    if (!classical) {
#pragma unroll
        for (int j = 0; j < NPL; ++j) sT[j] = pR[j] + pT[j];
    } else {
#pragma unroll
        for (int j = 0; j < NPL; ++j) {
            const bool used = (sw[j] >> lane) & 1ull;
            float v = j * 64 + lane < N ? polv[j] : 0.0f;
            if (lo.policy == kPolicyLRU) {
                if (used) v = (float)(2 * a.t + 2);
            } else if (lo.policy == kPolicyLFU) {
                if (used) v = v + 1.0f;
            } else {
                v = v * lo.lrfu_w;
                if (used) v = v + 1.0f;
            }
            sT[j] = v;
            const int e = j * 64 + lane;
            if (e < N) lo.pol[sl * N + e] = v;
        }
    }

    // access
    int count = 0, hits = 0;
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        count += __popcll(cw[j]);
        hits += __popcll(cw[j] & sw[j]);
    }
    const int nD = K - hits;
    // Algorithm 1 with the demand set D = S \ C taken before any insertion
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        unsigned long long dw = sw[j] & ~cw[j];
        while (dw) {
            const int b = __builtin_ctzll(dw);
            dw &= dw - 1;
            if (count < lo.C) {
                cw[j] |= 1ull << b;
                ++count;
            } else {
                unsigned long long vict[NPL];
#pragma unroll
                for (int jj = 0; jj < NPL; ++jj) vict[jj] = cw[jj] & ~sw[jj];
                const unsigned long long mn = argmin_member(sT, vict, N, lane);
                clear_bit(cw, (int)(mn & 0xFFFFFFFFull));
                cw[j] |= 1ull << b;
            }
        }
    }
    if (lane == 0) {
        for (int j = 0; j < lo.NW; ++j) lo.cache[sl * lo.NW + j] = cw[j];
        *reinterpret_cast<int4*>(lo.events + ((int64_t)l * lo.S + s) * 4) = int4{hits, nD, nP, 0};
        if (counted) {
            int64_t* c = lo.ctr + sl * kNctr;
            c[kCtrA] = ctr_a[kCtrA] + K;
            c[kCtrHits] = ctr_a[kCtrHits] + hits;
            c[kCtrD] = ctr_a[kCtrD] + nD;
            c[kCtrP] = ctr_a[kCtrP] + nP;
            c[kCtrT] = ctr_a[kCtrT] + 1;
        }
    }
    if (spatio) {  // the next token's a-score of this layer
        const bool spatio_only = lo.iT < 0;
#pragma unroll
        for (int j = 0; j < NPL; ++j) {
            const int e = j * 64 + lane;
            if (e < N) lo.aT[sl * N + e] = spatio_only ? pR[j] : sT[j];
        }
        if (bl == a.nl - 1) {  // p^S of the batch's last layer, for its successor
            float own[3][NPL], po[3][NPL];
            if (REF) {
#pragma unroll
                for (int j = 0; j < NPL; ++j) own[0][j] = z[NR - 1][j];
                softmax_fixed<NPL, 1>(own, N, lane, po);
            }
#pragma unroll
            for (int j = 0; j < NPL; ++j) {
                const int e = j * 64 + lane;
                if (e < N) lo.pS[((int64_t)a.psw * lo.S + s) * N + e] = REF ? po[0][j] : pz[NR - 1][j];
            }
        }
    }
    if (lane < K) lo.pairs[bucket * lo.S + bucket_pos] = (s << 8) | lane;
}

// grid: x = streams, y = layers of the batch; one wavefront per (stream,
// layer).  No step depends on another: a layer's refinement needs the previous
// token's state of that layer and the predecessor's Spatio logits of this
// token, which the router launch has left for every layer of the batch, so
// one launch takes a batch of layers.  A wavefront is a chain of dependent
// wave reductions (about 4 us); only the number of them in flight hides it.
// At 64 streams and 24 layers one launch replaces 24 of 5.9 us.  With a.snap one
// more workgroup copies the slot maps of the batch's one layer (the fill launch
// that follows reads the copy while it writes the maps).
template <int NPL, int NR, bool INJECT, int ZS, bool REF>
__global__ __launch_bounds__(64) void cache_step_kernel(Layout lo, StepArgs a) {
    if (!REF && (int)blockIdx.x == lo.S) {  // only with a.snap
        for (int i = threadIdx.x; i < lo.N; i += 64) lo.snap_of[i] = lo.slot_of[(int64_t)a.l0 * lo.N + i];
        for (int i = threadIdx.x; i < lo.n_slots; i += 64) lo.snap_exp[i] = lo.slot_exp[(int64_t)a.l0 * lo.n_slots + i];
        return;
    }
    stream_step<NPL, NR, INJECT, ZS, REF>(lo, a, blockIdx.x, blockIdx.y, threadIdx.x);
}

// ---------------------------------------------------------------- init
__global__ void init_kernel(Layout lo) {
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t gs = (int64_t)gridDim.x * blockDim.x;
    const int64_t nc = (int64_t)lo.S * lo.L * lo.NW;
    for (int64_t i = gid; i < nc; i += gs) lo.cache[i] = 0ull;
    const int64_t na = (int64_t)lo.S * lo.L * lo.N;
    for (int64_t i = gid; i < na; i += gs) {
        lo.aT[i] = 0.0f;
        lo.pol[i] = 0.0f;
    }
    for (int64_t i = gid; i < (int64_t)2 * lo.S * lo.N; i += gs) lo.pS[i] = 0.0f;
    for (int64_t i = gid; i < (int64_t)lo.S * lo.L * kNctr; i += gs) lo.ctr[i] = 0;
    for (int64_t i = gid; i < (int64_t)lo.L * 2; i += gs) lo.phys[i] = 0;
    for (int64_t i = gid; i < lo.L; i += gs) lo.active_sum[i] = 0ull;
    for (int64_t i = gid; i < (int64_t)lo.L * lo.N; i += gs) lo.selcount[i] = 0ull;
    for (int64_t i = gid; i < (int64_t)lo.L * lo.N; i += gs) lo.slot_of[i] = -1;
    for (int64_t i = gid; i < (int64_t)lo.L * lo.n_slots; i += gs) {
        lo.slot_exp[i] = -1;
        lo.slot_stamp[i] = 0;
    }
    if (lo.events == nullptr) return;  // no workspace bound (kernel-uniform)
    for (int64_t i = gid; i < (int64_t)lo.L * 2; i += gs) lo.step_fills[i] = 0;
    for (int64_t i = gid; i < (int64_t)lo.L * lo.S * 4; i += gs) lo.events[i] = 0;
    for (int64_t i = gid; i < (int64_t)lo.G * lo.N; i += gs) lo.bcount[i] = 0;
}

}  // namespace

hipError_t launch_init(const Layout& lo, hipStream_t st) {
    hipLaunchKernelGGL(init_kernel, dim3(256), dim3(256), 0, st, lo);
    return hipGetLastError();
}

template <int NPL, int NR, bool REF>
void launch_step_ref(const Layout& lo, const StepArgs& a, hipStream_t st, const Timing& tm) {
    const dim3 grid(lo.S + (a.snap ? 1 : 0), a.nl), block(64);
    if (a.flags & kFlagInject)
        launch_kernel(cache_step_kernel<NPL, NR, true, 1, REF>, grid, block, st, tm, lo, a);
    else if (lo.nsplit <= 2)
        launch_kernel(cache_step_kernel<NPL, NR, false, 2, REF>, grid, block, st, tm, lo, a);
    else
        launch_kernel(cache_step_kernel<NPL, NR, false, kMaxSplit, REF>, grid, block, st, tm, lo, a);
}

template <int NPL, int NR>
hipError_t launch_step_nr(const Layout& lo, const StepArgs& a, hipStream_t st, const Timing& tm) {
    if constexpr (NR > 1) {  // refinement needs a Spatio Router
        if (a.flags & kFlagRefine) {
            launch_step_ref<NPL, NR, true>(lo, a, st, tm);
            return hipGetLastError();
        }
    }
    launch_step_ref<NPL, NR, false>(lo, a, st, tm);
    return hipGetLastError();
}

template <int NPL>
hipError_t launch_step_npl(const Layout& lo, const StepArgs& a, hipStream_t st, const Timing& tm) {
    if (lo.n_r == 3) return launch_step_nr<NPL, 3>(lo, a, st, tm);
    if (lo.n_r == 2) return launch_step_nr<NPL, 2>(lo, a, st, tm);
    return launch_step_nr<NPL, 1>(lo, a, st, tm);
}

hipError_t launch_cache_step(const Layout& lo, const StepArgs& a, hipStream_t st, const Timing& tm) {
    if (lo.N <= 64) return launch_step_npl<1>(lo, a, st, tm);
    if (lo.N <= 128) return launch_step_npl<2>(lo, a, st, tm);
    return launch_step_npl<4>(lo, a, st, tm);
}

}  // namespace cmoe
