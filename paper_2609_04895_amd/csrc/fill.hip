// fill.hip - physical residency and expert copies (the demand loads and
// proactive loads of Section 2 / Algorithm 2 as transfers into HBM slots).
//
// A residency event of a layer follows the refinement (proactive loads) or the
// post-access update (demand loads): the layer's HBM slots must hold the union
// U of the streams' caches.  Experts that left U free their slot; each new
// expert, in ascending order, takes the lowest free slot and is copied there
// from the cold pool.
//
// Two kernels, each launched once for a batch of layers:
//   residency_kernel  one workgroup per layer decides the layer's events in
//                     order (the proactive one, if the token refined, then the
//                     demand one) on its slot maps in LDS, lists the copies of
//                     each and lays out the layer step's FFN work units;
//   copy_kernel       walks the listed copies of all layers of the batch in
//                     pieces of 16 or 32 KB;
// or, for a batch of one layer with a demand event only, one:
//   fill_kernel       every workgroup decides the event by itself and copies
//                     its share of the pieces.
// fill_kernel's workgroups read a copy of the slot maps that the cache step has
// made, and one of them writes the maps.
// The host never reads the lists.  The pool may be pinned host memory mapped
// into the device; copies then run over the host link.
#include "cmoe_internal.h"

namespace cmoe {

namespace {

// Threads of a fill workgroup (four wavefronts), a compile-time constant so
// that no loop bound has to be read from the dispatch packet.
constexpr int kFillThreads = 256;
static_assert(kFillThreads == kMaxN, "one expert, one slot and one ranking key per thread");

// Block-wide exclusive prefix counts and sums over the 256 threads of the
// block, each call with one barrier: the wavefront totals go to LDS slots
// (four per value), and consecutive calls use different slots, so no barrier
// is needed after one call before the next.
// NF flags at once: the ballot bits below the lane; total[f] gets the block
// total of flag f.  slot: 4 NF ints.
template <int NF>
__device__ void block_counts(const bool (&v)[NF], int (&below)[NF], int (&total)[NF], int* slot) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const unsigned long long b = __ballot(v[f]);
        below[f] = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
        if (lane == 0) slot[4 * f + w] = __popcll(b);
    }
    __syncthreads();
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        int off = 0, tot = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < w) off += slot[4 * f + i];
            tot += slot[4 * f + i];
        }
        below[f] += off;
        total[f] = tot;
    }
}

// Inclusive wavefront scan in DPP steps (shifts by 1, 2, 4 and 8 inside each
// 16-lane row, then the last lane of row 0 and of row 1 added to the rows
// after them); a lane whose source is outside its row adds 0.
__device__ inline int wave_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
    return x;
}

__device__ int block_scan(int v, int* total, int* slot) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int x = wave_scan(v);
    if (lane == 63) slot[w] = x;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < w) off += slot[i];
        tot += slot[i];
    }
    *total = tot;
    return off + x - v;
}

// bf16 experts are stored in their HBM slot in the order the FFN kernels
// consume them, so that every load instruction reads 1 KB of contiguous
// memory.  Units are 16 bytes (8 bf16); lane l of a wavefront takes unit l of
// a 64-unit run.
//   gate/up part, units [0, F d / 4):
//     ((((ft * (d/64) + c) * 2 + mat) * 2 + half) * 64 + lane)
//     = W_mat[16 ft + lane % 16][64 c + 32 half + 8 (lane / 16) .. + 8],
//     mat 0 = gate, 1 = up
//   down part, units [F d / 4, 3 F d / 8):
//     F d / 4 + ((((dt * (F/64) + c) * 2 + mt) * 2 + half) * 64 + lane)
//     = W_down[32 dt + 16 mt + lane % 16][64 c + 32 half + 8 (lane / 16) .. + 8]
// The cold pool keeps the plain row-major layout.  Every 128-unit block of
// the packed order (one run for each half) holds 16 source rows x 128
// contiguous bytes: rows 16 ft + r of W_mat at columns 64 c .. 64 c + 63 for
// the gate/up part, rows 32 dt + 16 mt + r of W_down at columns 64 c .. for
// the down part.
//
// A piece is up to CH k chunks c of one tile, both blocks (gate and up, or the
// two 16-row halves) of each chunk: 32 source row segments of up to 128 CH
// bytes, one contiguous run of up to 4 CH KB in the slot.  It passes through
// LDS, so that both the loads and the stores of a wavefront are contiguous, and
// the next piece's loads are in flight while this one is stored.  Measured on
// MI355X (read plus write, 96 experts of 9.4 MB and 16 of 49.8 MB): CH = 4 with
// 512 workgroups and nontemporal loads and stores 6.2 and 5.7 TB/s, without
// them 5.9 and 5.3; CH = 8 5.5 and 5.4, CH = 2 5.7; 1280 workgroups 5.7 and 5.2;
// without LDS, 128-byte row segments read straight into the packed order, 4.0
// to 4.5 one load a thread and at most 5.6 four loads a thread; a plain copy of
// the same bytes 6.0.
// Source unit w of a block (row w / 8, 16-byte unit w % 8 of the row's 128
// bytes) goes to packed unit (unit / 4) * 64 + row + 16 (unit % 4).
__device__ inline int packed_dest_in_block(int w) {
    const int r = w >> 3, j = w & 7;
    return (j >> 2) * 64 + r + 16 * (j & 3);
}

// LDS place of piece unit p = 256 c + 128 sub + packed unit.  A wavefront
// stores one row's units (bits 4-6 and 8-10 of p vary: a stride of 256 bytes
// or more, all in one bank group) and loads 64 consecutive p; the low four
// bits, xored with those six, spread the stores over the sixteen 16-byte bank
// groups and stay a permutation for the loads.
__device__ inline int piece_place(int p) { return p ^ (((p >> 4) & 7) ^ (((p >> 8) & 7) << 1)); }

// Expert copies are read once and written once: nontemporal both ways.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ inline uint4 load_once(const uint4* p) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return uint4{v.x, v.y, v.z, v.w};
}
__device__ inline void store_once(uint4* p, const uint4& v) {
    __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(p));
}

// Cache word i = s NW + j: word j of stream s's membership bits of the layer,
// after the refinement or (demand) after the access.
template <bool DEMAND>
__device__ inline unsigned long long cache_word(const Layout& lo, int layer, int i) {
    if constexpr (!DEMAND) {
        return lo.mid[(int64_t)layer * lo.S * lo.NW + i];
    } else {
        const int s = i / lo.NW, j = i - s * lo.NW;
        return lo.cache[((int64_t)s * lo.L + layer) * lo.NW + j];
    }
}

constexpr int kWords = 4;  // cache words per thread per batch of loads

// A layer's state during its residency events.
struct ResLds {
    unsigned long long U[2][4];  // unions of the caches: after the access, after the refinement
    int so[kMaxN], se[kMaxN], stp[kMaxN], rnd_s[kMaxN], free_list[kMaxN], victim_list[kMaxN];
    int lds4[8];         // block-scan slots
    int lds_cnt[2][20];  // block-count slots: round plan; free slots, entries, units
    __align__(16) int key[kMaxN];
    int by_rank[kMaxN], who[kMaxN], m_rank[kMaxN];
};

template <bool DEMAND>
__device__ inline void load_words(const Layout& lo, int layer, int i0, unsigned long long (&w)[kWords]) {
#pragma unroll
    for (int u = 0; u < kWords; ++u)
        w[u] = cache_word<DEMAND>(lo, layer, min(i0 + (int)threadIdx.x + u * kFillThreads, lo.S * lo.NW - 1));
}

// U gets the union of the layer's caches; w holds the first batch of words.
template <bool DEMAND>
__device__ inline void unite(const Layout& lo, int layer, unsigned long long (&w)[kWords], unsigned long long* U) {
    const int S_NW = lo.S * lo.NW, tid = threadIdx.x;
    const bool fixed = kFillThreads % lo.NW == 0;  // all of a thread's words are the same word of their stream
    unsigned long long acc = 0ull;
    for (int i0 = 0; i0 < S_NW; i0 += kWords * kFillThreads) {
        if (i0 > 0) {
            load_words<DEMAND>(lo, layer, i0, w);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 0; u < kWords; ++u) {
            const int i = i0 + tid + u * kFillThreads;
            if (i >= S_NW) continue;
            if (fixed)
                acc |= w[u];
            else if (w[u])
                atomicOr(&U[i % lo.NW], w[u]);
        }
    }
    if (fixed && acc) atomicOr(&U[tid % lo.NW], acc);
}

// One residency event of `layer`; the slot maps in sm are current on entry and
// on return, and list gets the copies ((slot << 8) | expert, in the experts'
// ascending order).  Returns their number.  Every thread of the workgroup runs
// it.  m_v, ro_v: this thread's expert's bucket size and (later rounds) its
// planned round.  writer: this workgroup stores the round plan and the units.
template <bool DEMAND>
__device__ __forceinline__ int residency_event(const Layout& lo, const ResidencyArgs& f, ResLds& sm, int bl, int m_v, int ro_v,
                                               bool writer, int clk, int32_t* list) {
    const bool units = DEMAND && writer && f.units;
    const int round = f.round;
    const unsigned long long* U = sm.U[DEMAND ? 0 : 1];
    int *so = sm.so, *se = sm.se, *stp = sm.stp, *rnd_s = sm.rnd_s, *free_list = sm.free_list;
    const int tid = threadIdx.x, e = tid, N = lo.N, P = lo.n_slots;
    const bool inU = e < N && ((U[e >> 6] >> (e & 63)) & 1ull);
    int cur = e < N ? so[e] : -1;
    if (e < N && cur >= 0 && !inU) {  // left every cache: free its slot
        se[cur] = -1;
        so[e] = -1;
        cur = -1;
    }
    int nU = 0;
    for (int j = 0; j < lo.NW; ++j) nU += __popcll(U[j]);
    const bool overflow = nU > P;  // the union does not fit the arena (block-uniform)
    __syncthreads();
    // FFN round of each expert the layer step executes.  While the union fits,
    // all run in round 0.  Otherwise round 0 plans the rounds: the executed
    // experts already resident first, then the others, each group ascending,
    // P per round; later rounds read the plan.
    const bool inE = DEMAND && e < N && m_v > 0;
    int rnd = -1;
    if (DEMAND) {
        if (!overflow) {
            rnd = inE ? 0 : -1;
        } else if (round == 0) {
            const bool res_e = inE && cur >= 0, mis_e = inE && cur < 0;
            const bool fl[2] = {res_e, mis_e};
            int rk[2], n[2];
            block_counts<2>(fl, rk, n, sm.lds_cnt[0]);
            rnd = res_e ? rk[0] / P : (mis_e ? (n[0] + rk[1]) / P : -1);
        } else {
            rnd = e < N ? ro_v : -1;
        }
        if (writer && round == 0 && e < N) lo.round_of[(int64_t)bl * N + e] = rnd;
    }
    if (e < N) rnd_s[e] = rnd;
    const bool now = DEMAND && rnd >= 0 && rnd == round;  // executed in this round
    bool enter;
    if (!DEMAND) enter = e < N && inU && cur < 0;
    else if (!overflow) enter = round == 0 && e < N && inU && cur < 0;
    else enter = now && cur < 0;
    const bool is_free = tid < P && se[tid] == -1;
    // The work units of this round (below) need to know whether any bucket
    // takes more than one pass, and rank the experts by their bucket sizes
    // if one does: the flags join the free-slot and entry counts, and the
    // ranking keys are stored before the same barrier.
    const int m_own = (units && now) ? m_v : 0;
    const int ut = lo.unit_tokens;
    const int mykey = (m_own << 8) | (255 - tid);
    if (units) sm.key[tid] = tid < N ? mykey : -1;  // kFillThreads == kMaxN: every entry is written
    const int light = lo.max_heavy > 0 ? kLightTokens : ut;  // tokens of the largest unit of the second list
    const bool fl[5] = {is_free, enter, m_own > ut, m_own > light, m_own > 0 && m_own <= light};
    int rk[5], n[5];
    block_counts<5>(fl, rk, n, sm.lds_cnt[1]);
    const int rf = rk[0], re = rk[1], nfree = n[0], nenter = n[1];
    const bool multi = n[2] > 0;
    if (is_free) free_list[rf] = tid;
    // A round that needs more than the free slots evicts the least recently
    // used experts that no remaining round needs (lower slot on ties), ranked
    // by (stamp, slot); after refinement only free slots are filled.
    int nvict = 0;
    if (DEMAND && overflow && nenter > nfree) {  // block-uniform
        bool vict = false;
        int rank = 0;
        if (tid < P && se[tid] >= 0) {
            vict = rnd_s[se[tid]] < round;
            if (vict) {
                const int sq = stp[tid];
                for (int q2 = 0; q2 < P; ++q2) {
                    const int v2 = se[q2];
                    if (v2 < 0 || rnd_s[v2] >= round) continue;
                    const int s2 = stp[q2];
                    rank += (s2 < sq || (s2 == sq && q2 < tid)) ? 1 : 0;
                }
            }
        }
        if (vict) sm.victim_list[rank] = tid;
        nvict = __syncthreads_count(vict);
    }
    const int nent = (!DEMAND && overflow) ? min(nenter, nfree) : nenter;
    __syncthreads();
    const bool takes = enter && re < nent;
    if (takes) {  // rank re among new experts takes the rank-re free slot, then the victims in rank order
        int q = -1;
        if (re < nfree)
            q = free_list[re];
        else if (re - nfree < nvict)
            q = sm.victim_list[re - nfree];
        if (q >= 0) {
            if (re >= nfree) so[se[q]] = -1;  // evicted
            so[e] = q;
            se[q] = e;
        }
        list[re] = (max(q, 0) << 8) | e;  // q < 0 cannot happen: a round fits the arena
    }
    __syncthreads();
    // last use: the experts executed in this round and every expert copied in
    if (e < N && (now || takes) && so[e] >= 0) stp[so[e]] = clk;
    __syncthreads();
    // FFN work units of this round: each of its experts' buckets cut into
    // passes of up to lo.unit_tokens tokens, each stored with its expert's new
    // slot and its token count, so that an FFN wavefront finds all three with
    // one load; {-1, -1, 0, 0} past the last unit.
    int4* big4 = reinterpret_cast<int4*>(lo.units) + (int64_t)bl * lo.max_units;
    int4* unit4 = big4 + lo.max_heavy;
    int nbig = n[3], nunit = n[4];
    if (units && !multi) {  // one unit per expert, in ascending order
        if (fl[3]) big4[rk[3]] = int4{e, so[e], m_own, 0};
        if (fl[4]) unit4[rk[4]] = int4{e, so[e], m_own, 0};
    } else if (units) {
        // otherwise experts with more tokens go first (lower index on ties),
        // so the longest units start first.  Rank of expert e = number of
        // larger keys (m << 8) | (255 - e), all distinct.
        // (the keys were stored before the barrier of the counts above)
        int *by_rank = sm.by_rank, *who = sm.who, *m_rank = sm.m_rank;
        const int m = m_own;
        int rank = 0;
        if (tid < N) {
            // batches of 32 keys, every LDS read of a batch issued before the
            // first compare; keys past N are -1 and never counted
            const int4* k4 = reinterpret_cast<const int4*>(sm.key);
            for (int u0 = 0; u0 < (N + 3) / 4; u0 += 8) {  // u0 + 7 < kMaxN / 4
                int4 v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = k4[u0 + i];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    rank += (v[i].x > mykey) + (v[i].y > mykey) + (v[i].z > mykey) + (v[i].w > mykey);
            }
        }
        if (tid < N) {
            by_rank[rank] = (m + ut - 1) / ut;
            who[rank] = tid;
            m_rank[rank] = m;
        }
        __syncthreads();
        // full passes of ut tokens, and the last pass, of either list
        const int passes = tid < N ? by_rank[tid] : 0;
        const int tail = passes > 0 ? m_rank[tid] - ut * (passes - 1) : 0;
        const int mine_big = lo.max_heavy > 0 ? (tail > light ? passes : max(passes - 1, 0)) : 0;
        const int off_big = block_scan(mine_big, &nbig, sm.lds4);
        const int off = block_scan(passes - mine_big, &nunit, sm.lds4 + 4);
        if (tid < N) {
            const int x = who[tid];
            for (int q = 0; q < passes; ++q) {
                int4* at = q < mine_big ? big4 + off_big + q : unit4 + off + (q - mine_big);
                *at = int4{(q << 8) | x, so[x], min(ut, m_rank[tid] - ut * q), 0};
            }
        }
    }
    if (units) {
        for (int i = nbig + tid; i < lo.max_heavy; i += kFillThreads) big4[i] = int4{-1, -1, 0, 0};
        for (int i = nunit + tid; i < lo.max_units - lo.max_heavy; i += kFillThreads) unit4[i] = int4{-1, -1, 0, 0};
    }
    return nent;
}

// The residency events of layer f.l0 + bl, decided by the whole workgroup; the
// copies go to dem and pro (PRO: the token may have refined).  Returns their
// numbers.  writer: this workgroup stores the new state.
template <bool PRO>
__device__ __forceinline__ int2 layer_events(const Layout& lo, const ResidencyArgs& f, ResLds& sm, int bl, bool writer,
                                             int32_t* dem, int32_t* pro) {
    const int layer = f.l0 + bl, tid = threadIdx.x, N = lo.N, P = lo.n_slots;
    const bool refined = PRO && f.refined && f.round == 0;
    int32_t* so_g = lo.slot_of + (int64_t)layer * N;
    int32_t* se_g = lo.slot_exp + (int64_t)layer * P;
    int32_t* st_g = lo.slot_stamp + (int64_t)layer * P;
    // Every global load is issued before the first is used (indices clamped; a
    // value that is not needed is not used): the slot maps and stamps, the
    // bucket sizes (the executed experts and the FFN work units), the round
    // plan of a later round, the fill counters, and the first batch of cache
    // words of each event.
    const int so_v = (PRO ? so_g : lo.snap_of)[min(tid, N - 1)], se_v = (PRO ? se_g : lo.snap_exp)[min(tid, P - 1)];
    const int st_v = writer ? st_g[min(tid, P - 1)] : 0;
    const int mb_v = lo.bcount[(int64_t)bl * N + min(tid, N - 1)];
    const int ro_v = lo.round_of[(int64_t)bl * N + min(tid, N - 1)];
    const int64_t phys0 = lo.phys[layer * 2], phys1 = lo.phys[layer * 2 + 1];
    const int32_t sf_v = lo.step_fills[layer * 2];
    const unsigned long long sel_v = lo.selcount[(int64_t)layer * N + min(tid, N - 1)], act_v = lo.active_sum[layer];
    unsigned long long w[kWords], wp[kWords];
    load_words<true>(lo, layer, 0, w);
    if (refined) load_words<false>(lo, layer, 0, wp);
    __builtin_amdgcn_sched_barrier(0);
    if (tid < 8) sm.U[tid >> 2][tid & 3] = 0ull;
    if (tid < N) sm.so[tid] = so_v;
    if (tid < P) {
        sm.se[tid] = se_v;
        sm.stp[tid] = st_v;
    }
    __syncthreads();
    unite<true>(lo, layer, w, sm.U[0]);
    if (refined) unite<false>(lo, layer, wp, sm.U[1]);
    __syncthreads();
    int npro = 0;
    if (refined) {
        npro = residency_event<false>(lo, f, sm, bl, 0, -1, writer, f.clk, pro);
        __syncthreads();
    }
    // the bucket sizes decide nothing but what the writer stores while the
    // union fits the arena
    const int ndem = residency_event<true>(lo, f, sm, bl, writer ? mb_v : 0, ro_v, writer, f.clk + (refined ? 1 : 0), dem);
    if (!writer) return int2{ndem, npro};
    // the layer step's selections and distinct experts, from the bucket sizes:
    // one atomic per selection in the cache step queued at the experts'
    // counters (cache step of 24 layers and 64 streams 12.2 us with them, 8.1
    // without; of 48 layers and 256 streams of given logits 36.2 and 32.0; this
    // launch stays within 0.2 us)
    if (f.counted && f.round == 0) {
        if (tid < N) lo.selcount[(int64_t)layer * N + tid] = sel_v + (unsigned)mb_v;
        const int distinct = __syncthreads_count(tid < N && mb_v > 0);
        if (tid == 0) lo.active_sum[layer] = act_v + (unsigned)distinct;
    }
    if (f.last && tid < N) lo.bcount[(int64_t)bl * N + tid] = 0;
    if (tid < N) so_g[tid] = sm.so[tid];
    if (tid < P) {
        se_g[tid] = sm.se[tid];
        st_g[tid] = sm.stp[tid];
    }
    if (tid == 0) {
        lo.step_fills[layer * 2] = (f.round > 0 ? sf_v : 0) + ndem;
        if (f.counted) lo.phys[layer * 2] = phys0 + ndem;
        if (f.round == 0) {
            lo.step_fills[layer * 2 + 1] = npro;
            if (f.counted && npro) lo.phys[layer * 2 + 1] = phys1 + npro;
        }
    }
    return int2{ndem, npro};
}

// grid: one workgroup per layer of the batch.  Latency-bound (one round trip
// of loads, then some twelve barriers), so the layers of a batch run side by
// side.
__global__ __launch_bounds__(kFillThreads) void residency_kernel(Layout lo, ResidencyArgs f) {
    __shared__ ResLds sm;
    const int layer = f.l0 + blockIdx.x;
    int32_t* list = lo.copy_list + (int64_t)layer * 2 * lo.N;
    const int2 n = layer_events<true>(lo, f, sm, blockIdx.x, true, list, list + lo.N);
    if (threadIdx.x == 0) {
        lo.copy_n[layer * 2] = n.x;
        if (f.round == 0) lo.copy_n[layer * 2 + 1] = n.y;
    }
}

// One piece of one copy: where its data comes from and goes.
struct Piece {
    const char* src;
    char* dst;
    int piece;  // -1: nothing to copy
};

// bf16: gate/up tiles first, then the down tiles.
template <int CH>
struct PackedCopy {
    static constexpr int kRows = 256 / (8 * CH);  // row segments that the workgroup loads at once
    static constexpr size_t kLds = sizeof(uint4) * 256 * CH;
    uint4 v[CH];
    int64_t d0;  // first packed unit
    int nc;      // chunks of this piece

    __host__ __device__ static int pieces(const Layout& lo) {
        const int gA = (lo.d / 64 + CH - 1) / CH, gB = (lo.F / 64 + CH - 1) / CH;
        return lo.F / 16 * gA + lo.d / 32 * gB;
    }
    __device__ void load(const Piece& pc, int d, int F) {
        const int nA = d / 64, gA = (nA + CH - 1) / CH, nB = F / 64, gB = (nB + CH - 1) / CH;
        const int partA = F / 16 * gA;
        int64_t s0, row, sub;  // source units: first, between rows, between the two blocks
        if (pc.piece < partA) {
            const int tile = pc.piece / gA, c0 = (pc.piece - tile * gA) * CH;
            nc = min(CH, nA - c0);
            row = d / 8;
            sub = (int64_t)F * row;
            s0 = (int64_t)16 * tile * row + 8 * c0;
            d0 = ((int64_t)tile * nA + c0) * 256;
        } else {
            const int q = pc.piece - partA, tile = q / gB, c0 = (q - tile * gB) * CH;
            nc = min(CH, nB - c0);
            row = F / 8;
            sub = 16 * row;
            s0 = (int64_t)2 * F * (d / 8) + (int64_t)32 * tile * row + 8 * c0;
            d0 = (int64_t)2 * F * (d / 8) + ((int64_t)tile * nB + c0) * 256;
        }
        const int u = threadIdx.x % (8 * CH), r0 = threadIdx.x / (8 * CH);
        const uint4* src = reinterpret_cast<const uint4*>(pc.src) + s0 + u;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = i * kRows + r0;  // rows 0-15: first block, 16-31: second
            if ((u >> 3) < nc) v[i] = load_once(src + (r >> 4) * sub + (r & 15) * row);
        }
    }
    __device__ void stage(uint4* buf) const {
        const int u = threadIdx.x % (8 * CH), c = u >> 3, r0 = threadIdx.x / (8 * CH);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = i * kRows + r0;
            if (c < nc)
                buf[piece_place(c * 256 + (r >> 4) * 128 + packed_dest_in_block(((r & 15) << 3) | (u & 7)))] = v[i];
        }
    }
    __device__ static void store(const uint4* buf, char* dst, int64_t d0, int nc) {
        uint4* o = reinterpret_cast<uint4*>(dst) + d0 + threadIdx.x;
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (i < nc) store_once(o + i * 256, buf[piece_place(i * 256 + (int)threadIdx.x)]);
    }
};

// fp32: each matrix transposed (W_gate^T, W_up^T [d][F], W_down^T [F][d]) so
// that the lanes of the FFN kernels, one output row each, read consecutive
// addresses; a piece is one 64 x 64 tile, through LDS.
struct TransposeCopy {
    static constexpr size_t kLds = sizeof(float) * 64 * 65 + 48;  // a multiple of 16
    float v[16];
    int64_t d0;  // first output float
    int nc;      // floats between output rows

    __host__ __device__ static int pieces(const Layout& lo) { return 3 * (lo.F / 64) * (lo.d / 64); }
    __device__ void load(const Piece& pc, int d, int F) {
        const int per = (F / 64) * (d / 64), mat = pc.piece / per, t = pc.piece - mat * per;
        const int rows = mat < 2 ? F : d, cols = mat < 2 ? d : F, ct = cols / 64;
        const int r0 = t / ct * 64, c0 = (t % ct) * 64;
        const float* s = reinterpret_cast<const float*>(pc.src) + (int64_t)mat * d * F +
                         (int64_t)(r0 + (threadIdx.x >> 6)) * cols + c0 + (threadIdx.x & 63);
        d0 = (int64_t)mat * d * F + (int64_t)c0 * rows + r0;
        nc = rows;
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = s[(int64_t)4 * i * cols];
    }
    __device__ void stage(uint4* buf) const {
        float* b = reinterpret_cast<float*>(buf) + (threadIdx.x >> 6) * 65 + (threadIdx.x & 63);
#pragma unroll
        for (int i = 0; i < 16; ++i) b[4 * i * 65] = v[i];
    }
    __device__ static void store(const uint4* buf, char* dst, int64_t d0, int nc) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        const float* b = reinterpret_cast<const float*>(buf) + lane * 65 + w;
        float* o = reinterpret_cast<float*>(dst) + d0 + (int64_t)w * nc + lane;
#pragma unroll
        for (int i = 0; i < 16; ++i) o[(int64_t)4 * i * nc] = b[4 * i];
    }
};

// The workgroups walk `total` pieces in turn; piece_of(item) finds one.
template <class COPY, class PIECE_OF>
__device__ __forceinline__ void copy_pieces(const Layout& lo, int64_t total, uint4* buf, PIECE_OF piece_of) {
    COPY cp;
    Piece pc = piece_of(blockIdx.x);
    if (pc.piece >= 0) cp.load(pc, lo.d, lo.F);
    for (int64_t item = blockIdx.x; item < total; item += gridDim.x) {
        __syncthreads();  // the previous piece has left the buffer
        cp.stage(buf);
        __syncthreads();
        char* dst = pc.dst;
        const int64_t d0 = cp.d0;
        const int nc = cp.nc;
        pc = piece_of(item + gridDim.x);
        if (pc.piece >= 0) cp.load(pc, lo.d, lo.F);
        COPY::store(buf, dst, d0, nc);
    }
}

__device__ inline int64_t expert_bytes(const Layout& lo) { return lo.expert_elems * (lo.dtype == 1 ? 2 : 4); }

// Piece number `piece` of the copy that list entry ent ((slot << 8) | expert)
// of a layer asks for.
__device__ inline Piece piece_at(const Layout& lo, int64_t bytes, int layer, int ent, int piece) {
    return Piece{static_cast<const char*>(lo.pool) + ((int64_t)layer * lo.N + (ent & 255)) * bytes,
                 static_cast<char*>(lo.arena) + ((int64_t)layer * lo.n_slots + (ent >> 8)) * bytes, piece};
}

// The listed copies of layers l0 .. l0 + nl - 1 (nl <= kMaxBatch, a layer per
// lane): every wavefront finds the copies of all layers from one load and a
// prefix sum, and the workgroups walk the pieces of all copies.  kind: 0
// demand, 1 proactive.
static_assert(kMaxBatch <= 64, "copy_kernel holds one layer of the batch per lane");
template <class COPY>
__global__ __launch_bounds__(kFillThreads) void copy_kernel(Layout lo, int l0, int nl, int kind) {
    __shared__ uint4 buf[COPY::kLds / sizeof(uint4)];
    const int lane = threadIdx.x & 63;
    const int mine = lane < nl ? lo.copy_n[(l0 + lane) * 2 + kind] : 0;
    const int below = wave_scan(mine);  // copies of this lane's layer and the ones before it
    const int ncopies = __builtin_amdgcn_readlane(below, 63);
    const int pieces = COPY::pieces(lo);
    const int64_t total = (int64_t)ncopies * pieces, bytes = expert_bytes(lo);
    copy_pieces<COPY>(lo, total, buf, [&](int64_t item) {  // workgroup-uniform
        if (item >= total) return Piece{nullptr, nullptr, -1};
        const int c = (int)(item / pieces);
        const int bl = __popcll(__ballot(below <= c));  // layers whose copies all come before this one
        const int layer = l0 + bl, k = c - (bl > 0 ? __builtin_amdgcn_readlane(below, bl - 1) : 0);
        return piece_at(lo, bytes, layer, lo.copy_list[((int64_t)layer * 2 + kind) * lo.N + k],
                        (int)(item - (int64_t)c * pieces));
    });
}

// The demand event of layer f.l0 and its copies, the arena always holding the
// union of the caches (so that the bucket sizes decide nothing).  With one layer
// there is nothing to run side by side, and a second launch for what is usually
// an empty copy list costs more than every workgroup deciding the event again,
// however many streams' caches it reads.
// Two launches against this one: 8.1 and 4.2 us at 64 streams of the 128-expert
// shape; a token of given logits 12.0 and 9.3 us at 1 stream, 14.0 and 12.6 at
// 256, 136 and 134.5 at 8192.
template <class COPY>
__global__ __launch_bounds__(kFillThreads) void fill_kernel(Layout lo, ResidencyArgs f) {
    __shared__ ResLds sm;
    __shared__ int32_t list[kMaxN];
    __shared__ uint4 buf[COPY::kLds / sizeof(uint4)];
    const int ncopies = layer_events<false>(lo, f, sm, 0, blockIdx.x == 0, list, nullptr).x;
    const int pieces = COPY::pieces(lo);
    const int64_t total = (int64_t)ncopies * pieces, bytes = expert_bytes(lo);
    copy_pieces<COPY>(lo, total, buf, [&](int64_t item) {  // workgroup-uniform
        if (item >= total) return Piece{nullptr, nullptr, -1};
        const int c = (int)(item / pieces);
        return piece_at(lo, bytes, f.l0, __builtin_amdgcn_readfirstlane(list[c]), (int)(item - (int64_t)c * pieces));
    });
}

// launch(copy type, workgroups) for the type of the weights and the pool
template <typename F>
void with_copy(const Layout& lo, F&& launch) {
    const dim3 blocks(lo.pool_host ? kCopyBlocksHost : kCopyBlocksDevice);
    if (lo.dtype != 1)
        launch(TransposeCopy{}, blocks);
    else if (lo.pool_host)
        launch(PackedCopy<8>{}, blocks);
    else
        launch(PackedCopy<4>{}, blocks);
}

}  // namespace

hipError_t launch_residency(const Layout& lo, const ResidencyArgs& f, hipStream_t st, const Timing& tm) {
    launch_kernel(residency_kernel, dim3(f.nl), dim3(kFillThreads), st, tm, lo, f);
    return hipGetLastError();
}

hipError_t launch_copies(const Layout& lo, int l0, int nl, int kind, hipStream_t st, const Timing& tm) {
    with_copy(lo, [&](auto copy, dim3 blocks) {
        launch_kernel(copy_kernel<decltype(copy)>, blocks, dim3(kFillThreads), st, tm, lo, l0, nl, kind);
    });
    return hipGetLastError();
}

hipError_t launch_fill(const Layout& lo, const ResidencyArgs& f, hipStream_t st, const Timing& tm) {
    with_copy(lo, [&](auto copy, dim3 blocks) {
        launch_kernel(fill_kernel<decltype(copy)>, blocks, dim3(kFillThreads), st, tm, lo, f);
    });
    return hipGetLastError();
}

}  // namespace cmoe
