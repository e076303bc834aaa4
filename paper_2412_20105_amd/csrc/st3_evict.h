// Exact top-k selection (radix select on the order-preserving image of the fp32 score, ties by
// id) and the per-sequence eviction plan of a decode step (Eq. 3, Eq. 7, Alg. 3 VTA branch), as
// device code of the selection and eviction kernels.
#pragma once

#include <cstddef>
#include <type_traits>

#include "st3_decode.h"

namespace st3 {
constexpr int kSelLdsKeys = 8192;

__device__ __forceinline__ uint32_t score_key(float f) {
    uint32_t u = __float_as_uint(f);
    if (u == 0x80000000u) u = 0u;                       // -0.0 ranks with +0.0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // larger float <-> larger key
}

struct EvictArgs {
    float* score_col;
    int32_t* id_col;
    int64_t col_stride;
    int32_t* vis_len;
    int32_t* kv_len;
    const int32_t* tail_start;  // [B] or null: the tail keeps its place (no tail moves, kv_len not lowered)
    int32_t sys_len, max_vis, max_kv, keep_count, mode;
    int32_t* move_cnt;          // [B]
    int32_t* moves;             // [B][max_moves][2] = (dst row, src row)
    int32_t max_moves;
    // extras used by the fused per-layer decode step
    int32_t appended;           // 1: the attention kernel has just written one more row than kv_len[b] says
    int32_t capacity;           // row stride of `logits` (capacity of the cache whose attention produced them)
    int32_t inline_apply;       // 1: HOLE_FILL moves are applied to K and V by this kernel
    char* k;
    char* v;
    int64_t stride_b, stride_h, stride_t;   // bytes
    int32_t H, vecs_per_row;
    // visual mass the attention kernel left to be finished here (all null: none)
    const float* part_ml;
    const float* logits;
    const int32_t* pending;     // [B][4] descriptor written by the attend kernel (read only: lazy layers share it)
    int32_t nsplit_cap;
    float* mass_dst;
    int64_t mass_stride;
    const int32_t* own_pending; // descriptor of this layer's own attention (its visual rows); `pending` unless the layer is lazy
    int32_t mass_apart;         // 1: score_col does not take this step's mass: whoever ranks it need not wait for the mass
};

// The plan of a layer of a whole step, from its table entry.
__device__ __forceinline__ EvictArgs plan_from_entry(const StepCommon& c, const StepLayer& e) {
    const DecodeWs wl = decode_ws_sized(c.B, c.H, c.D, e.capacity, e.nsplit_cap);
    EvictArgs a;
    a.score_col = e.score_col; a.id_col = e.id_col; a.col_stride = e.col_stride;
    a.vis_len = e.vis_len; a.kv_len = e.kv_len; a.tail_start = e.tail_start;
    a.sys_len = e.sys_len; a.max_vis = e.max_vis; a.max_kv = e.max_kv;
    a.keep_count = e.keep_count; a.mode = c.mode;
    a.move_cnt = reinterpret_cast<int32_t*>(e.ws + wl.moves_cnt);
    a.moves = reinterpret_cast<int32_t*>(e.ws + wl.moves);
    a.max_moves = wl.max_moves;
    a.appended = 1;
    a.inline_apply = (e.flags & kStepInlineApply) != 0;
    a.k = reinterpret_cast<char*>(e.k); a.v = reinterpret_cast<char*>(e.v);
    const int eb = (e.flags & kStepE4M3) ? 1 : c.elem_bytes;
    a.stride_b = e.stride_b * eb; a.stride_h = e.stride_h * eb; a.stride_t = (int64_t)e.stride_t * eb;
    a.H = c.H; a.vecs_per_row = c.D * eb / 16;
    // a lazy layer's mass is finished from what its source's launch left
    const bool lazy = (e.flags & kStepLazy) != 0;
    const DecodeWs ml = lazy ? decode_ws_sized(c.B, c.H, c.D, e.hint_base, e.src_nsplit_cap) : wl;
    const char* mws = lazy ? reinterpret_cast<const char*>(e.q) : e.ws;
    a.part_ml = reinterpret_cast<const float*>(mws + ml.part_ml);
    a.logits = reinterpret_cast<const float*>(mws + ml.logits);
    a.pending = reinterpret_cast<const int32_t*>(mws + ml.pending);
    a.nsplit_cap = ml.nsplit_cap; a.capacity = lazy ? e.hint_base : e.capacity;
    a.mass_dst = e.mass; a.mass_stride = e.mass_stride;
    a.own_pending = reinterpret_cast<const int32_t*>(e.ws + wl.pending);
    a.mass_apart = (e.flags & kStepApart) != 0;
    return a;
}

typedef uint32_t u32x4_v __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_a4_t __attribute__((ext_vector_type(4), aligned(4)));

// ---------------------------------------------------------------------------------------------
// The plan workgroup.  Latency bound: a chain of dependent steps over a few kilobytes per (layer, sequence), and at small
// batches there are fewer plans than compute units, so it takes as many threads as there is work for (plan_threads).  Its parts before
// -> after the 256-thread form, which kept eight head-strided loads in flight, ran six barriers per radix digit and went
// through a move list in global memory (us a launch: high resolution batch 8 77 -> 30, 13B batch 8 with fast annealing 66 ->
// 33, 7B batch 1 21 -> 13):
//   mass      heads are dealt to thread groups, 8 loads in flight per thread
//   select    two barriers per digit (one wave scans the histogram), and no further digit once the k-th key is apart
//   lists     ranks from ballots, the list of a small eviction in LDS
//   rows      moved past the caches: lines left dirty in L2 are written back between the reads of the next attention
//             (whole step, ordinary -> non-temporal: 13B batch 8 with fast annealing 541 -> 506 us, 7B batch 16 layer by layer
//             733 -> 704)
// ---------------------------------------------------------------------------------------------
constexpr int kPlanThreadsMost = 1024;
// Threads of a plan workgroup: what its chain of steps is spread over (mass: rows times heads, unless that has workgroups of its own;
// ranking: rows), against waves that start, meet at barriers and stop for nothing, and against plans that wait for each other when
// there are several per compute unit: one of 1024 threads, three of 512, seven of 256, by their scalar registers (a plan's LDS, 13
// KB and four bytes a row, allows more).  us a call with 256 / 512 / 1024 threads: layer step of 2 heads, 16 rows, evicting 8 14.1 /
// 14.1 / 15.2, 40 heads, 64 rows 16.1 / 16.6 / 17.5, 32 heads, 128 rows 17.6 / 17.7 / 18.6, 40 heads, 500 rows, batch 8 36.3 / 32.3 /
// 32.1; select-and-compact of 300 rows, batch 1 10.3 / 9.3 / 9.8, batch 512 12.2 / 11.6 / 18.6, 576 rows, batch 256 13.0 / 12.0 /
// 11.5, 16 rows, batch 2048 17.3 / 25.8 / 60.4; st3_decode_plans of 32 layers of 288 rows 21.8 / 20.2 / 21.2, 40 of 400 rows, batch 8
// 33.4 / 29.8 / 31.2, 32 of 2000 rows, batch 8 51.4 / 38.5 / 37.1, 40 of 576 rows, batch 12 37.7 / 33.7 / 40.7; whole steps whose columns
// take the mass, 7B batch 1 46.0 / 41.9 / 43.4, 13B batch 8 489 / 496 / 498, 2000 rows, batch 8 1512 / 1495 / 1487 (1024 in all three,
// which the first two would rather not).
inline int plan_threads(int64_t plans, int most_vis, int heads) {       // heads: 1 when no mass is to be finished
    const int64_t mass = (int64_t)most_vis * heads;
    if ((plans <= 512 && mass > 8192) || (plans <= 256 && most_vis > 512)) return 1024;
    return most_vis > 256 || mass >= 3072 ? 512 : 256;
}
// Threads of a workgroup that ranks one row of n scores.  us a call, 256 / 512 / 1024 threads (256-thread form of before): 256
// scores, batch 8 4.3 / 4.2 / 4.8 (5.3), batch 8192 27.9 / 30.6 / 64.0 (39.9), 365 scores 4.9 / 4.5 / 4.9 (6.3) and 35.4 / 34.3 / 68.4
// (53.9), 2880 scores, batch 8 14.4 / 10.1 / 9.0 (18.3), batch 1024 21.1 / 18.3 / 23.1 (27.0).
inline int topk_threads(int64_t rows, int n) { return n <= 256 ? 256 : n > 1024 && rows <= 512 ? 1024 : 512; }
// Runs go(NT) with that many threads as a constant.
template <typename Go>
void with_threads(int threads, Go go) {
    if (threads == 1024) go(std::integral_constant<int, 1024>{});
    else if (threads == 512) go(std::integral_constant<int, 512>{});
    else go(std::integral_constant<int, 256>{});
}
constexpr int kPlanMaxInline = 64;          // moves of an eviction that the plan workgroup applies itself (at most 48 evicted rows)

// What ranking a row of scores needs, and what a plan needs besides.  The keys lie in dynamic LDS (sel_keys(): a word for each row
// that is ranked, and for each thread of a plan), which takes no more of it than the call's rows need.
struct SelectShared {
    alignas(16) int hist[4][256];       // scanned as int4
    int wave_tot[2][kPlanThreadsMost / kWave];
    int sel_bin, sel_want, sel_cnt, red;
};
static_assert(alignof(SelectShared) == 16 && offsetof(SelectShared, hist) % 16 == 0, "plan_select reads four bins at once");
struct PlanShared : SelectShared {
    float hm[1024], hrl[1024];
    int mv[kPlanMaxInline][2];
};
__device__ __forceinline__ uint32_t* sel_keys() {
    extern __shared__ uint32_t sm_sel_keys[];
    return sm_sel_keys;
}
inline size_t plan_lds(int most_vis, int threads) { return sizeof(uint32_t) * (size_t)(most_vis > threads ? most_vis : threads); }

// Ranks of two flags over the workgroup in thread order: r1 / r2 = how many threads before this one have the flag,
// t1 / t2 = how many in all.  One barrier; calls in a row alternate `parity`.
template <int NT>
__device__ __forceinline__ void plan_ranks(bool f1, bool f2, int parity, SelectShared& sm, int& r1, int& r2, int& t1, int& t2) {
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const unsigned long long b1 = __ballot(f1), b2 = __ballot(f2), below = (1ull << lane) - 1;
    if (lane == 0) sm.wave_tot[parity][wave] = __popcll(b1) | (__popcll(b2) << 16);
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) {
        const int v = sm.wave_tot[parity][w];
        base += w < wave ? v : 0;
        tot += v;
    }
    r1 = (base & 0xffff) + __popcll(b1 & below);
    r2 = (base >> 16) + __popcll(b2 & below);
    t1 = tot & 0xffff; t2 = tot >> 16;
}

// Finds the key of rank `want` (1-based, descending) among the elements for which f(i, key) is true, 8 bits at a time.
// Returns its leading digits, zeros behind them: the search ends as soon as exactly the wanted elements share them.
// `want` becomes how many of the elements equal to the returned digits belong to the top set, `ties` how many there are.
// Ends with a barrier behind every use of sm.hist.
template <int NT, class F>
__device__ __forceinline__ uint32_t plan_select(F f, int n, int& want, int& ties, SelectShared& sm) {
    const int tid = threadIdx.x;
    for (int i = tid; i < 4 * 256; i += NT) (&sm.hist[0][0])[i] = 0;
    __syncthreads();
    uint32_t prefix = 0, pmask = 0;
    for (int r = 0; r < 4; ++r) {
        const int shift = 24 - 8 * r;
        for (int i = tid; i < n; i += NT) {
            uint32_t key;
            if (f(i, key) && (key & pmask) == prefix) atomicAdd(&sm.hist[r][(key >> shift) & 255u], 1);
        }
        __syncthreads();
        if (tid < kWave) {                              // lane l: bins 255 - 4 l ... 252 - 4 l
            const int4 c = *reinterpret_cast<const int4*>(&sm.hist[r][252 - 4 * tid]);
            const int sum = c.x + c.y + c.z + c.w;
            int incl = sum;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const int t = __shfl_up(incl, off);
                if (tid >= off) incl += t;
            }
            int before = incl - sum;
            if (incl >= want && before < want) {
                int bin = 255 - 4 * tid, cnt = c.w;
                if (want > before + cnt) { before += cnt; cnt = c.z; --bin; }
                if (want > before + cnt) { before += cnt; cnt = c.y; --bin; }
                if (want > before + cnt) { before += cnt; cnt = c.x; --bin; }
                sm.sel_bin = bin; sm.sel_want = want - before; sm.sel_cnt = cnt;
            }
        }
        __syncthreads();
        prefix |= (uint32_t)sm.sel_bin << shift;
        pmask |= 255u << shift;
        want = sm.sel_want;
        ties = sm.sel_cnt;
        if (want == ties) break;                        // uniform: sel_* are the workgroup's
    }
    __syncthreads();
    return prefix;
}

// Which elements are among the top k by (key descending, id ascending): those for which keeps() holds.  `key` may be the leading
// digits of the kept keys only (then `all` is set, and every key that is not below it stays).
struct TopSet {
    uint32_t key, idkey;        // idkey: ~id, so that the lowest ids rank first
    bool all;                   // all elements at `key` belong to the set
    // element i (its id is read only where the k-th key is shared)
    template <class Key, class IdKey>
    __device__ __forceinline__ bool keeps(Key key_at, IdKey idkey_at, int i) const {
        const uint32_t k = key_at(i);
        return k > key || (k == key && (all || idkey_at(i) >= idkey));
    }
};

// The set for 0 < k < n; key_at(i) and idkey_at(i) give element i's.  What the caller staged for them is read behind a barrier.
template <int NT, class Key, class IdKey>
__device__ __forceinline__ TopSet top_set(Key key_at, IdKey idkey_at, int n, int k, SelectShared& sm) {
    int want = k, ties = 0;
    TopSet t{0, 0, true};
    t.key = plan_select<NT>([&](int i, uint32_t& key) { key = key_at(i); return true; }, n, want, ties, sm);
    t.all = want == ties;
    if (!t.all) {                                       // the k-th key is shared: the lowest ids of its holders
        int want2 = want, ties2 = 0;
        t.idkey = plan_select<NT>([&](int i, uint32_t& key) { key = idkey_at(i); return key_at(i) == t.key; }, n, want2, ties2, sm);
    }
    return t;
}

// Copies rows move(i) = {destination, source}, i < count, on all strips of sequence b.  Callers guarantee that no destination of the batch is a
// source of it.  A wave moves one row of as many strips as 64 lanes of 16 bytes cover, kUR such pieces in flight.  The pieces are
// dealt to `parts` workgroups; by_strip: so that all pieces of a strip go to the same one.
// Bound by the trips to memory: the list's entries, then rows of 256 bytes here and there.  The entries of a round are fetched
// before the first of its rows (loads come back in order, so that an entry behind a row waits for it).  Rows are
// stored past the caches (ordinary stores: the launch 28 -> 23 us, but the next step's attention, which evicts them, 406 -> 464) and
// loaded through them.  us, entries one by one and non-temporal loads / entries together / and ordinary loads: launch behind the
// attention of 13B batch 8 with fast annealing (285 moves a sequence, 94 MB) 31.4 / 28.3 / 28.6, the attention behind it 404 / 406 / 402;
// whole steps of it 475 / 473 / 469, high resolution batch 2 E4M3 161.6 / 160.8 / 160.0, 8 layers of 12 heads, batch 32 52.0 / 50.0 / 49.2.
template <int NT, class Move>
__device__ __forceinline__ void copy_rows(const EvictArgs& a, int b, int part, int parts, bool by_strip, int count, Move move) {
    constexpr int kUR = 8, kWaves = NT / kWave;
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int strips = (a.k ? 2 : 1) * a.H;             // K may be absent (layers that keep V only)
    const int vpr = a.vecs_per_row, spw = kWave / vpr;  // 4 ... 32, a power of two
    const int all = (strips + spw - 1) / spw;           // pieces per row
    const int g0 = by_strip ? part : 0, gstep = by_strip ? parts : 1, groups = g0 < all ? (all - g0 + gstep - 1) / gstep : 1;
    const int total = g0 < all ? count * groups : 0;
    const int qstep = by_strip ? kWaves : parts * kWaves;
    for (int q0 = by_strip ? wave : part * kWaves + wave; q0 < total; q0 += kUR * qstep) {
        int2 m[kUR];
#pragma unroll
        for (int u = 0; u < kUR; ++u) m[u] = move(min(q0 + u * qstep, total - 1) / groups);
        u32x4_v tmp[kUR];
        char* to[kUR];
#pragma unroll
        for (int u = 0; u < kUR; ++u) {
            const int q = min(q0 + u * qstep, total - 1), strip = ((q % groups) * gstep + g0) * spw + lane / vpr;
            to[u] = nullptr;
            if (q0 + u * qstep >= total || strip >= strips) continue;
            const bool in_k = a.k && strip < a.H;
            char* base = (in_k ? a.k : a.v) + b * a.stride_b + (int64_t)(strip >= a.H ? strip - a.H : strip) * a.stride_h +
                         (lane % vpr) * 16;
            tmp[u] = *reinterpret_cast<const u32x4_v*>(base + m[u].y * a.stride_t);
            to[u] = base + m[u].x * a.stride_t;
        }
#pragma unroll
        for (int u = 0; u < kUR; ++u)
            if (to[u] != nullptr) __builtin_nontemporal_store(tmp[u], reinterpret_cast<u32x4_v*>(to[u]));
    }
}

// Merges the chunk partials of the output rows of heads [h0, h1) of sequence b in chunk order (what
// decode_finish_kernel does when the attention is called on its own).  Runs beside the plan
// workgroup of the same sequence, which rewrites the lengths: the number of rows the attend launch
// saw therefore comes from the descriptor that launch left (a lazy layer: its source's launch, which
// saw as many), not from the lengths.
__device__ __forceinline__ void merge_chunks(const StepCommon& c, const StepLayer& e, int b, int h0, int h1) {
    const bool lazy = (e.flags & kStepLazy) != 0;
    const DecodeWs wl = decode_ws_sized(c.B, c.H, c.D, e.capacity, e.nsplit_cap);
    const DecodeWs sl = lazy ? decode_ws_sized(c.B, c.H, c.D, e.hint_base, e.src_nsplit_cap) : wl;
    const int seen = reinterpret_cast<const int32_t*>((lazy ? reinterpret_cast<const char*>(e.q) : e.ws) + sl.pending)[b * 4] >> 1;
    const int ns = seen > 0 ? min((seen + e.chunk - 1) / e.chunk, (int)e.nsplit) : 0;
    if (ns <= 0) return;                                // an empty sequence had its zeros written by the attend launch
    const int D = c.D;
    h1 = min(h1, c.H);
    const float* part_o = reinterpret_cast<const float*>(e.ws + wl.part_o);
    const float* part_ml = reinterpret_cast<const float*>(e.ws + wl.part_ml);
    for (int idx = threadIdx.x; idx < (h1 - h0) * D; idx += blockDim.x) {
        const int h = h0 + idx / D, d = idx % D;
        const int64_t bh = (int64_t)b * c.H + h;
        const float* po = part_o + bh * wl.nsplit_cap * D + d;
        const float o = merge_partials(lazy, po, D, part_ml + bh * wl.nsplit_cap * 2, ns);
        if (c.elem_bytes == 2) reinterpret_cast<uint16_t*>(e.out)[bh * D + d] = (uint16_t)f32_to_bf16_bits(o);
        else reinterpret_cast<float*>(e.out)[bh * D + d] = o;
    }
}

// The visual mass that the attention launch left pending: mass_row[j] = (1/H) sum_h exp2(logit[h][j] - m_h) / l_h for
// j < n.  Heads are dealt to NT / keys groups of threads whose sums are added in group order: the result does not depend
// on scheduling.  ns: chunks per head of the attention launch.
template <int NT>
__device__ __forceinline__ void plan_mass(const EvictArgs& a, int b, int n, int ns, PlanShared& sm) {
    const int tid = threadIdx.x, H = a.H;
    head_norms<NT>(a.part_ml, b, H, ns, a.nsplit_cap, sm.hm, sm.hrl);
    // (few heads: one group, whose sums need not meet)
    const int keys = H <= 8 ? NT : NT == 256 && n <= 64 ? 64 : NT == 256 && n <= 128 ? 128 : min(NT, n <= 256 ? 256 : n <= 512 ? 512 : NT);
    const int groups = NT / keys, per = (H + groups - 1) / groups;
    const int g = __builtin_amdgcn_readfirstlane(tid / keys);     // (a wave lies in one group)
    const int h0 = g * per, h1 = min(H, h0 + per);
    const float* lg = a.logits + a.sys_len + (int64_t)b * H * a.capacity;
    float* row = a.mass_dst + b * a.mass_stride;
    float* part = reinterpret_cast<float*>(sel_keys());  // (the keys are staged later)
    for (int j = tid & (keys - 1); j < n; j += keys) {  // (one round unless n > NT, and then there is one group)
        // (8 loads in flight and not 12: 7B batch 1 57.9 us a step instead of 58.7; up to 4 heads do not take the work of 8)
        const float acc = h1 - h0 <= 4 ? prob_sum<4>(lg + j, a.capacity, sm.hm, sm.hrl, h0, h1)
                                       : prob_sum<8>(lg + j, a.capacity, sm.hm, sm.hrl, h0, h1);
        if (groups == 1) row[j] = acc * (1.0f / (float)H);
        else part[tid] = acc;
    }
    __syncthreads();                                    // the ranking may read these scores, or reuse the keys' place
    if (groups > 1) {
        if (tid < n && tid < keys) {
            float acc = part[tid];
            for (int i = 1; i < groups; ++i) acc += part[i * keys + tid];
            row[tid] = acc * (1.0f / (float)H);
        }
        __syncthreads();
    }
}

// What an eviction of sequence b starts from: visual rows, rows that exist (the appended one included), visual rows to keep.
struct EvictCounts {
    int n, len, k;
    bool evicts;        // something to evict, lengths consistent
};
__device__ __forceinline__ EvictCounts evict_counts(const EvictArgs& a, int b) {
    EvictCounts c;
    c.n = max(0, min(a.vis_len[b], a.max_vis));
    c.len = max(0, min(a.kv_len[b] + (a.appended ? 1 : 0), a.max_kv + (a.appended ? 1 : 0)));
    c.k = a.keep_count < 0 ? c.n : min(a.keep_count, c.n);
    c.evicts = c.k < c.n && a.sys_len + c.n <= c.len;
    return c;
}

// The moves of an eviction: `inner` inside the visual segment, then `tail` rows that close up behind it.
struct EvictMoves {
    int inner, tail;
};

// Ranks the visual rows of sequence b by score_col, compacts the columns to the kept rows and lists the row moves: in LDS
// (in_lds, at most kPlanMaxInline) or, for other workgroups, in global memory.  HOLE_FILL: a row move fills the i-th hole
// among the first k rows with the i-th survivor behind them (sources >= k, destinations < k: disjoint), and the vacated end
// [k, n) is refilled from the END of the cache when at least n - k rows follow the segment, else all rows that follow move down:
// either way sources and destinations are disjoint (r >= g -> src >= len - g >= sys + n; r < g -> dst < sys + k + r < sys + n).
// The global list holds both kinds, the LDS list the inner ones.
template <int NT>
__device__ __forceinline__ EvictMoves evict_rank(const EvictArgs& a, int b, const EvictCounts& c, SelectShared& sm, const bool in_lds,
                                                 int (*lds_list)[2]) {
    const int tid = threadIdx.x, n = c.n, k = c.k;
    uint32_t* keys = sel_keys();
    float* scores = a.score_col + b * a.col_stride;
    int32_t* ids = a.id_col + b * a.col_stride;
    int32_t* mv = a.moves + (int64_t)b * a.max_moves * 2;
    TopSet top{0, 0, true};
    auto key_at = [&](int i) { return keys[i]; };
    auto idkey_at = [&](int i) { return ~(uint32_t)ids[i]; };
    if (k > 0) {
        for (int i = tid; i < n; i += NT) keys[i] = score_key(scores[i]);
        top = top_set<NT>(key_at, idkey_at, n, k, sm);
    }
    auto kept_at = [&](int p) -> bool { return p < n && k > 0 && top.keeps(key_at, idkey_at, p); };
    const int n_pad = (n + NT - 1) / NT * NT;
    const int g = n - k;                                // rows evicted
    // rows behind the visual segment that have to close up; none when the tail keeps its place
    const int r = a.tail_start ? 0 : c.len - (a.sys_len + n);
    int parity = 0, r1, r2, t1, t2;
    if (a.mode == ST3_HOLE_FILL) {
        int base_h = 0, base_f = 0;
        for (int p0 = 0; p0 < n_pad; p0 += NT, parity ^= 1) {
            const int p = p0 + tid;
            const bool kept = kept_at(p);
            const bool hole = p < k && !kept;
            const bool fill = p >= k && kept;
            plan_ranks<NT>(hole, fill, parity, sm, r1, r2, t1, t2);
            if (in_lds) {                  // (ids that repeat could keep more rows than the list holds)
                if (hole && base_h + r1 < kPlanMaxInline) lds_list[base_h + r1][0] = a.sys_len + p;
                if (fill && base_f + r2 < kPlanMaxInline) lds_list[base_f + r2][1] = a.sys_len + p;
            } else {
                if (hole) mv[2 * (base_h + r1)] = a.sys_len + p;
                if (fill) mv[2 * (base_f + r2) + 1] = a.sys_len + p;
            }
            base_h += t1; base_f += t2;
        }
        const int m = min(min(base_h, base_f), in_lds ? kPlanMaxInline : n);  // all equal when the ids are distinct
        __syncthreads();                                // move list visible to the whole block
        for (int i = tid; i < m; i += NT) {
            const int dst = (in_lds ? lds_list[i][0] : mv[2 * i]) - a.sys_len;
            const int src = (in_lds ? lds_list[i][1] : mv[2 * i + 1]) - a.sys_len;
            scores[dst] = scores[src];
            ids[dst] = ids[src];
        }
        const int cnt = min(g, r);
        if (!in_lds) {
            const int src0 = (r >= g) ? c.len - g : a.sys_len + n;
            for (int j = tid; j < cnt; j += NT) {
                mv[2 * (m + j)] = a.sys_len + k + j;
                mv[2 * (m + j) + 1] = src0 + j;
            }
        }
        return EvictMoves{m, cnt};
    }
    // first hole = number of leading kept positions
    if (tid == 0) sm.red = n;
    __syncthreads();
    for (int p = tid; p < n; p += NT)
        if (!kept_at(p)) { atomicMin(&sm.red, p); break; }
    __syncthreads();
    const int fh = sm.red;
    int base = 0;
    for (int p0 = 0; p0 < n_pad; p0 += NT, parity ^= 1) {
        const int p = p0 + tid;
        const bool kept = kept_at(p);
        float sv = 0.f; int32_t iv = 0;
        if (kept) { sv = scores[p]; iv = ids[p]; }
        plan_ranks<NT>(kept, false, parity, sm, r1, r2, t1, t2);    // contains a barrier: loads precede stores
        const int rank = base + r1;
        if (kept && p > fh) {
            scores[rank] = sv; ids[rank] = iv;
            mv[2 * (rank - fh)] = a.sys_len + rank;
            mv[2 * (rank - fh) + 1] = a.sys_len + p;
        }
        base += t1;
    }
    const int m = k - fh;
    for (int j = tid; j < r; j += NT) {
        mv[2 * (m + j)] = a.sys_len + k + j;
        mv[2 * (m + j) + 1] = a.sys_len + n + j;
    }
    return EvictMoves{m, r};
}

// The lengths behind an eviction (or behind a step that evicts nothing); one thread.
__device__ __forceinline__ void evict_publish(const EvictArgs& a, int b, const EvictCounts& c) {
    if (c.evicts) a.vis_len[b] = c.k;
    a.kv_len[b] = c.evicts && !a.tail_start ? c.len - (c.n - c.k) : c.len;
}

// The whole per-sequence plan, run by one workgroup of NT threads for sequence b:
//   1. finish the visual mass the attention kernel left pending (unless workgroups of their own do, mass_block),
//   2. rank the visual rows by score_col and evict down to keep_count (columns, and - when
//      inline_apply - the K/V rows themselves),
//   3. publish the new lengths (including the row the attention kernel appended).
template <int NT>
__device__ __forceinline__ void evict_plan_body(const EvictArgs& a, int b, PlanShared& sm) {
    const int tid = threadIdx.x;
    const EvictCounts c = evict_counts(a, b);
    int moves_left = 0;
    if (a.pending != nullptr && a.mass_dst != nullptr && !a.mass_apart) {
        // the lengths are those the attention call saw
        const int4 d = *reinterpret_cast<const int4*>(a.pending + b * 4);
        if (d.x & 1) {
            const int chunk = max(d.z, 32);
            const int seen = seq_layout(a.sys_len, c.n, a.max_vis, c.len, a.tail_start, b).vlen;    // rows the attend launch saw
            const int ns = seen > 0 ? min((seen + chunk - 1) / chunk, min(d.y, a.nsplit_cap)) : 0;
            if (ns > 0) plan_mass<NT>(a, b, c.n, ns, sm);
        }
    }
    if (c.evicts) {
        const bool inl = a.mode == ST3_HOLE_FILL && a.inline_apply && c.n - c.k <= kPlanMaxInline;
        const EvictMoves m = evict_rank<NT>(a, b, c, sm, inl, sm.mv);
        if (inl) {
            const int g = c.n - c.k, r = c.len - (a.sys_len + c.n);
            const int src0 = (r >= g) ? c.len - g : a.sys_len + c.n;
            copy_rows<NT>(a, b, 0, 1, true, m.inner, [&](int i) { return make_int2(sm.mv[i][0], sm.mv[i][1]); });
            if (m.tail > 0) {
                __syncthreads();                        // those reads are done before [k, n) is overwritten
                copy_rows<NT>(a, b, 0, 1, true, m.tail, [&](int i) { return make_int2(a.sys_len + c.k + i, src0 + i); });
            }
        } else {
            moves_left = m.inner + m.tail;
        }
    }
    if (tid == 0) {
        a.move_cnt[b] = moves_left;
        evict_publish(a, b, c);
    }
}

// ---------------------------------------------------------------------------------------------
// The same plan in independent parts, for columns that do not take this step's mass (EvictArgs::mass_apart): the ranking needs
// nothing of the step's attention and the mass nothing of the ranking.  The whole-step call ranks in spare workgroups of its
// attention launch (evict_rank_early), whose chain of a dozen dependent steps is then hidden behind the reads of K and V, and
// what is left for the launch behind it - masses, row moves, lengths, merges - are short chains in many small workgroups.  The
// parts do not read the lengths that one of them advances: rows attended and visual rows come from the attention's descriptor,
// the number of moves from the ranking.  us a launch of plans, whole plan in one workgroup -> in parts: two layers of 64 rows in
// float32 8.5 -> 5.2, 7B batch 1 12.5 -> 8.9, batch 4 17.9 -> 13.2, 13B batch 8 with fast annealing 32.5 -> 30 (its row moves),
// batch 32 37 -> 29, high resolution batch 8 27.6 -> 20.
// ---------------------------------------------------------------------------------------------

// How many moves the ranking has left to the rows' workgroups: inner | tail << kMoveTailShift (at most 8192 rows are ranked).
constexpr int kMoveTailShift = 16;

// Ranking, columns and the move list of sequence b, beside the attention.  (Moves of a launch of their own: counted in one.)
template <int NT>
__device__ __forceinline__ void evict_rank_early(const EvictArgs& a, int b, SelectShared& sm) {
    const EvictCounts c = evict_counts(a, b);
    EvictMoves m{0, 0};
    if (c.evicts) m = evict_rank<NT>(a, b, c, sm, false, nullptr);
    if (threadIdx.x == 0) a.move_cnt[b] = a.inline_apply ? m.inner | (m.tail << kMoveTailShift) : m.inner + m.tail;
}

// Applies a part of the moves that evict_rank_early has listed.  Moves inside the segment are independent of each other; what closes
// up behind it overwrites their sources, so then a strip's moves stay with one workgroup.
template <int NT>
__device__ __forceinline__ void move_rows_block(const EvictArgs& a, int b, int part, int parts) {
    const int packed = a.move_cnt[b], inner = packed & ((1 << kMoveTailShift) - 1), tail = packed >> kMoveTailShift;
    const int32_t* mv = a.moves + (int64_t)b * a.max_moves * 2;
    auto apply = [&](int count) {
        copy_rows<NT>(a, b, part, parts, tail > 0, count, [&](int i) { return reinterpret_cast<const int2*>(mv)[i]; });
    };
    apply(inner);
    if (tail > 0) {                                     // (uniform)
        __syncthreads();                                // those reads are done before the segment's end is overwritten
        mv += 2 * inner;
        apply(tail);
    }
}

// kMassKeys mass entries of sequence b from key j0 on, by a workgroup of NT threads: a wave takes a share of the heads, a lane four
// keys of a row (one 16-byte load), and the shares are added in order.
constexpr int kMassKeys = 4 * kWave;
template <int NT>
struct MassShared {
    float hm[1024], hrl[1024];
    f32x4_t part[NT / kWave][kWave];
};
template <int NT>
__device__ __forceinline__ void mass_block(const EvictArgs& a, int b, int j0, MassShared<NT>& sm) {
    constexpr int kWaves = NT / kWave, kUR = 8;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x % kWave, j = j0 + 4 * lane;
    const int per = (a.H + kWaves - 1) / kWaves, h0 = min(a.H, wave * per), h1 = min(a.H, h0 + per);
    // (a load may reach three floats past the visual rows: more of the row, the next one or what lies behind the logits)
    const float* lg = a.logits + a.sys_len + (int64_t)b * a.H * a.capacity + j;
    f32x4_t v[kUR], acc = {0.f, 0.f, 0.f, 0.f};
    auto load = [&](int h) {
#pragma unroll
        for (int u = 0; u < kUR; ++u)
            if (j < a.max_vis && h + u < h1) v[u] = *reinterpret_cast<const f32x4_a4_t*>(lg + (int64_t)(h + u) * a.capacity);
    };
    load(h0);                                           // (on their way while the descriptor and the norms arrive)
    const int4 d = *reinterpret_cast<const int4*>(a.pending + b * 4);
    const int chunk = max(d.z, 32), seen = (d.x & 1) ? d.x >> 1 : 0;
    const int ns = seen > 0 ? min((seen + chunk - 1) / chunk, min(d.y, a.nsplit_cap)) : 0;
    const int n = ns > 0 ? min(a.own_pending[b * 4 + 3] >> 1, a.max_vis) : 0;      // (0: no mass is pending)
    if (j0 >= n) return;                                // (uniform; always so without chunks)
    head_norms<NT>(a.part_ml, b, a.H, ns, a.nsplit_cap, sm.hm, sm.hrl);
    for (int h = h0; h < h1; h += kUR) {
        if (h > h0) load(h);
#pragma unroll
        for (int u = 0; u < kUR; ++u) {
            if (h + u >= h1) break;
            const float m = sm.hm[h + u], rl = sm.hrl[h + u];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += exp2_fast(v[u][i] - m) * rl;
        }
    }
    sm.part[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && j < n) {
#pragma unroll
        for (int w = 1; w < kWaves; ++w) acc += sm.part[w][lane];
        float* out = a.mass_dst + b * a.mass_stride + j;
        for (int i = 0; i < min(4, n - j); ++i) out[i] = acc[i] * (1.0f / (float)a.H);
    }
}

// The same where the attention has left sums of probabilities over its groups of heads (kStepSums): `groups` rows, `step` heads apart.
template <int NT>
__device__ __forceinline__ void mass_sums_block(const EvictArgs& a, int b, int j0, int groups, int step, MassShared<NT>& sm) {
    constexpr int kWaves = NT / kWave, kUR = 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x % kWave, j = j0 + 4 * lane;
    const int per = (groups + kWaves - 1) / kWaves, g0 = min(groups, wave * per), g1 = min(groups, g0 + per);
    const float* at = a.logits + a.sys_len + (int64_t)b * a.H * a.capacity + j;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1                                        // (unrolled, the launch takes 241 registers instead of 125, and its rows move a quarter slower)
    for (int g = g0; g < g1; g += kUR) {
        f32x4_t v[kUR];
#pragma unroll
        for (int u = 0; u < kUR; ++u)
            if (j < a.max_vis && g + u < g1) v[u] = *reinterpret_cast<const f32x4_a4_t*>(at + (int64_t)(g + u) * step * a.capacity);
#pragma unroll
        for (int u = 0; u < kUR; ++u)
            if (g + u < g1) acc += v[u];
    }
    const int n = (a.pending[b * 4] & 1) ? min(a.own_pending[b * 4 + 3] >> 1, a.max_vis) : 0;      // (0: no mass is pending)
    if (j0 >= n) return;                                // (uniform)
    sm.part[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && j < n) {
#pragma unroll
        for (int w = 1; w < kWaves; ++w) acc += sm.part[w][lane];
        float* out = a.mass_dst + b * a.mass_stride + j;
        for (int i = 0; i < min(4, n - j); ++i) out[i] = acc[i] * (1.0f / (float)a.H);
    }
}

// ---- host side (defined in st3_select.hip) --------------------------------------------------
// Fills the plan arguments for one layer; needs_apply tells whether evict_apply_kernel must run
// after the plan (evictions too large for the plan workgroup to move, or STABLE mode).
// kv->k may be null (a layer that caches V only).  mass_workspace (null: `workspace`) is the
// workspace whose attend launch left the logits the mass is finished from - a lazy layer's
// source - and mass_capacity that cache's capacity.  batched: the plan will share its launch with
// the plans of other layers (decides how many row moves the plan workgroup does itself).
st3_status build_evict_args(const st3_attn_shape* shape, const st3_kv_layer* kv, const st3_segments* seg,
                            float* score_col, int32_t* id_col, int64_t col_stride, int32_t keep_count, int32_t mode,
                            void* workspace, size_t workspace_bytes, int appended, float* mass_dst,
                            int64_t mass_stride, EvictArgs& ea, bool& needs_apply, bool batched,
                            const void* mass_workspace = nullptr, int32_t mass_capacity = 0);
void launch_evict_plan(const EvictArgs& ea, int B, hipStream_t st);
constexpr int kPlanBatch = 16;     // plans that travel by value: 216 bytes each (the argument block would hold 18)
// Plans of n layers (device work of one decode step) with one launch per kPlanBatch layers.
void launch_evict_plan_batch(const EvictArgs* plans, int n, int B, hipStream_t st);
// The plans of the n layers of a whole step whose attention has been enqueued, as many per launch as a table holds.
struct PlanNeeds {
    int most_vis;       // the largest bound of any layer's visual rows
    bool merge;         // some strip was cut
    bool apart;         // every layer's rows have been ranked beside the attention (kStepApart)
    int64_t moves;      // 16-byte pieces of rows that the launch moves for a sequence of a layer, at most
};
void launch_evict_plan_table(const StepCommon& c, const StepLayer* entry, int n, const PlanNeeds& needs, hipStream_t st);
void launch_evict_apply(const EvictArgs& ea, int B, hipStream_t st);

}  // namespace st3
