// The layers of a whole decode step as they travel to its launches: by value, in the kernel arguments.
//
// A launch's argument block holds about 4 KB, and every launch of a step costs a ramp, a tail and a gap (about 9 us whatever it
// reads), so the entries are packed: pointers as 48 bits, strides in units of 16 bytes, counts in 16 bits where they fit.  A layer
// of 184 bytes takes 112 (124 with the scales of an E4M3 cache) in the attention's table and 96 (112 where the rows are still to
// be ranked) in the table of the launch behind it: 35, 32, 41 and 35 layers a launch.  us a step, 21 layers a launch and entries
// left in the workspaces for the launch behind it -> so: 7B batch 1 55 -> 45, 13B batch 8 with lazy layers 504 -> 496, high resolution batch
// 8 E4M3 629 -> 624; a generation of 16 steps, 7B batch 4, 4824 -> 4758.
//
// A table is wide where some layer needs it (token-major caches, whose rows can lie megabytes apart): three words more for each entry,
// from the table's end, have the upper halves of what the entry holds in 16 or 32 bits.  (Kernels of their own read such tables: a few
// scalar loads and a flag at the start of every workgroup cost the other steps 0.1 to 0.4 us.)  Rows of 2 MB, us a step, layer by
// layer -> wide: 32 layers of the 7B shape, batch 4 285 -> 93, 40 layers of 40 heads, batch 2 341 -> 85.
#pragma once

#include <stdint.h>

#ifndef __HIPCC__
#define __host__
#define __device__
#endif

namespace st3 {

struct StepCommon {
    int32_t B, H, D;
    int16_t mode;               // st3_compact_mode
    int16_t elem_bytes;         // of q, the new rows, the outputs and plain caches: 2 (bf16) or 4 (float32)
    float scale_l2;
    int32_t layers;             // entries of the table
    int8_t wide;                // 1: the table's entries are wide
    int8_t leave;               // 1: the attention leaves its entries in the layers' workspaces (kLeftWords)
    int16_t chunks;             // most chunks of any layer: the attention's grid is (H, chunks, rank_z + B * layers), without groups
    int32_t rank_z;             // the grid's first z, or with groups, in a grid that is a line, its first workgroups: they rank rows, one for each
                                // (layer, sequence); 0: no row is ranked
    int8_t groups[4];           // layers of an attention's table whose workgroups take 8, 4, 2 heads (in this order) one after the other, and 1: the
                                // others; groups[3]: 1 where the grid is for that (no strip is cut then), else 0
};

struct StepLayer {
    const void* q;              // lazy layer: the source layer's workspace
    void* k;                    // lazy layer: null unless it caches keys all the same (they move with an eviction)
    void* v;
    const void* k_new;          // lazy layer: unused
    const void* v_new;
    void* out;
    int32_t* kv_len;
    int32_t* vis_len;
    const int32_t* tail_start;
    float* score_col;
    int32_t* id_col;
    float* mass;                // null: no mass
    char* ws;
    const float* k_scale;
    const float* v_scale;
    int64_t stride_b, stride_h; // cache elements
    int32_t stride_t, col_stride, mass_stride;
    int32_t sys_len, max_vis, max_kv;       // bounds BEFORE the step (max_kv does not count the appended row)
    int32_t keep_count;         // < 0: no eviction
    int32_t chunk;              // rows per chunk of a strip, a multiple of 32
    int32_t hint_base, hint_gap;            // layout_hint; lazy layer: hint_base is the source cache's capacity
    int32_t capacity;
    uint8_t nsplit, nsplit_cap; // chunks per strip of this launch / that the workspace has room for (at most 64)
    uint8_t src_nsplit_cap;     // lazy layer: of the source's workspace; kStepSums: heads of a sum
    uint8_t flags;
};
constexpr uint8_t kStepInlineApply = 1, kStepKeepAll = 2, kStepLazy = 4, kStepWantMass = 8, kStepE4M3 = 16;
constexpr uint8_t kStepApart = 32;      // the next eviction does not rank by this step's mass
constexpr uint8_t kStepSums = 64;       // the attention leaves sums of probabilities over its groups of heads, in the logits' place, instead of logits

// Words of an entry: pointers (low words, then high halves in pairs), then ten or eleven words of numbers.
constexpr int kAttendPtrs = 12, kAttendPtrsE4M3 = 14, kFinishPtrs = 9, kPlanPtrs = 11;
constexpr int ptr_words(int n) { return n + (n + 1) / 2; }
constexpr int kAttendWords = ptr_words(kAttendPtrs) + 10, kAttendWordsE4M3 = ptr_words(kAttendPtrsE4M3) + 10;
constexpr int kFinishWords = ptr_words(kFinishPtrs) + 10, kPlanWords = ptr_words(kPlanPtrs) + 11;
constexpr int kWideWords = 3;
constexpr int kStepTableWords = 992;
// Where the rows are still to be ranked and that table does not hold all layers (36 of a 40-layer model do not fit), a second launch
// would rank the rest after the first has finished.  Then the attention leaves its own entries behind the layers' decode
// workspaces, where prefill scratch lies at other times, and the table holds where they are, the mass's place and stride.
// Columns that take the mass, us a step, two launches -> one: 40 layers of 32 heads, 300 rows, batch 1 72.9 -> 61.1,
// batch 8 317 -> 316.
constexpr int kLeftPtrs = 2, kLeftWords = ptr_words(kLeftPtrs) + 1, kLeftBytes = 256;
static_assert((kAttendWordsE4M3 + kWideWords) * 4 <= kLeftBytes, "what is left of an entry");
inline int entries_per_table(int words, int wide) { return kStepTableWords / (words + (wide ? kWideWords : 0)); }
template <typename W>
__host__ __device__ inline W* high_words(W* table, int i) { return table + kStepTableWords - kWideWords * (i + 1); }

struct StepTable {
    StepCommon c;
    uint32_t w[kStepTableWords];
};
static_assert(sizeof(StepTable) <= 4016, "the table travels by value, two words beside it in some launches");

// Slices (z) of the attention's grid that ranking takes: a workgroup for each (layer, sequence) of the launch.
inline int rank_rows_z(int B, int H, int chunks, int layers) {
    const int64_t slice = (int64_t)H * chunks;
    return (int)(((int64_t)B * layers + slice - 1) / slice);
}
// Layers that a launch may rank for: rank_z + B * layers is at most 65535 however few chunks there are.
inline int max_layers_ranked(int B, int H) { return (int)((int64_t)65534 * H / (H + 1) / B); }

inline void put_ptr(uint32_t* w, int n, int i, const void* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    w[i] = (uint32_t)v;
    uint32_t& hi = w[n + i / 2];
    hi = i % 2 ? (hi & 0xffffu) | ((uint32_t)(v >> 32) << 16) : (hi & 0xffff0000u) | (uint32_t)((v >> 32) & 0xffffu);
}
template <typename P>
__host__ __device__ inline void get_ptr(const uint32_t* w, int n, int i, P& p) {
    const uint64_t hi = (w[n + i / 2] >> (16 * (i % 2))) & 0xffffu;
    p = reinterpret_cast<P>(hi << 32 | w[i]);
}

// Whether an entry, wide or not, of a layer whose cache elements are eb bytes wide holds these values.
inline bool step_layer_fits(const StepLayer& e, int eb, bool wide = false) {
    const void* ptrs[] = {e.q, e.k, e.v, e.k_new, e.v_new, e.out, e.kv_len, e.vis_len, e.tail_start, e.score_col, e.id_col, e.mass, e.ws,
                          e.k_scale, e.v_scale};
    for (const void* p : ptrs)
        if (reinterpret_cast<uint64_t>(p) >> 48) return false;
    const bool lazy = (e.flags & kStepLazy) != 0, hinted = !lazy && e.hint_base != 0x7fffffff;
    const int64_t nv = (int64_t)e.hint_base - e.sys_len, unit = 16 / eb;
    const int more = wide ? 16 : 0;
    for (int64_t s : {e.stride_b, e.stride_h, (int64_t)e.stride_t})
        if (s < 0 || s % unit) return false;
    return (e.stride_b / unit) >> (32 + more) == 0 && (e.stride_h / unit) >> (32 + more) == 0 && (e.stride_t / unit) >> (16 + more) == 0 &&
           e.sys_len >= 0 && (int64_t)e.sys_len >> (16 + more) == 0 && e.max_vis >= 0 && e.max_vis >> 16 == 0 && e.keep_count < 0xffff &&
           e.chunk % 32 == 0 && (int64_t)(e.chunk / 32) >> (16 + more) == 0 && (!hinted || (nv >= 0 && nv < 0xffff));
}

inline uint32_t pair16(int lo, int hi) { return ((uint32_t)lo & 0xffffu) | (uint32_t)hi << 16; }
// The ten words that both tables have, but for two of them (a, b); high: where a wide entry's upper halves go (null: not wide).
inline void pack_numbers(uint32_t* w, const StepLayer& e, int eb, uint32_t a, uint32_t b, uint32_t* high) {
    const int64_t unit = 16 / eb, sb = e.stride_b / unit, sh = e.stride_h / unit, st = e.stride_t / unit;
    if (high != nullptr) {
        high[0] = pair16((int)(st >> 16), e.sys_len >> 16);
        high[1] = pair16((int)(sb >> 32), (int)(sh >> 32));
        high[2] = (uint32_t)(e.chunk / 32) >> 16;
    }
    w[0] = (uint32_t)sb; w[1] = (uint32_t)sh;
    w[2] = pair16((int)st, e.sys_len);
    w[3] = pair16(e.max_vis, e.keep_count < 0 ? 0 : e.keep_count + 1);
    w[4] = (uint32_t)e.max_kv; w[5] = (uint32_t)e.capacity;
    w[6] = (uint32_t)e.nsplit | (uint32_t)e.nsplit_cap << 8 | (uint32_t)e.src_nsplit_cap << 16 | (uint32_t)e.flags << 24;
    w[7] = pair16(e.chunk / 32, (e.flags & kStepLazy) || e.hint_base == 0x7fffffff ? 0xffff : e.hint_base - e.sys_len);
    w[8] = a; w[9] = b;
}
__host__ __device__ inline void unpack_numbers(const uint32_t* w, StepLayer& e, int eb, const uint32_t* high, bool wide) {
    const int64_t unit = 16 / eb;
    const uint32_t mask = wide ? 0xffffffffu : 0u, h0 = high[0] & mask, h1 = high[1] & mask, h2 = high[2] & mask;
    e.stride_b = (int64_t)((uint64_t)(h1 & 0xffffu) << 32 | w[0]) * unit; e.stride_h = (int64_t)((uint64_t)(h1 >> 16) << 32 | w[1]) * unit;
    e.stride_t = (int32_t)((h0 << 16 | (w[2] & 0xffffu)) * (uint32_t)unit); e.sys_len = (int32_t)((h0 & 0xffff0000u) | w[2] >> 16);
    e.max_vis = (int32_t)(w[3] & 0xffffu); e.keep_count = (int32_t)(w[3] >> 16) - 1;
    e.max_kv = (int32_t)w[4]; e.capacity = (int32_t)w[5];
    e.nsplit = (uint8_t)w[6]; e.nsplit_cap = (uint8_t)(w[6] >> 8); e.src_nsplit_cap = (uint8_t)(w[6] >> 16); e.flags = (uint8_t)(w[6] >> 24);
    e.chunk = (int32_t)((h2 << 16 | (w[7] & 0xffffu)) * 32u);
}

// The attention's entry: everything but the mass's place.
inline void pack_attend(uint32_t* w, const StepLayer& e, bool coded, int eb, uint32_t* high) {
    const int n = coded ? kAttendPtrsE4M3 : kAttendPtrs;
    const void* ptrs[kAttendPtrsE4M3] = {e.q, e.k, e.v, e.k_new, e.v_new, e.out, e.kv_len, e.vis_len, e.tail_start, e.ws, e.score_col,
                                         e.id_col, e.k_scale, e.v_scale};
    for (int i = 0; i < n; ++i) put_ptr(w, n, i, ptrs[i]);
    pack_numbers(w + ptr_words(n), e, eb, (uint32_t)e.col_stride, (uint32_t)((e.flags & kStepLazy) ? e.hint_base : e.hint_gap), high);
}
template <bool CODED>
__host__ __device__ inline StepLayer unpack_attend(const uint32_t* w, int eb, const uint32_t* high, bool wide) {
    constexpr int n = CODED ? kAttendPtrsE4M3 : kAttendPtrs;
    StepLayer e{};
    get_ptr(w, n, 0, e.q); get_ptr(w, n, 1, e.k); get_ptr(w, n, 2, e.v); get_ptr(w, n, 3, e.k_new); get_ptr(w, n, 4, e.v_new);
    get_ptr(w, n, 5, e.out); get_ptr(w, n, 6, e.kv_len); get_ptr(w, n, 7, e.vis_len); get_ptr(w, n, 8, e.tail_start);
    get_ptr(w, n, 9, e.ws); get_ptr(w, n, 10, e.score_col); get_ptr(w, n, 11, e.id_col);
    if (CODED) { get_ptr(w, n, 12, e.k_scale); get_ptr(w, n, 13, e.v_scale); }
    const uint32_t* num = w + ptr_words(n);
    unpack_numbers(num, e, eb, high, wide);
    e.col_stride = (int32_t)num[8];
    const int nv = (int)(num[7] >> 16);
    if (e.flags & kStepLazy) e.hint_base = (int32_t)num[9];
    else { e.hint_base = nv == 0xffff ? 0x7fffffff : e.sys_len + nv; e.hint_gap = (int32_t)num[9]; }
    return e;
}

// The entry of the launch behind the attention; ranking: with the columns.  (q is the source's workspace of a lazy layer, null else.)
inline void pack_plan(uint32_t* w, const StepLayer& e, bool ranking, int eb, uint32_t* high) {
    const int n = ranking ? kPlanPtrs : kFinishPtrs;
    const bool lazy = (e.flags & kStepLazy) != 0;
    const void* ptrs[kPlanPtrs] = {lazy ? e.q : nullptr, e.k, e.v, e.out, e.kv_len, e.vis_len, e.tail_start, e.ws, e.mass, e.score_col, e.id_col};
    for (int i = 0; i < n; ++i) put_ptr(w, n, i, ptrs[i]);
    uint32_t* num = w + ptr_words(n);
    pack_numbers(num, e, eb, (uint32_t)e.mass_stride, lazy ? (uint32_t)e.hint_base : 0u, high);
    if (ranking) num[10] = (uint32_t)e.col_stride;
}
template <bool RANKING>
__host__ __device__ inline StepLayer unpack_plan(const uint32_t* w, int plain_eb, const uint32_t* high, bool wide) {
    constexpr int n = RANKING ? kPlanPtrs : kFinishPtrs;
    StepLayer e{};
    get_ptr(w, n, 0, e.q); get_ptr(w, n, 1, e.k); get_ptr(w, n, 2, e.v); get_ptr(w, n, 3, e.out); get_ptr(w, n, 4, e.kv_len);
    get_ptr(w, n, 5, e.vis_len); get_ptr(w, n, 6, e.tail_start); get_ptr(w, n, 7, e.ws); get_ptr(w, n, 8, e.mass);
    const uint32_t* num = w + ptr_words(n);
    const bool coded = (num[6] >> 24 & kStepE4M3) != 0;
    unpack_numbers(num, e, coded ? 1 : plain_eb, high, wide);
    e.mass_stride = (int32_t)num[8]; e.hint_base = (int32_t)num[9];
    if (RANKING) { get_ptr(w, n, 9, e.score_col); get_ptr(w, n, 10, e.id_col); e.col_stride = (int32_t)num[10]; }
    return e;
}

// Where the attention has left a layer's entry (at `left`, its upper halves behind it), and what that lacks; the layer's cache format goes along, since the entry's
// layout depends on it.
inline void pack_left(uint32_t* w, const StepLayer& e, const void* left) {
    put_ptr(w, kLeftPtrs, 0, left); put_ptr(w, kLeftPtrs, 1, e.mass);
    w[ptr_words(kLeftPtrs)] = (uint32_t)e.mass_stride | ((e.flags & kStepE4M3) ? 0x80000000u : 0u);
}
__host__ __device__ inline StepLayer unpack_left(const uint32_t* w, int plain_eb, bool wide) {
    const uint32_t* left;
    get_ptr(w, kLeftPtrs, 0, left);
    const uint32_t last = w[ptr_words(kLeftPtrs)];
    StepLayer e = last >> 31 ? unpack_attend<true>(left, 1, left + kAttendWordsE4M3, wide) : unpack_attend<false>(left, plain_eb, left + kAttendWords, wide);
    get_ptr(w, kLeftPtrs, 1, e.mass);
    e.mass_stride = (int32_t)(last & 0x7fffffffu);
    return e;
}

}  // namespace st3
