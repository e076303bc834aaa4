// Decode attention over a ragged KV cache (Eq. 2 with a single query row that follows every
// cached key) with the visual mass of Sec. 3.2, plus KV append.
//
// decode_attend_kernel streams K and V exactly once.  Each (b,h) strip is cut into `nsplit`
// chunks (one workgroup each); nsplit is 1 as soon as B*H alone fills the chip and the strip is no
// longer than the logit staging area, and then the workgroup writes the finished output row itself.  With nsplit > 1 the workgroups leave
// un-normalised partials that decode_finish_kernel merges in chunk order.  For the visual mass the
// attend kernel saves the scaled logits of the visual keys (collected in LDS, written out as whole
// lines at the end of the workgroup) and every chunk's (max, sum); turning
// them into probabilities and adding them over heads - in a fixed order, so the sum is the same on
// every run - is done by prob_sum() in decode_finish_kernel for the stand-alone call, and behind the
// attention of a fused step: by workgroups of their own beside the plans (mass_block), or by the plan
// itself where it ranks by that mass, or is the only one (plan_mass).
// The whole-step call runs the same workgroups for many layers in one launch
// (decode_attend_layers_kernel, decode_inherit_layers_kernel), and ranks rows in the launch's first workgroups.
// The token being appended is read from k_new/v_new as cache row kv_len[b] by the workgroup that
// owns the end of the strip, which also stores it into the cache; kv_len itself is bumped by the
// eviction plan that follows the attention.
// (Letting that plan ride in spare workgroups of the next layer's attend launch was measured and
// dropped: a plan workgroup is a chain of dependent memory round trips that outlasts the attention of one
// layer and halves the streaming rate of the compute unit it sits on.  What rides in a whole step's attention
// is the ranking alone, beside the strips of all layers, and where those take longer: rank_beside().)
//
// No kernel here communicates between workgroups of one launch: device-scope fences cost a
// write-back and invalidate of the XCD-private L2 on this part and were measured to be ruinous.
#include <hip/hip_ext.h>

#include <atomic>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <utility>
#include <vector>

#include "st3_common.h"
#include "st3_attend.h"
#include "st3_evict.h"

#ifndef ST3_DECODE_THREADS
#define ST3_DECODE_THREADS 256      // threads per workgroup of the attend kernel
#endif
#ifndef ST3_DECODE_MIN_BLOCKS
#define ST3_DECODE_MIN_BLOCKS 2     // workgroups per CU the register budget must allow
#endif

namespace st3 {

bool profile_take(hipEvent_t* start, hipEvent_t* stop, int layers);     // st3_api.hip

namespace {

constexpr int kDecodeThreads = ST3_DECODE_THREADS;
constexpr int kDecodeWaves = kDecodeThreads / kWave;

struct DecodeArgs {
    const void* q;
    void* k;
    void* v;
    int64_t stride_b, stride_h, stride_t;
    const int32_t* kv_len;
    const int32_t* vis_len;
    const int32_t* tail_start;  // [B] or null (the tail follows the visual rows directly)
    int32_t B, sys_len, max_vis, max_kv, H, nsplit, nsplit_cap, chunk, capacity;
    int32_t hint_base, hint_gap;    // the host's guess at the layout of a fixed-tail cache (INT_MAX, 0: none)
    int32_t defer;          // 1: the mass of this call is finished by the eviction plan that follows; mark it pending
    int32_t keep_all_logits;  // 1: keep the logit of every key (a lazy layer will ask for them), else visual only
    float scale_l2;
    const float* k_scale;   // [B*H] value of one K code unit (E4M3 caches; null: 1)
    const float* v_scale;   // [B*H] likewise for V
    float* part_o;          // [B,H,nsplit_cap,D]   (nsplit > 1 only)
    float* part_ml;         // [B,H,nsplit_cap,2]
    float* logits;          // [B,H,capacity]; null when no mass is wanted
    int32_t stage_rows;     // floats of LDS in which a workgroup collects the logits it keeps (0 when it keeps none)
    int32_t* pending;       // [B][4]: {mass still to be finished | rows attended << 1, nsplit, chunk, logits of every key present | visual rows << 1}
    const void* k_new;      // [B,H,D] rows of the token being appended (null: none); the cache row
    const void* v_new;      //         kv_len[b] is then taken from here and written to the cache
    void* out;              // [B,H,D]
};

// A store that leaves the line in L2 (NT = false) or goes past the caches.  (A template parameter and not a flag: the
// compiler folds the two arms of a run-time choice into one ordinary store.)
template <bool NT, typename V>
__device__ __forceinline__ void store_hint(V* p, V v) {
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <typename T, bool NT = false>
__device__ __forceinline__ void store_out(void* out, int64_t idx, float o) {
    if (sizeof(T) == 4) store_hint<NT>(reinterpret_cast<float*>(out) + idx, o);
    else store_hint<NT>(reinterpret_cast<uint16_t*>(out) + idx, (uint16_t)f32_to_bf16_bits(o));
}

// This lane's 16-byte slice of a new token's row, in the format of the cache it is going into
// (lane map of RowMap<KT, D>): a plain copy when the cache holds elements of T, the E4M3 quantiser
// otherwise.  What the attention then reads is exactly what later steps will find in the cache.
// load(): each lane for itself.  load_by_wave(): the K and the V row (k_row may be null) of one token by a whole wave, for the
// one wave of an attention workgroup that takes the appended row while the others wait for it at the end: the quantiser costs
// about 45 instructions an element (an exactly rounded division), so every element is quantised by one lane only and the codes
// are exchanged, 4 elements a lane instead of 32.  E4M3 caches, us a step, before -> after: 7B batch 1 49.4 -> 43.5, 7B batch 16
// layer by layer 536 -> 443, 13B batch 8 with lazy layers 300 -> 282, batch 32 1304 -> 1275, high resolution batch 8 637 -> 630.
template <typename T, typename KT, int D>
struct NewRow {
    static __device__ __forceinline__ u32x4_t load(const T* row, int lane, float) {
        using M = RowMap<KT, D>;
        return *reinterpret_cast<const u32x4_t*>(row + (lane % M::LPR) * M::EPL);
    }
    static __device__ __forceinline__ void load_by_wave(const T* k_row, const T* v_row, int lane, float, float, u32x4_t& k, u32x4_t& v) {
        if (k_row != nullptr) k = load(k_row, lane, 1.0f);
        v = load(v_row, lane, 1.0f);
    }
};
template <typename T, int D>
struct NewRow<T, e4m3_t, D> {
    static __device__ __forceinline__ u32x4_t load(const T* row, int lane, float scale) {
        float f[16];
        load_row_slice<T, e4m3_t, D>(row, lane, f);
        u32x4_t r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = four(f + 4 * i, scale);
        return r;
    }
    static __device__ __forceinline__ void load_by_wave(const T* k_row, const T* v_row, int lane, float k_scale, float v_scale,
                                                        u32x4_t& k, u32x4_t& v) {
        static_assert(sizeof(T) == 2 && D / 4 <= 32, "half a wave covers a row, four bf16 elements a lane");
        const bool is_k = lane < 32 && k_row != nullptr;        // lanes 0..31: K, 32..63: V
        const T* src = (is_k ? k_row : v_row) + 4 * (lane % (D / 4));
        const uint2 raw = *reinterpret_cast<const uint2*>(src);
        const float f[4] = {bf16_lo(raw.x), bf16_hi(raw.x), bf16_lo(raw.y), bf16_hi(raw.y)};
        const int word = (int)four(f, is_k ? k_scale : v_scale);
        const int first = 4 * (lane % RowMap<e4m3_t, D>::LPR);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (k_row != nullptr) k[i] = (uint32_t)__shfl(word, first + i);
            v[i] = (uint32_t)__shfl(word, 32 + first + i);
        }
    }

private:
    static __device__ __forceinline__ uint32_t four(const float* f, float scale) {
        return quantize_e4m3(f[0], scale) | (quantize_e4m3(f[1], scale) << 8) | (quantize_e4m3(f[2], scale) << 16) |
               (quantize_e4m3(f[3], scale) << 24);
    }
};

// One workgroup: chunk `split` of strip (b, h).  T: element type of q, k_new, v_new and out; KT: element type of the cache.
// NTS: what the workgroup writes (output row, appended row, logits) goes past the caches.
template <typename T, typename KT, int D, int U, bool NTS>
__device__ __forceinline__ void attend_chunk(const DecodeArgs& a, const int split, const int h, const int b) {
    using M = RowMap<KT, D>;
    constexpr int EPL = M::EPL, LPR = M::LPR, TILE = U * M::RPL;
    const int c0 = split * a.chunk;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int64_t bh = (int64_t)b * a.H + h;
    const T* qrow = reinterpret_cast<const T*>(a.q) + bh * D;
    KT* kbase = reinterpret_cast<KT*>(a.k) + b * a.stride_b + h * a.stride_h;
    KT* vbase = reinterpret_cast<KT*>(a.v) + b * a.stride_b + h * a.stride_h;
    if (a.max_kv > 0 && c0 >= a.max_kv) return;     // (the host launches no such chunk; the early loads below rely on it)
    // The first tile's loads go out before the sequence length has arrived: the host bound keeps
    // them inside the strip (rows the length later rules out are masked when the tile is consumed).
    // Takes one dependent memory round trip off the front of every workgroup.  Where the cache keeps
    // a gap behind its visual segment the rows are placed by the host's guess at it.
    uint4 kr[U], vr[U];
    const RowShift guess{a.hint_base, a.hint_gap};
    issue_tile_within<KT, D, U, true>(kbase, vbase, a.stride_t, c0 + wave * TILE, c0 + a.chunk,
                                     a.max_kv - (a.k_new != nullptr ? 1 : 0), c0, lane, kr, vr, guess);
    float qf[EPL];
    load_row_slice<T, KT, D>(qrow, lane, qf);
    // a code unit of K is worth k_scale: folded into the logit scale; V's goes onto the output
    const float k_unit = a.k_scale ? a.k_scale[bh] : 1.0f, v_unit = a.v_scale ? a.v_scale[bh] : 1.0f;
    const float scale_l2 = a.scale_l2 * k_unit;
    // the row being appended sits at index kv_len[b]; never trust a device length past the host bound
    const int len_phys = min(a.kv_len[b] + (a.k_new != nullptr ? 1 : 0), a.max_kv);
    // `len` and every row index below are in the gap-free numbering (a cache with a fixed tail keeps
    // dead rows between the visual segment and the tail); `sh` maps a row to where it is stored
    const SeqLayout lay = seq_layout(a.sys_len, a.vis_len[b], a.max_vis, len_phys, a.tail_start, b);
    const int len = lay.vlen;
    const RowShift sh = lay.shift();
    if (split == 0 && h == 0 && tid == 0 && a.pending != nullptr) {
        // bit 0: the mass of this launch is still to be finished; above it: the rows this launch attends over
        a.pending[b * 4 + 0] = ((a.logits != nullptr && len > 0 && a.defer) ? 1 : 0) | (max(len, 0) << 1);
        a.pending[b * 4 + 1] = a.nsplit;
        a.pending[b * 4 + 2] = a.chunk;
        a.pending[b * 4 + 3] = ((a.logits != nullptr && len > 0 && a.keep_all_logits) ? 1 : 0) | (lay.nv << 1);
    }
    if (len <= 0) {                                  // empty sequence: out = 0, no mass
        if (split == 0 && tid < D) store_out<T>(a.out, bh * D + tid, 0.f);
        return;
    }
    if (c0 >= len) return;
    const int c1 = min(c0 + a.chunk, len);

    WaveState<EPL> st;

    // Scaled logits kept for later: those of the visual keys become the mass; a layer with lazy
    // followers (QK heredity, Eq. 6) keeps the logit of EVERY key for them.  Keeping all of them
    // always was measured at +5 % on this kernel (4 bytes stored against 512 read per key, but as
    // partial-line writes), so it is done only where it is needed.  Index = cache row either way.
    float* lg = a.logits ? a.logits + bh * a.capacity : nullptr;
    const int vis_lo = a.keep_all_logits ? 0 : a.sys_len;
    const int vis_hi = a.keep_all_logits ? len : a.sys_len + lay.nv;
    if (lg) lg += vis_lo;           // the wave loop indexes by (row - vis_lo)
    // this workgroup owns the appended row (stored at the physical end, which a fixed tail must have reached)
    const bool has_new = a.k_new != nullptr && c1 == len && len_phys - 1 >= lay.base + lay.gap;
    const int c1_cached = has_new ? c1 - 1 : c1;
    // the appended token's row is fetched now and used after the cached rows: off the critical path
    u32x4_t kn_raw = {0, 0, 0, 0}, vn_raw = {0, 0, 0, 0};       // native vectors: the uint4 class would live in scratch
    if (has_new && wave == 0) {
        NewRow<T, KT, D>::load_by_wave(reinterpret_cast<const T*>(a.k_new) + bh * D, reinterpret_cast<const T*>(a.v_new) + bh * D,
                                       lane, k_unit, v_unit, kn_raw, vn_raw);
    }
    // waves take the tiles of the chunk round-robin, so all four stay busy to the end
    // the early tile placed its rows by the host's guess: fetch it again if that put a row this
    // sequence attends to in the wrong place (a sequence that differs from the guess, in a tile that
    // reaches behind its visual segment or the guessed one)
    {
        const int tile_end = min(c0 + wave * TILE + TILE, c1_cached);
        const bool same = lay.gap == guess.gap && (lay.gap == 0 || lay.base == guess.split_row);
        const bool in_front = tile_end <= lay.base && (guess.gap == 0 || tile_end <= guess.split_row);
        if (!same && !in_front)
            issue_tile<KT, D, U, true>(kbase, vbase, a.stride_t, c0 + wave * TILE, c1_cached, c0, lane, kr, vr, sh);
    }
    // rows of the early tile that the length rules out came from beyond the sequence: their V may
    // hold anything (NaN included), and 0 * NaN would poison the accumulator
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (c0 + wave * TILE + u * M::RPL + lane / LPR >= c1_cached) vr[u] = make_uint4(0, 0, 0, 0);
    // The logits this workgroup keeps (rows [lg_lo, lg_hi) of its chunk) are collected in LDS and leave
    // as whole lines after the waves have merged: stored one by one from the loop (16 bytes per wave
    // and tile) they cost 2 us of a 66 us launch at the 13B shape.  The launcher cuts strips so that a
    // chunk's rows fit the staging area (kLogitStageMaxRows) whenever logits are kept.
    extern __shared__ float sm_lg[];
    const int lg_lo = max(c0, vis_lo), lg_hi = min(c1, vis_hi);
    float* lg_stage = lg != nullptr ? sm_lg : nullptr;
    wave_attend_primed<KT, D, U, true>(qf, kbase, vbase, a.stride_t, c0 + wave * TILE, c1_cached, kDecodeWaves * TILE,
                                       c0, scale_l2, lane, st, lg_stage, lg_lo, vis_hi, kr, vr, sh);
    if (has_new && wave == 0) {
        wave_attend_row<KT, D>(qf, make_uint4(kn_raw.x, kn_raw.y, kn_raw.z, kn_raw.w),
                               make_uint4(vn_raw.x, vn_raw.y, vn_raw.z, vn_raw.w), len - 1, scale_l2, lane, st, lg_stage, lg_lo,
                               vis_hi);
        if (lane < 2 * LPR) {                       // store the row into the cache: lanes [0,LPR) K, [LPR,2*LPR) V
            KT* dst = (lane < LPR ? kbase : vbase) + (int64_t)(len_phys - 1) * a.stride_t + (lane % LPR) * EPL;
            store_hint<NTS>(reinterpret_cast<u32x4_t*>(dst), lane < LPR ? kn_raw : vn_raw);
        }
    }
    finish_wave<KT, D>(st);

    __shared__ float sm_acc[kDecodeWaves][D];
    __shared__ float sm_m[kDecodeWaves], sm_l[kDecodeWaves];
    if (lane < LPR) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) sm_acc[wave][lane * EPL + e] = st.acc[e];
    }
    if (lane == 0) { sm_m[wave] = st.m; sm_l[wave] = st.l; }
    __syncthreads();
    if (lg != nullptr) {
        for (int i = tid; i < lg_hi - lg_lo; i += kDecodeThreads)
            store_hint<NTS>(lg + (lg_lo - vis_lo + i), sm_lg[i]);
    }
    if (tid < D) {
        float m = sm_m[0];
#pragma unroll
        for (int w = 1; w < kDecodeWaves; ++w) m = fmaxf(m, sm_m[w]);   // finite (WaveState)
        float o = 0.f, l = 0.f;
#pragma unroll
        for (int w = 0; w < kDecodeWaves; ++w) {
            float f = exp2_fast(sm_m[w] - m);           // wave without rows: its sums are 0
            o = fmaf(sm_acc[w][tid], f, o);
            l = fmaf(sm_l[w], f, l);
        }
        const int64_t slot = bh * a.nsplit_cap + split;
        if (a.nsplit == 1) store_out<T, NTS>(a.out, bh * D + tid, o / l * v_unit);
        else a.part_o[slot * D + tid] = o * v_unit;
        if (tid == 0) { a.part_ml[slot * 2] = m; a.part_ml[slot * 2 + 1] = l; }
    }
}

// One workgroup: the whole strips of heads [h0, h1) of sequence b, one after the other (nsplit is 1).  What attend_chunk does for each, with
// the next head's first tile on its way while the waves of the current one merge; and with `sums`, the mass's share of these heads is
// added up here, since a whole strip's normaliser is known: instead of a logit for every head and visual row, one sum of probabilities for every
// visual row leaves, in the place of head h0's logits.  Why: a write costs a streaming launch as much as reading ten times its bytes
// (a plain kernel reads strips of 380 KB at 7.07 TB/s, with one KB written for each at 6.87, with two at 6.61, wherever the KB goes, whatever the store's policy
// and moment).  Whole steps, us, with a logit for each head, with none (no mass wanted), with sums over up to 8 heads, and the same with mass_sums_block's
// loop not unrolled, as it is now: 13B batch 32 2431, 2304, 2363, 2326, high resolution batch 8 E4M3 638, 547, 594, 585, 13B batch 8 with lazy
// layers 496, 470, 484, 476.
template <typename T, typename KT, int D, int U, bool NTS>
__device__ __forceinline__ void attend_heads(const DecodeArgs& a, const int h0, const int h1, const int b, const bool sums, const int n_sums) {
    using M = RowMap<KT, D>;
    constexpr int EPL = M::EPL, LPR = M::LPR, TILE = U * M::RPL;
    const int tid = threadIdx.x, lane0 = tid % kWave, wave = tid / kWave;
    const int64_t bh0 = (int64_t)b * a.H + h0;
    const KT* kb = reinterpret_cast<const KT*>(a.k) + b * a.stride_b;
    const KT* vb = reinterpret_cast<const KT*>(a.v) + b * a.stride_b;
    uint4 kr[U], vr[U];
    const RowShift guess{a.hint_base, a.hint_gap};
    issue_tile_within<KT, D, U, true>(kb + h0 * a.stride_h, vb + h0 * a.stride_h, a.stride_t, wave * TILE, a.chunk,
                                     a.max_kv - (a.k_new != nullptr ? 1 : 0), 0, lane0, kr, vr, guess);
    const int len_phys = min(a.kv_len[b] + (a.k_new != nullptr ? 1 : 0), a.max_kv);
    const SeqLayout lay = seq_layout(a.sys_len, a.vis_len[b], a.max_vis, len_phys, a.tail_start, b);
    const int len = lay.vlen;
    const RowShift sh = lay.shift();
    if (h0 == 0 && tid == 0 && a.pending != nullptr) {
        a.pending[b * 4 + 0] = ((a.logits != nullptr && len > 0 && a.defer) ? 1 : 0) | (max(len, 0) << 1);
        a.pending[b * 4 + 1] = a.nsplit;
        a.pending[b * 4 + 2] = a.chunk;
        a.pending[b * 4 + 3] = ((a.logits != nullptr && len > 0 && a.keep_all_logits) ? 1 : 0) | (lay.nv << 1);
    }
    if (len <= 0) {                                     // empty sequence: out = 0, no mass
        for (int i = tid; i < (h1 - h0) * D; i += kDecodeThreads) store_out<T>(a.out, bh0 * D + i, 0.f);
        return;
    }
    const int vis_lo = a.keep_all_logits ? 0 : a.sys_len;
    const int vis_hi = a.keep_all_logits ? len : a.sys_len + lay.nv;
    const bool has_new = a.k_new != nullptr && len_phys - 1 >= lay.base + lay.gap;
    const int c1_cached = has_new ? len - 1 : len;
    extern __shared__ float sm_lg[];
    const int lg_lo = max(0, vis_lo), n_lg = min(len, vis_hi) - lg_lo;
    float* lg_stage = a.logits != nullptr ? sm_lg : nullptr;
    float* acc = sm_lg + n_sums;                        // a thread's own entries: i = tid, tid + 256, ...
    __shared__ float sm_acc[kDecodeWaves][D];
    __shared__ float sm_m[kDecodeWaves], sm_l[kDecodeWaves];
    {
        const int tile_end = min(wave * TILE + TILE, c1_cached);
        const bool same = lay.gap == guess.gap && (lay.gap == 0 || lay.base == guess.split_row);
        const bool in_front = tile_end <= lay.base && (guess.gap == 0 || tile_end <= guess.split_row);
        if (!same && !in_front)
            issue_tile<KT, D, U, true>(kb + h0 * a.stride_h, vb + h0 * a.stride_h, a.stride_t, wave * TILE, c1_cached, 0, lane0, kr, vr, sh);
    }
    for (int h = h0; h < h1; ++h) {
        // (opaque: else what a lane works out for its first tile waits in registers from head to head)
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        const int64_t bh = (int64_t)b * a.H + h;
        const KT* kbase = kb + h * a.stride_h;
        const KT* vbase = vb + h * a.stride_h;
        float qf[EPL];
        load_row_slice<T, KT, D>(reinterpret_cast<const T*>(a.q) + bh * D, lane, qf);
        const float k_unit = a.k_scale ? a.k_scale[bh] : 1.0f, v_unit = a.v_scale ? a.v_scale[bh] : 1.0f;
        const float scale_l2 = a.scale_l2 * k_unit;
        u32x4_t kn_raw = {0, 0, 0, 0}, vn_raw = {0, 0, 0, 0};
        if (has_new && wave == 0)
            NewRow<T, KT, D>::load_by_wave(reinterpret_cast<const T*>(a.k_new) + bh * D, reinterpret_cast<const T*>(a.v_new) + bh * D,
                                           lane, k_unit, v_unit, kn_raw, vn_raw);
#pragma unroll
        for (int u = 0; u < U; ++u)                     // (rows past the end may hold anything)
            if (wave * TILE + u * M::RPL + lane / LPR >= c1_cached) vr[u] = make_uint4(0, 0, 0, 0);
        WaveState<EPL> st;
        wave_attend_primed<KT, D, U, true>(qf, kbase, vbase, a.stride_t, wave * TILE, c1_cached, kDecodeWaves * TILE, 0, scale_l2, lane, st,
                                           lg_stage, lg_lo, vis_hi, kr, vr, sh);
        if (has_new && wave == 0) {
            wave_attend_row<KT, D>(qf, make_uint4(kn_raw.x, kn_raw.y, kn_raw.z, kn_raw.w), make_uint4(vn_raw.x, vn_raw.y, vn_raw.z, vn_raw.w),
                                   len - 1, scale_l2, lane, st, lg_stage, lg_lo, vis_hi);
            if (lane < 2 * LPR) {
                KT* dst = const_cast<KT*>(lane < LPR ? kbase : vbase) + (int64_t)(len_phys - 1) * a.stride_t + (lane % LPR) * EPL;
                store_hint<NTS>(reinterpret_cast<u32x4_t*>(dst), lane < LPR ? kn_raw : vn_raw);
            }
        }
        finish_wave<KT, D>(st);
        if (lane < LPR) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) sm_acc[wave][lane * EPL + e] = st.acc[e];
        }
        if (lane == 0) { sm_m[wave] = st.m; sm_l[wave] = st.l; }
        asm volatile("" : "+v"(lane));
        if (h + 1 < h1)
            issue_tile<KT, D, U, true>(kbase + a.stride_h, vbase + a.stride_h, a.stride_t, wave * TILE, c1_cached, 0, lane, kr, vr, sh);
        __syncthreads();
        float m = sm_m[0], l = 0.f, f[kDecodeWaves];
#pragma unroll
        for (int w = 1; w < kDecodeWaves; ++w) m = fmaxf(m, sm_m[w]);   // finite (WaveState)
#pragma unroll
        for (int w = 0; w < kDecodeWaves; ++w) {
            f[w] = exp2_fast(sm_m[w] - m);              // wave without rows: its sums are 0
            l = fmaf(sm_l[w], f[w], l);
        }
        if (tid < D) {
            float o = 0.f;
#pragma unroll
            for (int w = 0; w < kDecodeWaves; ++w) o = fmaf(sm_acc[w][tid], f[w], o);
            store_out<T, NTS>(a.out, bh * D + tid, o / l * v_unit);
        }
        if (sums) {
            const float rl = 1.0f / l;
            for (int i = tid; i < n_lg; i += kDecodeThreads) {
                const float p = exp2_fast(sm_lg[i] - m) * rl, s = h == h0 ? p : acc[i] + p;
                if (h + 1 < h1) acc[i] = s;
                else store_hint<NTS>(a.logits + bh0 * a.capacity + lg_lo + i, s);
            }
        } else if (lg_stage != nullptr) {
            float* lg = a.logits + bh * a.capacity + lg_lo;
            for (int i = tid; i < n_lg; i += kDecodeThreads) store_hint<NTS>(lg + i, sm_lg[i]);
            if (tid == 0) { a.part_ml[bh * a.nsplit_cap * 2] = m; a.part_ml[bh * a.nsplit_cap * 2 + 1] = l; }
        }
        __syncthreads();                                // (the next head's waves write the logits' and the sums' places)
    }
}

// grid (nsplit, H, B)
template <typename T, typename KT, int D, int U>
__global__ __launch_bounds__(kDecodeThreads, ST3_DECODE_MIN_BLOCKS)
__attribute__((amdgpu_waves_per_eu(ST3_DECODE_MIN_BLOCKS, ST3_DECODE_MIN_BLOCKS)))    // do not spill to reach a third wave
void decode_attend_kernel(DecodeArgs a) {
    attend_chunk<T, KT, D, U, false>(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// What a workgroup of a whole-step launch does: chunk `split` of strip (b, h) of the table's entry li, or, with the launch's first
// workgroups, the ranking of (li, b) for a layer whose next eviction does not wait for the mass of this step (kStepApart,
// evict_rank_early).  A ranking takes as long as the attention of a small step (2048 rows 15 us), so all of them have to start at
// once: as workgroups behind the attention's of their sequence, the last ones started when the launch's last strips did, and with them
// the grid was one head wider.  us a step, so -> first: 16 layers of 16 heads, 2880 visual rows 82.5 -> 74.0, 32 layers of 8 heads, batch 2,
// 2048 rows, E4M3 60.7 -> 56.0, 32 layers of 4 heads 44.3 -> 45.7, 4 layers of 40 heads 49.6 -> 53.0 (behind a first slice of strips:
// 82.4, 61.9, 45.5, 48.9); without evictions 8 layers of 8 heads, batch 4, 1500 rows 44.5 -> 39.7, 40 layers of 12 heads, 2000 rows 110 ->
// 94.0, 32 layers of 8 heads, batch 4, 2880 rows 267 -> 254.
struct StepWork {
    bool ranks;
    int li, b, split, h;
};
__device__ __forceinline__ StepWork step_work(const StepCommon& c) {
    StepWork w;
    w.split = blockIdx.y; w.h = blockIdx.x;
    w.ranks = (int)blockIdx.z < c.rank_z;
    const int z = w.ranks ? ((int)blockIdx.z * c.chunks + w.split) * c.H + w.h : (int)blockIdx.z - c.rank_z;
    w.li = __builtin_amdgcn_readfirstlane(z / c.B);
    w.b = z - w.li * c.B;
    return w;
}
// The same of a launch of groups of heads, whose grid is a line: rank_z workgroups that rank, then the layers' groups, of 8, 4, 2 and 1 heads
// (w.h is the first one, `heads` how many).
__device__ __forceinline__ StepWork step_work_grouped(const StepCommon& c, int& heads) {
    StepWork w;
    w.split = 0;
    int x = (int)blockIdx.x, first = 0, per = 1;        // per: workgroups of a (layer, sequence)
    w.ranks = x < c.rank_z;
    heads = 1;
    if (!w.ranks) {
        x -= c.rank_z;
        per = c.H;
#pragma unroll
        for (int i = 0, g = 8; i < 3; ++i, g /= 2) {
            const int p = (c.H + g - 1) / g, all = c.groups[i] * c.B * p;
            if (heads == 1) {
                if (x < all) { heads = g; per = p; }
                else { x -= all; first += c.groups[i]; }
            }
        }
    }
    const int y = __builtin_amdgcn_readfirstlane(x / per), z = __builtin_amdgcn_readfirstlane(y / c.B);
    w.h = (x - y * per) * heads;
    w.li = first + z;
    w.b = y - z * c.B;
    return w;
}
__device__ __forceinline__ void rank_workgroup(const StepCommon& c, const StepLayer& e, int b) {
    if (!(e.flags & kStepApart) || e.keep_count < 0) return;
    __shared__ SelectShared sm;
    evict_rank_early<kDecodeThreads>(plan_from_entry(c, e), b, sm);
}
// The first workgroup of a layer leaves the layer's entry, as it stands in the table, behind the layer's decode workspace.
__device__ __forceinline__ void leave_entry(const StepTable& t, const StepLayer& e, const DecodeWs& wl, const StepWork& w, int words) {
    const int i = threadIdx.x;
    if (!t.c.leave || w.split != 0 || w.h != 0 || w.b != 0 || i >= words + kWideWords) return;
    reinterpret_cast<uint32_t*>(e.ws + wl.total)[i] = t.w[i < words ? w.li * words + i : kStepTableWords - kWideWords * (w.li + 1) + i - words];
}

// The attention of several layers of a step that do not depend on each other; grid (H, most chunks of any of them, rank_z +
// B * layers), layers in order, so the longest strips (early layers keep the most rows) start first.  Bound by HBM; as a
// launch per layer it was bound by the ramp and the tail of each launch and the gap behind it (about 9 us a layer, whatever
// its bytes).  Whole step, us, one launch per layer -> up to 35 layers per launch: 7B batch 1 191 -> 42 (209 MB), 13B batch 8
// with lazy layers 707 -> 496 (2.9 GB), high resolution batch 8 E4M3 830 -> 618 (3.6 GB), 13B batch 32 2514 -> 2407 (15.4 GB,
// 6.4 TB/s; a kernel that only reads the same rows takes 2155).
// FORM: kStepPlain; kStepAny: the table may be wide, and the entries may be left for the plans (a build of its own: these cost 0.1 to 0.4 us a step at the
// start of every workgroup); kStepGroups: workgroups of whole strips of several heads (c.groups), in a grid that is a line.
enum StepForm { kStepPlain, kStepAny, kStepGroups };
template <typename T, typename KT, int D, int U, bool NTS, StepForm FORM>
__global__ __launch_bounds__(kDecodeThreads, ST3_DECODE_MIN_BLOCKS)
__attribute__((amdgpu_waves_per_eu(ST3_DECODE_MIN_BLOCKS, ST3_DECODE_MIN_BLOCKS)))
void decode_attend_layers_kernel(StepTable t) {
    constexpr bool ANY = FORM == kStepAny;
    const StepCommon& c = t.c;
    int heads = 1;
    const StepWork w = FORM == kStepGroups ? step_work_grouped(c, heads) : step_work(c);
    if (w.li >= c.layers) return;
    constexpr bool coded = sizeof(KT) == 1;
    constexpr int words = coded ? kAttendWordsE4M3 : kAttendWords;
    const StepLayer e = unpack_attend<coded>(t.w + w.li * words, sizeof(KT), high_words(t.w, w.li), ANY && c.wide != 0);
    if (w.ranks) return rank_workgroup(c, e, w.b);
    if (w.split >= e.nsplit) return;
    const DecodeWs wl = decode_ws_sized(c.B, c.H, D, e.capacity, e.nsplit_cap);
    if (ANY) leave_entry(t, e, wl, w, words);
    const bool want = (e.flags & kStepWantMass) != 0, all = (e.flags & kStepKeepAll) != 0;
    DecodeArgs a;
    a.q = e.q; a.k = e.k; a.v = e.v;
    a.stride_b = e.stride_b; a.stride_h = e.stride_h; a.stride_t = e.stride_t;
    a.kv_len = e.kv_len; a.vis_len = e.vis_len; a.tail_start = e.tail_start;
    a.B = c.B; a.sys_len = e.sys_len; a.max_vis = e.max_vis; a.max_kv = e.max_kv + 1; a.H = c.H;
    a.nsplit = e.nsplit; a.nsplit_cap = e.nsplit_cap; a.chunk = e.chunk; a.capacity = e.capacity;
    a.hint_base = e.hint_base; a.hint_gap = e.hint_gap;
    a.defer = want; a.keep_all_logits = all;
    a.scale_l2 = c.scale_l2; a.k_scale = e.k_scale; a.v_scale = e.v_scale;
    a.part_o = reinterpret_cast<float*>(e.ws + wl.part_o);
    a.part_ml = reinterpret_cast<float*>(e.ws + wl.part_ml);
    a.logits = (want || all) ? reinterpret_cast<float*>(e.ws + wl.logits) : nullptr;
    a.stage_rows = 0;           // (the launcher's)
    a.pending = reinterpret_cast<int32_t*>(e.ws + wl.pending);
    a.k_new = e.k_new; a.v_new = e.v_new; a.out = e.out;
    if constexpr (FORM == kStepGroups) {
        const bool sums = (e.flags & kStepSums) != 0;
        attend_heads<T, KT, D, U, NTS>(a, w.h, min(c.H, w.h + heads), w.b, sums, sums ? e.max_vis : 0);
    } else {
        attend_chunk<T, KT, D, U, NTS>(a, w.split, w.h, w.b);
    }
}

// ---------------------------------------------------------------------------------------------
// Lazy layer (QK heredity, Eq. 6 / Alg. 2): o = sum_j p_j V[j] with the probabilities p of the
// SOURCE layer's attention of the same step, rebuilt from the logits and chunk (max, sum) pairs
// that the source's attend launch left in its workspace.  Streams V once: half the bytes.
// ---------------------------------------------------------------------------------------------
struct InheritArgs {
    void* v;
    int64_t stride_b, stride_h, stride_t;
    const int32_t* kv_len;
    const int32_t* vis_len;
    const int32_t* tail_start;  // [B] or null
    int32_t B, max_kv, H, nsplit, nsplit_cap, chunk, sys_len, max_vis;
    const float* src_logits;    // [B,H,src_capacity]
    const float* src_part_ml;   // [B,H,src_nsplit_cap,2]
    const int32_t* src_pending; // [B][4]
    int32_t src_capacity, src_nsplit_cap;
    int32_t* own_pending;       // [B][4] of this layer: the visual rows are left there for a plan (the rest is the source's); null where
                                // no plan follows: then the workspace may be the source's own, whose descriptor other workgroups read
    float* part_o;              // [B,H,nsplit_cap,D]   (nsplit > 1 only)
    const void* v_new;          // [B,H,D] value row of the token being appended (null: none)
    const float* v_scale;       // [B*H] value of one V code unit (E4M3 caches; null: 1)
    void* out;
};

// One wave over the tiles of U*RPL value rows starting at r0, r0+step, ... below r1; next tile's
// loads are issued before the current tile is consumed.
template <typename T, int D, int U>
__device__ __forceinline__ void wave_inherit(const T* vbase, int64_t stride_t, int r0, int r1, int step, int safe_row,
                                             const float* lg, float m, float rl, int lane, float* acc,
                                             const RowShift sh) {
    using M = RowMap<T, D>;
    constexpr int EPL = M::EPL, LPR = M::LPR, RPL = M::RPL;
    const int grp = lane / LPR;
    const int64_t col = (int64_t)(lane % LPR) * EPL;
    if (r0 >= r1) return;
    u32x4_t vr[U], vn[U];
    float sr[U], sn[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int row = r0 + u * RPL + grp;
        const int rr = row < r1 ? row : safe_row;
        vr[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(vbase + (int64_t)sh.physical(rr) * stride_t + col));
        sr[u] = lg[rr];
    }
    for (int t0 = r0; t0 < r1; t0 += step) {
        const int tn = t0 + step;
        if (tn < r1) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int row = tn + u * RPL + grp;
                const int rr = row < r1 ? row : safe_row;
                vn[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(vbase + (int64_t)sh.physical(rr) * stride_t + col));
                sn[u] = lg[rr];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = t0 + u * RPL + grp;
            const float p = row < r1 ? exp2_fast(sr[u] - m) * rl : 0.f;
            float vf[EPL];
            ElemTraits<T>::unpack(make_uint4(vr[u].x, vr[u].y, vr[u].z, vr[u].w), vf);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
        }
        if (tn < r1) {
#pragma unroll
            for (int u = 0; u < U; ++u) { vr[u] = vn[u]; sr[u] = sn[u]; }
        }
    }
}

// One workgroup: chunk `split` of strip (b, h) of a lazy layer.
template <typename T, typename KT, int D, int U>
__device__ __forceinline__ void inherit_chunk(const InheritArgs& a, const int split, const int h, const int b) {
    using M = RowMap<KT, D>;
    constexpr int EPL = M::EPL, LPR = M::LPR, TILE = U * M::RPL;
    const int len_phys = min(a.kv_len[b] + (a.v_new != nullptr ? 1 : 0), a.max_kv);
    // rows are numbered without the gap a fixed-tail cache keeps behind its visual segment, as in the
    // source layer's attend launch (same lengths, same layout): its logits are indexed the same way
    const SeqLayout lay = seq_layout(a.sys_len, a.vis_len[b], a.max_vis, len_phys, a.tail_start, b);
    const int len = lay.vlen;
    const int c0 = split * a.chunk;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int64_t bh = (int64_t)b * a.H + h;
    // (called last: loads behind a store that could have written what they read are not scalar ones; 4096 strips of 100 rows, D = 64,
    // 12.8 us a call with the store here instead of 11.7)
    auto leave_rows = [&] {
        if (a.own_pending != nullptr && split == 0 && h == 0 && tid == 0) a.own_pending[b * 4 + 3] = lay.nv << 1;
    };
    const bool have = (a.src_pending[b * 4 + 3] & 1) != 0;        // the source attended a non-empty sequence
    if (len <= 0 || !have) {                                // nothing to inherit: out = 0
        if (split == 0 && tid < D) store_out<T>(a.out, bh * D + tid, 0.f);
        if (len > 0 && a.nsplit > 1 && c0 < len && tid < D) a.part_o[(bh * a.nsplit_cap + split) * D + tid] = 0.f;
        leave_rows();
        return;
    }
    if (c0 >= len) return;
    const int c1 = min(c0 + a.chunk, len);
    // the source row's maximum and sum from its chunk pairs, in chunk order (every thread alike)
    const int s_nsplit = min(a.src_pending[b * 4 + 1], a.src_nsplit_cap);
    const int s_chunk = max(a.src_pending[b * 4 + 2], 32);
    const int s_ns = min((len + s_chunk - 1) / s_chunk, s_nsplit);
    const float* ml = a.src_part_ml + bh * a.src_nsplit_cap * 2;
    float m = ml[0];
    for (int s = 1; s < s_ns; ++s) m = fmaxf(m, ml[2 * s]);
    float l = 0.f;
    for (int s = 0; s < s_ns; ++s) l = fmaf(ml[2 * s + 1], exp2_fast(ml[2 * s] - m), l);
    const float rl = 1.0f / l;

    KT* vbase = reinterpret_cast<KT*>(a.v) + b * a.stride_b + h * a.stride_h;
    const float* lg = a.src_logits + bh * a.src_capacity;
    const float v_unit = a.v_scale ? a.v_scale[bh] : 1.0f;
    float acc[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
    const bool has_new = a.v_new != nullptr && c1 == len && len_phys - 1 >= lay.base + lay.gap;
    const int c1_cached = has_new ? c1 - 1 : c1;
    wave_inherit<KT, D, U>(vbase, a.stride_t, c0 + wave * TILE, c1_cached, kDecodeWaves * TILE, c0, lg, m, rl, lane, acc,
                           lay.shift());
    if (has_new && wave == 0) {
        u32x4_t none = {0, 0, 0, 0}, raw = {0, 0, 0, 0};
        NewRow<T, KT, D>::load_by_wave(nullptr, reinterpret_cast<const T*>(a.v_new) + bh * D, lane, 1.0f, v_unit, none, raw);
        if (lane < LPR) {
            const float p = exp2_fast(lg[len - 1] - m) * rl;
            float vf[EPL];
            ElemTraits<KT>::unpack(make_uint4(raw.x, raw.y, raw.z, raw.w), vf);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
            *reinterpret_cast<u32x4_t*>(vbase + (int64_t)(len_phys - 1) * a.stride_t + lane * EPL) = raw;
        }
    }
#pragma unroll
    for (int off = LPR; off < kWave; off <<= 1) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] += __shfl_xor(acc[e], off);
    }
    __shared__ float sm_acc[kDecodeWaves][D];
    if (lane < LPR) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) sm_acc[wave][lane * EPL + e] = acc[e];
    }
    __syncthreads();
    if (tid < D) {
        float o = 0.f;
#pragma unroll
        for (int w = 0; w < kDecodeWaves; ++w) o += sm_acc[w][tid];
        if (a.nsplit == 1) store_out<T>(a.out, bh * D + tid, o * v_unit);
        else a.part_o[(bh * a.nsplit_cap + split) * D + tid] = o * v_unit;
    }
    leave_rows();
}

// grid (nsplit, H, B)
template <typename T, typename KT, int D, int U>
__global__ __launch_bounds__(kDecodeThreads, ST3_DECODE_MIN_BLOCKS) void decode_inherit_kernel(InheritArgs a) {
    inherit_chunk<T, KT, D, U>(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// Several lazy layers of a step (their sources have all attended); grid as in decode_attend_layers_kernel.
template <typename T, typename KT, int D, int U, bool ANY>
__global__ __launch_bounds__(kDecodeThreads, ST3_DECODE_MIN_BLOCKS) void decode_inherit_layers_kernel(StepTable t) {
    const StepCommon& c = t.c;
    const StepWork w = step_work(c);
    if (w.li >= c.layers) return;
    constexpr bool coded = sizeof(KT) == 1;
    constexpr int words = coded ? kAttendWordsE4M3 : kAttendWords;
    const StepLayer e = unpack_attend<coded>(t.w + w.li * words, sizeof(KT), high_words(t.w, w.li), ANY && c.wide != 0);
    if (w.ranks) return rank_workgroup(c, e, w.b);
    if (w.split >= e.nsplit) return;
    const DecodeWs wl = decode_ws_sized(c.B, c.H, D, e.capacity, e.nsplit_cap);
    if (ANY) leave_entry(t, e, wl, w, words);
    const DecodeWs sl = decode_ws_sized(c.B, c.H, D, e.hint_base, e.src_nsplit_cap);
    const char* sws = reinterpret_cast<const char*>(e.q);
    InheritArgs a;
    a.v = e.v; a.stride_b = e.stride_b; a.stride_h = e.stride_h; a.stride_t = e.stride_t;
    a.kv_len = e.kv_len; a.vis_len = e.vis_len; a.tail_start = e.tail_start;
    a.B = c.B; a.max_kv = e.max_kv + 1; a.H = c.H; a.nsplit = e.nsplit; a.nsplit_cap = e.nsplit_cap; a.chunk = e.chunk;
    a.sys_len = e.sys_len; a.max_vis = e.max_vis;
    a.src_logits = reinterpret_cast<const float*>(sws + sl.logits);
    a.src_part_ml = reinterpret_cast<const float*>(sws + sl.part_ml);
    a.src_pending = reinterpret_cast<const int32_t*>(sws + sl.pending);
    a.src_capacity = e.hint_base; a.src_nsplit_cap = e.src_nsplit_cap;
    a.own_pending = reinterpret_cast<int32_t*>(e.ws + wl.pending);
    a.part_o = reinterpret_cast<float*>(e.ws + wl.part_o);
    a.v_new = e.v_new; a.v_scale = e.v_scale; a.out = e.out;
    inherit_chunk<T, KT, D, U>(a, w.split, w.h, w.b);
}

struct FinishArgs {
    const float* part_o;
    const float* part_ml;
    const float* logits;
    const int32_t* kv_len;
    const int32_t* vis_len;
    const int32_t* tail_start;  // [B] or null
    int32_t H, nsplit, nsplit_cap, chunk, capacity, max_vis, max_kv, sys_len;
    int32_t plain_sum;      // 1: the partial outputs are already normalised, just add them (lazy layers)
    int32_t appended;       // 1: the attend kernel took one more row than kv_len[b] says (the token being appended)
    void* out;              // null: outputs already written (nsplit == 1)
    float* mass;            // null: no mass
    int64_t mass_stride;
};

// grid (out_blocks + mass_blocks, B), 256 threads.  Blocks x < H (when out != null) merge the
// chunk partials of head x; the rest produce kFinishKeys mass entries each.
constexpr int kFinishKeys = kWave;
template <typename T, int D>
__global__ __launch_bounds__(256) void decode_finish_kernel(FinishArgs a) {
    const int b = blockIdx.y, tid = threadIdx.x;
    const SeqLayout lay = seq_layout(a.sys_len, a.vis_len[b], a.max_vis, min(a.kv_len[b] + a.appended, a.max_kv),
                                     a.tail_start, b);
    const int len = lay.vlen;                           // rows the attend launch saw
    const int ns = len > 0 ? min((len + a.chunk - 1) / a.chunk, a.nsplit) : 0;
    const int out_blocks = a.out ? a.H : 0;
    if ((int)blockIdx.x < out_blocks) {
        const int h = blockIdx.x;
        const int64_t bh = (int64_t)b * a.H + h;
        if (tid >= D || ns == 0) return;                // empty sequence: the attend kernel wrote zeros
        const float* po = a.part_o + bh * a.nsplit_cap * D + tid;
        store_out<T>(a.out, bh * D + tid, merge_partials(a.plain_sum, po, D, a.part_ml + bh * a.nsplit_cap * 2, ns));
        return;
    }
    if (a.mass == nullptr) return;
    // kFinishKeys mass entries: a wave takes a quarter of the heads, the quarters are added in order
    __shared__ float sm_m[1024], sm_rl[1024], sm_part[4][kFinishKeys];
    const int nv = lay.nv;
    const int j = ((int)blockIdx.x - out_blocks) * kFinishKeys + tid % kWave;
    if (ns == 0) {                                      // an empty sequence: no probabilities
        if (j < nv && tid < kWave) a.mass[(int64_t)b * a.mass_stride + j] = 0.f;
        return;
    }
    head_norms<256>(a.part_ml, b, a.H, ns, a.nsplit_cap, sm_m, sm_rl);
    const int g = __builtin_amdgcn_readfirstlane(tid / kWave), per = (a.H + 3) / 4, h0 = g * per, h1 = min(a.H, h0 + per);
    if (j < nv)
        // (12 loads in flight: a quarter of 40 heads in one round; with 8 such a call takes 0.5 us more)
        sm_part[g][tid % kWave] = prob_sum<12>(a.logits + a.sys_len + (int64_t)b * a.H * a.capacity + j, a.capacity, sm_m, sm_rl, h0, h1);
    __syncthreads();
    if (j < nv && tid < kWave)
        a.mass[(int64_t)b * a.mass_stride + j] = ((sm_part[0][tid] + sm_part[1][tid]) + (sm_part[2][tid] + sm_part[3][tid])) *
                                                 (1.0f / (float)a.H);
}

struct AppendArgs {
    void* k;
    void* v;
    int64_t stride_b, stride_h, stride_t;
    const void* k_new;
    const void* v_new;
    const int32_t* kv_len;
    const float* k_scale;
    const float* v_scale;
    int32_t H, capacity;
};

// grid (H, B), 64 threads: lanes [0, LPR) write the K row, lanes [LPR, 2*LPR) the V row.
template <typename T, typename KT, int D>
__global__ __launch_bounds__(64) void append_kernel(AppendArgs a) {
    using M = RowMap<KT, D>;
    const int h = blockIdx.x, b = blockIdx.y, lane = threadIdx.x;
    const int row = a.kv_len[b];
    if (row < 0 || row >= a.capacity || lane >= 2 * M::LPR) return;
    const bool is_v = lane >= M::LPR;
    if (!is_v && a.k == nullptr) return;                // a layer that caches V only
    const int64_t bh = (int64_t)b * a.H + h;
    const float* sc = is_v ? a.v_scale : a.k_scale;
    const T* src = reinterpret_cast<const T*>(is_v ? a.v_new : a.k_new) + bh * D;
    const u32x4_t raw = NewRow<T, KT, D>::load(src, lane % M::LPR, sc ? sc[bh] : 1.0f);
    KT* dst = reinterpret_cast<KT*>(is_v ? a.v : a.k) + b * a.stride_b + h * a.stride_h + row * a.stride_t +
              (lane % M::LPR) * M::EPL;
    *reinterpret_cast<u32x4_t*>(dst) = raw;
}

// Rows [0, n) of a [B,H,n,D] tensor of T into rows [0, n) of one half of a cache, in its format.
struct QuantArgs {
    const void* src;
    int64_t s_sb, s_sh, s_st;       // elements of T
    void* dst;
    int64_t d_sb, d_sh, d_st;       // cache elements
    const float* scale;             // [B*H] or null
    int32_t H, n;
};

// grid (ceil(n / rows per block), H, B), 256 threads: LPR lanes per row.
template <typename T, typename KT, int D>
__global__ __launch_bounds__(256) void quantize_rows_kernel(QuantArgs a) {
    using M = RowMap<KT, D>;
    const int h = blockIdx.y, b = blockIdx.z;
    const int row = blockIdx.x * (256 / M::LPR) + threadIdx.x / M::LPR;
    if (row >= a.n) return;
    const int64_t bh = (int64_t)b * a.H + h;
    const T* src = reinterpret_cast<const T*>(a.src) + b * a.s_sb + h * a.s_sh + row * a.s_st;
    const u32x4_t raw = NewRow<T, KT, D>::load(src, threadIdx.x % M::LPR, a.scale ? a.scale[bh] : 1.0f);
    KT* dst = reinterpret_cast<KT*>(a.dst) + b * a.d_sb + h * a.d_sh + row * a.d_st + (threadIdx.x % M::LPR) * M::EPL;
    *reinterpret_cast<u32x4_t*>(dst) = raw;
}

__global__ void bump_len_kernel(int32_t* kv_len, int32_t B, int32_t capacity) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B && kv_len[b] >= 0 && kv_len[b] < capacity) kv_len[b] += 1;
}

// ---------------------------------------------------------------------------------------------
// Tile size (U = 16-byte loads of K, and of V, in flight per lane and tile; a wave-wide load is 1 KB).
// While every workgroup of a launch is resident at once, a tile of 8 KB per wave is the fastest for
// two- and four-byte caches (U = 4: 16 bf16 rows; room for four workgroups per compute unit, short
// strips pipelined in finer steps: 5-9 % faster than U = 8 at B*H = 40 ... 640 strips), 6 KB for E4M3
// (U = 3: 24 rows).  With more workgroups than the device holds, what counts is how full the last
// round of workgroups is: B*H = 1280 bf16 strips are 1.25 rounds at U = 4 (slowest), 1.67 at U = 6,
// 2.5 at U = 8, and fit at once at U = 1 (66 registers, seven workgroups per unit: fastest, though
// much the slowest build for small launches).  So the launcher asks the runtime how many workgroups
// of each build the device holds and takes the build that wastes least of its last round; the
// candidate lists below are in order of preference for ties.
// ---------------------------------------------------------------------------------------------
// The current device's id when it indexes the per-device caches below, else -1 (then nothing is cached).
int current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -1;
    return dev;
}

int compute_units(int dev) {
    static std::atomic<int> cached[kMaxDevices];    // 0 = not asked yet; a race only repeats the query
    if (dev >= 0 && cached[dev].load(std::memory_order_relaxed) != 0) return cached[dev].load(std::memory_order_relaxed);
    int n = 0;
    if (dev < 0 || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
    if (dev >= 0) cached[dev].store(n, std::memory_order_relaxed);
    return n;
}

// Workgroups of `kernel` (256 threads, no dynamic LDS) the current device holds at once; `cache` is
// the kernel's own array of one entry per device.
template <typename K>
int resident_workgroups(K kernel, std::atomic<int>* cache) {
    const int dev = current_device();
    if (dev >= 0 && cache[dev].load(std::memory_order_relaxed) != 0) return cache[dev].load(std::memory_order_relaxed);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kDecodeThreads, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    const int n = per_cu * compute_units(dev);
    if (dev >= 0) cache[dev].store(n, std::memory_order_relaxed);
    return n;
}

// Time of a launch of `items` equal workgroups on `slots` concurrent ones, relative to a launch whose
// last round is full.
inline double last_round_cost(int64_t items, int slots) {
    const double rounds = (double)items / (double)slots;
    return rounds <= 1.0 ? 1.0 : std::ceil(rounds) / rounds;
}

// Index of the cheapest of n candidates (ordered by preference: the first wins ties).
inline int cheapest(const double* cost, int n) {
    int best = 0;
    for (int i = 1; i < n; ++i)
        if (cost[i] < cost[best] - 1e-9) best = i;
    return best;
}

// Launches `kernel` with the profiler's event pair attached when one is to be had; `layers` is how many layers'
// attention the launch does.
template <typename K, typename A>
void launch_timed(K kernel, dim3 grid, size_t lds, hipStream_t st, int layers, const A& args) {
    hipEvent_t e0, e1;
    if (profile_take(&e0, &e1, layers))     // timed launch: the events receive the kernel's own start and end
        hipExtLaunchKernelGGL(kernel, grid, dim3(kDecodeThreads), lds, st, e0, e1, 0, args);
    else
        kernel<<<grid, kDecodeThreads, lds, st>>>(args);
}

// go(U) with the forced tile size when one is set and built, else with build number `pick` of Us...
template <int... Us, typename Go>
void with_tile(std::integer_sequence<int, Us...>, int pick, Go go) {
    const int us[] = {Us...};
    int u = debug_state().attend_tile;          // 0 unless the debug block is enabled
    if (!((u == Us) || ...)) u = us[pick];
    ((u == Us ? (go(std::integral_constant<int, Us>{}), 0) : 0), ...);
}

// The cheapest of the builds Us... (in order of preference) for a launch of `items` workgroups.
template <typename T, typename KT, int D, int... Us>
int best_tile(int64_t items, std::integer_sequence<int, Us...>) {
    constexpr int N = sizeof...(Us);
    static std::atomic<int> slots[N][kMaxDevices];  // resident workgroups of each build, per device
    double cost[N];
    int i = 0;
    ((cost[i] = last_round_cost(items, resident_workgroups(decode_attend_kernel<T, KT, D, Us>, slots[i])), ++i), ...);
    return cheapest(cost, N);
}

template <typename KT>
using AttendTiles = std::conditional_t<sizeof(KT) == 1, std::integer_sequence<int, 3, 4, 1>, std::integer_sequence<int, 4, 6, 8, 1>>;

template <int U0, int... Us>
constexpr int first_tile(std::integer_sequence<int, U0, Us...>) { return U0; }

template <typename T, typename KT, int D>
void launch_attend(const DecodeArgs& da, int B, hipStream_t st) {
    const dim3 grid(da.nsplit, da.H, B);
    const size_t lds = (size_t)da.stage_rows * sizeof(float);       // dynamic LDS: the logit staging area
    with_tile(AttendTiles<KT>{}, best_tile<T, KT, D>((int64_t)da.nsplit * da.H * B, AttendTiles<KT>{}), [&](auto u) {
        launch_timed(decode_attend_kernel<T, KT, D, decltype(u)::value>, grid, lds, st, 1, da);
    });
}

// `most`: the largest chunk count of any layer of the table.  One build: a launch over many layers runs many rounds of
// workgroups of unequal length, there is no last round to fill.  Measured at U = 4 / 1 / 6 / 8 (E4M3: 3 / 4 / 1), us per step:
// 7B batch 1 72.6 / 71.8 / 75.6 / 78.9, 13B batch 8 with lazy layers 563 / 571 / 560 / 565, 13B batch 32 2441 / 2457 / 2433 /
// 2421, 13B batch 32 E4M3 1327 / 1404 / 1423, high resolution batch 8 E4M3 700 / 696 / 721.
template <typename T, typename KT, int D>
void launch_attend_layers(const StepTable& t, int lds_words, bool stream, hipStream_t st) {
    const dim3 grid(t.c.H, t.c.chunks, t.c.rank_z + t.c.B * t.c.layers);
    const size_t lds = (size_t)lds_words * sizeof(float);
    constexpr int U0 = first_tile(AttendTiles<KT>{});
    if (t.c.wide || t.c.leave) {
        if (stream) launch_timed(decode_attend_layers_kernel<T, KT, D, U0, true, kStepAny>, grid, lds, st, t.c.layers, t);
        else launch_timed(decode_attend_layers_kernel<T, KT, D, U0, false, kStepAny>, grid, lds, st, t.c.layers, t);
        return;
    }
    if (t.c.groups[3]) {
        int per_sequence = 0, left = t.c.layers;
        for (int i = 0, g = 8; i < 3; ++i, g /= 2) { per_sequence += t.c.groups[i] * ((t.c.H + g - 1) / g); left -= t.c.groups[i]; }
        const dim3 line(t.c.rank_z + t.c.B * (per_sequence + left * t.c.H));
        if (stream) launch_timed(decode_attend_layers_kernel<T, KT, D, U0, true, kStepGroups>, line, lds, st, t.c.layers, t);
        else launch_timed(decode_attend_layers_kernel<T, KT, D, U0, false, kStepGroups>, line, lds, st, t.c.layers, t);
        return;
    }
    with_tile(AttendTiles<KT>{}, 0, [&](auto u) {
        if (stream) launch_timed(decode_attend_layers_kernel<T, KT, D, decltype(u)::value, true, kStepPlain>, grid, lds, st, t.c.layers, t);
        else launch_timed(decode_attend_layers_kernel<T, KT, D, decltype(u)::value, false, kStepPlain>, grid, lds, st, t.c.layers, t);
    });
}

template <typename T, typename KT, int D>
void launch_inherit_layers(const StepTable& t, int lds_words, hipStream_t st) {
    const dim3 grid(t.c.H, t.c.chunks, t.c.rank_z + t.c.B * t.c.layers);
    const size_t lds = (size_t)lds_words * sizeof(uint32_t);
    if (t.c.wide || t.c.leave) decode_inherit_layers_kernel<T, KT, D, 4, true><<<grid, kDecodeThreads, lds, st>>>(t);
    else decode_inherit_layers_kernel<T, KT, D, 4, false><<<grid, kDecodeThreads, lds, st>>>(t);
}

// The V-only kernel of lazy layers: 4 loads per lane and tile (4 KB per wave) were the fastest or
// within 2 % of it at every batch size and for both cache formats (8, 12 and 16 loads lose up to
// 17 % where the launch has more workgroups than fit at once; 2 loads lose at small batches).
template <typename T, typename KT, int D>
void launch_inherit(const InheritArgs& ia, int B, hipStream_t st) {
    decode_inherit_kernel<T, KT, D, 4><<<dim3(ia.nsplit, ia.H, B), kDecodeThreads, 0, st>>>(ia);
}

template <typename T, int D>
void launch_finish(const FinishArgs& fa, int B, hipStream_t st) {
    const int blocks = (fa.out ? fa.H : 0) + (fa.mass ? (fa.max_vis + kFinishKeys - 1) / kFinishKeys : 0);
    if (blocks > 0) decode_finish_kernel<T, D><<<dim3(blocks, B), 256, 0, st>>>(fa);
}

template <typename T, typename KT, int D>
void launch_append(const AppendArgs& aa, int B, int32_t* kv_len, hipStream_t st) {
    append_kernel<T, KT, D><<<dim3(aa.H, B), 64, 0, st>>>(aa);
    bump_len_kernel<<<(B + 255) / 256, 256, 0, st>>>(kv_len, B, aa.capacity);
}

template <typename T, typename KT, int D>
void launch_quantize(const QuantArgs& qa, int B, hipStream_t st) {
    using M = RowMap<KT, D>;
    const int rpb = 256 / M::LPR;
    quantize_rows_kernel<T, KT, D><<<dim3((qa.n + rpb - 1) / rpb, qa.H, B), 256, 0, st>>>(qa);
}

// Launchers that depend on the cache element type: KT = T for plain caches, e4m3_t (bf16 I/O only,
// checked on the host) for E4M3 caches.
#define ST3_DISPATCH_KV(fn, shape, kv, ...)                                                                    \
    do {                                                                                                       \
        if ((kv)->format == ST3_KV_E4M3) {                                                                     \
            if ((shape)->head_dim == 128) fn<bf16_t, e4m3_t, 128>(__VA_ARGS__);                                \
            else fn<bf16_t, e4m3_t, 64>(__VA_ARGS__);                                                          \
        } else if ((shape)->dtype == ST3_BF16) {                                                               \
            if ((shape)->head_dim == 128) fn<bf16_t, bf16_t, 128>(__VA_ARGS__);                                \
            else fn<bf16_t, bf16_t, 64>(__VA_ARGS__);                                                          \
        } else {                                                                                               \
            if ((shape)->head_dim == 128) fn<float, float, 128>(__VA_ARGS__);                                  \
            else fn<float, float, 64>(__VA_ARGS__);                                                            \
        }                                                                                                      \
    } while (0)

#define ST3_DISPATCH(fn, shape, ...)                                                                   \
    do {                                                                                               \
        if ((shape)->dtype == ST3_BF16) {                                                              \
            if ((shape)->head_dim == 128) fn<bf16_t, 128>(__VA_ARGS__); else fn<bf16_t, 64>(__VA_ARGS__); \
        } else {                                                                                       \
            if ((shape)->head_dim == 128) fn<float, 128>(__VA_ARGS__); else fn<float, 64>(__VA_ARGS__);   \
        }                                                                                              \
    } while (0)

st3_status check_kv(const st3_attn_shape* s, const st3_kv_layer* kv, const st3_segments* seg, bool value_only = false) {
    if (!kv || !seg || (!kv->k && !value_only) || !kv->v || !seg->kv_len || !seg->vis_len) return ST3_ERR_INVALID_ARG;
    if (kv->capacity <= 0 || seg->sys_len < 0 || seg->max_vis_len < 0 || seg->max_kv_len < 0)
        return ST3_ERR_INVALID_ARG;
    if (seg->max_kv_len > kv->capacity) return ST3_ERR_INVALID_ARG;
    if (seg->sys_len + seg->max_vis_len > kv->capacity) return ST3_ERR_INVALID_ARG;
    if (kv->stride_t < s->head_dim || kv->stride_h < 0 || kv->stride_b < 0) return ST3_ERR_INVALID_ARG;
    if (kv->format != ST3_KV_PLAIN && kv->format != ST3_KV_E4M3) return ST3_ERR_INVALID_ARG;
    if (kv->format == ST3_KV_E4M3) {
        if (s->dtype != ST3_BF16) return ST3_ERR_UNSUPPORTED;
        if ((kv->k && !kv->k_scale) || !kv->v_scale) return ST3_ERR_INVALID_ARG;
    }
    const int eb = kv_elem_bytes(s, kv);
    if ((kv->k && !aligned16(kv->k)) || !aligned16(kv->v)) return ST3_ERR_INVALID_ARG;
    if ((kv->stride_t * eb) % 16 || (kv->stride_h * eb) % 16 || (kv->stride_b * eb) % 16)
        return ST3_ERR_INVALID_ARG;
    return ST3_OK;
}

}  // namespace

// The caller's guess at the layout of a fixed-tail cache, as the attend kernel takes it (none: INT_MAX, 0).
static void layout_hint(const st3_segments* seg, int capacity, int32_t& hint_base, int32_t& hint_gap) {
    hint_base = 0x7fffffff; hint_gap = 0;
    if (seg->tail_start == nullptr || seg->tail_start_hint <= 0) return;
    const int nv = std::max(0, std::min(seg->vis_len_hint, seg->max_vis_len));
    const int base = seg->sys_len + nv;
    const int ts = std::min(seg->tail_start_hint, capacity);        // (keeps row + gap far from overflow)
    if (ts > base) { hint_base = base; hint_gap = ts - base; }
}

// Enqueues attention (+ the finish kernel when it is needed).  max_kv_len bounds the length the
// kernels will see (kv_len[b], plus one when a token is appended: k_new/v_new non-null).
// defer_mass: leave the head reduction of the mass to the eviction plan that follows.
st3_status enqueue_decode(const st3_attn_shape* shape, const void* q, const st3_kv_layer* kv,
                          const st3_segments* seg, int32_t max_kv_len, const void* k_new, const void* v_new,
                          void* out, float* vis_mass, int64_t mass_stride, bool want_mass, bool defer_mass,
                          bool keep_all_logits, void* workspace, size_t workspace_bytes, hipStream_t st) {
    const int B = shape->batch, H = shape->heads, D = shape->head_dim;
    const DecodeWs wl = decode_ws(B, H, D, kv->capacity);
    if (workspace_bytes < wl.total) return ST3_ERR_WORKSPACE_TOO_SMALL;
    char* ws = reinterpret_cast<char*>(workspace);
    want_mass = want_mass && seg->max_vis_len > 0;
    DecodeArgs da{};
    da.q = q; da.k = kv->k; da.v = kv->v;
    da.stride_b = kv->stride_b; da.stride_h = kv->stride_h; da.stride_t = kv->stride_t;
    da.kv_len = seg->kv_len; da.vis_len = seg->vis_len; da.tail_start = seg->tail_start;
    da.B = B; da.sys_len = seg->sys_len; da.max_vis = seg->max_vis_len; da.max_kv = max_kv_len; da.H = H;
    layout_hint(seg, kv->capacity, da.hint_base, da.hint_gap);
    const bool mass_now = want_mass && !defer_mass;
    // a call that finishes its mass has a second launch anyway, so that a cut costs it no launch (13B shape, five sequences
    // of 173 to 1111 rows, attention + finish: 26 us in 200 workgroups, 20.5 us in 1000)
    const int target = mass_now ? merged_target((int64_t)B * H, max_kv_len, D, kv_elem_bytes(shape, kv)) : kDecodeTargetWgs;
    da.nsplit = decode_nsplit(B, H, max_kv_len, target);
    if (da.nsplit > wl.nsplit_cap) da.nsplit = wl.nsplit_cap;
    da.nsplit_cap = wl.nsplit_cap;
    da.chunk = decode_chunk(max_kv_len, da.nsplit);
    da.nsplit = (max_kv_len + da.chunk - 1) / da.chunk;         // rounding the chunk up to 32 rows can leave chunks empty
    if (da.nsplit < 1) da.nsplit = 1;
    da.capacity = kv->capacity;
    da.scale_l2 = scale_log2(shape);
    if (kv->format == ST3_KV_E4M3) { da.k_scale = kv->k_scale; da.v_scale = kv->v_scale; }
    da.part_o = reinterpret_cast<float*>(ws + wl.part_o);
    da.part_ml = reinterpret_cast<float*>(ws + wl.part_ml);
    da.logits = (want_mass || keep_all_logits) ? reinterpret_cast<float*>(ws + wl.logits) : nullptr;
    da.keep_all_logits = keep_all_logits ? 1 : 0;
    // a workgroup keeps at most this many logits: all rows of its chunk, or the visual ones (chunk <= kLogitStageMaxRows)
    if (da.logits != nullptr) da.stage_rows = keep_all_logits ? da.chunk : std::min(da.chunk, seg->max_vis_len);
    if (da.stage_rows > 3 * kLogitStageMaxRows) return ST3_ERR_UNSUPPORTED;    // 48 KB of LDS: a cache of more than 64 x 3 x 4096 rows
    da.pending = reinterpret_cast<int32_t*>(ws + wl.pending);
    da.k_new = k_new; da.v_new = v_new;
    da.out = out;
    da.defer = (want_mass && defer_mass) ? 1 : 0;
    ST3_DISPATCH_KV(launch_attend, shape, kv, da, B, st);
    if (da.nsplit > 1 || mass_now) {
        FinishArgs fa{};
        fa.part_o = da.part_o; fa.part_ml = da.part_ml; fa.logits = da.logits;
        fa.kv_len = seg->kv_len; fa.vis_len = seg->vis_len; fa.tail_start = seg->tail_start;
        fa.H = H; fa.nsplit = da.nsplit; fa.nsplit_cap = wl.nsplit_cap; fa.chunk = da.chunk;
        fa.capacity = kv->capacity; fa.max_vis = seg->max_vis_len; fa.max_kv = max_kv_len; fa.sys_len = seg->sys_len;
        fa.appended = k_new != nullptr ? 1 : 0;
        fa.out = da.nsplit > 1 ? out : nullptr;
        fa.mass = mass_now ? vis_mass : nullptr; fa.mass_stride = mass_stride;
        ST3_DISPATCH(launch_finish, shape, fa, B, st);
    }
    return check_launch();
}

st3_status enqueue_append(const st3_attn_shape* shape, const st3_kv_layer* kv, const st3_segments* seg,
                          const void* k_new, const void* v_new, hipStream_t st) {
    const int B = shape->batch, H = shape->heads;
    AppendArgs aa{};
    aa.k = kv->k; aa.v = kv->v;
    aa.stride_b = kv->stride_b; aa.stride_h = kv->stride_h; aa.stride_t = kv->stride_t;
    aa.k_new = k_new; aa.v_new = v_new; aa.kv_len = seg->kv_len; aa.H = H; aa.capacity = kv->capacity;
    if (kv->format == ST3_KV_E4M3) { aa.k_scale = kv->k_scale; aa.v_scale = kv->v_scale; }
    ST3_DISPATCH_KV(launch_append, shape, kv, aa, B, seg->kv_len, st);
    return check_launch();
}

st3_status validate_kv(const st3_attn_shape* s, const st3_kv_layer* kv, const st3_segments* seg) {
    return check_kv(s, kv, seg);
}

st3_status validate_kv_value_only(const st3_attn_shape* s, const st3_kv_layer* kv, const st3_segments* seg) {
    return check_kv(s, kv, seg, true);
}

// Enqueues a lazy layer's attention (Eq. 6): the probabilities come from the attend launch that last
// used `src_workspace` (same batch, heads and lengths; cache capacity src_capacity), the values
// from `kv->v` plus - when v_new is given - the row being appended, which is stored on the way.  plan_follows: the layer's mass
// is finished by a plan, and the workspace is another than the source's.
st3_status enqueue_inherit(const st3_attn_shape* shape, const st3_kv_layer* kv, const st3_segments* seg,
                           int32_t max_kv_len, const void* v_new, const void* src_workspace,
                           size_t src_workspace_bytes, int32_t src_capacity, void* out, void* workspace,
                           size_t workspace_bytes, bool plan_follows, hipStream_t st) {
    const int B = shape->batch, H = shape->heads, D = shape->head_dim;
    const DecodeWs wl = decode_ws(B, H, D, kv->capacity);
    const DecodeWs sl = decode_ws(B, H, D, src_capacity);
    if (workspace_bytes < wl.total || src_workspace_bytes < sl.total) return ST3_ERR_WORKSPACE_TOO_SMALL;
    if (max_kv_len > src_capacity) return ST3_ERR_INVALID_ARG;       // the source kept a logit per cached key
    char* ws = reinterpret_cast<char*>(workspace);
    const char* sws = reinterpret_cast<const char*>(src_workspace);
    InheritArgs ia{};
    ia.v = kv->v; ia.stride_b = kv->stride_b; ia.stride_h = kv->stride_h; ia.stride_t = kv->stride_t;
    ia.kv_len = seg->kv_len; ia.vis_len = seg->vis_len; ia.tail_start = seg->tail_start;
    ia.sys_len = seg->sys_len; ia.max_vis = seg->max_vis_len;
    ia.B = B; ia.max_kv = max_kv_len; ia.H = H;
    ia.nsplit = decode_nsplit(B, H, max_kv_len);
    if (ia.nsplit > wl.nsplit_cap) ia.nsplit = wl.nsplit_cap;
    ia.nsplit_cap = wl.nsplit_cap;
    ia.chunk = decode_chunk(max_kv_len, ia.nsplit);
    ia.nsplit = (max_kv_len + ia.chunk - 1) / ia.chunk;
    if (ia.nsplit < 1) ia.nsplit = 1;
    ia.src_logits = reinterpret_cast<const float*>(sws + sl.logits);
    ia.src_part_ml = reinterpret_cast<const float*>(sws + sl.part_ml);
    ia.src_pending = reinterpret_cast<const int32_t*>(sws + sl.pending);
    ia.src_capacity = src_capacity; ia.src_nsplit_cap = sl.nsplit_cap;
    if (plan_follows) ia.own_pending = reinterpret_cast<int32_t*>(ws + wl.pending);
    ia.part_o = reinterpret_cast<float*>(ws + wl.part_o);
    ia.v_new = v_new; ia.out = out;
    if (kv->format == ST3_KV_E4M3) ia.v_scale = kv->v_scale;
    ST3_DISPATCH_KV(launch_inherit, shape, kv, ia, B, st);
    if (ia.nsplit > 1) {
        FinishArgs fa{};
        fa.part_o = ia.part_o; fa.kv_len = seg->kv_len; fa.vis_len = seg->vis_len; fa.tail_start = seg->tail_start;
        fa.sys_len = seg->sys_len; fa.max_vis = seg->max_vis_len;
        fa.H = H; fa.nsplit = ia.nsplit; fa.nsplit_cap = wl.nsplit_cap; fa.chunk = ia.chunk;
        fa.capacity = kv->capacity; fa.max_kv = max_kv_len; fa.plain_sum = 1;
        fa.appended = v_new != nullptr ? 1 : 0;
        fa.out = out;
        ST3_DISPATCH(launch_finish, shape, fa, B, st);
    }
    return check_launch();
}

// ---------------------------------------------------------------------------------------------
// All layers of a step, several per launch (the caller has checked them and knows that they share no buffers).
// ---------------------------------------------------------------------------------------------
// A launch writes one output row and two cache rows per strip, and the logits.  Left to the caches, those lines are evicted
// between the reads of K and V, and every turn of the memory from reading to writing costs: with ordinary stores a plain
// strip-reading kernel that writes as little (0.4 % of what it reads) falls from 7.04 to 6.18 TB/s, with non-temporal ones
// to 6.61.  But what stays in the caches is found there by the launch that follows.  Measured, us per step, ordinary ->
// non-temporal, by the bytes a launch writes: 13B batch 2 (3 MB) 170 -> 175, 7B batch 2 (3 MB) 74.0 -> 77.0, 13B batch 4 (6 MB) 317.5 ->
// 320, 7B batch 4 (6.4 MB) 143.2 -> 144.8, batch 6 (9.7 MB) 213.4 -> 211.9, 13B batch 8 (12 MB) 636 -> 622, high resolution batch 2
// (15 MB) 298.7 -> 300, batch 4 (29 MB) 599 -> 584, batch 8 (58 MB) 1201 -> 1154, E4M3 batch 4 (28 MB) 312 -> 311, batch 8 (57 MB) 624 -> 618,
// 13B batch 16 1265 -> 1219, batch 24 1892 -> 1815.
constexpr int64_t kStreamStoreBytes = (int64_t)8 << 20;

// Whether a step's rows are ranked beside its attention, by 256 threads a plan, or in the plans behind it, by up to 1024.  Beside it
// a ranking is hidden as long as the attention lasts (that grows with the strips of all layers), and the masses have workgroups of
// their own, which a plan finishes by itself, heads times rows of them; a layer that evicts more rows than a plan moves takes a
// launch more behind it.  The line is fitted to these, us a step, beside / behind, bf16 d = 128, one sequence, by layers x heads:
//   1024 rows  1 x 4 17.8 / 19.3, 8 x 4 20.2 / 21.9, 1 x 32 21.7 / 24.4
//   2048 rows  1 x 4 24.3 / 22.6, 4 x 4 25.7 / 24.8, 8 x 4 26.5 / 27.9, 1 x 32 26.4 / 30.4
//   2880 rows  1 x 4 28.0 / 24.2, 4 x 4 30.1 / 28.3, 8 x 4 31.9 / 30.6, 16 x 4 35.7 / 37.9, 1 x 32 32.3 / 37.0
//   4096 rows  1 x 4 32.3 / 27.9, 4 x 4 37.7 / 32.8, 8 x 4 40.7 / 39.0, 16 x 4 46.5 / 47.3, 1 x 32 37.3 / 44.8
//   8192 rows  1 x 4 53.7 / 39.4, 8 x 4 66.2 / 61.4, 16 x 4 84.6 / 77.8, 32 x 4 112 / 122, 1 x 32 46.3 / 75.7
//   200 rows evicted: 2880 rows 1 x 4 30.1 / 27.0, 4 x 4 31.2 / 34.7, 8192 rows 1 x 4 57.3 / 45.2, 4 x 4 62.1 / 57.7, 8 x 4 69.8 / 75.9
// Of 176 such steps of 2048 rows or more (4 to 32 heads, 4 to 128 strips, batch 1 to 16, both cache formats) it takes the slower side
// in 18, by 4 % in the middle and by 13 % at most.
static bool rank_beside(int rows, int heads, int64_t strips, int many_moves) {
    return rows <= 1024 || (187 - 10 * heads - strips - 20 * (int64_t)many_moves) * rows <= 270000;
}

// Heads that the workgroups of a layer of so many rows take one after the other (attend_heads), where rows are ranked beside the attention
// and no strip is cut: the more, the fewer sums of the mass are written; but the launch must not end waiting for a long workgroup, so one takes no more
// rows than a 384th of what the launch has behind the layer (`behind`), and the last layers go head by head.  Layers are visited in order: the number falls from layer
// to layer.  us a step, head by head / a share of 768 / 384 / 256 / 128 (or 8 heads always): 13B batch 32 2399 / 2314 / 2314 / 2316 / 2315 (2342), high
// resolution batch 8 E4M3 634 / 595 / 582 / 578 / 588 (584), bf16 1144 / 1084 / 1069 / 1063 / 1095 (1086), 13B batch 8 with fast annealing 522 / 505 / 504 / 502 / 508
// (570), with lazy layers 489 / 471 / 468 / 483 / 478 (474), 7B batch 4 146 / 143 / 142 / 157 / 155 (150), 8 layers of 12 heads, batch 32 133 / 133 / 131 / 132 /
// 151 (149), 32 layers of D = 64, batch 16 330 / 313 / 310 / 313 / 314 (314).  Float32 rows are twice as long for the same logit and go head by head; a share of
// 768 / 384 would gain them little: batch 8 of 16 heads, 8 layers 87.1 / 87.2 / 87.2, 32 layers 307 / 305 / 304, of D = 64, batch 16 318 / 309 / 308.
static int heads_together(int H, int64_t rows, int64_t behind) {
    int g = 8;
    while (g > 1 && (g > H || g * rows * 384 > behind)) g /= 2;
    return g;
}

// Attention of every layer of a checked step: the ordinary layers, as many per launch as its table holds, then the lazy ones, caches of
// either format in launches of their own (32 layers of the 7B shape, every other cache E4M3, us a step, layer by layer -> so:
// batch 1 377 -> 60, batch 8 482 -> 290).
// e[i] receives layer i's entry, for the launch behind them; needs: what is left for that launch; needs_apply[i] is cleared where
// it moves the layer's rows.  The ranking goes along with the attention when no layer's columns take its mass.  Returns ST3_ERR_UNSUPPORTED, with nothing enqueued, for a step that a table
// cannot describe.
st3_status enqueue_step_attend(const st3_attn_shape* shape, int n_layers, const st3_layer_step* layers, int mode,
                               const char* has_heirs, const EvictArgs* plan, char* needs_apply, StepCommon& common, StepLayer* e,
                               PlanNeeds& needs, hipStream_t st) {
    const int B = shape->batch, H = shape->heads, D = shape->head_dim;
    common = StepCommon{B, H, D, (int16_t)mode, (int16_t)elem_bytes(shape->dtype), scale_log2(shape), 0, 0, 0, 0, 0, {0, 0, 0, 0}};
    int64_t rows[2] = {0, 0};           // of the ordinary and of the lazy layers
    int as_long = 0, shorter = 0;       // layers in which most sequences hold as many rows as the bound says, by the hint, or may not
    for (int i = 0; i < n_layers; ++i) {
        const st3_layer_step& L = layers[i];
        const int64_t most32 = 0x7fffffff;
        if (L.kv.stride_t > most32 || L.col_stride < 0 || L.col_stride > most32 || L.mass_stride < 0 || L.mass_stride > most32)
            return ST3_ERR_UNSUPPORTED;
        rows[L.inherit_from >= 0] += L.seg.max_kv_len + 1;
        if (L.seg.max_vis_len > 0) (L.seg.vis_len_hint >= L.seg.max_vis_len ? as_long : shorter) += 1;
    }
    const bool alike = B == 1 || (as_long > 0 && shorter == 0);
    if (B > 65535) return ST3_ERR_UNSUPPORTED;
    std::vector<char> moves_here((size_t)n_layers, 0);
    std::vector<int> stage((size_t)n_layers, 0), groups[4];     // layers that may share launches, in launch order
    // (grid z is rank_z + B * layers, at most 65535)
    bool cut = false;                   // some ordinary layer's strips are
    needs = PlanNeeds{0, false, max_layers_ranked(B, H) > 0, 0};
    int most_ranked = 0, many_moves = 0;        // rows of a layer that evicts; layers that evict more rows than a plan moves by itself
    for (int i = 0; i < n_layers; ++i) {
        needs.most_vis = std::max(needs.most_vis, plan[i].max_vis);
        needs.apart = needs.apart && plan[i].mass_apart;
        if (plan[i].keep_count >= 0) most_ranked = std::max(most_ranked, plan[i].max_vis);
        many_moves += needs_apply[i];
    }
    needs.apart = needs.apart && rank_beside(most_ranked, H, (int64_t)B * H * n_layers, many_moves);
    for (int i = 0; i < n_layers; ++i) {
        const st3_layer_step& L = layers[i];
        const bool lazy = L.inherit_from >= 0, coded = L.kv.format == ST3_KV_E4M3;
        const int len = L.seg.max_kv_len + 1;
        const DecodeWs wl = decode_ws(B, H, D, L.kv.capacity);
        StepLayer& s = e[i];
        s = StepLayer{};
        s.v = L.kv.v; s.v_new = L.v_new; s.out = L.out;
        s.kv_len = L.seg.kv_len; s.vis_len = L.seg.vis_len; s.tail_start = L.seg.tail_start;
        s.score_col = L.score_col; s.id_col = L.id_col; s.mass = plan[i].mass_dst; s.ws = reinterpret_cast<char*>(L.workspace);
        if (coded) { s.k_scale = L.kv.k_scale; s.v_scale = L.kv.v_scale; }
        s.stride_b = L.kv.stride_b; s.stride_h = L.kv.stride_h; s.stride_t = (int32_t)L.kv.stride_t;
        s.col_stride = (int32_t)L.col_stride; s.mass_stride = (int32_t)L.mass_stride;
        s.sys_len = L.seg.sys_len; s.max_vis = L.seg.max_vis_len; s.max_kv = L.seg.max_kv_len;
        s.keep_count = plan[i].keep_count; s.capacity = L.kv.capacity;
        int nsplit = step_nsplit(B, H, len, rows[lazy], alike);
        if (nsplit > wl.nsplit_cap) nsplit = wl.nsplit_cap;
        s.chunk = decode_chunk(len, nsplit);
        nsplit = (len + s.chunk - 1) / s.chunk;
        s.nsplit = (uint8_t)nsplit; s.nsplit_cap = (uint8_t)wl.nsplit_cap;
        needs.merge = needs.merge || nsplit > 1;
        cut = cut || (!lazy && nsplit > 1);
        // Rows are moved by as many workgroups as they need, so however many an eviction moves, unless the order of the moves
        // matters (STABLE) or a strip's moves must stay together (a tail that closes up) and are many.  A launch of its own per
        // layer for more than 48 rows, as the other forms have it, before -> after, us a step: 7B shape evicting 50 rows a layer, batch 1
        // 106 -> 41, batch 8 301 -> 266, 3 layers 43 -> 19; high resolution batch 8 E4M3, 90 rows 559 -> 449.
        const bool moved = plan[i].inline_apply ||
                           (needs.apart && plan[i].keep_count >= 0 && mode == ST3_HOLE_FILL && L.seg.tail_start != nullptr);
        if (moved) needs.moves = std::max(needs.moves, (int64_t)(plan[i].max_vis - plan[i].keep_count) * 2 * H * plan[i].vecs_per_row);
        moves_here[(size_t)i] = moved;
        s.flags = (uint8_t)((moved ? kStepInlineApply : 0) | (coded ? kStepE4M3 : 0) | (needs.apart ? kStepApart : 0));
        if (lazy) {
            const st3_layer_step& S = layers[L.inherit_from];
            const DecodeWs sl = decode_ws(B, H, D, S.kv.capacity);
            if (L.workspace_bytes < wl.total || S.workspace_bytes < sl.total) return ST3_ERR_WORKSPACE_TOO_SMALL;
            if (len > S.kv.capacity) return ST3_ERR_INVALID_ARG;        // the source kept a logit per cached key
            s.q = S.workspace; s.hint_base = S.kv.capacity; s.src_nsplit_cap = (uint8_t)sl.nsplit_cap;
            s.k = L.kv.k;               // its rows move with an eviction when the layer caches keys after all
            s.flags |= kStepLazy;
        } else {
            s.q = L.q; s.k = L.kv.k; s.k_new = L.k_new;
            layout_hint(&L.seg, L.kv.capacity, s.hint_base, s.hint_gap);
            const bool want = L.vis_mass != nullptr && L.seg.max_vis_len > 0;
            if (want) s.flags |= kStepWantMass;
            if (has_heirs[i]) s.flags |= kStepKeepAll;
            if (has_heirs[i]) stage[(size_t)i] = s.chunk;
            else if (want) stage[(size_t)i] = std::min(s.chunk, L.seg.max_vis_len);
            if (stage[(size_t)i] > 3 * kLogitStageMaxRows) return ST3_ERR_UNSUPPORTED;
        }
        const int eb = kv_elem_bytes(shape, &L.kv);
        if (!step_layer_fits(s, eb)) common.wide = 1;
        if (!step_layer_fits(s, eb, true)) return ST3_ERR_UNSUPPORTED;
        groups[2 * lazy + coded].push_back(i);
    }
    if (!needs.apart && n_layers > entries_per_table(kPlanWords, common.wide)) {
        common.leave = 1;                               // (not where a workspace ends with what the decode calls need)
        for (int i = 0; i < n_layers; ++i)
            if (layers[i].workspace_bytes < decode_ws(B, H, D, layers[i].kv.capacity).total + kLeftBytes) common.leave = 0;
    }
    for (int i = 0; i < n_layers; ++i)                  // (from here on nothing is refused)
        if (moves_here[(size_t)i]) needs_apply[i] = 0;
    // (the builds that the diagnostic switch asks for have no groups)
    const bool whole = needs.apart && !common.wide && !cut && debug_state().attend_tile == 0;
    for (const std::vector<int>& members : groups) {
        const int n = (int)members.size();
        if (n == 0) continue;
        const bool coded = layers[members[0]].kv.format == ST3_KV_E4M3;
        const int words = coded ? kAttendWordsE4M3 : kAttendWords;
        const int per = std::min(entries_per_table(words, common.wide), needs.apart ? max_layers_ranked(B, H) : 65535 / B);
        const int launches = (n + per - 1) / per;
        for (int g = 0, i0 = 0; g < launches; ++g) {
            const int cnt = (n - i0 + launches - g - 1) / (launches - g);       // as equal as can be
            const int first = members[(size_t)i0];
            const bool lazy = layers[first].inherit_from >= 0;
            const st3_kv_layer* kv = &layers[first].kv;
            StepTable t;
            t.c = common; t.c.layers = cnt;
            if (whole && !lazy && kv_elem_bytes(shape, kv) <= 2) {
                int64_t behind = 0;                     // rows of the launch behind a layer
                for (int j = 0; j < cnt; ++j) behind += (int64_t)B * H * (e[members[(size_t)(i0 + j)]].max_kv + 1);
                int g = 8;
                for (int j = 0; j < cnt; ++j) {
                    StepLayer& s = e[members[(size_t)(i0 + j)]];
                    behind -= (int64_t)B * H * (s.max_kv + 1);
                    g = std::min(g, heads_together(H, s.max_kv + 1, behind));
                    if (g == 1) break;
                    t.c.groups[g == 8 ? 0 : g == 4 ? 1 : 2] += 1;
                    t.c.groups[3] = 1;
                    if ((s.flags & (kStepWantMass | kStepKeepAll)) != kStepWantMass || s.max_vis > kLogitStageMaxRows) continue;
                    s.flags |= kStepSums;
                    s.src_nsplit_cap = (uint8_t)g;
                    stage[(size_t)members[(size_t)(i0 + j)]] = 2 * s.max_vis;   // a head's logits and the sums
                }
            }
            int64_t written = (int64_t)cnt * B * H * D * (2 * kv_elem_bytes(shape, kv) + elem_bytes(shape->dtype));
            int most = 1, lds_words = 0, ranked = 0;    // dynamic LDS: the logits a workgroup collects, or the keys it ranks
            for (int j = 0; j < cnt; ++j) {
                const int i = members[(size_t)(i0 + j)];
                pack_attend(t.w + j * words, e[i], coded, kv_elem_bytes(shape, kv), common.wide ? high_words(t.w, j) : nullptr);
                most = std::max(most, (int)e[i].nsplit);
                lds_words = std::max(lds_words, stage[(size_t)i]);
                if (e[i].flags & kStepKeepAll) written += (int64_t)B * H * e[i].max_kv * sizeof(float);
                else if (e[i].flags & kStepWantMass) written += (int64_t)B * ((e[i].flags & kStepSums) ? (H + e[i].src_nsplit_cap - 1) / e[i].src_nsplit_cap : H) * e[i].max_vis * sizeof(float);
                if ((e[i].flags & kStepApart) && e[i].keep_count >= 0) { lds_words = std::max(lds_words, e[i].max_vis); ranked += 1; }
            }
            t.c.chunks = (int16_t)most;
            t.c.rank_z = ranked == 0 ? 0 : t.c.groups[3] ? B * cnt : rank_rows_z(B, H, most, cnt);
            if (lazy) ST3_DISPATCH_KV(launch_inherit_layers, shape, kv, t, lds_words, st);
            else ST3_DISPATCH_KV(launch_attend_layers, shape, kv, t, lds_words, written > kStreamStoreBytes, st);
            i0 += cnt;
        }
    }
    return check_launch();
}

}  // namespace st3

extern "C" st3_status st3_decode_attention(const st3_attn_shape* shape, const void* q, const st3_kv_layer* kv,
                                           const st3_segments* seg, void* out, float* vis_mass, int64_t mass_stride,
                                           void* workspace, size_t workspace_bytes, void* stream) {
    st3_status s = st3::check_shape(shape);
    if (s != ST3_OK) return s;
    s = st3::validate_kv(shape, kv, seg);
    if (s != ST3_OK) return s;
    if (!q || !out || !workspace) return ST3_ERR_INVALID_ARG;
    if (!st3::aligned16(q) || !st3::aligned16(workspace)) return ST3_ERR_INVALID_ARG;
    if (vis_mass && mass_stride < seg->max_vis_len) return ST3_ERR_INVALID_ARG;
    return st3::enqueue_decode(shape, q, kv, seg, seg->max_kv_len, nullptr, nullptr, out, vis_mass, mass_stride,
                               vis_mass != nullptr, false, true, workspace, workspace_bytes,
                               reinterpret_cast<hipStream_t>(stream));
}

extern "C" st3_status st3_decode_attention_inherit(const st3_attn_shape* shape, const st3_kv_layer* kv,
                                                   const st3_segments* seg, const void* src_workspace,
                                                   size_t src_workspace_bytes, int32_t src_kv_capacity, void* out,
                                                   void* workspace, size_t workspace_bytes, void* stream) {
    st3_status s = st3::check_shape(shape);
    if (s != ST3_OK) return s;
    s = st3::validate_kv_value_only(shape, kv, seg);
    if (s != ST3_OK) return s;
    if (!out || !workspace || !src_workspace || src_kv_capacity <= 0) return ST3_ERR_INVALID_ARG;
    if (!st3::aligned16(workspace) || !st3::aligned16(src_workspace)) return ST3_ERR_INVALID_ARG;
    return st3::enqueue_inherit(shape, kv, seg, seg->max_kv_len, nullptr, src_workspace, src_workspace_bytes,
                                src_kv_capacity, out, workspace, workspace_bytes, false,
                                reinterpret_cast<hipStream_t>(stream));
}

extern "C" st3_status st3_quantize_rows(const st3_attn_shape* shape, const st3_tensor4* src, const st3_kv_layer* kv,
                                        int32_t which, int32_t n, void* stream) {
    using namespace st3;
    st3_status s = check_shape(shape);
    if (s != ST3_OK) return s;
    if (!src || !src->data || !kv || (which != 0 && which != 1) || n < 0) return ST3_ERR_INVALID_ARG;
    if (kv->format != ST3_KV_PLAIN && kv->format != ST3_KV_E4M3) return ST3_ERR_INVALID_ARG;
    if (kv->format == ST3_KV_E4M3 && shape->dtype != ST3_BF16) return ST3_ERR_UNSUPPORTED;
    void* dst = which == 0 ? kv->k : kv->v;
    const float* scale = kv->format == ST3_KV_E4M3 ? (which == 0 ? kv->k_scale : kv->v_scale) : nullptr;
    if (!dst || (kv->format == ST3_KV_E4M3 && !scale) || n > kv->capacity) return ST3_ERR_INVALID_ARG;
    const int eb = elem_bytes(shape->dtype), ceb = kv_elem_bytes(shape, kv);
    if (!aligned16(src->data) || !aligned16(dst)) return ST3_ERR_INVALID_ARG;
    if ((src->stride_t * eb) % 16 || (src->stride_h * eb) % 16 || (src->stride_b * eb) % 16) return ST3_ERR_INVALID_ARG;
    if ((kv->stride_t * ceb) % 16 || (kv->stride_h * ceb) % 16 || (kv->stride_b * ceb) % 16) return ST3_ERR_INVALID_ARG;
    if (src->stride_t < shape->head_dim || kv->stride_t < shape->head_dim) return ST3_ERR_INVALID_ARG;
    if (n == 0) return ST3_OK;
    QuantArgs qa{};
    qa.src = src->data; qa.s_sb = src->stride_b; qa.s_sh = src->stride_h; qa.s_st = src->stride_t;
    qa.dst = dst; qa.d_sb = kv->stride_b; qa.d_sh = kv->stride_h; qa.d_st = kv->stride_t;
    qa.scale = scale; qa.H = shape->heads; qa.n = n;
    ST3_DISPATCH_KV(launch_quantize, shape, kv, qa, shape->batch, reinterpret_cast<hipStream_t>(stream));
    return check_launch();
}

extern "C" st3_status st3_kv_append(const st3_attn_shape* shape, const st3_kv_layer* kv, const st3_segments* seg,
                                    const void* k_new, const void* v_new, void* stream) {
    st3_status s = st3::check_shape(shape);
    if (s != ST3_OK) return s;
    // a layer that caches V only (lazy layer of Alg. 2) passes kv->k == NULL and k_new == NULL
    const bool value_only = kv && !kv->k && !k_new;
    s = value_only ? st3::validate_kv_value_only(shape, kv, seg) : st3::validate_kv(shape, kv, seg);
    if (s != ST3_OK) return s;
    if ((!value_only && (!k_new || !st3::aligned16(k_new))) || !v_new || !st3::aligned16(v_new))
        return ST3_ERR_INVALID_ARG;
    if (seg->max_kv_len >= kv->capacity) return ST3_ERR_INVALID_ARG;
    return st3::enqueue_append(shape, kv, seg, k_new, v_new, reinterpret_cast<hipStream_t>(stream));
}
