// Top-k selection of visual tokens by attention mass (Eq. 3), the in-place compaction of rows
// that follows it (Alg. 1/3: V = V[T]), and the per-layer, per-step eviction of visual KV rows
// (Eq. 7, Alg. 3 VTA branch).
//
// Selection is an exact radix select on the order-preserving 32-bit image of the float32 score
// (8 bits a pass, at most four, histograms in LDS), followed - only when the k-th score is shared -
// by a second radix select on the tie ids, so that the result is the unique top-k set under the
// total order (score descending, id ascending).  One workgroup per sequence.
#include <algorithm>

#include "st3_evict.h"

namespace st3 {

namespace {

// ---------------------------------------------------------------------------------------------
// st3_select_topk
// ---------------------------------------------------------------------------------------------
struct TopkArgs {
    const float* scores;
    int64_t score_stride;
    const int32_t* ids;
    int64_t id_stride;
    const int32_t* n_dev;
    int32_t n, k;
    uint8_t* mask;
    int32_t* idx;
    int64_t idx_stride;
    float* out_scores;      // the kept entries themselves, in ascending order of position (null: not wanted)
    int64_t out_score_stride;
    int32_t* out_ids;
    int64_t out_id_stride;
};

// One workgroup per row, latency bound (topk_threads).  COLUMNS: the kept entries are wanted, else the mask and the positions.  (In
// one kernel their arguments took it to more than 80 scalar registers, with which no two workgroups of 1024 threads fit a compute
// unit: 512 rows of 8192 scores 32.4 us instead of 24.3.)
template <int NT, bool COLUMNS>
__global__ __launch_bounds__(NT) void select_topk_kernel(TopkArgs a) {
    __shared__ SelectShared sm;
    const int b = blockIdx.x, tid = threadIdx.x;
    uint32_t* keys = sel_keys();
    int n = a.n_dev ? a.n_dev[b] : a.n;
    n = max(0, min(n, a.n));
    const int k = min(a.k, n);
    const float* scores = a.scores + b * a.score_stride;
    const int32_t* ids = a.ids ? a.ids + b * a.id_stride : nullptr;
    uint8_t* mask = !COLUMNS && a.mask ? a.mask + (int64_t)b * a.n : nullptr;
    int32_t* idx = !COLUMNS && a.idx ? a.idx + (int64_t)b * a.idx_stride : nullptr;
    const bool staged = n <= kSelLdsKeys;
    auto key_at = [&](int i) -> uint32_t { return staged ? keys[i] : score_key(scores[i]); };
    auto idkey_at = [&](int i) { return ~(uint32_t)(ids ? ids[i] : i); };
    TopSet top{0, 0, true};
    if (k > 0 && k < n) {
        if (staged)
            for (int i = tid; i < n; i += NT) keys[i] = score_key(scores[i]);
        top = top_set<NT>(key_at, idkey_at, n, k, sm);
    }
    int base = 0, parity = 0, r1, r2, t1, t2;
    const int n_pad = (a.n + NT - 1) / NT * NT;
    for (int p0 = 0; p0 < n_pad; p0 += NT, parity ^= 1) {
        const int p = p0 + tid;
        const bool keep = p < n && (k >= n || (k > 0 && top.keeps(key_at, idkey_at, p)));
        if (mask && p < a.n) mask[p] = keep ? 1 : 0;
        plan_ranks<NT>(keep, false, parity, sm, r1, r2, t1, t2);
        if (keep && base + r1 < a.k) {
            if (idx) idx[base + r1] = p;
            if (COLUMNS) {
                a.out_ids[b * a.out_id_stride + base + r1] = ids[p];
                a.out_scores[b * a.out_score_stride + base + r1] = scores[p];
            }
        }
        base += t1;
    }
    if (idx) for (int i = k + tid; i < a.k; i += NT) idx[i] = -1;
}

void launch_topk(const TopkArgs& a, int batch, hipStream_t st) {
    with_threads(topk_threads(batch, a.n), [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        const size_t lds = sizeof(uint32_t) * std::min(a.n, kSelLdsKeys);
        if (a.out_ids) select_topk_kernel<NT, true><<<batch, NT, lds, st>>>(a);
        else select_topk_kernel<NT, false><<<batch, NT, lds, st>>>(a);
    });
}

// ---------------------------------------------------------------------------------------------
// st3_compact_rows: stable in-place gather.  grid (slabs, inner, batch).
// Destination rows are produced in ascending chunks; a chunk is loaded completely before any of
// it is stored, and since keep_idx is ascending with keep_idx[r] >= r no later chunk reads a row
// an earlier chunk has overwritten.
// ---------------------------------------------------------------------------------------------
struct CompactArgs {
    char* rows;
    int64_t stride_b, stride_inner, stride_row;     // bytes
    int32_t row_units, slab_units, unit_bytes;      // a unit is 16 or 4 bytes
    const int32_t* idx;
    int64_t idx_stride;
    int32_t k, n, tail;
};
constexpr int kCompactUR = 4;       // rows a thread moves in a pass

template <typename V>
__global__ __launch_bounds__(256) void compact_rows_kernel(CompactArgs a) {
    constexpr int UR = kCompactUR;
    __shared__ int sm_kb;
    __shared__ int sm_cnt[4];
    const int tid = threadIdx.x, b = blockIdx.z;
    const int32_t* idx = a.idx + (int64_t)b * a.idx_stride;
    // length of the leading run of valid indices (0 <= idx < n): position of the first invalid entry
    int local = a.k;
    for (int i = tid; i < a.k; i += 256)
        if (idx[i] < 0 || idx[i] >= a.n) { local = i; break; }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) local = min(local, __shfl_xor(local, off));
    if (tid % kWave == 0) sm_cnt[tid / kWave] = local;
    __syncthreads();
    if (tid == 0) sm_kb = min(min(sm_cnt[0], sm_cnt[1]), min(sm_cnt[2], sm_cnt[3]));
    __syncthreads();
    const int kb = sm_kb;
    const int total = kb + a.tail;
    char* strip = a.rows + b * a.stride_b + (int64_t)blockIdx.y * a.stride_inner;
    const int rows_per_pass = 256 / a.slab_units;
    const int rr = tid / a.slab_units;
    const int cu = blockIdx.x * a.slab_units + tid % a.slab_units;
    const bool col_ok = cu < a.row_units;
    for (int r0 = 0; r0 < total; r0 += UR * rows_per_pass) {
        V tmp[UR];
        int dst[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            int r = r0 + u * rows_per_pass + rr;
            dst[u] = -1;
            if (r < total && col_ok) {
                int src = r < kb ? idx[r] : a.n + (r - kb);
                if (src > r && src < a.n + a.tail) {     // src == r: already in place
                    tmp[u] = *reinterpret_cast<const V*>(strip + src * a.stride_row + (int64_t)cu * sizeof(V));
                    dst[u] = r;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < UR; ++u)
            if (dst[u] >= 0) *reinterpret_cast<V*>(strip + dst[u] * a.stride_row + (int64_t)cu * sizeof(V)) = tmp[u];
        __syncthreads();
    }
}

// The same where no tail follows and the rows are one pass of a workgroup (columns of ids and scores).  Such a call is one chain of
// memory trips: indices for the length of the valid run, indices again, rows.  Here a thread keeps the indices it has looked at
// and loads its rows beside the reduction; a row behind the first invalid index is loaded for nothing and not stored.
// us a launch, three trips -> one: 8 columns of 365 entries to 350 2.8 -> 2.6, 4 of 2000 to 1500 4.3 -> 2.9, 8 of 2880 to 2800 6.3 -> 3.1;
// 200 of 220 rows of 256 bytes, 32 strips 10.0 -> 7.2; 16 of 40 rows of 8 KB, 8 strips 9.2 -> 5.9.
template <typename V, int NT>
__global__ __launch_bounds__(NT) void compact_short_kernel(CompactArgs a) {
    __shared__ int sm_first[NT / kWave];
    const int tid = threadIdx.x, b = blockIdx.z;
    const int32_t* idx = a.idx + (int64_t)b * a.idx_stride;
    char* strip = a.rows + b * a.stride_b + (int64_t)blockIdx.y * a.stride_inner;
    const int rows_per_pass = NT / a.slab_units, rr = tid / a.slab_units;
    const int cu = blockIdx.x * a.slab_units + tid % a.slab_units;
    V tmp[kCompactUR];
    int src[kCompactUR];
#pragma unroll
    for (int u = 0; u < kCompactUR; ++u) {
        const int r = u * rows_per_pass + rr;
        src[u] = r < a.k ? idx[r] : 0;
    }
    int first = a.k;                                    // position of the first invalid index
#pragma unroll
    for (int u = 0; u < kCompactUR; ++u) {
        const int r = u * rows_per_pass + rr;
        const bool valid = src[u] >= 0 && src[u] < a.n;
        if (r < a.k && !valid) first = min(first, r);
        if (!valid || src[u] <= r || cu >= a.row_units || r >= a.k) src[u] = -1;       // src == r: already in place
        else tmp[u] = *reinterpret_cast<const V*>(strip + src[u] * a.stride_row + (int64_t)cu * sizeof(V));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) first = min(first, __shfl_xor(first, off));
    if (tid % kWave == 0) sm_first[tid / kWave] = first;
    __syncthreads();                                    // (all rows have been loaded, too)
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) first = min(first, sm_first[w]);
#pragma unroll
    for (int u = 0; u < kCompactUR; ++u) {
        const int r = u * rows_per_pass + rr;
        if (src[u] >= 0 && r < first) *reinterpret_cast<V*>(strip + r * a.stride_row + (int64_t)cu * sizeof(V)) = tmp[u];
    }
}

template <typename V>
void launch_compact(const CompactArgs& a, int inner, int batch, hipStream_t st) {
    const dim3 grid((a.row_units + a.slab_units - 1) / a.slab_units, inner, batch);
    const int64_t slots = (int64_t)a.k * a.slab_units;  // of a workgroup's pass
    if (a.tail == 0 && slots <= kCompactUR * 256) compact_short_kernel<V, 256><<<grid, 256, 0, st>>>(a);
    else if (a.tail == 0 && slots <= kCompactUR * 1024) compact_short_kernel<V, 1024><<<grid, 1024, 0, st>>>(a);
    else compact_rows_kernel<V><<<grid, 256, 0, st>>>(a);
}

// ---------------------------------------------------------------------------------------------
// Decode-time eviction: ranking + move list + column update (one workgroup per sequence), then
// a second kernel that applies the move list to every (b,h) strip of K and V.
// ---------------------------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(NT) void evict_plan_kernel(EvictArgs a) {
    __shared__ PlanShared sm;
    evict_plan_body<NT>(a, blockIdx.x, sm);
}

// ---- st3_gather_rows: out-of-place gather of kept rows, several tensors per launch -------------
struct GatherArgs {
    st3_gather_pair pair[ST3_MAX_GATHER];
    const int32_t* idx;
    int64_t idx_stride;
    int32_t n_pairs, vecs_per_row, vpr_shift, head, k, n, tail;     // vpr_shift >= 0: vecs_per_row == 1 << vpr_shift
};

// grid (ceil(rows*vecs_per_row / (256*UR)), inner, batch*n_pairs); a thread moves UR 16-byte vectors.
#ifndef ST3_GATHER_UR
// Bound by HBM.  Two vectors a thread: workgroups in flight at the same time then touch addresses close to each other.
// us at 1 / 2 / 3 / 4 / 8, three tensors of bf16 d = 128: 32 heads x batch 4, 527 of 671 rows 21.4 / 21.1 / 21.7 / 22.9 / 37.2;
// 40 x 8, 395 rows 37.5 / 37.1 / 37.9 / 39.7 / 74.7 (194 MB read and written at 5.2 TB/s, the launch itself included); 40 x 32,
// 527 rows 174 / 167 / 167 / 176 / 302 (1.04 GB, 6.2 TB/s).
// The index lookups of a thread's vectors taken together before its loads change nothing.
#define ST3_GATHER_UR 2
#endif
#ifndef ST3_GATHER_NT
#define ST3_GATHER_NT 1
#endif
constexpr int kGatherUR = ST3_GATHER_UR;
// Written bytes above which the rows go past the caches.  The launch itself is 8 % faster so from 128 MB on, but what reads the
// rows next (the layer's attention) finds most of them in the last-level cache (256 MB) after ordinary stores, up to somewhat
// beyond its size.  us, ordinary -> non-temporal stores, gather alone and gather + one read of its output, buffers in rotation:
// 123 MB written 47.6 -> 43.7, 94 -> 99; 185 MB 70 -> 64, 126 -> 128; 247 MB 92 -> 85, 152 -> 158; 370 MB 138 -> 126, 232 -> 219;
// 432 MB 158 -> 146, 270 -> 248.  So for this reader the sides cross between 250 and 370 MB; the line lies beyond that, where the launch alone
// gains most and no reader was seen to lose.  At 300 MB whole prefills would gain little: 13B batch 28 10.32 -> 10.23 ms, batch 32 11.79 ->
// 11.75, batch 36 13.2 -> 13.0.
constexpr int64_t kGatherStreamBytes = (int64_t)400 << 20;
template <bool NTS>        // NTS: non-temporal stores
__global__ __launch_bounds__(256) void gather_rows_kernel(GatherArgs a) {
    constexpr int UR = kGatherUR;
    const int p = blockIdx.z % a.n_pairs, b = blockIdx.z / a.n_pairs;
    const st3_gather_pair& pr = a.pair[p];
    const char* src = reinterpret_cast<const char*>(pr.src) + b * pr.src_stride_b + (int64_t)blockIdx.y * pr.src_stride_inner;
    char* dst = reinterpret_cast<char*>(pr.dst) + b * pr.dst_stride_b + (int64_t)blockIdx.y * pr.dst_stride_inner;
    const int32_t* idx = a.idx ? a.idx + (int64_t)b * a.idx_stride : nullptr;
    const int rows = a.head + a.k + a.tail;
    const uint32_t total = (uint32_t)rows * (uint32_t)a.vecs_per_row;      // < 2^31, checked on the host
    const uint32_t base = blockIdx.x * (256u * UR) + threadIdx.x;
    u32x4_v tmp[UR];
    int64_t doff[UR];
#pragma unroll
    for (int u = 0; u < UR; ++u) {
        const uint32_t e = base + (uint32_t)u * 256u;
        doff[u] = -1;
        if (e < total) {
            // 32-bit index arithmetic, a shift when the row is a power of two vectors long: a 64-bit
            // division per 16 bytes moved made this kernel ALU bound
            const int r = a.vpr_shift >= 0 ? (int)(e >> a.vpr_shift) : (int)(e / (uint32_t)a.vecs_per_row);
            const int vec = (int)(e - (uint32_t)r * (uint32_t)a.vecs_per_row);
            int sr;
            if (r < a.head) sr = r;
            else if (r < a.head + a.k) {
                const int j = idx ? idx[r - a.head] : r - a.head;
                sr = (j >= 0 && j < a.n) ? a.head + j : -1;
            } else sr = r - a.k + a.n;
            if (sr >= 0) {
#if ST3_GATHER_NT
                tmp[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_v*>(src + sr * pr.src_stride_row + (int64_t)vec * 16));
#else
                tmp[u] = *reinterpret_cast<const u32x4_v*>(src + sr * pr.src_stride_row + (int64_t)vec * 16);
#endif
                doff[u] = r * pr.dst_stride_row + (int64_t)vec * 16;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < UR; ++u)
        if (doff[u] >= 0) {
            if (NTS) __builtin_nontemporal_store(tmp[u], reinterpret_cast<u32x4_v*>(dst + doff[u]));
            else *reinterpret_cast<u32x4_v*>(dst + doff[u]) = tmp[u];
        }
}

struct ApplyArgs {
    char* k;
    char* v;
    int64_t stride_b, stride_h, stride_t;   // bytes
    const int32_t* move_cnt;
    const int32_t* moves;
    int32_t max_moves, H, vecs_per_row;
    int32_t vecs_per_part;      // 16-byte vectors of a row that one workgroup moves (vecs_per_row / gridDim.z)
};

// grid (2*H, B, parts): x < H moves K rows of head x, x >= H moves V rows of head x-H; z picks the
// columns [z * vecs_per_part, (z+1) * vecs_per_part) of every row.  The parts of a strip share
// nothing - each applies the whole list, in order, to its own columns - so when the strips are few
// each is moved by two workgroups, half a row per workgroup.
// Moves are applied in list order in chunks; a chunk is loaded completely before it is stored.
// The plan kernel orders the list so that no move reads a row that an earlier chunk has written
// unless that is the intended (already shifted) content.
#ifndef ST3_APPLY_UR
#define ST3_APPLY_UR 16     // 4 -> 16: 4.1 -> 4.8 TB/s read+write (plan launch included) for a stable eviction of 288 rows
#endif
__global__ __launch_bounds__(256) void evict_apply_kernel(ApplyArgs a) {
    constexpr int UR = ST3_APPLY_UR;        // 16-byte loads in flight per thread: a chunk is UR * 256 * 16 bytes
    const int b = blockIdx.y, tid = threadIdx.x;
    const int M = min(a.move_cnt[b], a.max_moves);
    if (M <= 0) return;
    if ((int)blockIdx.x < a.H && a.k == nullptr) return;    // a layer that caches V only
    const int h = blockIdx.x % a.H;
    char* strip = (blockIdx.x < a.H ? a.k : a.v) + b * a.stride_b + h * a.stride_h;
    const int32_t* mv = a.moves + (int64_t)b * a.max_moves * 2;
    const int rpp = 256 / a.vecs_per_part;
    const int rr = tid / a.vecs_per_part;
    const int64_t cb = (int64_t)((int)blockIdx.z * a.vecs_per_part + tid % a.vecs_per_part) * 16;
    for (int c0 = 0; c0 < M; c0 += UR * rpp) {
        u32x4_v tmp[UR];
        int dst[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            int i = c0 + u * rpp + rr;
            dst[u] = -1;
            if (i < M) {
                dst[u] = mv[2 * i];
                // every row is read once and written once: keep it out of the way of the caches' other tenants
                tmp[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_v*>(strip + mv[2 * i + 1] * a.stride_t + cb));
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < UR; ++u)
            if (dst[u] >= 0) *reinterpret_cast<u32x4_v*>(strip + dst[u] * a.stride_t + cb) = tmp[u];
        __syncthreads();
    }
}

}  // namespace

st3_status validate_kv(const st3_attn_shape* s, const st3_kv_layer* kv, const st3_segments* seg);
st3_status validate_kv_value_only(const st3_attn_shape* s, const st3_kv_layer* kv, const st3_segments* seg);

// Rows are moved inside the plan kernel when the mode is HOLE_FILL and few rows can be evicted per
// sequence; larger evictions and STABLE mode go through evict_apply_kernel, which has a workgroup
// per strip but is a launch of its own per layer.  A plan workgroup moves a row on all 2*H strips in
// about 2 us (measured, H = 40, bf16 d = 128), a plan + apply pair costs about 10 us more than a plan
// alone: so up to 48 evicted rows stay in the plan when the plans of many layers share a launch
// (the apply launches they save are per layer), and only a handful when a layer is planned alone
// (each evicted row is one move with a fixed tail, two without).
constexpr int kInlineEvictBatched = 48;
constexpr int kInlineEvictAloneFixedTail = 8;
constexpr int kInlineEvictAlone = 4;

// Whether the mass of this step may land in what the eviction ranks by, or moves (mode "current" writes it into the score column).
static bool columns_take_mass(const EvictArgs& ea, int B) {
    if (ea.mass_dst == nullptr || ea.keep_count < 0) return false;
    const uintptr_t bytes = sizeof(float);
    const uintptr_t m0 = reinterpret_cast<uintptr_t>(ea.mass_dst), m1 = m0 + ((uintptr_t)(B - 1) * ea.mass_stride + ea.max_vis) * bytes;
    const uintptr_t span = ((uintptr_t)(B - 1) * ea.col_stride + ea.max_vis) * bytes;
    for (const void* col : {(const void*)ea.score_col, (const void*)ea.id_col}) {
        const uintptr_t c0 = reinterpret_cast<uintptr_t>(col);
        if (m0 < c0 + span && c0 < m1) return true;
    }
    return false;
}

st3_status build_evict_args(const st3_attn_shape* shape, const st3_kv_layer* kv, const st3_segments* seg,
                            float* score_col, int32_t* id_col, int64_t col_stride, int32_t keep_count, int32_t mode,
                            void* workspace, size_t workspace_bytes, int appended, float* mass_dst,
                            int64_t mass_stride, EvictArgs& ea, bool& needs_apply, bool batched,
                            const void* mass_workspace, int32_t mass_capacity) {
    const int B = shape->batch, H = shape->heads, D = shape->head_dim;
    if (seg->max_vis_len > kSelLdsKeys) return ST3_ERR_UNSUPPORTED;
    const DecodeWs wl = decode_ws(B, H, D, kv->capacity);
    if (workspace_bytes < wl.total) return ST3_ERR_WORKSPACE_TOO_SMALL;
    char* ws = reinterpret_cast<char*>(workspace);
    const int eb = kv_elem_bytes(shape, kv);
    const bool evicting = keep_count >= 0 && keep_count < seg->max_vis_len;
    ea = EvictArgs{};
    ea.score_col = score_col; ea.id_col = id_col; ea.col_stride = col_stride;
    ea.vis_len = seg->vis_len; ea.kv_len = seg->kv_len; ea.tail_start = seg->tail_start;
    ea.sys_len = seg->sys_len; ea.max_vis = seg->max_vis_len; ea.max_kv = seg->max_kv_len;
    ea.keep_count = evicting ? keep_count : -1; ea.mode = mode;
    ea.move_cnt = reinterpret_cast<int32_t*>(ws + wl.moves_cnt);
    ea.moves = reinterpret_cast<int32_t*>(ws + wl.moves);
    ea.max_moves = wl.max_moves;
    ea.appended = appended; ea.capacity = kv->capacity;
    const int inline_limit = batched ? kInlineEvictBatched
                                     : (seg->tail_start != nullptr ? kInlineEvictAloneFixedTail : kInlineEvictAlone);
    ea.inline_apply = evicting && mode == ST3_HOLE_FILL && (seg->max_vis_len - keep_count) <= inline_limit;
    ea.k = reinterpret_cast<char*>(kv->k); ea.v = reinterpret_cast<char*>(kv->v);
    ea.stride_b = kv->stride_b * eb; ea.stride_h = kv->stride_h * eb; ea.stride_t = kv->stride_t * eb;
    ea.H = H; ea.vecs_per_row = D * eb / 16;
    if (mass_dst != nullptr) {
        const char* mws = mass_workspace ? reinterpret_cast<const char*>(mass_workspace) : ws;
        const DecodeWs ml = mass_workspace ? decode_ws(B, H, D, mass_capacity) : wl;
        ea.part_ml = reinterpret_cast<const float*>(mws + ml.part_ml);
        ea.logits = reinterpret_cast<const float*>(mws + ml.logits);
        ea.pending = reinterpret_cast<const int32_t*>(mws + ml.pending);
        ea.nsplit_cap = ml.nsplit_cap;
        if (mass_workspace) ea.capacity = mass_capacity;
        ea.mass_dst = mass_dst; ea.mass_stride = mass_stride;
    }
    ea.own_pending = reinterpret_cast<const int32_t*>(ws + wl.pending);
    ea.mass_apart = batched && !columns_take_mass(ea, B);
    needs_apply = evicting && !ea.inline_apply;
    return ST3_OK;
}

void launch_evict_plan(const EvictArgs& ea, int B, hipStream_t st) {
    with_threads(plan_threads(B, ea.max_vis, ea.mass_dst != nullptr ? ea.H : 1), [&](auto nt) {
        constexpr int NT = decltype(nt)::value;
        evict_plan_kernel<NT><<<B, NT, plan_lds(ea.max_vis, NT), st>>>(ea);
    });
}

// Up to kPlanBatch plans travel by value in the kernel arguments; grid (B, layers of the batch).
struct EvictBatch {
    EvictArgs layer[kPlanBatch];
};
static_assert(sizeof(EvictBatch) <= 4000, "plans of one batch must fit the kernel argument segment");

// grid (B, layers of the batch, 1 + mass workgroups): z = 0 runs the plan, z >= 1 finish kMassKeys entries of the mass each where
// the plan need not wait for them.
template <int NT>
__global__ __launch_bounds__(NT) void evict_plan_batch_kernel(EvictBatch batch) {
    __shared__ union { PlanShared plan; MassShared<NT> mass; } sm;
    const EvictArgs& a = batch.layer[blockIdx.y];
    if (blockIdx.z == 0) evict_plan_body<NT>(a, blockIdx.x, sm.plan);
    else if (a.mass_apart && a.mass_dst != nullptr) mass_block<NT>(a, blockIdx.x, ((int)blockIdx.z - 1) * kMassKeys, sm.mass);
}

void launch_evict_plan_batch(const EvictArgs* plans, int n, int B, hipStream_t st) {
    for (int i0 = 0; i0 < n; i0 += kPlanBatch) {
        const int cnt = n - i0 < kPlanBatch ? n - i0 : kPlanBatch;
        EvictBatch batch;
        int most_vis = 0, apart_vis = 0;
        bool mass_in_plan = false;
        for (int i = 0; i < cnt; ++i) {
            const EvictArgs& p = plans[i0 + i];
            batch.layer[i] = p;
            most_vis = std::max(most_vis, p.max_vis);
            if (p.mass_apart && p.mass_dst != nullptr) apart_vis = std::max(apart_vis, p.max_vis);
            mass_in_plan = mass_in_plan || !p.mass_apart;
        }
        for (int i = cnt; i < kPlanBatch; ++i) batch.layer[i] = EvictArgs{};
        const dim3 grid(B, cnt, 1 + (apart_vis + kMassKeys - 1) / kMassKeys);
        with_threads(plan_threads((int64_t)B * cnt, most_vis, mass_in_plan ? plans[i0].H : 1), [&](auto nt) {
            constexpr int NT = decltype(nt)::value;
            evict_plan_batch_kernel<NT><<<grid, NT, plan_lds(most_vis, NT), st>>>(batch);
        });
    }
}

constexpr int kMergeHeads = 8;      // heads whose chunk partials one merge workgroup of the plan launch combines
// ... and of the finish launch: an output for each of its 256 threads, who take their chunks' partials in rounds of loads.  (Eight
// heads, four outputs one after the other for each thread -> so, us a step of one layer of 8 heads: 1024 visual rows, 17 chunks 26.1 -> 18.3,
// 2048 rows, 33 chunks 24.5 -> 13.2, 4096 rows, 64 chunks 26.7 -> 15.3; 32 heads, 100 rows, 2 chunks 11.7 -> 10.5.)
inline __host__ __device__ int finish_merge_heads(int D) { return D == 64 ? 4 : 2; }

// grid (B, layers, 1 + merge workgroups): z = 0 runs the plan of (sequence x, layer y); z >= 1 merges the chunk partials
// of that layer's attention output for kMergeHeads heads (only launched when some layer left partials to merge).
// FORM: entries of the table, wide entries, or the entries that the attention has left in the layers' workspaces.
enum { kFormTable, kFormWide, kFormLeft };
template <int NT, int FORM>
__global__ __launch_bounds__(NT) void evict_plan_table_kernel(StepTable t) {
    __shared__ PlanShared sm;
    const StepLayer e = FORM == kFormLeft
        ? unpack_left(t.w + blockIdx.y * kLeftWords, t.c.elem_bytes, t.c.wide != 0)
        : unpack_plan<true>(t.w + blockIdx.y * kPlanWords, t.c.elem_bytes, high_words(t.w, blockIdx.y), FORM == kFormWide);
    if (blockIdx.z == 0) {
        EvictArgs a = plan_from_entry(t.c, e);
        a.mass_apart = 0;
        evict_plan_body<NT>(a, blockIdx.x, sm);
    } else if (e.nsplit > 1) {
        const int h0 = ((int)blockIdx.z - 1) * kMergeHeads;
        if (h0 < t.c.H) merge_chunks(t.c, e, blockIdx.x, h0, h0 + kMergeHeads);
    }
}

// What is left of the plans when the rows have been ranked beside the attention.  grid (B, layers, moves + masses + merges), 256
// threads: workgroups z < move_wgs move rows (the first one advances the lengths too), the next mass_wgs finish kMassKeys
// entries of the mass each, the rest merge the chunk partials of finish_merge_heads heads each.
template <bool WIDE>
__global__ __launch_bounds__(256) void step_finish_kernel(StepTable t, int move_wgs, int mass_wgs) {
    __shared__ MassShared<256> sm;
    const StepLayer e = unpack_plan<false>(t.w + blockIdx.y * kFinishWords, t.c.elem_bytes, high_words(t.w, blockIdx.y), WIDE);
    const int z = blockIdx.z, b = blockIdx.x;
    if (z < move_wgs + mass_wgs) {
        const EvictArgs a = plan_from_entry(t.c, e);
        if (z >= move_wgs) {
            const int j0 = (z - move_wgs) * kMassKeys;
            if (a.mass_dst == nullptr) return;
            if (e.flags & kStepSums) mass_sums_block<256>(a, b, j0, (t.c.H + e.src_nsplit_cap - 1) / e.src_nsplit_cap, e.src_nsplit_cap, sm);
            else mass_block<256>(a, b, j0, sm);
            return;
        }
        if (z == 0 && threadIdx.x == 0) evict_publish(a, b, evict_counts(a, b));
        if (a.inline_apply) move_rows_block<256>(a, b, z, move_wgs);
    } else if (e.nsplit > 1) {
        const int heads = finish_merge_heads(t.c.D), h0 = (z - move_wgs - mass_wgs) * heads;
        if (h0 < t.c.H) merge_chunks(t.c, e, b, h0, h0 + heads);
    }
}

// Workgroups that move rows, over all plans of a launch.  us a step at 512 / 1024 / 2048 / 4096: 7B batch 1 54.4 / 55.0 / 55.0 / 55.9,
// 13B batch 8 with fast annealing 533 / 507 / 504 / 503, batch 32 2403 / 2408 / 2402 / 2403, high resolution batch 8 630 / 628 / 628 / 627.
constexpr int kFinishMoveWgs = 2048;
void launch_evict_plan_table(const StepCommon& c, const StepLayer* entry, int n, const PlanNeeds& needs, hipStream_t st) {
    const int words = c.leave ? kLeftWords : needs.apart ? kFinishWords : kPlanWords, per = entries_per_table(words, c.wide && !c.leave);
    const int launches = (n + per - 1) / per;
    for (int g = 0, i0 = 0; g < launches; ++g) {
        const int cnt = (n - i0 + launches - g - 1) / (launches - g);       // as equal as can be
        StepTable t;
        t.c = c; t.c.layers = cnt;
        for (int i = 0; i < cnt; ++i) {
            const StepLayer& e = entry[i0 + i];
            if (c.leave) pack_left(t.w + i * words, e, e.ws + decode_ws(c.B, c.H, c.D, e.capacity).total);
            else pack_plan(t.w + i * words, e, !needs.apart, (e.flags & kStepE4M3) ? 1 : c.elem_bytes, c.wide ? high_words(t.w, i) : nullptr);
        }
        i0 += cnt;
        const int merge_heads = needs.apart ? finish_merge_heads(c.D) : kMergeHeads;
        const int merge_wgs = needs.merge ? (c.H + merge_heads - 1) / merge_heads : 0;
        const int64_t plans = (int64_t)c.B * cnt;
        if (needs.apart) {
            // (a round of a workgroup's loads: eight of 16 bytes for each thread)
            const int64_t rounds = (needs.moves + 8 * 256 - 1) / (8 * 256), strips = 2 * c.H * (c.D * c.elem_bytes / 16) / 256;
            const int move_wgs = (int)std::max<int64_t>(1, std::min<int64_t>(std::max(rounds, strips), kFinishMoveWgs / plans));
            const int mass_wgs = (needs.most_vis + kMassKeys - 1) / kMassKeys;
            const dim3 grid(c.B, cnt, move_wgs + mass_wgs + merge_wgs);
            if (c.wide) step_finish_kernel<true><<<grid, 256, 0, st>>>(t, move_wgs, mass_wgs);
            else step_finish_kernel<false><<<grid, 256, 0, st>>>(t, move_wgs, mass_wgs);
        } else {
            const dim3 grid(c.B, cnt, 1 + merge_wgs);
            with_threads(plan_threads(plans, needs.most_vis, c.H), [&](auto nt) {
                constexpr int NT = decltype(nt)::value;
                const size_t lds = plan_lds(needs.most_vis, NT);
                if (c.leave) evict_plan_table_kernel<NT, kFormLeft><<<grid, NT, lds, st>>>(t);
                else if (c.wide) evict_plan_table_kernel<NT, kFormWide><<<grid, NT, lds, st>>>(t);
                else evict_plan_table_kernel<NT, kFormTable><<<grid, NT, lds, st>>>(t);
            });
        }
    }
}

void launch_evict_apply(const EvictArgs& ea, int B, hipStream_t st) {
    ApplyArgs aa{};
    aa.k = ea.k; aa.v = ea.v;
    aa.stride_b = ea.stride_b; aa.stride_h = ea.stride_h; aa.stride_t = ea.stride_t;
    aa.move_cnt = ea.move_cnt; aa.moves = ea.moves; aa.max_moves = ea.max_moves; aa.H = ea.H;
    aa.vecs_per_row = ea.vecs_per_row;
    // two column halves per strip while the strips are few and a half is whole 128-byte lines: measured read+write rate of a
    // stable eviction, one part -> two, 512 strips (high-resolution shape, batch 8) 3.0 -> 3.9 TB/s, 640 strips (13B shape,
    // batch 8) 3.0 -> 3.8, 1280 strips (batch 16) 4.8 -> 4.7
    const int parts = (2 * ea.H * B <= 1024 && ea.vecs_per_row % 16 == 0) ? 2 : 1;
    aa.vecs_per_part = ea.vecs_per_row / parts;
    evict_apply_kernel<<<dim3(2 * ea.H, B, parts), 256, 0, st>>>(aa);
}


// Eviction plan (+ optional append bookkeeping, finishing of the mass and in-kernel row moves),
// then the separate move kernel when the plan kernel does not move the rows itself.
//   appended:   the attention kernel has just written one row beyond kv_len[b]; it is counted here
//   mass_dst:   where the mass of the attention launch before this call is finished (null: skip)
st3_status enqueue_select_compact(const st3_attn_shape* shape, const st3_kv_layer* kv, const st3_segments* seg,
                                  float* score_col, int32_t* id_col, int64_t col_stride, int32_t keep_count,
                                  int32_t mode, void* workspace, size_t workspace_bytes, hipStream_t st,
                                  int appended, float* mass_dst, int64_t mass_stride) {
    EvictArgs ea;
    bool needs_apply = false;
    st3_status s = build_evict_args(shape, kv, seg, score_col, id_col, col_stride, keep_count, mode, workspace,
                                    workspace_bytes, appended, mass_dst, mass_stride, ea, needs_apply, false);
    if (s != ST3_OK) return s;
    launch_evict_plan(ea, shape->batch, st);
    if (needs_apply) launch_evict_apply(ea, shape->batch, st);
    return check_launch();
}

// ---------------------------------------------------------------------------------------------
// Diagnostics on mass vectors: Overlap_n (Eq. 10) and cosine similarity (Eq. 4-5).
// ---------------------------------------------------------------------------------------------
namespace {

constexpr int kDiagIdSpace = 16384;
constexpr int kDiagThreads = 256;

struct OverlapArgs {
    const float* score_a; const int32_t* ids_a; int64_t stride_a; const int32_t* n_a_dev; int32_t n_a;
    const float* score_b; const int32_t* ids_b; int64_t stride_b; const int32_t* n_b_dev; int32_t n_b;
    int32_t k, id_space;
    int32_t* overlap;       // [B] |TopK(a) ^ TopK(b)|
    int32_t* topk_a;        // [B] |TopK(a)| = min(k, n_a[b])
};

// One workgroup per sequence.  TopK(a) is marked in an LDS bitmap indexed by token id; the
// members of TopK(b) whose id is marked are counted.
__global__ __launch_bounds__(kDiagThreads) void overlap_topk_kernel(OverlapArgs a) {
    __shared__ SelectShared sm;
    __shared__ uint32_t seen[kDiagIdSpace / 32];
    __shared__ int sm_count;
    const int b = blockIdx.x, tid = threadIdx.x;
    uint32_t* keys = sel_keys();
    for (int i = tid; i < kDiagIdSpace / 32; i += kDiagThreads) seen[i] = 0u;
    if (tid == 0) sm_count = 0;
    __syncthreads();
    for (int side = 0; side < 2; ++side) {
        const float* scores = (side ? a.score_b + b * a.stride_b : a.score_a + b * a.stride_a);
        const int32_t* ids = (side ? a.ids_b + b * a.stride_b : a.ids_a + b * a.stride_a);
        const int32_t* n_dev = side ? a.n_b_dev : a.n_a_dev;
        int n = n_dev ? n_dev[b] : (side ? a.n_b : a.n_a);
        n = max(0, min(n, side ? a.n_b : a.n_a));
        const int k = min(a.k, n);
        auto key_at = [&](int i) { return keys[i]; };
        auto idkey_at = [&](int i) { return ~(uint32_t)ids[i]; };
        TopSet top{0, 0, true};
        if (k > 0 && k < n) {
            for (int i = tid; i < n; i += kDiagThreads) keys[i] = score_key(scores[i]);
            top = top_set<kDiagThreads>(key_at, idkey_at, n, k, sm);
        }
        int local = 0;
        for (int p = tid; p < n; p += kDiagThreads) {
            const bool keep = k >= n || (k > 0 && top.keeps(key_at, idkey_at, p));
            const int id = ids[p];
            if (!keep || id < 0 || id >= a.id_space) continue;
            if (side == 0) atomicOr(&seen[id >> 5], 1u << (id & 31));
            else local += (seen[id >> 5] >> (id & 31)) & 1u;
        }
        if (side == 0 && tid == 0) a.topk_a[b] = k;
        if (side == 1 && local) atomicAdd(&sm_count, local);
        __syncthreads();
    }
    if (tid == 0) a.overlap[b] = sm_count;
}

struct CosineArgs {
    const float* va; const int32_t* ids_a; int64_t stride_a; const int32_t* n_a_dev; int32_t n_a;
    const float* vb; const int32_t* ids_b; int64_t stride_b; const int32_t* n_b_dev; int32_t n_b;
    int32_t id_space;
    float* cosine;          // [B]
};

__device__ __forceinline__ float block_sum(float v, float* sm4) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if (threadIdx.x % kWave == 0) sm4[threadIdx.x / kWave] = v;
    __syncthreads();
    return (sm4[0] + sm4[1]) + (sm4[2] + sm4[3]);
}

// One workgroup per sequence.  Entries are matched by token id (ids_x == null: by position);
// tokens present on one side only count as zero on the other.  fp32 sums in a fixed order.
__global__ __launch_bounds__(kDiagThreads) void cosine_kernel(CosineArgs a) {
    __shared__ int16_t pos_b[kDiagIdSpace];
    __shared__ float sm4[4];
    const int b = blockIdx.x, tid = threadIdx.x;
    const float* va = a.va + b * a.stride_a;
    const float* vb = a.vb + b * a.stride_b;
    const int32_t* ia = a.ids_a ? a.ids_a + b * a.stride_a : nullptr;
    const int32_t* ib = a.ids_b ? a.ids_b + b * a.stride_b : nullptr;
    const int na = max(0, min(a.n_a_dev ? a.n_a_dev[b] : a.n_a, a.n_a));
    const int nb = max(0, min(a.n_b_dev ? a.n_b_dev[b] : a.n_b, a.n_b));
    for (int i = tid; i < a.id_space; i += kDiagThreads) pos_b[i] = -1;
    __syncthreads();
    float sbb = 0.f;
    for (int p = tid; p < nb; p += kDiagThreads) {
        const int id = ib ? ib[p] : p;
        if (id >= 0 && id < a.id_space) pos_b[id] = (int16_t)p;
        sbb = fmaf(vb[p], vb[p], sbb);
    }
    __syncthreads();
    float saa = 0.f, sab = 0.f;
    for (int p = tid; p < na; p += kDiagThreads) {
        const int id = ia ? ia[p] : p;
        const float x = va[p];
        saa = fmaf(x, x, saa);
        if (id >= 0 && id < a.id_space && pos_b[id] >= 0) sab = fmaf(x, vb[pos_b[id]], sab);
    }
    const float taa = block_sum(saa, sm4), tbb = block_sum(sbb, sm4), tab = block_sum(sab, sm4);
    if (tid == 0) a.cosine[b] = (taa > 0.f && tbb > 0.f) ? tab / (sqrtf(taa) * sqrtf(tbb)) : 0.f;
}

}  // namespace

}  // namespace st3

extern "C" st3_status st3_overlap_topk(const float* score_a, const int32_t* ids_a, int64_t stride_a,
                                       const int32_t* n_a_dev, int32_t n_a, const float* score_b,
                                       const int32_t* ids_b, int64_t stride_b, const int32_t* n_b_dev, int32_t n_b,
                                       int32_t batch, int32_t k, int32_t id_space, int32_t* overlap, int32_t* topk_a,
                                       void* stream) {
    if (!score_a || !ids_a || !score_b || !ids_b || !overlap || !topk_a) return ST3_ERR_INVALID_ARG;
    if (batch <= 0 || n_a < 0 || n_b < 0 || k < 0 || stride_a < n_a || stride_b < n_b) return ST3_ERR_INVALID_ARG;
    if (n_a > st3::kSelLdsKeys || n_b > st3::kSelLdsKeys || id_space <= 0 || id_space > st3::kDiagIdSpace)
        return ST3_ERR_UNSUPPORTED;
    st3::OverlapArgs a{score_a, ids_a, stride_a, n_a_dev, n_a, score_b, ids_b, stride_b, n_b_dev, n_b, k, id_space,
                       overlap, topk_a};
    st3::overlap_topk_kernel<<<batch, st3::kDiagThreads, sizeof(uint32_t) * std::max(n_a, n_b), reinterpret_cast<hipStream_t>(stream)>>>(a);
    return st3::check_launch();
}

extern "C" st3_status st3_cosine_similarity(const float* va, const int32_t* ids_a, int64_t stride_a,
                                            const int32_t* n_a_dev, int32_t n_a, const float* vb,
                                            const int32_t* ids_b, int64_t stride_b, const int32_t* n_b_dev,
                                            int32_t n_b, int32_t batch, int32_t id_space, float* cosine, void* stream) {
    if (!va || !vb || !cosine) return ST3_ERR_INVALID_ARG;
    if (batch <= 0 || n_a < 0 || n_b < 0 || stride_a < n_a || stride_b < n_b) return ST3_ERR_INVALID_ARG;
    if (id_space <= 0 || id_space > st3::kDiagIdSpace || n_a > 32767 || n_b > 32767) return ST3_ERR_UNSUPPORTED;
    st3::CosineArgs a{va, ids_a, stride_a, n_a_dev, n_a, vb, ids_b, stride_b, n_b_dev, n_b, id_space, cosine};
    st3::cosine_kernel<<<batch, st3::kDiagThreads, 0, reinterpret_cast<hipStream_t>(stream)>>>(a);
    return st3::check_launch();
}

extern "C" st3_status st3_select_topk(const float* scores, int64_t score_stride, const int32_t* tie_ids,
                                      int64_t id_stride, int32_t batch, const int32_t* n_dev, int32_t n, int32_t k,
                                      uint8_t* keep_mask, int32_t* keep_idx, int64_t idx_stride, void* stream) {
    if (!scores || batch <= 0 || n < 0 || k < 0 || k > n) return ST3_ERR_INVALID_ARG;
    if (keep_idx && idx_stride < k) return ST3_ERR_INVALID_ARG;
    if (n > 16384 || batch > 65535 * 32) return ST3_ERR_UNSUPPORTED;
    if (score_stride < n || (tie_ids && id_stride < n)) return ST3_ERR_INVALID_ARG;
    if (n == 0) return ST3_OK;
    st3::TopkArgs a{};
    a.scores = scores; a.score_stride = score_stride; a.ids = tie_ids; a.id_stride = id_stride;
    a.n_dev = n_dev; a.n = n; a.k = k; a.mask = keep_mask; a.idx = keep_idx; a.idx_stride = idx_stride;
    st3::launch_topk(a, batch, reinterpret_cast<hipStream_t>(stream));
    return st3::check_launch();
}

extern "C" st3_status st3_select_columns(const float* scores, int64_t score_stride, const int32_t* ids, int64_t id_stride,
                                         int32_t batch, int32_t n, int32_t k, float* out_scores, int64_t out_score_stride,
                                         int32_t* out_ids, int64_t out_id_stride, void* stream) {
    if (!scores || !ids || !out_scores || !out_ids || batch <= 0 || n < 0 || k < 0 || k > n) return ST3_ERR_INVALID_ARG;
    if (n > 16384 || batch > 65535 * 32) return ST3_ERR_UNSUPPORTED;
    if (score_stride < n || id_stride < n || out_score_stride < k || out_id_stride < k) return ST3_ERR_INVALID_ARG;
    if (k == 0) return ST3_OK;
    // whether a row of x shares memory with a row of y (rows of one buffer may alternate); rows follow each other without overlap
    auto meet = [&](const void* x, int64_t xs, int64_t xn, const void* y, int64_t ys, int64_t yn) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(x), b = reinterpret_cast<uintptr_t>(y);
        if (a >= b + ((uintptr_t)(batch - 1) * ys + yn) * 4 || b >= a + ((uintptr_t)(batch - 1) * xs + xn) * 4) return false;
        for (int32_t i = 0, j = 0; i < batch && j < batch;) {
            const uintptr_t p = a + (uintptr_t)i * xs * 4, q = b + (uintptr_t)j * ys * 4, p1 = p + xn * 4, q1 = q + yn * 4;
            if (p < q1 && q < p1) return true;
            p1 <= q ? ++i : ++j;
        }
        return false;
    };
    if (meet(scores, score_stride, n, out_scores, out_score_stride, k) || meet(scores, score_stride, n, out_ids, out_id_stride, k) ||
        meet(ids, id_stride, n, out_scores, out_score_stride, k) || meet(ids, id_stride, n, out_ids, out_id_stride, k) ||
        meet(out_scores, out_score_stride, k, out_ids, out_id_stride, k))
        return ST3_ERR_INVALID_ARG;
    st3::TopkArgs a{};
    a.scores = scores; a.score_stride = score_stride; a.ids = ids; a.id_stride = id_stride; a.n = n; a.k = k;
    a.out_scores = out_scores; a.out_score_stride = out_score_stride; a.out_ids = out_ids; a.out_id_stride = out_id_stride;
    st3::launch_topk(a, batch, reinterpret_cast<hipStream_t>(stream));
    return st3::check_launch();
}

extern "C" st3_status st3_compact_rows(void* rows, int32_t batch, int32_t inner, int64_t stride_b_bytes,
                                       int64_t stride_inner_bytes, int64_t stride_row_bytes, int32_t row_bytes,
                                       const int32_t* keep_idx, int64_t idx_stride, int32_t k, int32_t n,
                                       int32_t tail_rows, void* stream) {
    if (!rows || !keep_idx || batch <= 0 || inner <= 0 || k < 0 || n < 0 || k > n || tail_rows < 0)
        return ST3_ERR_INVALID_ARG;
    if (idx_stride < k) return ST3_ERR_INVALID_ARG;
    if (row_bytes <= 0 || row_bytes % 4 || stride_row_bytes < row_bytes) return ST3_ERR_INVALID_ARG;
    if (batch > 65535 || inner > 65535) return ST3_ERR_UNSUPPORTED;
    if (k + tail_rows == 0) return ST3_OK;
    const bool vec16 = (row_bytes % 16 == 0) && (stride_row_bytes % 16 == 0) && (stride_b_bytes % 16 == 0) &&
                       (stride_inner_bytes % 16 == 0) && st3::aligned16(rows);
    if (!vec16 && ((stride_row_bytes % 4) || (stride_b_bytes % 4) || (stride_inner_bytes % 4) ||
                   (reinterpret_cast<uintptr_t>(rows) & 3)))
        return ST3_ERR_INVALID_ARG;
    st3::CompactArgs a{};
    a.rows = reinterpret_cast<char*>(rows);
    a.stride_b = stride_b_bytes; a.stride_inner = stride_inner_bytes; a.stride_row = stride_row_bytes;
    a.unit_bytes = vec16 ? 16 : 4;
    a.row_units = row_bytes / a.unit_bytes;
    int slab = 1;
    while (slab * 2 <= a.row_units && slab * 2 <= 256) slab *= 2;
    a.slab_units = slab;
    a.idx = keep_idx; a.idx_stride = idx_stride; a.k = k; a.n = n; a.tail = tail_rows;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (vec16) st3::launch_compact<uint4>(a, inner, batch, st);
    else st3::launch_compact<uint32_t>(a, inner, batch, st);
    return st3::check_launch();
}

extern "C" st3_status st3_gather_rows(const st3_gather_pair* pairs, int32_t n_pairs, int32_t batch, int32_t inner,
                                      int32_t row_bytes, int32_t head_rows, const int32_t* keep_idx, int64_t idx_stride,
                                      int32_t k, int32_t n, int32_t tail_rows, void* stream) {
    using namespace st3;
    if (!pairs || n_pairs <= 0 || n_pairs > ST3_MAX_GATHER || batch <= 0 || inner <= 0) return ST3_ERR_INVALID_ARG;
    if (row_bytes <= 0 || row_bytes % 16 || head_rows < 0 || k < 0 || n < 0 || k > n || tail_rows < 0)
        return ST3_ERR_INVALID_ARG;
    if (!keep_idx && k != n) return ST3_ERR_INVALID_ARG;
    if (keep_idx && idx_stride < k) return ST3_ERR_INVALID_ARG;
    if ((int64_t)batch * n_pairs > 65535 || inner > 65535) return ST3_ERR_UNSUPPORTED;
    const int64_t src_rows = (int64_t)head_rows + n + tail_rows, dst_rows = (int64_t)head_rows + k + tail_rows;
    GatherArgs a{};
    for (int p = 0; p < n_pairs; ++p) {
        const st3_gather_pair& g = pairs[p];
        if (!g.src || !g.dst || !aligned16(g.src) || !aligned16(g.dst)) return ST3_ERR_INVALID_ARG;
        const int64_t st[6] = {g.src_stride_b, g.src_stride_inner, g.src_stride_row,
                               g.dst_stride_b, g.dst_stride_inner, g.dst_stride_row};
        for (int64_t v : st) if (v < 0 || v % 16) return ST3_ERR_INVALID_ARG;
        if (g.src_stride_row < row_bytes || g.dst_stride_row < row_bytes) return ST3_ERR_INVALID_ARG;
        // the whole source and destination regions of this pair must be disjoint
        const char* s0 = reinterpret_cast<const char*>(g.src);
        const char* d0 = reinterpret_cast<const char*>(g.dst);
        const int64_t s_ext = (batch - 1) * g.src_stride_b + (inner - 1) * g.src_stride_inner +
                              (src_rows > 0 ? (src_rows - 1) * g.src_stride_row + row_bytes : 0);
        const int64_t d_ext = (batch - 1) * g.dst_stride_b + (inner - 1) * g.dst_stride_inner +
                              (dst_rows > 0 ? (dst_rows - 1) * g.dst_stride_row + row_bytes : 0);
        if (s0 < d0 + d_ext && d0 < s0 + s_ext) return ST3_ERR_INVALID_ARG;
        a.pair[p] = g;
    }
    if (dst_rows == 0) return ST3_OK;
    a.idx = keep_idx; a.idx_stride = idx_stride; a.n_pairs = n_pairs; a.vecs_per_row = row_bytes / 16;
    a.head = head_rows; a.k = k; a.n = n; a.tail = tail_rows;
    const int64_t total = dst_rows * a.vecs_per_row;
    if (total >= 0x7fffffff) return ST3_ERR_UNSUPPORTED;           // the kernel indexes a strip with 32 bits
    a.vpr_shift = -1;
    for (int sh = 0; sh < 31; ++sh)
        if ((1 << sh) == a.vecs_per_row) a.vpr_shift = sh;
    const int64_t blocks = (total + 256 * kGatherUR - 1) / (256 * kGatherUR);
    const dim3 grid((unsigned)blocks, inner, batch * n_pairs);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (dst_rows * row_bytes * inner * batch * n_pairs > kGatherStreamBytes) gather_rows_kernel<true><<<grid, 256, 0, st>>>(a);
    else gather_rows_kernel<false><<<grid, 256, 0, st>>>(a);
    return check_launch();
}

extern "C" st3_status st3_select_compact_layer(const st3_attn_shape* shape, const st3_kv_layer* kv,
                                               const st3_segments* seg, float* score_col, int32_t* id_col,
                                               int64_t col_stride, int32_t keep_count, int32_t mode,
                                               void* workspace, size_t workspace_bytes, void* stream) {
    st3_status s = st3::check_shape(shape);
    if (s != ST3_OK) return s;
    s = (kv && !kv->k) ? st3::validate_kv_value_only(shape, kv, seg) : st3::validate_kv(shape, kv, seg);
    if (s != ST3_OK) return s;
    if (!score_col || !id_col || !workspace || keep_count < 0) return ST3_ERR_INVALID_ARG;
    if (col_stride < seg->max_vis_len) return ST3_ERR_INVALID_ARG;
    if (mode != ST3_STABLE && mode != ST3_HOLE_FILL) return ST3_ERR_INVALID_ARG;
    if (!st3::aligned16(workspace)) return ST3_ERR_INVALID_ARG;
    return st3::enqueue_select_compact(shape, kv, seg, score_col, id_col, col_stride, keep_count, mode, workspace,
                                       workspace_bytes, reinterpret_cast<hipStream_t>(stream), 0, nullptr, 0);
}
