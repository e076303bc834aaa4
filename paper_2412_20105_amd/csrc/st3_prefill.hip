// Prefill attention (Eq. 2, causal) with the visual mass of the last query rows (Sec. 3.2).
//
// Two kernels produce the attention output:
//   * prefill_rows_kernel  - float32 arithmetic on any supported element type, one wavefront per
//                            query row streaming the keys it may see.  Used for float32 inputs.
//   * prefill_mfma_kernel  - bf16 inputs, MFMA contraction with LDS-staged K/V tiles (st3_prefill_mfma.hip).
// Both leave, for the last W query rows, the scaled logits of the visual keys and the row's
// (max, sum) in the workspace; prefill_mass_kernel turns them into probabilities and adds them
// over heads and rows in a fixed order.
#include "st3_attend.h"
#include "st3_prefill.h"

namespace st3 {

namespace {

constexpr int kRowsPerBlock = 4;

// grid (ceil(n/4), H, B); wave w of block x handles query row n-1-(4x+w): longest rows first.
template <typename T, int D>
__global__ __launch_bounds__(256) void prefill_rows_kernel(PrefillArgs a) {
    using M = RowMap<T, D>;
    constexpr int EPL = M::EPL, LPR = M::LPR;
    const int h = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int i = a.n - 1 - ((int)blockIdx.x * kRowsPerBlock + wave);
    if (i < 0) return;
    const T* qrow = reinterpret_cast<const T*>(a.q) + b * a.q_sb + h * a.q_sh + (int64_t)query_row(a, b, i) * a.q_st;
    const T* kbase = reinterpret_cast<const T*>(a.k) + b * a.k_sb + h * a.k_sh;
    const T* vbase = reinterpret_cast<const T*>(a.v) + b * a.v_sb + h * a.v_sh;
    float qf[EPL];
    load_q_slice<T, D>(qrow, lane, qf);
    WaveState<EPL> st;
    const int64_t bh = (int64_t)b * a.H + h;
    const int w_idx = i - (a.n - a.window);
    float* lg = nullptr;
    if (a.pre_logits && w_idx >= 0) lg = a.pre_logits + (bh * a.window + w_idx) * a.vis_len;
    // K and V may have different strides; wave_attend takes one stride, so require equality here
    wave_attend<T, D, 4, false>(qf, kbase, vbase, a.k_st, 0, i + 1, 4 * M::RPL, 0, a.scale_l2, lane, st, lg, a.sys_len,
                         a.sys_len + a.vis_len);
    finish_wave<T, D>(st);
    if (lane < LPR) {
        float o[EPL];
        const float rl = 1.0f / st.l;
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[e] = st.acc[e] * rl;
        T* orow = reinterpret_cast<T*>(a.out) + b * a.o_sb + h * a.o_sh + (int64_t)i * a.o_st;
        *reinterpret_cast<uint4*>(orow + lane * EPL) = ElemTraits<T>::pack(o);
    }
    if (lg && lane == 0) {
        a.pre_ml[(bh * a.window + w_idx) * 2] = st.m;
        a.pre_ml[(bh * a.window + w_idx) * 2 + 1] = st.l;
    }
}

struct PrefillMassArgs {
    const float* pre_logits;
    const float* pre_ml;
    float* mass;
    int64_t mass_stride;
    int32_t n, sys_len, vis_len, window, H;
};

// grid (ceil(vis_len/64), B).  mass[b,j] = (1/H) sum_h sum_w p_{h,w}[sys_len+j]; a window row
// that precedes key sys_len+j cannot see it (causal mask) and contributes nothing.  Latency bound (4 bytes per head, window
// row and key): one of 16 waves takes a sixteenth of the (head, row) pairs, kUR loads in flight (eight, or the power of two that
// covers its pairs when they are fewer: each pair left over costs a division), and the sixteenths are added in order.  One thread per key that walked all heads took 12 us for one sequence and 24 us for 32; a prefill call
// of one 7B layer, 310 tokens, went from 30.9 to 21.2 us, of one 13B layer, batch 32, 739 tokens, from 403 to 398.
constexpr int kMassWaves = 16;
template <int kUR>
__global__ __launch_bounds__(kMassWaves * kWave) void prefill_mass_kernel(PrefillMassArgs a) {
    __shared__ float part[kMassWaves][kWave];
    const int b = blockIdx.y, lane = threadIdx.x % kWave, g = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int j = blockIdx.x * kWave + lane;
    const int rows = a.H * a.window, per = (rows + kMassWaves - 1) / kMassWaves;
    const int r0 = g * per, r1 = min(rows, r0 + per);
    const float* lg = a.pre_logits + (int64_t)b * rows * a.vis_len + min(j, a.vis_len - 1);
    const float* ml = a.pre_ml + (int64_t)b * rows * 2;
    const int first = a.sys_len + j - (a.n - a.window);     // the first window row that sees the key
    float acc = 0.f;
    for (int r = r0; r < r1; r += kUR) {
        float v[kUR];
#pragma unroll
        for (int u = 0; u < kUR; ++u) v[u] = lg[(int64_t)min(r + u, r1 - 1) * a.vis_len];
#pragma unroll
        for (int u = 0; u < kUR; ++u) {
            const int rr = min(r + u, r1 - 1);
            const float p = exp2_fast(v[u] - ml[rr * 2]) / ml[rr * 2 + 1];
            acc += r + u < r1 && rr % a.window >= first ? p : 0.f;      // (a row that cannot see the key has left no logit)
        }
    }
    part[g][lane] = acc;
    __syncthreads();
    if (g == 0 && j < a.vis_len) {
        acc = 0.f;
#pragma unroll
        for (int w = 0; w < kMassWaves; ++w) acc += part[w][lane];
        a.mass[(int64_t)b * a.mass_stride + j] = acc / (float)a.H;
    }
}

template <typename T, int D>
void launch_rows(const PrefillArgs& a, int B, hipStream_t st) {
    dim3 grid((a.n + kRowsPerBlock - 1) / kRowsPerBlock, a.H, B);
    prefill_rows_kernel<T, D><<<grid, 256, 0, st>>>(a);
}

bool tensor_ok(const st3_tensor4* t, int eb, int d) {
    if (!t || !t->data || !aligned16(t->data)) return false;
    if (t->stride_t < d || t->stride_h < 0 || t->stride_b < 0) return false;
    return (t->stride_t * eb) % 16 == 0 && (t->stride_h * eb) % 16 == 0 && (t->stride_b * eb) % 16 == 0;
}

// Whether one of the nx rows of a strip of x shares memory with one of the ny rows of a strip of y.  Tensors of equal strides may be parts of one
// buffer, whose rows alternate; of others, all that lies between the first byte and the last counts.
bool rows_meet(const st3_tensor4* x, int64_t nx, const st3_tensor4* y, int64_t ny, int B, int H, int D, int eb) {
    const int64_t row = (int64_t)D * eb, d = (int64_t)(reinterpret_cast<intptr_t>(y->data) - reinterpret_cast<intptr_t>(x->data));
    auto extent = [&](const st3_tensor4* t, int64_t n) { return ((B - 1) * t->stride_b + (H - 1) * t->stride_h + (n - 1) * t->stride_t) * eb + row; };
    if (d >= extent(x, nx) || -d >= extent(y, ny)) return false;
    if (x->stride_b != y->stride_b || x->stride_h != y->stride_h || x->stride_t != y->stride_t) return true;
    const int64_t sb = x->stride_b * eb, sh = x->stride_h * eb, st = x->stride_t * eb;
    for (int64_t b = 1 - B; b < B; ++b)
        for (int64_t h = 1 - H; h < H; ++h) {
            // rows i of x and j of y begin gap + (j - i) * st apart; the two nearest values of j - i on either side of -gap / st
            const int64_t gap = d + b * sb + h * sh, near = -gap / st;
            for (int64_t k = near - 1; k <= near + 1; ++k)
                if (k > -nx && k < ny && gap + k * st < row && -(gap + k * st) < row) return true;
        }
    return false;
}

}  // namespace
}  // namespace st3

namespace st3 {
static st3_status prefill_attention(const st3_attn_shape* shape, const st3_tensor4* q, const int32_t* q_ids, int64_t q_ids_stride, int32_t q_vis,
                                    const st3_tensor4* k, const st3_tensor4* v, int32_t n, int32_t sys_len, int32_t vis_len,
                                    int32_t score_window, const st3_tensor4* out, float* vis_mass, int64_t mass_stride, void* workspace,
                                    size_t workspace_bytes, void* stream) {
    st3_status s = check_shape(shape);
    if (s != ST3_OK) return s;
    const int B = shape->batch, H = shape->heads, D = shape->head_dim, eb = elem_bytes(shape->dtype);
    if (!tensor_ok(q, eb, D) || !tensor_ok(k, eb, D) || !tensor_ok(v, eb, D) || !tensor_ok(out, eb, D))
        return ST3_ERR_INVALID_ARG;
    if (n <= 0 || sys_len < 0 || vis_len < 0 || sys_len + vis_len > n) return ST3_ERR_INVALID_ARG;
    if (n > 32768) return ST3_ERR_UNSUPPORTED;
    if (score_window < 1 || score_window > n || score_window > kMaxWindow) return ST3_ERR_INVALID_ARG;
    if (k->stride_t != v->stride_t) return ST3_ERR_UNSUPPORTED;
    // queries by id: a workgroup reads rows in whose places of the output others write
    if (q_ids && rows_meet(q, (int64_t)n - vis_len + q_vis, out, n, B, H, D, eb)) return ST3_ERR_INVALID_ARG;
    const bool want_mass = vis_mass != nullptr && vis_len > 0;
    if (want_mass && mass_stride < vis_len) return ST3_ERR_INVALID_ARG;
    const PrefillWs wl = prefill_ws(B, H, vis_len, score_window);
    // the prefill scratch sits at the END of the workspace, clear of the decode-path region
    if (want_mass) {
        if (!workspace || !aligned16(workspace)) return ST3_ERR_INVALID_ARG;
        if (workspace_bytes < wl.total) return ST3_ERR_WORKSPACE_TOO_SMALL;
    }
    const size_t ws_base = want_mass ? (workspace_bytes - wl.total) / 256 * 256 : 0;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    PrefillArgs a{};
    a.q = q->data; a.k = k->data; a.v = v->data; a.out = out->data;
    a.q_sb = q->stride_b; a.q_sh = q->stride_h; a.q_st = q->stride_t;
    a.k_sb = k->stride_b; a.k_sh = k->stride_h; a.k_st = k->stride_t;
    a.v_sb = v->stride_b; a.v_sh = v->stride_h; a.v_st = v->stride_t;
    a.o_sb = out->stride_b; a.o_sh = out->stride_h; a.o_st = out->stride_t;
    a.n = n; a.sys_len = sys_len; a.vis_len = vis_len; a.window = score_window; a.H = H;
    a.scale_l2 = scale_log2(shape);
    a.q_ids = q_ids; a.q_ids_sb = q_ids_stride; a.q_vis = q_vis;
    if (want_mass) {
        char* ws = reinterpret_cast<char*>(workspace) + ws_base;
        a.pre_logits = reinterpret_cast<float*>(ws + wl.pre_logits);
        a.pre_ml = reinterpret_cast<float*>(ws + wl.pre_ml);
    }
    // diagnostic override of the kernel choice (0 unless the debug block is enabled): 1 = the row
    // kernel also for bf16, 2 = the MFMA kernel or fail
    const int g_prefill_path = debug_state().prefill_path;
    bool use_mfma = shape->dtype == ST3_BF16;
    if (g_prefill_path == 1) use_mfma = false;
    if (g_prefill_path == 2 && shape->dtype != ST3_BF16) return ST3_ERR_UNSUPPORTED;
    if (use_mfma) {
        s = launch_prefill_mfma(a, B, D, st);
        if (s == ST3_ERR_UNSUPPORTED && g_prefill_path != 2) use_mfma = false;    // shape outside the MFMA kernel
        else if (s != ST3_OK) return s;
    }
    if (!use_mfma) {
        if (shape->dtype == ST3_BF16) {
            if (D == 128) launch_rows<bf16_t, 128>(a, B, st); else launch_rows<bf16_t, 64>(a, B, st);
        } else {
            if (D == 128) launch_rows<float, 128>(a, B, st); else launch_rows<float, 64>(a, B, st);
        }
    }
    if (want_mass) {
        PrefillMassArgs m{a.pre_logits, a.pre_ml, vis_mass, mass_stride, n, sys_len, vis_len, score_window, H};
        const dim3 grid((vis_len + kWave - 1) / kWave, B);
        const int per = (H * score_window + kMassWaves - 1) / kMassWaves;
        if (per <= 1) prefill_mass_kernel<1><<<grid, kMassWaves * kWave, 0, st>>>(m);
        else if (per <= 2) prefill_mass_kernel<2><<<grid, kMassWaves * kWave, 0, st>>>(m);
        else if (per <= 4) prefill_mass_kernel<4><<<grid, kMassWaves * kWave, 0, st>>>(m);
        else prefill_mass_kernel<8><<<grid, kMassWaves * kWave, 0, st>>>(m);
    }
    return check_launch();
}
}  // namespace st3

extern "C" st3_status st3_prefill_attention(const st3_attn_shape* shape, const st3_tensor4* q, const st3_tensor4* k,
                                            const st3_tensor4* v, int32_t n, int32_t sys_len, int32_t vis_len,
                                            int32_t score_window, const st3_tensor4* out, float* vis_mass,
                                            int64_t mass_stride, void* workspace, size_t workspace_bytes,
                                            void* stream) {
    return st3::prefill_attention(shape, q, nullptr, 0, 0, k, v, n, sys_len, vis_len, score_window, out, vis_mass, mass_stride, workspace,
                                  workspace_bytes, stream);
}

extern "C" st3_status st3_prefill_attention_kept(const st3_attn_shape* shape, const st3_tensor4* q, const int32_t* q_ids,
                                                 int64_t q_ids_stride, int32_t q_vis, const st3_tensor4* k, const st3_tensor4* v, int32_t n,
                                                 int32_t sys_len, int32_t vis_len, int32_t score_window, const st3_tensor4* out,
                                                 float* vis_mass, int64_t mass_stride, void* workspace, size_t workspace_bytes,
                                                 void* stream) {
    if (!q_ids || vis_len < 0 || q_vis < vis_len || q_ids_stride < vis_len) return ST3_ERR_INVALID_ARG;
    return st3::prefill_attention(shape, q, q_ids, q_ids_stride, q_vis, k, v, n, sys_len, vis_len, score_window, out, vis_mass, mass_stride,
                                  workspace, workspace_bytes, stream);
}
