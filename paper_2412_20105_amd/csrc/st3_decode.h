// Head reduction of the visual mass (Sec. 3.2: last-row attention on the visual keys, here
// averaged over heads), shared by the decode finish kernel and by the eviction-plan kernel, which
// finishes the mass of the attention launch that preceded it.
#pragma once

#include "st3_attend.h"

namespace st3 {

#if defined(__HIPCC__)

// One output element from its chunks' partials po[s * stride], s < ns, in chunk order.  UR chunks' loads are in flight at a time: a
// load and its wait for each chunk in turn were most of what a merge took (us a step, min-sized chunks: 2 layers of the 7B shape, 8
// chunks, 20.5 -> 14.8, 12 layers of 8 heads 22.8 -> 17.8).
template <int UR>
__device__ __forceinline__ float merged_sum(const float* po, int64_t stride, int ns) {
    float o = 0.f;
    for (int s0 = 0; s0 < ns; s0 += UR) {
        float v[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) v[u] = po[min(s0 + u, ns - 1) * stride];
#pragma unroll
        for (int u = 0; u < UR; ++u) o += s0 + u < ns ? v[u] : 0.f;
    }
    return o;
}
// The same of un-normalised partials with their (max, sum) pairs ml[2 s], ml[2 s + 1].
template <int UR>
__device__ __forceinline__ float merged_output(const float* po, int64_t stride, const float* ml, int ns) {
    float m = -3.402823466e38f, l = 0.f, o = 0.f;       // (no chunk's maximum is lower)
    for (int s0 = 0; s0 < ns; s0 += UR) {
        float v[UR];
        float2 x[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const int s = min(s0 + u, ns - 1);
            x[u] = *reinterpret_cast<const float2*>(ml + 2 * s);
            v[u] = po[s * stride];
        }
        float m_new = m;
#pragma unroll
        for (int u = 0; u < UR; ++u) m_new = fmaxf(m_new, x[u].x);
        const float f0 = exp2_fast(m - m_new);          // first round: sums of 0
        l *= f0; o *= f0; m = m_new;
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const float f = exp2_fast(x[u].x - m);
            l = s0 + u < ns ? fmaf(x[u].y, f, l) : l;   // (a chunk that is not there adds nothing, whatever its place holds)
            o = s0 + u < ns ? fmaf(v[u], f, o) : o;
        }
    }
    return o / l;
}
// normalised: the partials are finished outputs of their chunks' share of the probabilities (a lazy layer's).  Eight loads in flight
// or, for more chunks, sixteen (8 / 12 / 16 always: 4 layers of 8 heads, 11 chunks, 16.3 / 14.8 / 15.2; 2 layers of 32 heads, 8 chunks,
// 14.5 / 15.0 / 15.7).
__device__ __forceinline__ float merge_partials(bool normalised, const float* po, int64_t stride, const float* ml, int ns) {
    if (normalised) return ns <= 8 ? merged_sum<8>(po, stride, ns) : merged_sum<16>(po, stride, ns);
    return ns <= 8 ? merged_output<8>(po, stride, ml, ns) : merged_output<16>(po, stride, ml, ns);
}

// Row maximum and reciprocal row sum of every head of sequence b, rebuilt from the per-chunk (max, sum) pairs (ns > 0 of
// them, at most 64; a power of two of lanes per head), into two LDS arrays of H entries.  Ends with a barrier.
template <int NT>
__device__ __forceinline__ void head_norms(const float* part_ml, int b, int H, int ns, int nsplit_cap, float* sm_m,
                                           float* sm_rl) {
    int nsp = 1;
    while (nsp < ns) nsp *= 2;                          // a head's lanes lie in one wave
    for (int base = 0; base < H * nsp; base += NT) {
        const int x = base + (int)threadIdx.x, h = x / nsp, c = x & (nsp - 1);
        float m = -INFINITY, l = 0.f;
        if (h < H && c < ns) {
            const float2 ml = *reinterpret_cast<const float2*>(part_ml + (((int64_t)b * H + h) * nsplit_cap + c) * 2);
            m = ml.x; l = ml.y;
        }
        const float own = m;
        for (int off = 1; off < nsp; off <<= 1) m = fmaxf(m, __shfl_xor(m, off));
        l = c < ns ? l * exp2_fast(own - m) : 0.f;
        for (int off = 1; off < nsp; off <<= 1) l += __shfl_xor(l, off);
        if (h < H && c == 0) { sm_m[h] = m; sm_rl[h] = 1.0f / l; }
    }
    __syncthreads();
}

// acc + the sum over rows [r, r1) of exp2(x[r * stride] - m[r]) * rl[r], in row order, at most U of them and U loads in flight.
template <int U>
__device__ __forceinline__ float prob_sum_some(float acc, const float* x, int64_t stride, const float* m, const float* rl, int r, int r1) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = x[(int64_t)min(r + u, r1 - 1) * stride];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int rr = min(r + u, r1 - 1);
        const float p = exp2_fast(v[u] - m[rr]) * rl[rr];
        acc += r + u < r1 ? p : 0.f;
    }
    return acc;
}

// The same over rows [r0, r1), U loads in flight.  r0 and r1 are the same for the lanes of a wave.
template <int U>
__device__ __forceinline__ float prob_sum(const float* x, int64_t stride, const float* m, const float* rl, int r0, int r1) {
    float acc = 0.f;
    for (int r = r0; r < r1; r += U) acc = prob_sum_some<U>(acc, x, stride, m, rl, r, r1);
    return acc;
}

#endif  // __HIPCC__

}  // namespace st3
