// Head reduction of the visual mass (Sec. 3.2: last-row attention on the visual keys, here
// averaged over heads), shared by the decode finish kernel and by the eviction-plan kernel, which
// finishes the mass of the attention launch that preceded it.
#pragma once

#include "st3_attend.h"

namespace st3 {

#if defined(__HIPCC__)

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
