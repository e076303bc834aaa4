// bf16 prefill attention (Eq. 2, causal) on the MFMA units of gfx950, with the logits of the last
// W query rows saved for the visual mass (Sec. 3.2).
//
// Tiling.  A workgroup of 4 wavefronts owns 128 consecutive query rows (32 per wave) of one (b,h)
// and walks the key tiles (32 or 64 keys) up to its diagonal.  K and V tiles live in LDS, row-major, in
// a ring of buffers.  They get there by direct global-to-LDS loads (no staging registers; a strip's base
// address in scalar registers, 32 bits of offset per lane): later tiles are in
// flight while the current one is consumed, and a tile costs one barrier.
// A direct load writes the 64 x 16 bytes of a wave to consecutive LDS addresses, so rows cannot be
// padded against bank conflicts; instead every lane chooses WHICH 16 bytes of its row it fetches,
// which stores the row's 16-byte units permuted (unit u of row r holds column unit u ^ swz(r)).
//
// Per wave, with v_mfma_f32_16x16x32_bf16 (A: 16 x 32, B: 32 x 16, C: 16 x 16; lane l = 16 g + c holds
// A[c][8g..8g+7], B[8g..8g+7][c] and C[4g..4g+3][c]); its 32 queries are two columns of 16:
//   S^T = K Q^T   A = K rows from LDS (one 16-byte read per lane), B = Q fragments kept in
//                 registers.  A lane then holds, of ONE query of either column (c), 8 of a sub-tile's 32
//                 keys: 4g..4g+3 and 16+4g..16+4g+3.
//   O^T = V^T P^T B = P^T taken straight from the S^T accumulator registers, which fixes which keys
//                 sit in which contraction slot: slots 8g..8g+3 are keys 4g..4g+3 of the sub-tile, slots 8g+4..8g+7 keys
//                 16+4g..16+4g+3.  A = V^T in the same
//                 pattern: a lane needs, for ONE column of V, two runs of four consecutive keys,
//                 which is what the LDS transpose read of gfx950 (ds_read_b64_tr_b16) returns from
//                 a row-major tile: within 16 lanes, lane i passes the address of elements
//                 4*(i%4)..+3 of row i/4 of a 4 x 16 block and receives column i of that block
//                 (layout checked on the device with an index pattern).
// Why this shape of MFMA.  Under this kernel the card is at its power limit: with inputs of zeros (nothing toggles) the 13B layer takes
// 257 us instead of 330, the high-resolution one 615 instead of 820.  What counts is therefore the energy of a product as much as
// the time of one, and the shapes differ in both (loops of nothing but MFMAs, TFLOP/s, zeros / normal values):
//   32x32x16, one wave a SIMD 2463 / 1762, two waves 1650 / 1310 (two waves that take turns lose a third of the matrix unit)
//   16x16x32, two or three waves 2440 / 2010 to 2250, the more the longer products in a row add to the same accumulator
// So P_hi V and P_lo V follow each other on one accumulator, and the contraction steps of S^T too; the compiler is kept from mixing the
// chains (it would, to hide a latency that the hardware does not have: 862 us instead of 838 at the high-resolution shape).
// A tile that lies entirely below a wave's diagonal is consumed whole (one softmax
// update); on the diagonal the 32-key sub-tile that holds it is masked and a sub-tile above it is
// skipped.  Online softmax in the log2 domain, fp32; the softmax scale is folded into the
// exponent's multiply-add.  For the second MFMA P is split into two bf16 terms, P = P_hi + P_lo
// (P_hi the upper 16 bits of the float, P_lo the rounded rest: 16 mantissa bits together), and both
// are multiplied by V: rounding P to one bf16 would put an error of 2^-9 of the row's magnitude on
// every output element, far above the element-wise tolerance for outputs that happen to be small.
#include <algorithm>

#include "st3_prefill.h"

namespace st3 {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

constexpr int kBM = 128;            // queries per workgroup
constexpr int kBN = 64;             // keys per tile where a tile is two sub-tiles

// An LDS tile is BN rows of D elements, no padding.  The 64 banks are 256 bytes wide together, so
// RPB rows share one pass over the banks.  K rows are read 16 bytes per lane by lanes holding
// consecutive rows: unit u ^ ((r / RPB) % UPR) spreads 16 consecutive rows over all banks.  V rows
// are read by the transpose read, 32 lanes covering 8 consecutive rows x 32 bytes (2 units): the
// permutation 2 * ((r / RPB) % (UPR / 2)) puts the eight rows on disjoint eighths of the banks.
template <int D, int BN = kBN> struct TileLayout {
    static constexpr int UPR = D / 8;                   // 16-byte units per row
    static constexpr int RPB = 256 / (2 * D);           // rows per 256 bytes: 1 or 2
    static constexpr int RPI = 1024 / (2 * D);          // rows per wave-wide direct load (1 KB): 4 or 8
    static constexpr int NI = BN / (RPI * 4);           // direct loads of K, and of V, per wave and tile
    static constexpr int TILE = BN * D;                // elements of one K (or V) tile
    __device__ static __forceinline__ int k_swz(int row) { return (row / RPB) & (UPR - 1); }
    __device__ static __forceinline__ int v_swz(int row) { return 2 * ((row / RPB) & (UPR / 2 - 1)); }
};

union Frag {
    bf16x8 v;
    u32x4 u4;
    uint32_t w[4];
    i16x4 h[2];
};

// One wave-wide direct load: every lane fetches the 16 bytes at base + lane_byte_off (global memory;
// the base is the same for all lanes and sits in scalar registers, the offset is 32 bits wide) and
// the wave's 64 x 16 bytes land at LDS byte address lds_byte_addr .. + 1023 in lane order (gfx950:
// global_load_lds_dwordx4, LDS base in M0).  Issued through inline assembly: the compiler treats the
// builtin form as an access that is outstanding on the LDS counter as well, and then makes every
// later wait for an LDS read a wait for ALL LDS reads in flight, which serialises the fragment
// reads of the whole tile.  What it does not know about is handled here: wait_direct_loads() before
// the barrier that publishes a buffer; M0 is declared clobbered; "memory" keeps LDS reads in place.
__device__ __forceinline__ void direct_load16(const uint16_t* base, uint32_t lane_byte_off, uint32_t lds_byte_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_byte_addr), "v"(lane_byte_off), "s"(base)
                 : "memory", "m0");
}

// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ const uint16_t* uniform_ptr(const uint16_t* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const uint16_t*>(((uint64_t)hi << 32) | lo);
}

// LDS byte address of a __shared__ object.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void*)p);
}

// Starts the direct loads of the K/V tile at key k0 into the buffer at LDS byte address `lds_buf` (K
// tile, then V tile).  Rows past n-1 are clamped: such keys lie above every valid query's diagonal
// and are masked there.  Every address read is a row of the caller's tensors; every LDS address
// written lies inside the buffer.
// Kp / Vp: row 0 of the strip (uniform).  k_lane / v_lane: byte offset of this lane's 16 bytes within
// the first 1 KB group of a tile at key 0 (row min(row0, n-1) and permuted unit folded in).
// Offsets from the strip's row 0 fit 32 bits (checked by the launcher).  wave_s: the wave's index, scalar.
template <int D, int BN = kBN>
__device__ __forceinline__ void issue_tile(uint32_t lds_buf, const uint16_t* Kp, const uint16_t* Vp, uint32_t k_lane,
                                           uint32_t v_lane, int64_t k_st, int64_t v_st, int k0, int n, int lane, int wave,
                                           int wave_s) {
    using L = TileLayout<D, BN>;
    const int row0 = wave * L::RPI + lane / L::UPR;     // this lane's row in the wave's first group
    if (k0 + BN <= n) {                                // all rows of the tile exist: plain strides
#pragma unroll
        for (int i = 0; i < L::NI; ++i) {
            const uint32_t dst = lds_buf + (4 * i + wave_s) * 1024;    // which 1 KB of the tile this wave-wide load fills
            const int key = k0 + 4 * i * L::RPI;
            direct_load16(uniform_ptr(Kp + key * k_st), k_lane, dst);
            direct_load16(uniform_ptr(Vp + key * v_st), v_lane, dst + 2 * L::TILE);
        }
    } else {
        const uint16_t* Ku = uniform_ptr(Kp);
        const uint16_t* Vu = uniform_ptr(Vp);
#pragma unroll
        for (int i = 0; i < L::NI; ++i) {
            const uint32_t dst = lds_buf + (4 * i + wave_s) * 1024;
            const int key = max(0, min(k0 + 4 * i * L::RPI, n - 1 - row0));     // this lane's row, key + row0, stays <= n - 1
            direct_load16(Ku, k_lane + (uint32_t)key * (uint32_t)(2 * k_st), dst);
            direct_load16(Vu, v_lane + (uint32_t)key * (uint32_t)(2 * v_st), dst + 2 * L::TILE);
        }
    }
}

// All direct loads this wave has issued have landed in LDS (vmcnt(0); other counters untouched).
__device__ __forceinline__ void wait_direct_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// The same but for this wave's last N direct loads.
template <int N>
__device__ __forceinline__ void wait_direct_loads_but() {
    static_assert(N < 16, "the counter's low bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | N);
}

// LDS reads at a byte address: 16 bytes, and the transpose read (4 consecutive rows of one column; see the header comment for the lane map).
__device__ __forceinline__ u32x4 lds_read16(uint32_t at) { return *reinterpret_cast<__attribute__((address_space(3))) const u32x4*>(at); }
__device__ __forceinline__ i16x4 lds_read_tr(uint32_t at) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<__attribute__((address_space(3))) i16x4*>(at));
}

// Where a lane finds its operands in a tile (byte offsets, fixed for the whole kernel).  K fragment s of row c: unit (4s + g) ^ k_swz(c),
// which is the first one's address ^ 64 s; transpose read of the 16 columns dt: row 4g + c/4, unit (2dt + (c%4)/2) ^ v_swz(row),
// half c%2: the first one's ^ 32 dt.  (g < 4 and (c%4)/2 < 2, so the + is an ^ too; tiles start at multiples of a row's bytes, so the ^ may
// come last: two registers, not twelve.)
template <int D>
struct LaneMap {
    uint32_t k, v;
    __device__ __forceinline__ void init(int c, int g) {
        using L = TileLayout<D>;
        k = (uint32_t)(2 * (c * D + (g ^ L::k_swz(c)) * 8));
        const int row = 4 * g + (c >> 2);
        v = (uint32_t)(2 * (row * D + (((c & 3) >> 1) ^ L::v_swz(row)) * 8 + 4 * (c & 1)));
    }
};

// The score window (the last W query rows), as the wave with first query q0 sees it: uniform values only, so that it costs the wave no
// vector registers while it works on other tiles.
struct Window {
    float* rows;            // logits of the strip's window rows, vis_len each; null: none of the wave's queries is in the window
    int shift;              // q0 - (n - W): a lane's query c is window row shift + c
    int rows_end;           // W
    int vis_lo, vis_hi;
};

// A wave's 32 queries, as two columns of 16: lane (c, g) holds query 16 qc + c of either, and of its output the columns
// 16 dt + 4 g .. + 3.
template <int D>
struct WaveRows {
    f32x4 o[D / 16][2];     // un-normalised output, transposed
    float m[2];             // reference point of the exponents; the same for the four lanes that share a query
    float l[2];             // sum of this lane's probabilities
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt)
#pragma unroll
            for (int qc = 0; qc < 2; ++qc) o[dt][qc] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int qc = 0; qc < 2; ++qc) { m[qc] = -3.402823466e38f; l[qc] = 0.f; }
    }
};

// NSUB 32-key sub-tiles for one wave: S^T, one online-softmax update over all NSUB * 32 keys, O^T += V^T P^T.  Kt, Vt: LDS byte
// addresses of the tile's K and V, this lane's part (LaneMap) included.  DIAG: the last sub-tile lies on the wave's diagonal (its keys
// start at the wave's first query), the only place where some keys are invisible to some rows.
template <int D, int NSUB, bool DIAG, bool LONE = false>
__device__ __forceinline__ void tile_step(uint32_t Kt, uint32_t Vt, const Frag (&qf)[2][D / 32], WaveRows<D>& st, float scale_l2, int c,
                                          int g, int k0, const Window& win) {
    constexpr int KS = D / 32, DT = D / 16, NG = 2 * NSUB;
    __builtin_amdgcn_s_setprio(1);
    // ---- S^T = K Q^T, 16 keys at a time; the next 16 keys' fragments are on their way meanwhile ----------------
    Frag ka[2][KS];
    f32x4 sacc[NSUB][2][2];             // [sub-tile][half of its keys][query column]
    auto load_k = [&](int grp) {
#pragma unroll
        for (int s = 0; s < KS; ++s) ka[grp & 1][s].u4 = lds_read16((Kt ^ (64 * s)) + 32 * grp * D);
    };
    load_k(0);
#pragma unroll
    for (int grp = 0; grp < NG; ++grp) {
        if (grp + 1 < NG) load_k(grp + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int qc = 0; qc < 2; ++qc) {
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) x = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[grp & 1][s].v, qf[qc][s].v, x, 0, 0, 0);
            sacc[grp / 2][grp % 2][qc] = x;
            if (!LONE) __builtin_amdgcn_sched_barrier(0);
        }
    }
    constexpr int VB = LONE ? DT : DT < 4 ? DT : 4;     // V^T fragments in flight
    Frag va[VB];
    auto load_v = [&](int i) {              // i-th of NSUB * DT: sub-tile i / DT, columns 16 (i % DT)
        const uint32_t at = (Vt ^ (32 * (i % DT))) + 64 * (i / DT) * D;
        va[i % VB].h[0] = lds_read_tr(at);
        va[i % VB].h[1] = lds_read_tr(at + 32 * D);
    };
#pragma unroll
    for (int i = 0; i < VB; ++i) load_v(i);             // these land while the softmax runs
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    // ---- causal mask (diagonal sub-tile only), row maximum ----------------------------------------
    if (DIAG) {
        int last = c - 4 * g;                           // (opaque: else the comparisons wait in registers for this one tile)
        asm volatile("" : "+v"(last));
#pragma unroll
        for (int kr = 0; kr < 2; ++kr)
#pragma unroll
            for (int qc = 0; qc < 2; ++qc)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (16 * kr - 16 * qc + r > last) sacc[NSUB - 1][kr][qc][r] = -INFINITY;
    }
    // A row of the score window keeps the scaled logits of its visual keys.  The wave that holds it sets the pace of the
    // strip's heaviest workgroup, so the usual case - every key of the tile visible and visual - is 16-byte stores.
    // (With a comparison and a store per key such a tile took 7200 cycles instead of 4250; 13B layer, batch 32: 396 -> 380 us a
    // call, high resolution, batch 8: 1010 -> 940.)
    if (win.rows != nullptr) {
        int cw = c, first = 4 * g;                      // (opaque: what follows is not worked out ahead of the one wave that needs it)
        asm volatile("" : "+v"(cw), "+v"(first));
        first += k0 - win.vis_lo;                       // this lane's first key among the visual ones
        const int n_vis = win.vis_hi - win.vis_lo;
        const bool whole = !DIAG && k0 >= win.vis_lo && k0 + 32 * NSUB <= win.vis_hi;
#pragma unroll
        for (int qc = 0; qc < 2; ++qc) {
            const int w = win.shift + 16 * qc + cw;     // window row
            if (w < 0 || w >= win.rows_end) continue;
            float* row = win.rows + (int64_t)w * n_vis;
            // (a masked key's logit is -inf here and is not kept)
            const int end = DIAG ? min(n_vis, k0 + 32 * (NSUB - 1) + 16 * qc + cw + 1 - win.vis_lo) : n_vis;
#pragma unroll
            for (int x = 0; x < 2 * NSUB; ++x) {
                const f32x4 v = sacc[x / 2][x % 2][qc] * scale_l2;
                if (whole) {
                    *reinterpret_cast<f32x4_a4*>(row + first + 16 * x) = v;     // (4-byte aligned, which is all a global store asks for)
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int j = first + 16 * x + r;
                        if (j >= 0 && j < end) row[j] = v[r];
                    }
                }
            }
        }
    }
    // The reference point m of the exponents only follows the row maximum when that has moved by
    // more than kLazy (probabilities then reach 2^kLazy at most, far inside fp32 and bf16 range):
    // a softmax is invariant to the reference point, and the accumulator rescaling it triggers
    // becomes rare instead of happening in nearly every tile.  Only then do the four lanes of a query need each other's maxima.
    // (Every row sees the first key of every tile it gets here, k0 <= q0: a maximum is -inf only where keys of logit -inf are all it
    // sees; they weigh nothing, whatever the reference.)
    constexpr float kLazy = 8.0f;
    float mx[2];
#pragma unroll
    for (int qc = 0; qc < 2; ++qc) {
        mx[qc] = sacc[0][0][qc][0];
#pragma unroll
        for (int x = 0; x < 2 * NSUB; ++x)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx[qc] = fmaxf(mx[qc], sacc[x / 2][x % 2][qc][r]);
        mx[qc] *= scale_l2;
    }
    if (__any(mx[0] - st.m[0] > kLazy || mx[1] - st.m[1] > kLazy)) {   // m is the lowest float before the first key of a finite logit: it moves
#pragma unroll
        for (int qc = 0; qc < 2; ++qc) {
            const float m_cand = fmaxf(st.m[qc], wave_max_from<16>(mx[qc]));
            const float m_new = m_cand - st.m[qc] > kLazy ? m_cand : st.m[qc];
            const float alpha = exp2_fast(st.m[qc] - m_new);            // 1 when not moved; 0 before the first key
            st.m[qc] = m_new;
            st.l[qc] *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) st.o[dt][qc] *= alpha;
        }
    }
    Frag pb[NSUB][2], pl[NSUB][2];
#pragma unroll
    for (int sub = 0; sub < NSUB; ++sub)
#pragma unroll
        for (int qc = 0; qc < 2; ++qc)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4& x = sacc[sub][j / 2][qc];
                const float p0 = exp2_fast(fmaf(x[2 * (j & 1)], scale_l2, -st.m[qc]));        // masked: exp2(-inf) = 0
                const float p1 = exp2_fast(fmaf(x[2 * (j & 1) + 1], scale_l2, -st.m[qc]));
                st.l[qc] += p0 + p1;
                const uint32_t b0 = __float_as_uint(p0), b1 = __float_as_uint(p1);
                pb[sub][qc].w[j] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);      // upper halves of (p0, p1)
                const f32x2 lo = {p0 - __uint_as_float(b0 & 0xffff0000u), p1 - __uint_as_float(b1 & 0xffff0000u)};
                pl[sub][qc].w[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
            }
    // ---- O^T += V^T P^T, 16 columns at a time; a fragment's place takes the one VB further on as soon as it is used ----------
#pragma unroll
    for (int i = 0; i < NSUB * DT; ++i) {
        const int sub = i / DT, dt = i % DT;
        if (i + VB - 1 < NSUB * DT && i > 0) load_v(i + VB - 1);
        if (!LONE) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int qc = 0; qc < 2; ++qc) {
            st.o[dt][qc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[i % VB].v, pb[sub][qc].v, st.o[dt][qc], 0, 0, 0);
            st.o[dt][qc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[i % VB].v, pl[sub][qc].v, st.o[dt][qc], 0, 0, 0);
            if (!LONE) __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// The part of the tile of BN keys at k0 (at LDS byte address `tile`) that the wave with first query q0 can see (k0 <= q0).
template <int D, int BN, bool LONE = false>
__device__ __forceinline__ void consume_tile(uint32_t tile, int k0, int q0, const Frag (&qf)[2][D / 32], WaveRows<D>& st, float scale_l2,
                                             const LaneMap<D>& lm, int c, int g, const Window& win) {
    const uint32_t Kt = tile + lm.k, Vt = tile + 2 * BN * D + lm.v;
    if constexpr (BN == 32) {
        if (k0 < q0) tile_step<D, 1, false, LONE>(Kt, Vt, qf, st, scale_l2, c, g, k0, win);
        else tile_step<D, 1, true, LONE>(Kt, Vt, qf, st, scale_l2, c, g, k0, win);
    } else {
        if (k0 + BN <= q0)          // below the diagonal: all 64 keys visible to all 32 rows
            tile_step<D, 2, false, LONE>(Kt, Vt, qf, st, scale_l2, c, g, k0, win);
        else if (k0 + 32 == q0)     // first half visible, second half on the diagonal
            tile_step<D, 2, true, LONE>(Kt, Vt, qf, st, scale_l2, c, g, k0, win);
        else                        // k0 == q0: first half on the diagonal, second half above it
            tile_step<D, 1, true, LONE>(Kt, Vt, qf, st, scale_l2, c, g, k0, win);
    }
}

// Normalises and stores a wave's 32 x D block of outputs.
// The accumulator holds O transposed (a lane owns one query and, per register quad, 4 consecutive
// columns): stored straight from there, a wave-wide store would touch 32 rows with 8 bytes each.
// So the wave's 32 x D block goes through LDS (obuf: 32 rows of D + 8 elements, this wave's own)
// and leaves as whole rows, 16 bytes per lane.
template <int D>
__device__ __forceinline__ void store_block(const PrefillArgs& a, int b, int h, uint16_t* obuf, const WaveRows<D>& st, const float (&l)[2],
                                            int q0, int n, bool wave_live, int lane, int g, int c) {
    constexpr int DT = D / 16;
    constexpr int OSTR = D + 8;                     // padded row, 16-byte aligned
    constexpr int VPR = D / 8;                      // 16-byte vectors (lanes) per row
    constexpr int RPI = 64 / VPR;                   // rows per wave-wide store
#pragma unroll
    for (int qc = 0; qc < 2; ++qc) {
        const float rl = 1.0f / l[qc];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const f32x4 o = st.o[dt][qc] * rl;
            const f32x2 o01 = {o[0], o[1]}, o23 = {o[2], o[3]};
            uint2 pk;                               // packed conversion, round to nearest even
            pk.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(o01, bf16x2));
            pk.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(o23, bf16x2));
            *reinterpret_cast<uint2*>(obuf + (16 * qc + c) * OSTR + 16 * dt + 4 * g) = pk;
        }
    }
    uint16_t* obase = reinterpret_cast<uint16_t*>(a.out) + b * a.o_sb + h * a.o_sh;
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int r = i * RPI + lane / VPR;
        const u32x4 val = *reinterpret_cast<const u32x4*>(obuf + r * OSTR + (lane % VPR) * 8);
        if (wave_live && q0 + r < n) *reinterpret_cast<u32x4*>(obase + (int64_t)(q0 + r) * a.o_st + (lane % VPR) * 8) = val;
    }
}

// q0 is the same for all lanes of a wave.
__device__ __forceinline__ Window window_of(const PrefillArgs& a, int64_t bh, int q0) {
    const int q = __builtin_amdgcn_readfirstlane(q0);
    const bool any = a.pre_logits != nullptr && q + 31 >= a.n - a.window && q < a.n && q >= 0;
    return Window{any ? a.pre_logits + bh * a.window * a.vis_len : nullptr, q - (a.n - a.window), a.window, a.sys_len, a.sys_len + a.vis_len};
}

// The window rows' maxima and sums.
__device__ __forceinline__ void keep_row_sums(const PrefillArgs& a, const Window& win, int64_t bh, int c, int g, const float (&m)[2],
                                              const float (&l)[2]) {
    if (win.rows == nullptr || g != 0) return;
#pragma unroll
    for (int qc = 0; qc < 2; ++qc) {
        const int w = win.shift + 16 * qc + c;
        if (w < 0 || w >= win.rows_end) continue;
        a.pre_ml[(bh * a.window + w) * 2] = m[qc];
        a.pre_ml[(bh * a.window + w) * 2 + 1] = l[qc];
    }
}

// A wave's query fragments: 32 rows from q0 on (rows that do not exist: the nearest that does).  Qp: the strip's row 0.
template <int D>
__device__ __forceinline__ void load_queries(const PrefillArgs& a, const uint16_t* Qp, int b, int q0, int c, int g, Frag (&qf)[2][D / 32]) {
#pragma unroll
    for (int qc = 0; qc < 2; ++qc) {
        const uint16_t* qrow = Qp + (int64_t)query_row(a, b, max(0, min(q0 + 16 * qc + c, a.n - 1))) * a.q_st;
#pragma unroll
        for (int s = 0; s < D / 32; ++s) qf[qc][s].u4 = *reinterpret_cast<const u32x4*>(qrow + 32 * s + 8 * g);
    }
}

constexpr int kLanes = 32;

// Workgroup -> (query tile, strip).  Workgroups go round-robin by linear id to the 8 XCDs (checked
// with a probe: XCC id == id % 8) and, within an XCD, in turn to its 4 shader engines; each XCD
// has an L2 of its own; a causal query tile costs in proportion to its index.  With the query
// tile as the fastest index, a tile count of 2 or 4 hands all heavy tiles to the same engines
// (measured: 4 tiles per strip ran slower than 5).  So each of the 32 dispatch lanes
// (id % 32) owns the strips congruent to it and receives the tiles of one strip back to back,
// heaviest first: all lanes see the same cost sequence and a strip's K and V stay in one L2.
__device__ __forceinline__ void place_workgroup(const PrefillArgs& a, int& strip, int& qt) {
    const int n_qt = a.n_qt, strips = a.H * a.B;
    const int full = strips / kLanes * kLanes;
    const int lin = blockIdx.x;
    if (lin < full * n_qt) {
        const int dl = lin % kLanes, m = lin / kLanes;
        strip = (m / n_qt) * kLanes + dl;
        qt = n_qt - 1 - m % n_qt;
    } else {                                    // the strips left over when H*B is no multiple of 32
        const int r = lin - full * n_qt;
        strip = full + r / n_qt;
        qt = n_qt - 1 - r % n_qt;
    }
}

// The same where not all workgroups find a place at once.  Such a launch ends with its last tiles, and a strip's heaviest tile can
// take as long as the strip's whole share of a compute unit: so the last strips of each lane (spread_strips) are dealt heaviest
// tiles first over all of them, and the strips left over come first of all, heaviest tiles first, instead of last.  us a call,
// before -> so (strips x tokens, with 32x32x16 MFMAs): 128 x 675 45.6 -> 37.4, 128 x 400 27.5 -> 23.4, 256 x 675 74.2 -> 62.7, 320 x 739 97.8 -> 88.6, 1280 x 739
// 371.5 -> 368.3, 80 x 739 42.0 -> 35.9, 140 x 1500 151.6 -> 127.4, 72 x 900 49.1 -> 38.5, 64 x 3136 234 -> 225.  (The kernel with key
// groups has all its workgroups in place at once and keeps the plain order: this one took its smallest calls 0.2 of 17 us.)
__device__ __forceinline__ void place_spread(const PrefillArgs& a, int& strip, int& qt) {
    const uint32_t n_qt = (uint32_t)a.n_qt, strips = (uint32_t)(a.H * a.B);
    const uint32_t per = strips / kLanes, over = strips % kLanes;       // strips of a lane, strips left over
    const uint32_t ahead = over * n_qt, spread = (uint32_t)a.spread, whole = (per - spread) * n_qt;
    const bool left = blockIdx.x < ahead;
    const uint32_t lin = blockIdx.x - ahead, m = lin / kLanes;          // (not used of a left-over strip)
    const bool apart = !left && m < whole;                              // a strip whose tiles come one after the other
    // (one division and no branch: behind a branch the other arguments are loaded in a second trip to memory)
    const uint32_t x = left ? blockIdx.x : apart ? m : m - whole, by = left ? over : apart ? n_qt : spread;
    const uint32_t quot = x / by, rest = x - quot * by;
    const uint32_t q = apart ? rest : quot;                             // the tile, counted from the heaviest
    strip = (int)(left ? per * kLanes + rest : ((apart ? quot : per - spread + rest) * kLanes + lin % kLanes));
    qt = (int)(n_qt - 1 - q);
}

// One-dimensional grid of ceil(n/128) * H * B workgroups (the mapping to query tile and strip is in the kernel).
// BN = 32: three waves per SIMD (168 registers, none spilled: a spill's reload would wait for every direct load in flight), three tiles
// of 16 KB in LDS (D = 128).  The tile two ahead is loaded behind the current one's products: issued in front of them, the loads hold
// up all waves of a compute unit at the same point (zeros, 13B layer / high resolution: 263 / 608 us behind, 289 / 648 in front).  The
// products of S^T run at raised wave priority, so that one wave's softmax meets another's products (normal values 354 / 866 with,
// 357 / 880 without).
// BN = 64: two waves per SIMD, two tiles of 32 KB; a wave that is alone on its SIMD takes a tile of 64 keys faster than two of 32.
// us a call, 32x32x16 MFMAs on 64-key tiles at two waves per SIMD -> BN = 32 (where not every launch below is at its rule's side: long_tiles):
// 13B layer batch 32 370 -> 330, high resolution batch 8 908 -> 820, 320 strips x 739 94.4 -> 85.8, 1280 x 200 64.6 -> 52.2, 96 x 8192 2170 ->
// 1921, D = 64: 1280 x 739 208 -> 196.
template <int D, bool SPREAD, int BN>
__global__ __launch_bounds__(256, BN == 32 ? 3 : 2) void prefill_mfma_kernel(PrefillArgs a) {
    using L = TileLayout<D, BN>;
    constexpr int kRing = BN == 32 ? 3 : 2;             // tiles in LDS
    __shared__ __attribute__((aligned(1024))) uint16_t buf[kRing * 2 * L::TILE];

    int strip, qt;
    if (SPREAD) place_spread(a, strip, qt);
    else place_workgroup(a, strip, qt);
    const int h = strip % a.H, b = strip / a.H;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, c = lane & 15;
    const int n = a.n;
    // Query tiles are cut from the END of the prompt in whole 32-row blocks: the blocks that a prompt
    // of no multiple of 128 rows leaves empty then sit at the front of a strip's FIRST tile, the one
    // that walks the fewest key tiles, and not behind its last (the one that walks them all).  Such a
    // wave has q0 < 0 and only helps to load tiles.  (Blocks stay aligned to 32 rows and key tiles to
    // their size, which is what the diagonal handling relies on.)
    const int q0 = qt * kBM + wave * 32 - a.q_shift;
    const int64_t bh = (int64_t)b * a.H + h;

    const uint16_t* Qp = reinterpret_cast<const uint16_t*>(a.q) + b * a.q_sb + h * a.q_sh;
    const uint16_t* Kp = reinterpret_cast<const uint16_t*>(a.k) + b * a.k_sb + h * a.k_sh;
    const uint16_t* Vp = reinterpret_cast<const uint16_t*>(a.v) + b * a.v_sb + h * a.v_sh;

    // this lane's part of the direct loads' source: row (wave * RPI + lane / UPR) of a 1 KB group, and the
    // 16-byte unit that the permutation assigns to its LDS slot (the permutations repeat every RPI * 4
    // rows or sooner, so they are the same for every group and every tile), as a byte offset
    uint32_t k_lane, v_lane;
    {
        const int row0 = wave * L::RPI + lane / L::UPR, u = lane % L::UPR;
        const int rowc = min(row0, n - 1);              // a prompt shorter than one group of rows
        k_lane = (uint32_t)(2 * (rowc * a.k_st + (u ^ L::k_swz(row0)) * 8));
        v_lane = (uint32_t)(2 * (rowc * a.v_st + (u ^ L::v_swz(row0)) * 8));
    }
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);     // for scalar address arithmetic only
    const uint32_t lds0 = lds_addr(buf);
    constexpr int kBufBytes = 4 * L::TILE;
    const int k_end = min(n, qt * kBM + kBM - a.q_shift);   // keys this workgroup can see
    const int nt = (k_end + BN - 1) / BN;
    auto issue = [&](int t, int slot) {
        issue_tile<D, BN>(lds0 + slot * kBufBytes, Kp, Vp, k_lane, v_lane, a.k_st, a.v_st, t * BN, n, lane, wave, wave_s);
    };
    issue(0, 0);
    Frag qf[2][D / 32];
    load_queries<D>(a, Qp, b, q0, c, g, qf);
    LaneMap<D> lm;
    lm.init(c, g);
    WaveRows<D> rows;
    rows.init();

    const Window win = window_of(a, bh, q0);
    const bool wave_live = q0 >= 0 && q0 < n;           // else all 32 queries lie outside the prompt
    // Tile t is in slot t % kRing.  A slot is refilled only behind a barrier that every wave has passed since its last read, and a
    // tile is read behind a barrier in front of which every wave has waited for its own loads of it.
    if (kRing == 3 && nt > 1) { issue(1, 1); wait_direct_loads_but<2 * L::NI>(); }
    else wait_direct_loads();
    __syncthreads();
    int slot = 0, next = kRing - 1;
    for (int t = 0; t < nt; ++t) {
        if (kRing == 2 && t + 1 < nt) issue(t + 1, next);
        const int k0 = t * BN;
        if (wave_live && k0 <= q0) consume_tile<D, BN>(lds0 + slot * kBufBytes, k0, q0, qf, rows, a.scale_l2, lm, c, g, win);
        if (kRing == 3 && t + 2 < nt) {
            issue(t + 2, next);
            wait_direct_loads_but<2 * L::NI>();
        } else {
            wait_direct_loads();
        }
        __syncthreads();
        slot = slot == kRing - 1 ? 0 : slot + 1;
        next = next == kRing - 1 ? 0 : next + 1;
    }
    // ---- normalise and store -----------------------------------------------------------------
    const float l_tot[2] = {wave_sum_from<16>(rows.l[0]), wave_sum_from<16>(rows.l[1])};
    uint16_t* obuf = buf + wave * (32 * (D + 8));      // (the tile buffers are free after the last barrier)
    static_assert(4 * 32 * (D + 8) <= kRing * 2 * L::TILE, "the waves' output blocks fit the tile buffers");
    store_block<D>(a, b, h, obuf, rows, l_tot, q0, n, wave_live, lane, g, c);
    keep_row_sums(a, win, bh, c, g, rows.m, l_tot);
}

// The same attention for launches that leave compute units idle (a short prompt, a few sequences).  128 / KS queries per
// workgroup: its four waves are KS groups that own the same query blocks and take the key tiles in turn, tile i to group
// i % KS, KS tiles at a time in LDS.  There are KS times the workgroups and each walks its tiles in a KS-th of the steps; at
// the end group 0 merges the groups' (maximum, sum, accumulator) through LDS.  Bound by the latencies of a step: two workgroups per
// compute unit (64 KB of LDS: tiles of 32 keys, KS = 2 keeps the next two in flight, KS = 4 has room for the current four only) hide
// them from each other, and a wave, at two per SIMD, orders its reads and products as the compiler likes.  us a call, 32x32x16 MFMAs on
// tiles of 64 keys and 128 KB, or without groups where those gained nothing -> so: 32 strips x 310 tokens 16.8 -> 13.5, 16 x 420 14.8 -> 13.4, 64 x 739
// 35.6 -> 27.8, 40 x 739 33.9 -> 25.8, 20 x 1200 49.1 -> 35.5, 8 x 3000 106.7 -> 69.4; D = 64: 32 x 420 12.3 -> 10.8, 16 x 1500 36.8 -> 26.2.
template <int D, int KS>
__global__ __launch_bounds__(256, 2) void prefill_mfma_split_kernel(PrefillArgs a) {
    constexpr int BN = 32, NBUF = KS == 2 ? 2 : 1;
    using L = TileLayout<D, BN>;
    constexpr int DT = D / 16;
    constexpr int NB = 4 / KS;                          // 32-query blocks per workgroup
    constexpr int TILE2 = 2 * L::TILE;                  // elements of a K tile and its V tile
    __shared__ __attribute__((aligned(1024))) uint16_t buf[NBUF * KS * TILE2];
    __shared__ float sm_m[KS][NB][2][64], sm_l[KS][NB][2][64];

    int strip, qt;
    place_workgroup(a, strip, qt);
    const int h = strip % a.H, b = strip / a.H;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, c = lane & 15;
    const int blk = wave % NB, kg = wave / NB;
    const int n = a.n;
    const int q0 = qt * (32 * NB) + blk * 32 - a.q_shift;
    const int64_t bh = (int64_t)b * a.H + h;
    const uint16_t* Qp = reinterpret_cast<const uint16_t*>(a.q) + b * a.q_sb + h * a.q_sh;
    const uint16_t* Kp = reinterpret_cast<const uint16_t*>(a.k) + b * a.k_sb + h * a.k_sh;
    const uint16_t* Vp = reinterpret_cast<const uint16_t*>(a.v) + b * a.v_sb + h * a.v_sh;
    uint32_t k_lane, v_lane;
    {
        const int row0 = wave * L::RPI + lane / L::UPR, u = lane % L::UPR;
        const int rowc = min(row0, n - 1);
        k_lane = (uint32_t)(2 * (rowc * a.k_st + (u ^ L::k_swz(row0)) * 8));
        v_lane = (uint32_t)(2 * (rowc * a.v_st + (u ^ L::v_swz(row0)) * 8));
    }
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t lds0 = lds_addr(buf);
    const int k_end = min(n, qt * (32 * NB) + 32 * NB - a.q_shift);     // keys this workgroup can see
    const int nt = (k_end + BN - 1) / BN;
    // the tiles of step s into buffer half s % NBUF (a tile past the last one is not loaded and not consumed)
    auto load_step = [&](int s) {
#pragma unroll
        for (int i = 0; i < KS; ++i)
            if (s * KS + i < nt)
                issue_tile<D, BN>(lds0 + (uint32_t)(((s % NBUF) * KS + i) * TILE2 * 2), Kp, Vp, k_lane, v_lane, a.k_st, a.v_st,
                              (s * KS + i) * BN, n, lane, wave, wave_s);
    };
    load_step(0);
    Frag qf[2][D / 32];
    load_queries<D>(a, Qp, b, q0, c, g, qf);
    LaneMap<D> lm;
    lm.init(c, g);
    WaveRows<D> rows;
    rows.init();
    const Window win = window_of(a, bh, q0);
    const bool wave_live = q0 >= 0 && q0 < n;

    const int steps = (nt + KS - 1) / KS;
    for (int s = 0; s < steps; ++s) {
        wait_direct_loads();
        __syncthreads();
        if (NBUF == 2 && s + 1 < steps) load_step(s + 1);
        const int t = s * KS + kg;
        if (wave_live && t < nt && t * BN <= q0)       // else the tile lies entirely above this wave's diagonal
            consume_tile<D, BN, true>(lds0 + ((s % NBUF) * KS + kg) * TILE2 * 2, t * BN, q0, qf, rows, a.scale_l2, lm, c, g, win);
        if (NBUF == 1 && s + 1 < steps) {
            __syncthreads();                            // every wave is done with the buffer
            load_step(s + 1);
        }
    }
    // ---- merge the key groups ----------------------------------------------------------------
    // (a lane of every group holds the same query and the same columns)
    __syncthreads();
    f32x4* merge = reinterpret_cast<f32x4*>(buf);       // [KS - 1][NB][2 * DT][64]
#pragma unroll
    for (int qc = 0; qc < 2; ++qc) { sm_m[kg][blk][qc][lane] = rows.m[qc]; sm_l[kg][blk][qc][lane] = rows.l[qc]; }
    if (kg > 0) {
        f32x4* dst = merge + ((kg - 1) * NB + blk) * (2 * DT * 64) + lane;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int qc = 0; qc < 2; ++qc) dst[(2 * dt + qc) * 64] = rows.o[dt][qc];
    }
    __syncthreads();
    if (kg > 0 || !wave_live) return;                   // (no barrier below)
    float l_tot[2];
#pragma unroll
    for (int qc = 0; qc < 2; ++qc) {
        float m = rows.m[qc];                           // (a group without tiles, or with keys of logit -inf only, has sum 0 at the lowest float)
#pragma unroll
        for (int k = 1; k < KS; ++k) m = fmaxf(m, sm_m[k][blk][qc][lane]);
        const float f0 = exp2_fast(rows.m[qc] - m);
        float l = rows.l[qc] * f0;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) rows.o[dt][qc] *= f0;
#pragma unroll
        for (int k = 1; k < KS; ++k) {
            const float f = exp2_fast(sm_m[k][blk][qc][lane] - m);
            l = fmaf(sm_l[k][blk][qc][lane], f, l);
            const f32x4* src = merge + ((k - 1) * NB + blk) * (2 * DT * 64) + lane;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) rows.o[dt][qc] += src[(2 * dt + qc) * 64] * f;
        }
        rows.m[qc] = m;
        l_tot[qc] = wave_sum_from<16>(l);
    }
    constexpr int kMergeElems = (KS - 1) * NB * 2 * DT * 64 * 8;       // of the merge area, in 16-bit elements
    static_assert(kMergeElems + NB * 32 * (D + 8) <= NBUF * KS * TILE2, "merge area and output blocks fit the tile buffers");
    store_block<D>(a, b, h, buf + kMergeElems + blk * (32 * (D + 8)), rows, l_tot, q0, n, true, lane, g, c);
    keep_row_sums(a, win, bh, c, g, rows.m, l_tot);
}

// Key groups for a launch (1: the kernel without groups).  The device holds 512 workgroups of the split kernel at D = 128, twice as many at
// D = 64; groups pay while all workgroups find a place at once, and a little beyond where few strips are long.  us a call, 1 / 2 / 4 groups
// (strips x tokens), D = 128:
//   four while (n / 32) strips <= 256, or <= 768 with up to 12 strips: 8 x 739 30.4 / 21.4 / 17.2, 32 x 250 14.8 / 11.9 / 10.9, 8 x 2000 70.1 / 45.9 /
//   39.1, 12 x 1500 54.1 / 42.2 / 37.3, 8 x 3000 100 / 71.4 / 69.4, 32 x 310 17.1 / 13.5 / 13.2, but 40 x 250 15.4 / 12.4 / 13.2, 20 x 500 22.9 / 17.2 / 18.1, 16 x 1500
//   54.1 / 43.0 / 47.6, 8 x 5000 168 / 124 / 144
//   two while (n / 64) strips <= 512, or <= 768 with up to 64 strips: 128 x 250 16.1 / 15.6, 80 x 300 18.2 / 16.5, 96 x 224 15.1 / 14.9, 64 x 739 33.4 / 27.8, 40 x
//   1000 41.6 / 40.2, 32 x 1500 57.1 / 40.7, 16 x 3000 104 / 95.9, but 80 x 420 21.7 / 22.7, 160 x 200 16.0 / 17.7, 120 x 300 20.1 / 22.0; prompts of one
//   query tile up to 128 strips: 128 x 100 10.9 / 10.6, 200 x 100 11.3 / 11.8
// D = 64 (four up to 1024 or 1536, two up to 768 or 1536): 20 x 1000 30.8 / 24.6 / 21.5, 32 x 1000 31.3 / 21.7 / 17.7, 128 x 200 12.3 / 11.1 / 10.9, 16 x 3000 79.4 / 65.0 /
// 59.4; 128 x 300 14.9 / 12.8 / 13.5, 256 x 150 11.7 / 10.8 / 13.5, 64 x 1500 47.7 / 45.7, but 256 x 200 14.5 / 15.8, 128 x 500 21.1 / 24.5, 160 x 380 17.6 / 18.9.
// Prompts of up to 64 tokens are one key tile or two: a second group saves a step and the merge takes it back, or more.  us a launch without the mass, 1 / 2 / 4
// groups, D = 128: 32 x 33 5.0 / 5.2 / 6.0, 32 x 64 5.2 / 5.5 / 6.0, 128 x 48 5.3 / 5.5 / 6.2, 320 x 64 8.4 / 9.4 / 13.4, 1280 x 33 15.2 / 16.9 / 30.3; D = 64: 32 x 33
// 3.9 / 3.9 / 4.3, 128 x 64 4.1 / 4.1 / 4.4, 640 x 48 6.5 / 7.0 / 9.0, 1280 x 48 10.1 / 9.6 / 13.7.
int key_groups(int D, int n, int64_t strips) {
    if (n <= 64) return 1;
    const bool d128 = D == 128;
    const int64_t four = (n + 31) / 32 * strips, two = (n + 63) / 64 * strips;
    if (four <= (d128 ? 256 : 1024) || (strips <= (d128 ? 12 : 16) && four <= (d128 ? 768 : 1536))) return 4;
    if (n <= 128 && strips > (d128 ? 128 : 256)) return 1;
    return two <= (d128 ? 512 : 768) || (strips <= 64 && two <= (d128 ? 768 : 1536)) ? 2 : 1;
}

// Whether a launch without key groups takes tiles of 64 keys (two workgroups per compute unit, shorter per workgroup) or of 32 (three,
// four at D = 64: more work at a time).  The 64 win while the launch lasts not much longer than its heaviest workgroup: strips * (query
// tiles + 1) / 2 is the number of those that its work amounts to.  us a call, 32 / 64 (strips x tokens), D = 128: 128 x 310 19.9 / 18.7,
// 128 x 675 38.2 / 35.1, 80 x 1500 79.1 / 74.5, 40 x 3000 150 / 130, 320 x 200 20.4 / 19.5, 256 x 300 24.8 / 22.7, 224 x 500 37.0 / 37.3,
// 200 x 600 40.9 / 42.2, 192 x 675 46.6 / 49.9, 320 x 300 29.5 / 31.9, 128 x 1200 76.5 / 78.6, 1280 x 200 52.2 / 59.0, but 256 x 500 40.8 / 39.8, 160 x
// 800 52.0 / 50.2, 120 x 1200 76.0 / 74.4; D = 64: 320 x 739 55.8 / 53.2, 512 x 400 38.1 / 36.2, 256 x 1000 67.3 / 66.7, 384 x 739 61.3 / 62.4, 1280 x
// 200 34.2 / 35.7.
bool long_tiles(int D, int n_qt, int64_t strips) { return strips * (n_qt + 1) < (D == 128 ? 1200 : 2600); }

// Strips of a dispatch lane whose tiles are dealt together at the end of a launch: as many as keep the K and V of an XCD's four
// lanes within about twice its L2 (4 MB), but two to four, or one where one strip of each is more than that.  us a call at 1 / 2 / 4 / 8 strips, D = 128: 256 x 675 66.8 / 62.9 / 56.9 /
// 60.0, 320 x 739 89.5 / 85.2 / 83.1 / 81.0, 1280 x 739 330.5 / 326.6 / 326.5 / 324.9, 140 x 1500 128.6 / 115.2 / 114.1 / 115.6, but 256 x 3136
// 821 / 809 / 822 / 895.  One / two strips, long prompts: 64 x 4096 337 / 330, 128 x
// 4096 677 / 673, 96 x 5120 775 / 780, 128 x 5120 1023 / 1034, 64 x 6144 732 / 738, 96 x 8192 1921 / 1943, 64 x 12288 2862 / 2919.  (Left-over
// strips come first either way, with 32x32x16 MFMAs: 40 x 8192 1103 -> 927.)
int spread_strips(int D, int n, int64_t strips) {
    const int64_t bytes = (int64_t)n * D * 16;          // of one strip of each of the four lanes
    const int64_t fit = ((int64_t)8 << 20) / bytes;
    return (int)std::min<int64_t>(strips / kLanes, fit < 1 ? 1 : std::max<int64_t>(2, std::min<int64_t>(4, fit)));
}

template <int D>
void launch_whole(const PrefillArgs& a, dim3 grid, bool long_t, hipStream_t st) {
    // (prompts of one query tile have no order to choose, and the choice costs them 0.2 of 11 us)
    if (a.n_qt > 1 && long_t) prefill_mfma_kernel<D, true, 64><<<grid, 256, 0, st>>>(a);
    else if (a.n_qt > 1) prefill_mfma_kernel<D, true, 32><<<grid, 256, 0, st>>>(a);
    else if (long_t) prefill_mfma_kernel<D, false, 64><<<grid, 256, 0, st>>>(a);
    else prefill_mfma_kernel<D, false, 32><<<grid, 256, 0, st>>>(a);
}

}  // namespace

st3_status launch_prefill_mfma(const PrefillArgs& a, int B, int D, hipStream_t st) {
    // 8-byte output stores and 16-byte input loads need these alignments (rows are 16-byte aligned already)
    PrefillArgs pa = a;
    const int ks = key_groups(D, a.n, (int64_t)a.H * B);
    const int bm = kBM / ks;
    pa.n_qt = (a.n + bm - 1) / bm;
    pa.q_shift = (pa.n_qt * bm - a.n) / 32 * 32;        // whole empty 32-row blocks, moved to the front
    pa.B = B;
    const int64_t strips = (int64_t)a.H * B, wgs = pa.n_qt * strips;
    if (wgs > 0x7fffffff) return ST3_ERR_UNSUPPORTED;
    pa.spread = spread_strips(D, a.n, strips);
    // the direct loads address a strip as a scalar base plus a 32-bit byte offset
    if ((int64_t)a.n * a.k_st * 2 >= (int64_t)1 << 31 || (int64_t)a.n * a.v_st * 2 >= (int64_t)1 << 31) return ST3_ERR_UNSUPPORTED;
    dim3 grid((unsigned)wgs);
    if (D != 128 && D != 64) return ST3_ERR_UNSUPPORTED;
    if (ks == 1) {
        if (D == 128) launch_whole<128>(pa, grid, long_tiles(D, pa.n_qt, strips), st);
        else launch_whole<64>(pa, grid, long_tiles(D, pa.n_qt, strips), st);
    } else if (ks == 2) {
        if (D == 128) prefill_mfma_split_kernel<128, 2><<<grid, 256, 0, st>>>(pa);
        else prefill_mfma_split_kernel<64, 2><<<grid, 256, 0, st>>>(pa);
    } else {
        if (D == 128) prefill_mfma_split_kernel<128, 4><<<grid, 256, 0, st>>>(pa);
        else prefill_mfma_split_kernel<64, 4><<<grid, 256, 0, st>>>(pa);
    }
    return ST3_OK;
}

}  // namespace st3
