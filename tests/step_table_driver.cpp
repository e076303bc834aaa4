// Packs random layers into the entries of a step's tables and unpacks them again: what fits comes back as it was, for both kinds of
// either table, and what does not fit is refused.
#include <cstdio>
#include <cstring>
#include <random>

#include "st3_step.h"

using namespace st3;

static std::mt19937_64 rng(7);
static int64_t upto(int64_t n) { return (int64_t)(rng() % (uint64_t)(n + 1)); }
template <typename P>
static void ptr(P& p) { p = reinterpret_cast<P>(upto(3) == 0 ? 0 : (rng() >> (16 + upto(20))) & ~15ull); }

static StepLayer random_layer(int eb, bool wide = false) {
    StepLayer e{};
    ptr(e.q); ptr(e.k); ptr(e.v); ptr(e.k_new); ptr(e.v_new); ptr(e.out); ptr(e.kv_len); ptr(e.vis_len); ptr(e.tail_start);
    ptr(e.score_col); ptr(e.id_col); ptr(e.mass); ptr(e.ws); ptr(e.k_scale); ptr(e.v_scale);
    const int64_t unit = 16 / eb;
    e.stride_b = (upto(1) ? 0xffffffffll : upto(1 << 20)) * unit; e.stride_h = upto(0xffffffffll) * unit;
    e.stride_t = (int32_t)((upto(1) ? 0xffff : 1 + upto(100)) * unit);
    e.col_stride = (int32_t)upto(0x7fffffff); e.mass_stride = (int32_t)upto(0x7fffffff);
    e.sys_len = (int32_t)(upto(1) ? 0xffff : upto(50)); e.max_vis = (int32_t)upto(8192); e.max_kv = (int32_t)upto(0x7ffffff0);
    e.keep_count = (int32_t)upto(8193) - 1; e.chunk = 32 * (int32_t)(1 + upto(0xfffe)); e.capacity = (int32_t)upto(0x7fffffff);
    e.nsplit = (uint8_t)(1 + upto(63)); e.nsplit_cap = (uint8_t)(1 + upto(63)); e.src_nsplit_cap = (uint8_t)upto(64);
    if (wide) {         // beyond what the other entries hold, up to what a cache can have
        e.stride_b = upto((1ll << 47)) * unit; e.stride_h = upto(1ll << 40) * unit; e.stride_t = (int32_t)(upto(0x7fffffff) / unit * unit);
        e.sys_len = (int32_t)upto(0x7fff0000 - 0x10000); e.chunk = 32 * (int32_t)(1 + upto((1 << 26) - 2));
    }
    e.flags = (uint8_t)(upto(63) & ~kStepE4M3) | (eb == 1 ? kStepE4M3 : 0);
    if (e.flags & kStepLazy) { e.hint_base = e.capacity / 2; e.hint_gap = 0; }
    else if (upto(2) == 0) { e.hint_base = 0x7fffffff; e.hint_gap = 0; }
    else { e.hint_base = e.sys_len + (int32_t)upto(8192); e.hint_gap = (int32_t)upto(0x7fffffff); }
    return e;
}

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
#define SAME(f) CHECK(a.f == e.f)

static int check(int eb, bool wide) {
    for (int i = 0; i < 20000; ++i) {
        const StepLayer e = random_layer(eb, wide && i % 4 != 0);
        CHECK(step_layer_fits(e, eb, wide));
        uint32_t w[64];
        std::memset(w, i % 2 ? 0xff : 0, sizeof(w));        // (a table's words start out as anything)
        const uint32_t guard = w[63];
        const int words = eb == 1 ? kAttendWordsE4M3 : kAttendWords;
        uint32_t* high = w + words;                         // (as an entry is left in a workspace)
        pack_attend(w, e, eb == 1, eb, wide ? high : nullptr);
        CHECK(w[words + (wide ? kWideWords : 0)] == guard);
        StepLayer a = eb == 1 ? unpack_attend<true>(w, eb, high, wide) : unpack_attend<false>(w, eb, high, wide);
        SAME(q); SAME(k); SAME(v); SAME(k_new); SAME(v_new); SAME(out); SAME(kv_len); SAME(vis_len); SAME(tail_start); SAME(score_col);
        SAME(id_col); SAME(ws); SAME(stride_b); SAME(stride_h); SAME(stride_t); SAME(col_stride); SAME(sys_len); SAME(max_vis);
        SAME(max_kv); SAME(keep_count); SAME(chunk); SAME(hint_base); SAME(hint_gap); SAME(capacity); SAME(nsplit); SAME(nsplit_cap);
        SAME(src_nsplit_cap); SAME(flags);
        if (eb == 1) { SAME(k_scale); SAME(v_scale); }
        uint32_t lw[kLeftWords + 1];
        lw[kLeftWords] = 0x55u;
        pack_left(lw, e, w);
        a = unpack_left(lw, eb == 1 ? 2 : eb, wide);
        CHECK(lw[kLeftWords] == 0x55u);
        SAME(k); SAME(v); SAME(out); SAME(kv_len); SAME(vis_len); SAME(tail_start); SAME(ws); SAME(mass); SAME(score_col); SAME(id_col);
        SAME(stride_b); SAME(stride_h); SAME(stride_t); SAME(mass_stride); SAME(col_stride); SAME(sys_len); SAME(max_vis); SAME(max_kv);
        SAME(keep_count); SAME(chunk); SAME(capacity); SAME(nsplit); SAME(nsplit_cap); SAME(src_nsplit_cap); SAME(flags);
        if (e.flags & kStepLazy) { SAME(q); SAME(hint_base); }
        for (int ranking = 0; ranking < 2; ++ranking) {
            std::memset(w, i % 2 ? 0xff : 0, sizeof(w));
            uint32_t* high = w + (ranking ? kPlanWords : kFinishWords) + 5;
            pack_plan(w, e, ranking, eb, wide ? high : nullptr);
            CHECK(w[ranking ? kPlanWords : kFinishWords] == guard && (wide || high[0] == guard) && high[kWideWords] == guard);
            a = ranking ? unpack_plan<true>(w, eb == 1 ? 2 : eb, high, wide) : unpack_plan<false>(w, eb == 1 ? 2 : eb, high, wide);
            SAME(k); SAME(v); SAME(out); SAME(kv_len); SAME(vis_len); SAME(tail_start); SAME(ws); SAME(mass); SAME(stride_b);
            SAME(stride_h); SAME(stride_t); SAME(mass_stride); SAME(sys_len); SAME(max_vis); SAME(max_kv); SAME(keep_count); SAME(chunk);
            SAME(capacity); SAME(nsplit); SAME(nsplit_cap); SAME(src_nsplit_cap); SAME(flags);
            if (e.flags & kStepLazy) { SAME(q); SAME(hint_base); }
            if (ranking) { SAME(score_col); SAME(id_col); SAME(col_stride); }
        }
    }
    StepLayer e = random_layer(eb);
    const StepLayer good = e;
    e.q = reinterpret_cast<const void*>(1ull << 48); CHECK(!step_layer_fits(e, eb) && !step_layer_fits(e, eb, true)); e = good;
    if (wide) {         // what a wide entry is for, and what it does not hold either
        e.stride_t = (1 << 16) * 16 / eb; CHECK(!step_layer_fits(e, eb) && step_layer_fits(e, eb, true)); e = good;
        e.stride_t = 0x7fffffff / 16 * 16; CHECK(step_layer_fits(e, eb, true)); e = good;
        e.sys_len = 0x7fff0000; e.hint_base = 0x7fffffff; CHECK(step_layer_fits(e, eb, true)); e = good;
        e.chunk = 0x7fffffe0; CHECK(step_layer_fits(e, eb, true)); e = good;
        e.stride_b = (1ll << 48) * 16 / eb; CHECK(!step_layer_fits(e, eb, true)); e = good;
        e.stride_t += 1; CHECK(!step_layer_fits(e, eb, true));
        return 0;
    }
    e.stride_b = (1ll << 32) * 16 / eb; CHECK(!step_layer_fits(e, eb)); e = good;
    e.stride_h = (1ll << 32) * 16 / eb; CHECK(!step_layer_fits(e, eb)); e = good;
    e.stride_t = (1 << 16) * 16 / eb; CHECK(!step_layer_fits(e, eb)); e = good;
    e.stride_t = 16 / eb + 1; CHECK(eb == 16 || !step_layer_fits(e, eb)); e = good;
    e.sys_len = 1 << 16; CHECK(!step_layer_fits(e, eb)); e = good;
    e.chunk = 32 << 16; CHECK(!step_layer_fits(e, eb)); e = good;
    e.flags &= (uint8_t)~kStepLazy; e.hint_base = e.sys_len + 0xffff; CHECK(!step_layer_fits(e, eb));
    return 0;
}

// A full table: the last entry ends where the upper halves begin.
static int check_room() {
    static uint32_t table[kStepTableWords];
    for (int words : {kAttendWords, kAttendWordsE4M3, kFinishWords, kPlanWords}) {
        const int wide = entries_per_table(words, 1), narrow = entries_per_table(words, 0);
        CHECK(high_words(table, wide - 1) >= table + wide * words && narrow * words <= kStepTableWords);
        CHECK(high_words(table, narrow - 1) >= table && high_words(table, 0) + kWideWords == table + kStepTableWords);      // (loaded always)
    }
    CHECK(entries_per_table(kAttendWords, 0) == 35 && entries_per_table(kAttendWordsE4M3, 0) == 32 && entries_per_table(kFinishWords, 0) == 41 &&
          entries_per_table(kPlanWords, 0) == 35);
    return 0;
}

// The attention's grid has at most 65535 slices, whatever batch a shape may have.
static int check_grid() {
    for (int H = 1; H <= 1024; H += H < 70 ? 1 : 53)
        for (int B = 1; B <= 65535; B += B < 300 || B > 32000 ? 1 : 97) {
            const int most = max_layers_ranked(B, H);
            for (int layers = most > 2 ? most - 2 : 1; layers <= most; ++layers)
                for (int chunks : {1, 2, 64}) {
                    const int64_t z = rank_rows_z(B, H, chunks, layers);
                    CHECK(z * H * chunks >= (int64_t)B * layers && z + (int64_t)B * layers <= 65535);
                }
        }
    CHECK(max_layers_ranked(43690, 2) == 0 && max_layers_ranked(43689, 2) == 1 && max_layers_ranked(1, 32) > 35);
    return 0;
}

int main() {
    if (check_room() || check_grid()) return 1;
    for (int eb : {1, 2, 4})
        if (check(eb, false) || check(eb, true)) return 1;
    std::printf("ok\n");
    return 0;
}
