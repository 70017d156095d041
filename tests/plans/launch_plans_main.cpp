// Walks the launch plans of the attention kernels (csrc/ecco_plan.h) over their whole range of sizes and prints the first one that
// the kernels could not run: spans are positive multiples of 32 that make progress, everything fits the LDS that the plan asks for.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "ecco_plan.h"

using namespace ecco;

static long checked = 0;

static void expect(bool ok, const char* what, const char* which, int S, bool lng, int grp, size_t wgs, long long tokens, int waves, int span, size_t lds) {
    ++checked;
    if (ok) return;
    std::printf("%s: %s at S %d long %d group %d workgroups %zu tokens %lld: waves %d span %d lds %zu\n", which, what, S, lng, grp, wgs, tokens, waves, span, lds);
    std::exit(1);
}

int main() {
    const int most = 0x7FFFFFFF;
    const std::vector<int> sizes = {1, 31, 32, 33, 256, 257, 300, 384, 385, 512, 513, 960, 961, 1000, 1024, 1025, 2048, 4096, 8191, 8192, 8193, 8224, 8225, 9000, 100000, 1 << 30,
                                    most - 63, most - 32, most - 31, most - 30, most - 1, most};
    for (int S = 1; S <= kMaxS; ++S)
        for (int lk = 0; lk < 2; ++lk)
            for (int lv = 0; lv < 2; ++lv)
                for (int Sv : {S, 1, kMaxS})
                    for (size_t wgs : {(size_t)1, (size_t)256, (size_t)257, (size_t)512, (size_t)1024, (size_t)100000})
                        for (int T : sizes) {
                            const bool lng = lk || lv;
                            const AttnPlan p = attn_plan(S, lk, Sv, lv, wgs, T, 256);
                            const auto check = [&](bool ok, const char* what) { expect(ok, what, "plain", S, lng, 1, wgs, T, p.waves, p.span, p.lds); };
                            check(lng ? p.waves == 12 : p.waves == 8 || p.waves == 12 || p.waves == 16, "wavefronts");
                            check(p.span >= kUnitBlocks && p.span % kUnitBlocks == 0, "span");
                            const int wk = decode_table_words(S, lk), wv = decode_table_words(Sv, lv);
                            check(p.table_words >= (p.both ? wk + wv : std::max(wk, wv)), "tables");
                            check(p.lds <= 160 * 1024, "limit");
                            check(p.lds == 4 * ((size_t)p.table_words + (size_t)p.waves * (kUnitWords + 2) + (size_t)p.span), "room");
                            for (int grp : {1, 2, 4, 7, 8, 9, 16})
                                for (int n_splits : {1, 2, 3, 16, 256}) {
                                    const int units = ((T - 1) / kUnitBlocks + n_splits) / n_splits;
                                    const GqaPlan g = gqa_plan(S, lk, Sv, lv, grp, wgs, units, 256);
                                    const auto checkg = [&](bool ok, const char* what) { expect(ok, what, "grouped", S, lng, grp, wgs, (long long)units * 32, g.waves, g.span, g.lds); };
                                    checkg(g.waves == 12 || (!lng && g.waves == 8), "wavefronts");
                                    checkg(g.span >= kUnitBlocks && g.span % kUnitBlocks == 0, "span");
                                    checkg(g.step >= kUnitBlocks && g.step % kUnitBlocks == 0 && g.step <= g.span, "step");
                                    checkg(g.table_words >= (g.both ? wk + wv : std::max(wk, wv)), "tables");
                                    checkg(g.lds <= 160 * 1024, "limit");
                                    checkg(g.lds >= 4 * ((size_t)g.table_words + (size_t)g.waves * (kUnitWords + kTileWords) + gqa_state_words(g.waves) + (size_t)grp * gqa_score_stride(g.span)), "room");
                                    checkg(g.lds >= 4 * ((size_t)gqa_state_words(g.waves) + (size_t)g.waves * 8 * kRedTile), "room of the sums");
                                }
                        }
    // Two workgroups share a compute unit (half of its LDS each) where no single sequence can outlast the work of
    // a compute unit otherwise, not where a few long ones decide.
    struct Shared { size_t wgs; int tokens; bool shared; };
    for (const Shared c : {Shared{256, 512, false}, {257, 512, true}, {257, 513, false}, {288, 4096, false}, {384, 1024, false}, {512, 1024, true}, {1024, 4096, false}, {2048, 4096, true}, {2048, 500, true}}) {
        const AttnPlan p = attn_plan(16, false, 16, false, c.wgs, c.tokens, 256);
        expect((p.lds <= 80 * 1024 && p.waves == 8 && p.both) == c.shared, "sharing", "plain", 16, false, 1, c.wgs, c.tokens, p.waves, p.span, p.lds);
        const GqaPlan g = gqa_plan(16, false, 16, false, 4, c.wgs, units_of(c.tokens), 256);
        expect((g.lds <= 80 * 1024 && g.waves == 8 && g.both) == c.shared, "sharing", "grouped", 16, false, 4, c.wgs, c.tokens, g.waves, g.span, g.lds);
    }
    // a range that the LDS holds whole is one span, however long the capacity is; of longer ones every span but the last is whole rounds
    const GqaPlan g = gqa_plan(64, false, 64, false, 8, 256, 32, 256);
    expect(g.span >= 928 && g.step % (g.waves * kUnitBlocks) == 0, "spans", "grouped", 64, false, 8, 256, 1024, g.waves, g.span, g.lds);
    std::printf("%ld conditions hold\n", checked);
    return 0;
}
