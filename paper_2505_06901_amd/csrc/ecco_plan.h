// How the attention kernels of the two-chain format are launched: wavefronts, tables and spans by sizes alone.  Host code without a
// runtime call, so that every size can be looked at without a GPU; the constants are shared with the kernels (ecco_kernels.hip).
#pragma once

#include <algorithm>
#include <cstddef>

#include "ecco_internal.h"

namespace ecco {

constexpr int kStride = kBlockWords + 1;  // LDS words per staged block (last one is a zero pad)
constexpr int kUnitBlocks = 32;
// private payload buffer of a wavefront, and behind it two words that a chain of whole windows reads, though it does not use them
constexpr int kUnitWords = kUnitBlocks * kStride + 4;
constexpr int kLdsWords = 160 * 1024 / 4;              // of a compute unit
// LDS words of the decode tables: the long-code lists and the centroids are only copied for models that need them
constexpr int decode_table_words(int S, bool lng) { return S * (kPeekEntries + kK + (lng ? kK + kK / 2 : 0)); }
// Units of 32 tokens in a capacity of `tokens`, which may be any positive number up to 2^31 - 1: of that many units, the tokens no longer
// fit an int.
constexpr int units_of(int tokens) { return (tokens - 1) / kUnitBlocks + 1; }
// Tokens of `units` units, or more than a span ever holds
constexpr int kSpanMax = 8192, kSpanLeast = 2048;
constexpr int span_tokens(int units) { return std::min(units, kSpanMax / kUnitBlocks + 1) * kUnitBlocks; }

// Whether two workgroups are to share a compute unit, each with half of the wavefronts that one alone would have: the other's decoding
// then covers what is fixed per workgroup, but a sequence by itself takes longer.  `units`: of the longest sequence (or range) that may come.
// It is taken where that one, if it is the only long one, is no more than the work of a compute unit otherwise: 16 units per workgroup there.
// 16 patterns, alone -> shared, in us, at full capacity / lengths drawn evenly / one sequence of full length beside others of an eighth of it:
//    288 workgroups of 500 tokens   32.0 -> 25.0     26.3 -> 20.3     23.8 -> 18.9     shared
//    512 of 1024                    50.7 -> 43.2     36.6 -> 33.7     34.7 -> 30.7     shared
//   1024 of 1024                    96.2 -> 79.9     76.8 -> 63.3     55.9 -> 32.2     shared
//    288 of 4096                   149.9 -> 140.8    87.5 -> 126.5    75.9 -> 102.6
//    384 of 2048                    82.4 -> 75.4     55.9 -> 58.0     41.8 -> 53.9
//    512 of 4096                   153.6 -> 145.0   133.6 -> 133.4    76.0 -> 103.6
//    768 of 2048                   123.6 -> 118.3   104.1 -> 96.3     49.6 -> 55.6
// Grouped queries, ranges of as many tokens: 320 of 3000 133.8 -> 125.2, 85.2 -> 102.0, 67.5 -> 82.8; 512 of 500 36.7 -> 29.3, 35.1 -> 28.0,
// 30.5 -> 20.1; 512 of 2000 97.5 -> 87.7, 79.7 -> 74.0, 49.0 -> 57.9; 1024 of 1000 108.6 -> 88.9, 97.0 -> 75.2, 60.3 -> 34.8.
inline bool share_units(size_t wgs, int units, int cus) { return wgs > (size_t)cus && (size_t)units * (size_t)cus <= 16 * wgs; }

// ---- kv_attend_kernel
// Two workgroups of eight wavefronts share a compute unit where there are workgroups for it and both models' tables fit half its
// LDS: each decodes while the other builds or sums.  Otherwise one workgroup takes it, of as few wavefronts as take the fewest rounds over the units
// of the capacity: a table read costs less the more wavefronts wait for theirs (one workgroup, 8192 tokens: 166.7 us with sixteen,
// 177.9 us with twelve), barriers and sums the more the more meet (64 patterns, ten units: 21.5 us with twelve, 22.2 us with sixteen;
// two units: 15.8 us with eight, 16.5 us with twelve).  The decoders of long codes need the registers of twelve.
struct AttnPlan {
    int waves;
    int table_words;  // LDS words of the tables: both models', or the larger one's
    int both;         // the V tables have their own place, behind those of K
    int span;         // tokens per span, a multiple of 32
    size_t lds;
};
inline AttnPlan attn_plan(int Sk, bool lk, int Sv, bool lv, size_t wgs, int T_max, int cus) {
    const int wk = decode_table_words(Sk, lk), wv = decode_table_words(Sv, lv), units = units_of(T_max), tokens = span_tokens(units);
    const auto plan = [&](int waves, int lds_words) {
        AttnPlan p;
        const int fixed = waves * (kUnitWords + 2);
        p.waves = waves;
        p.both = wk + wv + fixed + std::min(kSpanLeast, tokens) <= lds_words;
        p.table_words = p.both ? wk + wv : std::max(wk, wv);
        p.span = std::min({kSpanMax, tokens, (lds_words - p.table_words - fixed) / kUnitBlocks * kUnitBlocks});
        p.lds = (size_t)(p.table_words + fixed + p.span) * 4;
        return p;
    };
    if (lk || lv) return plan(12, kLdsWords);
    const AttnPlan two = plan(8, kLdsWords / 2);
    if (two.both && share_units(wgs, units, cus)) return two;
    const auto rounds = [&](int waves) { return (units + waves - 1) / waves; };
    const int waves = rounds(8) == rounds(16) ? 8 : rounds(12) == rounds(16) ? 12 : 16;
    return plan(waves, kLdsWords);
}

// ---- kv_attend_gqa_kernel
constexpr int kGqaMaxGroup = 16;
constexpr int kTileStride = 20;                 // words per row of the transposition tile: 32 tokens (16 words) + 4 of padding
constexpr int kTileWords = 16 * kTileStride;
constexpr int kGqaScoreWords = 7936;            // query heads x tokens of a span kept in LDS, at most
constexpr int kRedTile = 276, kRedRow = 68;     // words of a tile, and of 16 lanes of it, in the sum over wavefronts (skewed over the banks)
constexpr int gqa_state_words(int waves) { return 2 * waves * kGqaMaxGroup; }  // per wavefront and head: maximum, denominator

constexpr int gqa_score_stride(int span) { return span + 4; }   // words: 16-byte aligned, and 4 modulo 32 so that heads fall on different banks
// As AttnPlan, but eight wavefronts up to 8 units of a range (17.9 us, 19.3 us with twelve) and twelve beyond.  (Sixteen, in us for a quarter of the
// capacity / all of it: 16 units, 16 patterns, groups of 4 15.4 -> 16.5 / 21.6 -> 21.2, groups of 8 16.5 -> 18.2 / 22.7 -> 22.7, 64 patterns 17.6 -> 19.1
// / 24.1 -> 24.2; 32 units at all of it 31.7 -> 32.7, 64 patterns 33.1 -> 34.6, groups of 8 38.6 -> 40.6.)
struct GqaPlan {
    int waves;
    int table_words;  // LDS words of the tables: both models', or the larger one's
    int both;         // the V tables have their own place, behind those of K
    int span;         // tokens of a span that the LDS holds, a multiple of 32
    int step;         // tokens per span of a range that takes several: whole rounds of the wavefronts, where a span holds one
    size_t lds;
};
inline GqaPlan gqa_plan(int Sk, bool lk, int Sv, bool lv, int grp, size_t wgs, int units, int cus) {
    const int wk = decode_table_words(Sk, lk), wv = decode_table_words(Sv, lv), tokens = span_tokens(units);
    const auto plan = [&](int waves, int lds_words) {
        const int fixed = waves * (kUnitWords + kTileWords) + gqa_state_words(waves);
        GqaPlan p;
        p.waves = waves;
        const int round = std::min(units, waves) * kUnitBlocks;  // tokens that the wavefronts take at a time
        p.both = wk + wv + fixed + grp * gqa_score_stride(round) <= lds_words;
        p.table_words = p.both ? wk + wv : std::max(wk, wv);
        const int scores = std::min(kGqaScoreWords, lds_words - p.table_words - fixed);
        p.span = std::min((scores / grp - 4) & ~(kUnitBlocks - 1), tokens);
        p.step = p.span < tokens && p.span > round ? p.span - p.span % round : p.span;
        p.lds = (size_t)std::max(p.table_words + fixed + grp * gqa_score_stride(p.span), gqa_state_words(waves) + waves * 8 * kRedTile) * 4;
        return p;
    };
    if (lk || lv) return plan(12, kLdsWords);
    const GqaPlan two = plan(8, kLdsWords / 2);
    if (two.both && share_units(wgs, units, cus)) return two;
    return plan(units <= 8 ? 8 : 12, kLdsWords);
}

}  // namespace ecco
