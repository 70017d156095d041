// How the attention kernels of the two-chain format are launched: wavefronts, tables and spans by sizes alone.  Host code without a
// runtime call, so that every size can be looked at without a GPU; the constants are shared with the kernels (ecco_kernels.hip).
#pragma once

#include <algorithm>
#include <cstddef>

#include "ecco_internal.h"

namespace ecco {

constexpr int kStride = kBlockWords + 1;  // LDS words per staged block (last one is a zero pad)
constexpr int kUnitBlocks = 32;
constexpr int kUnitWords = kUnitBlocks * kStride + 4;  // private payload buffer of a wavefront, in whole pieces of 16 bytes
constexpr int kLdsWords = 160 * 1024 / 4;              // of a compute unit
// LDS words of the decode tables: the long-code lists and the centroids are only copied for models that need them
constexpr int decode_table_words(int S, bool lng) { return S * (kPeekEntries + kK + (lng ? kK + kK / 2 : 0)); }
// Units of 32 tokens in a capacity of `tokens`, which may be any positive number up to 2^31 - 1: of that many units, the tokens no longer
// fit an int.
constexpr int units_of(int tokens) { return (tokens - 1) / kUnitBlocks + 1; }
// Tokens of `units` units, or more than a span ever holds
constexpr int kSpanMax = 8192, kSpanLeast = 2048;
constexpr int span_tokens(int units) { return std::min(units, kSpanMax / kUnitBlocks + 1) * kUnitBlocks; }

// ---- kv_attend_kernel
// Two workgroups of eight wavefronts share a compute unit where there are workgroups for it and both models' tables fit half its
// LDS: each decodes while the other builds or sums (16 patterns, 16 x 32 sequences and heads of 1024 tokens 59.2 -> 48.1 us).  Otherwise
// one of as few wavefronts as take the fewest rounds over the units of a span: a table read costs less the more wavefronts
// wait for theirs (one workgroup, 8192 tokens: 166.7 us with sixteen, 177.9 us with twelve), barriers and sums the more the more
// meet (64 patterns, ten units: 21.5 us with twelve, 22.2 us with sixteen; two units: 15.8 us with eight, 16.5 us with twelve).  The
// decoders of long codes need the registers of twelve.
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
    if (wgs > (size_t)cus && two.both) return two;
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
// Two workgroups of eight wavefronts share a compute unit where there are workgroups for it and both models' tables fit half its
// LDS (16 patterns, 16 x 32 heads in groups of 2, 1000 tokens: 57.4 -> 44.9 us).  Otherwise one of as few wavefronts as take the fewest
// rounds over the units of a range (with 16 patterns: 16 units 23.6 us with sixteen, 24.6 us with twelve; 8 units 17.9 us with eight,
// 19.3 us with twelve, 20.6 us with sixteen).  The decoders of long codes need the registers of twelve.
struct GqaPlan {
    int waves;
    int table_words;  // LDS words of the tables: both models', or the larger one's
    int both;         // the V tables have their own place, behind those of K
    int span;         // tokens per span, a multiple of 32
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
        if (p.span < tokens && p.span > round) p.span -= p.span % round;
        p.lds = (size_t)std::max(p.table_words + fixed + grp * gqa_score_stride(p.span), gqa_state_words(waves) + waves * 8 * kRedTile) * 4;
        return p;
    };
    if (lk || lv) return plan(12, kLdsWords);
    const GqaPlan two = plan(8, kLdsWords / 2);
    if (wgs > (size_t)cus && two.both) return two;
    const auto rounds = [&](int waves) { return (units + waves - 1) / waves; };
    const int waves = rounds(8) == rounds(16) ? 8 : rounds(12) == rounds(16) ? 12 : 16;
    return plan(waves, kLdsWords);
}

}  // namespace ecco
