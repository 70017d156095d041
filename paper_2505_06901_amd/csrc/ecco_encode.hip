// Encoders of the two-chain block format for gfx950: bulk (ecco_encode, ecco_encode_minmax) and appended tokens
// (ecco_kv_append, ecco_kv_append_minmax).
//
// What bounds them.  Rating all S patterns value by value is 24 vector instructions per value and pattern for 16
// candidates: 48 wavefront instructions per group and pattern, 4 ns per group on the whole chip at S = 64, where reading
// the group and writing its block takes 0.06 ns.  The search is therefore done in two steps (ecco_search.h): bounds on
// every pattern's error from a matrix product of the group's histogram with tables of the model, 16 groups x 16 patterns at
// a time on the matrix cores, and the exact FP32 error only for the patterns whose bounds overlap the best (1.3 to 2 of 64 on
// weights, keys and values).  The chosen pattern, the indices and the block are those of the plain search, bit for bit.
// A group lies in a row of 16 lanes (ecco_rows.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ecco_launch.h"
#include "ecco_rows.h"
#include "ecco_stream.h"

using namespace ecco;
using namespace ecco_rows;

namespace {

constexpr int kHalf = kGroup / 2;
constexpr int kMinmaxThreads = 256;                                    // workgroup of the min/max encoder: 16 groups at a time
constexpr int kMinmaxBatch = kMinmaxThreads / 64 * kWaveRows;

// where a kernel finds group i and where its block goes
struct BulkIo {
    static constexpr bool kDense = true;  // blocks are written one behind the other
    const uint32_t* src;
    uint32_t* blocks;
    uint32_t* meta;
    size_t n;
    __device__ __forceinline__ size_t groups() const { return n; }
    __device__ __forceinline__ const uint32_t* values() const { return src; }
    __device__ __forceinline__ bool place(size_t i, size_t& at) const {
        at = i;
        return i < n;
    }
};
// one new token per sequence and head: group (b, h) goes to the slot seq_len[b] of its cache, if there is one
struct AppendIo {
    static constexpr bool kDense = false;
    const uint32_t* src;
    uint32_t* blocks;
    uint32_t* meta;
    const int32_t* seq_len;
    int n, heads, t_max;
    __device__ __forceinline__ size_t groups() const { return (size_t)n; }
    __device__ __forceinline__ const uint32_t* values() const { return src; }
    __device__ __forceinline__ bool place(size_t i, size_t& at) const {
        if (i >= (size_t)n) return false;
        const int t = seq_len[(uint32_t)i / (uint32_t)heads];
        at = i * t_max + t;
        return t >= 0 && t < t_max;
    }
};
template <class Io>
struct Job {  // one model and the groups it encodes; blockIdx.y picks one of two (keys and values)
    const uint32_t* dev;
    int S;
    Io io;
};

// tables of a model in LDS: near [S][64] (full search) or the min/max selector's bins, near or fine, pair [S][16], codes [S][16] with the
// code on top and 32 - length in the low byte: joined to a stream by one v_alignbit, which takes the word as the shift count
// as well, and the low bytes of up to eight words can be summed with the codes still on top
struct EncTables {
    const uint8_t* near;
    uint32_t pair, fine, enc;  // LDS addresses; pair and enc multiples of 64
};
constexpr int kTableWords = kSearchBins / 4 + 16 + kK;  // per pattern, with near
constexpr size_t minmax_table_words(int S, bool fine) { return (fine ? search_fine_words(S) : search_near_words(S)) + (size_t)S * (16 + kK); }
__device__ __forceinline__ uint32_t code_word(uint32_t enc) { return (enc << (32u - (enc >> 16))) | (32u - (enc >> 16)); }
template <int kThreads, bool kFine>
__device__ __forceinline__ EncTables stage_enc_tables(uint32_t* lds, const uint32_t* __restrict__ dev, int S) {
    const DevLayout D{S};
    const uint4* a = reinterpret_cast<const uint4*>(dev + (kFine ? D.pair() : D.near()));  // near and pair, or pair and fine, follow each other
    const uint4* e = reinterpret_cast<const uint4*>(dev + D.enc());
    uint4* d = reinterpret_cast<uint4*>(lds);
    const int n0 = (int)(S * 16 + (kFine ? search_fine_words(S) : search_near_words(S))) / 4, n1 = S * kK / 4, tid = threadIdx.x;
    constexpr int kMost = kMaxS * (kSearchBins / 4 + 16) / 4;
    static_assert(search_fine_words(kMaxS) == search_near_words(kMaxS), "of the same size");
    constexpr int kPieces = kMost / kThreads + (kMost % kThreads != 0);
    static_assert(kMaxS * kK / 4 <= kThreads, "one piece of the codes per thread");
    // all pieces requested before the first is stored; indices past the end repeat the last piece
    uint4 v[kPieces];
    const uint4 w = e[min(tid, n1 - 1)];
#pragma unroll
    for (int i = 0; i < kPieces; ++i) v[i] = a[min(tid + i * kThreads, n0 - 1)];
    if (tid < n1) d[n0 + tid] = make_uint4(code_word(w.x), code_word(w.y), code_word(w.z), code_word(w.w));
#pragma unroll
    for (int i = 0; i < kPieces; ++i)
        if (tid + i * kThreads < n0) d[tid + i * kThreads] = v[i];
    EncTables t;
    t.near = reinterpret_cast<const uint8_t*>(lds);
    t.pair = lds_address(lds + (kFine ? 0 : S * (kSearchBins / 4)));
    t.fine = lds_address(lds + S * 16);
    t.enc = lds_address(lds + 4 * n0);
    return t;
}

// Packs the row's group with the codes at the LDS address `enc` (a multiple of 64) of its pattern: lane l returns payload word l
// and the meta word.  idx: the lane's eight indices as nibbles, which is also the lane's payload word in raw mode.  image: 18
// words of LDS of the row.  A lane's codes are joined in one 64-bit word (two where the model has codes beyond 8 bits) and go
// into the image with two or three ORs (in runs of 32 bits with two each: min/max selector, 2 x 131072 groups, 16 patterns,
// 37.5 us with that and a scale found apart from the group's ends, 32.7 us so).
template <bool kLong>
__device__ __forceinline__ uint32_t pack_row(uint32_t enc, uint32_t* image, uint32_t idx, int l, uint32_t smax, uint32_t pattern, uint32_t& meta) {
    image[l] = 0u;
    if (l < 2) image[kRowLanes + l] = 0u;
    uint32_t e[kRowValues];
#pragma unroll
    for (int i = 0; i < kRowValues; ++i) e[i] = lds_word(enc | ((i < 7 ? idx >> (26 - 4 * i) : idx << 2) & 60u));
    constexpr int kParts = kLong ? 2 : 1, kRun = kRowValues / kParts;  // codes of kRun values always fit 64 bits together
    uint64_t bits[kParts];
    uint32_t n[kParts], lane_bits = 0;
#pragma unroll
    for (int r = 0; r < kParts; ++r) {
        uint32_t h[2], pad[2];  // the codes of half a run; 32 per value less their bits, in the low byte
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t* c = e + r * kRun + j * (kRun / 2);
            h[j] = c[0] >> (c[0] & 31u);
            pad[j] = c[0];
#pragma unroll
            for (int i = 1; i < kRun / 2; ++i) {
                h[j] = __builtin_amdgcn_alignbit(h[j], c[i], c[i]);
                pad[j] += c[i];
            }
        }
        bits[r] = ((uint64_t)h[0] << (16u * kRun - (pad[1] & 0xFFu))) | h[1];
        n[r] = 32u * kRun - ((pad[0] + pad[1]) & 0xFFu);
        lane_bits += n[r];
    }
    const uint32_t end = row_scan(lane_bits);
    const uint32_t total = row_lane<15>(end), mid = row_lane<7>(end);  // bits of all values, of values 0..63
    const bool raw = total > 8u * ECCO_BLOCK_BYTES;
    wave_fence();
    if (!raw) {
        uint32_t at = end - lane_bits;
#pragma unroll
        for (int r = 0; r < kParts; ++r) {
            const uint64_t v = bits[r] << (64u - n[r]);  // at least two bits: the shift is below 64
            const uint32_t hi = (uint32_t)(v >> 32), lo = (uint32_t)v, third = __builtin_amdgcn_alignbit(lo, 0u, at);
            uint32_t* to = image + (at >> 5);
            atomicOr(to, hi >> (at & 31u));
            atomicOr(to + 1, __builtin_amdgcn_alignbit(hi, lo, at));
            if (third != 0u) atomicOr(to + 2, third);
            at += n[r];
        }
    }
    wave_fence();
    meta = smax | (pattern << 16) | (raw ? 1u << 22 : 0u) | ((raw ? 4u * kHalf : mid) << 23);
    const uint32_t word = raw ? idx : image[l];
    wave_fence();
    return word;
}

// ---- the full search ---------------------------------------------------------------------------------------------------
// Up to 16 patterns the partial sums lie over the histogram: three workgroups then fit a compute unit instead of two (131072
// groups 48.1 -> 44.3 us, 262144 91.3 -> 82.8 us, below 16384 the same).  More patterns take registers for two workgroups only.
constexpr bool search_over(int tiles) { return tiles == 1; }
constexpr size_t search_lds_bytes(int S) {
    const int tiles = search_tiles(S);
    return ((size_t)S * kTableWords + (search_over(tiles) ? search_lds_words<true>(tiles) : search_lds_words<false>(tiles))) * 4;
}

// (six wavefronts per SIMD: the three workgroups)
template <int kTiles, bool kLong, class Io>
__global__ __launch_bounds__(kSearchThreads) __attribute__((amdgpu_waves_per_eu(search_over(kTiles) ? 6 : 4))) void encode_search_kernel(Job<Io> j0, Job<Io> j1) {
    extern __shared__ __align__(16) uint32_t smem[];
    const Job<Io>& job = blockIdx.y ? j1 : j0;
    const int S = job.S, tiles = search_tiles(S);
    const Io io = job.io;
    const int lane = threadIdx.x & 63, l = lane & 15, row = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const SearchLds L = search_lds<search_over(kTiles)>(smem + S * kTableWords, kTiles);
    uint32_t* hist = L.hist + (wave * kWaveRows + row) * kHistStride;
    const size_t batches = (io.groups() + kSearchBatch - 1) / kSearchBatch;
    RowValues v;
    load_values<kSearchBatch>(v, io.values(), io.groups(), blockIdx.x, wave * kWaveRows + row, l);
    Coefs<kTiles> C;
    C.load(job.dev + DevLayout{S}.coef(), wave, tiles, lane);
    const EncTables T = stage_enc_tables<kSearchThreads, false>(smem, job.dev, S);
    // Dealt out (rate_left) where there are more than 16 patterns: 131072 groups under 64 patterns 63.9 -> 60.3 us, 8192 groups 9.7 -> 8.4 us.
    // Of up to 16 the most of four groups is 1.7 where the deal's share is 0.9: it does not pay for itself (44.0 -> 44.6 us, 6.7 -> 6.9 us).
    constexpr bool kDeal = kTiles > 1;
    bool slack_set = false;
    if (l == 0) L.slack[wave * kWaveRows + row] = 0.0f;
    for (size_t b = blockIdx.x; b < batches; b += gridDim.x) {
        __builtin_amdgcn_s_setprio(priority_hist(search_over(kTiles)));
        const uint32_t smax = row_max(lane_absmax(v));
        const float s = half_bits_f(smax);
        const half2_t s2 = splat_half(smax);
        set_slack(L.slack + wave * kWaveRows + row, s, l, slack_set);
        clear_hist(L.hist + wave * kWaveRows * kHistStride, lane);
        wave_fence();
        set_bins<true>(v, kSearchStep * __builtin_amdgcn_rcpf(s), hist, -1);
        wave_fence();
        convert_hist(L.hist + wave * kWaveRows * kHistStride, lane);
        uint64_t left = patterns_left<kTiles, search_over(kTiles)>(L, C, tiles, wave, lane);
        __builtin_amdgcn_s_setprio(kPriorityRate);
        // What the table of nearest centroids does not serve is rated value by value (scan_patterns), scales too small for it
        // from the start.  Of scale 0 all patterns are alike: the first wins with index 0.
        uint64_t later = 0;
        if (!(s >= kSearchLeastScale)) {
            later = smax == 0u ? 0ull : left;
            left = 0;
        }
        uint32_t pattern = 0, idx = 0;
        float best = __builtin_inff();
        if constexpr (kDeal) {
            uint64_t crowded;
            pattern = rate_left<false, 8>(L.hist + wave * kWaveRows * kHistStride, T.near, T.pair, v, smax, -1, left, S, lane, best, crowded);
            later |= crowded;
        } else {
            int rated = 0;
            while (__builtin_amdgcn_ballot_w64(left != 0) != 0ull) {  // the patterns left, ascending; a row that has none left repeats its last one
                const uint32_t p = left != 0 ? (uint32_t)__builtin_ctzll(left) : pattern;
                float sse;
                uint32_t id;
                const uint32_t marks = rate_pattern<true, true>(T.near + p * kSearchBins, T.pair + p * 64u, s2, v, -1, sse, id);
                const uint64_t lanes = __builtin_amdgcn_ballot_w64((marks & ecco::kNearWide) != 0u);
                if (lanes != 0ull && row_any(lanes, row)) {  // this pattern and those after it value by value
                    later |= left;
                    left = 0;
                }
                if (left != 0 && sse < best) {  // strict <: the lowest pattern wins a tie
                    best = sse;
                    pattern = p;
                    idx = id;
                }
                left &= left - 1ull;
                if (++rated == kLookAfter && __builtin_amdgcn_ballot_w64(most_left(left, S)) != 0ull) {
                    later |= left;
                    left = 0;
                }
            }
        }
        bool won = false;  // by the comparison value by value
        if (__builtin_amdgcn_ballot_w64(later != 0) != 0ull)
            scan_patterns(reinterpret_cast<float*>(L.hist + wave * kWaveRows * kHistStride), smem + S * (kSearchBins / 4), v, smax, kGroup, later, lane,
                          best, pattern, won);
        bool scan = won;  // whether the table gives no indices
        if constexpr (kDeal) {
            if (__builtin_amdgcn_ballot_w64(!won && smax != 0u) != 0ull) {
                float none;
                const uint32_t marks = rate_pattern<false, true>(T.near + pattern * kSearchBins, T.pair + pattern * 64u, s2, v, -1, none, idx);
                scan = won || ((marks & ecco::kNearWide) != 0u && smax != 0u);
                idx = smax == 0u ? 0u : idx;
            }
        }
        const uint64_t scans = __builtin_amdgcn_ballot_w64(scan);
        if (scans != 0ull) {
            const uint32_t id = scan_indices(T.pair + pattern * 64u, s2, v, -1);
            idx = row_any(scans, row) ? id : idx;
        }
        __builtin_amdgcn_s_setprio(kPriorityPack);
        // the next group is requested here, when the search has given its registers back
        int last = threadIdx.x & 63;  // the lane taken afresh: what is derived from it is formed here, not kept through the search
        asm volatile("" : "+v"(last));
        const int place = last & 15, group = wave * kWaveRows + (last >> 4);
        load_values<kSearchBatch>(v, io.values(), io.groups(), b + gridDim.x, group, place);
        uint32_t mw;
        const uint32_t word = pack_row<kLong>(T.enc + pattern * (kK * 4u), L.hist + group * kHistStride, idx, place, smax, pattern, mw);
        size_t at;
        if (io.place(b * kSearchBatch + (uint32_t)group, at)) {
            io.blocks[at * kBlockWords + place] = word;
            if (place == 0) io.meta[at] = mw;
        }
    }
}

// ---- the min/max selector ------------------------------------------------------------------------------------------------
// Pattern selector of the online compressor (Section 3.2 "KV Cache Compression", pattern selector of Section 4.3): only the
// group's least and greatest value are compared with each pattern's ends, taken in the group's scale as fp16(centroid * s):
// fitness = (min - first)^2 + (max - last)^2, every operation rounded to FP32 on its own.  The lanes of a row rate the
// patterns l, l + 16, ...; the least fitness wins, the lowest pattern on a tie (pattern 0 if the input held a NaN, against
// the contract).
// (least value, least negated value) of the row; a NaN stays one.  Their magnitudes' greater is the group's scale.
__device__ __forceinline__ half2_t row_ends(const RowValues& v) {
    half2_t lo2 = as_half2(v.x[0]), hi2 = lo2;
#pragma unroll
    for (int i = 1; i < 4; ++i) {
        lo2 = __builtin_elementwise_minimum(lo2, as_half2(v.x[i]));
        hi2 = __builtin_elementwise_maximum(hi2, as_half2(v.x[i]));
    }
    const half2_t ends2 = __builtin_elementwise_minimum(as_half2(__builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, -hi2), __builtin_bit_cast(uint32_t, lo2), 0x05040100u)),
                                                        as_half2(__builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, -hi2), __builtin_bit_cast(uint32_t, lo2), 0x07060302u)));
    return row_all(ends2, [](half2_t a, half2_t b) { return __builtin_elementwise_minimum(a, b); });
}
__device__ __forceinline__ uint32_t select_minmax(const uint32_t* cent, int stride, int S, half2_t s2, half2_t ends2, int l) {
    const float lo = (float)ends2[0], hi = -(float)ends2[1];
    const auto fitness = [&](int p) {
        // first and last centroid: of the words with the ends (stride 1), or of a row of the pattern's pairs
        const uint32_t c = stride == 1 ? cent[p] : __builtin_amdgcn_perm(cent[p * stride + stride - 1], cent[p * stride], 0x07060100u);
        const half2_t e = as_half2(c) * s2;
        const float dlo = __fsub_rn(lo, (float)e[0]), dhi = __fsub_rn(hi, (float)e[1]);
        return __fadd_rn(__fmul_rn(dlo, dlo), __fmul_rn(dhi, dhi));
    };
    uint32_t at = (uint32_t)min(l, S - 1);  // lanes beyond the patterns rate the last one
    float least = fitness((int)at);
    for (int p = l + kRowLanes; p < S; p += kRowLanes) {
        const float f = fitness(p);
        if (f < least) {
            least = f;
            at = (uint32_t)p;
        }
    }
    const float all = row_min_pos(least);
    const uint32_t p = row_min(least == all ? at : 0xFFFFu);
    return p < (uint32_t)S ? p : 0u;
}

// ---- few groups ------------------------------------------------------------------------------------------------------------
// One workgroup per group: its 16 rows of lanes hold the same values and rate a sixteenth of the patterns each, value by
// value.  The search above starts with 120 KB of tables per workgroup and passes through four barriers for 32 groups at a
// time: appending 2 x 256 groups took 9.9 us with it.  Rating with the table of nearest centroids took as long here: among
// all 64 patterns there are always some whose centroids crowd a bin.  With the min/max selector every row selects alike and
// only the index step is left to share.
constexpr int kFewThreads = 256;
constexpr int kFewRows = kFewThreads / kRowLanes;

// least of d and the distances of x's kX-th half to both halves of r
template <int kX>
__device__ __forceinline__ float nearer(float d, uint32_t x, uint32_t r) {
    const float a = half_diff<kX, 0>(x, r), b = half_diff<kX, 1>(x, r);
    float m;
    asm("v_min3_f32 %0, %1, |%2|, |%3|" : "=v"(m) : "v"(d), "v"(a), "v"(b));
    return m;
}

template <bool kMinMax, bool kLong, class Io>
__global__ __launch_bounds__(kFewThreads) void encode_few_kernel(Job<Io> j0, Job<Io> j1) {
    __shared__ __align__(16) uint32_t cent[kMaxS * kK / 2];  // pairs of neighbouring centroids
    __shared__ __align__(64) uint32_t enc[kMaxS * kK];
    __shared__ __align__(16) uint32_t values[kGroup / 2];
    __shared__ __align__(16) uint8_t index[kGroup];
    __shared__ uint32_t row_sse[kFewRows], row_pattern[kFewRows], image[20];
    const Job<Io>& job = blockIdx.y ? j1 : j0;
    const int S = job.S;
    const Io io = job.io;
    const int tid = threadIdx.x, l = tid & 15, row = tid >> 4;
    const size_t g = blockIdx.x;
    size_t at;
    if (!io.place(g, at)) return;  // uniform
    RowValues v;
    load_values<1>(v, io.values(), io.groups(), g, 0, l);
    static_assert(kMaxS * kK / 4 <= kFewThreads, "a piece of each table per thread");
    {
        const DevLayout D{S};
        const int n0 = S * kK / 8, n1 = S * kK / 4;
        const uint4 c = reinterpret_cast<const uint4*>(job.dev + D.cent())[min(tid, n0 - 1)];
        const uint4 e = reinterpret_cast<const uint4*>(job.dev + D.enc())[min(tid, n1 - 1)];
        if (tid < n0) reinterpret_cast<uint4*>(cent)[tid] = c;
        if (tid < n1) reinterpret_cast<uint4*>(enc)[tid] = make_uint4(code_word(e.x), code_word(e.y), code_word(e.z), code_word(e.w));
    }
    if (row == 0) *reinterpret_cast<uint4*>(values + 4 * l) = make_uint4(v.x[0], v.x[1], v.x[2], v.x[3]);
    const uint32_t smax = row_max(lane_absmax(v));
    const half2_t s2 = splat_half(smax);
    __syncthreads();
    uint32_t win;
    if (kMinMax) {
        win = select_minmax(cent, kK / 2, S, s2, row_ends(v), l);
    } else {
        uint32_t pattern = 0;
        float best = __builtin_inff();
        for (int p0 = 0; p0 < S; p0 += kFewRows) {
            const uint32_t p = (uint32_t)min(p0 + row, S - 1);
            const uint4* c = reinterpret_cast<const uint4*>(cent + p * (kK / 2));
            const uint4 c0 = c[0], c1 = c[1];
            const uint32_t pairs[kK / 2] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
            float d[kRowValues];
#pragma unroll
            for (int i = 0; i < kRowValues; ++i) d[i] = __builtin_inff();
#pragma unroll
            for (int k = 0; k < kK / 2; ++k) {
                const uint32_t r = __builtin_bit_cast(uint32_t, as_half2(pairs[k]) * s2);
#pragma unroll
                for (int i = 0; i < kRowValues / 2; ++i) {
                    d[2 * i] = nearer<0>(d[2 * i], v.x[i], r);
                    d[2 * i + 1] = nearer<1>(d[2 * i + 1], v.x[i], r);
                }
            }
            const float sse = tree_sum(d, -1);
            if (p0 + row < S && (sse < best || p0 == 0)) {  // strict <: the lowest pattern wins a tie
                best = sse;
                pattern = p;
            }
        }
        if (l == 0) {
            row_sse[row] = __builtin_bit_cast(uint32_t, best);
            row_pattern[row] = pattern;
        }
        __syncthreads();
        static_assert(kFewRows == kRowLanes, "lane l compares row l");
        const uint32_t sse_l = row_sse[l], least = row_min(sse_l);
        win = row_min(sse_l == least ? row_pattern[l] : 0xFFFFFFFFu);
    }
    // its indices, a value per thread: the last k at which the distance strictly drops (rate_pattern)
    if (tid < kGroup) {
        const uint32_t x = values[tid >> 1] >> (16 * (tid & 1));
        const uint4* c = reinterpret_cast<const uint4*>(cent + win * (kK / 2));
        const uint4 c0 = c[0], c1 = c[1];
        const uint32_t pairs[kK / 2] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
        uint32_t k = 0;
        float last = __builtin_inff();
#pragma unroll
        for (int j = 0; j < kK / 2; ++j) {
            const uint32_t r = __builtin_bit_cast(uint32_t, as_half2(pairs[j]) * s2);
            const float a = fabsf(half_diff<0, 0>(x, r)), b = fabsf(half_diff<0, 1>(x, r));
            k = a < last ? 2u * j : k;
            k = b < a ? 2u * j + 1u : k;
            last = b;
        }
        index[tid] = (uint8_t)k;
    }
    __syncthreads();
    if (row != 0) return;
    const uint2 b = *reinterpret_cast<const uint2*>(index + 8 * l);  // eight indices, a byte each, to nibbles, first on top
    const auto nibbles = [](uint32_t w) { return (w & 15u) << 12 | (w & 0xF00u) | (w >> 12 & 0xF0u) | (w >> 24 & 15u); };
    uint32_t mw;
    const uint32_t word = pack_row<kLong>(lds_address(enc) + win * (kK * 4u), image, nibbles(b.x) << 16 | nibbles(b.y), l, smax, win, mw);
    io.blocks[at * kBlockWords + l] = word;
    if (l == 0) io.meta[at] = mw;
}

// ---- bulk encoder with the min/max selector --------------------------------------------------------------------------------
constexpr int kImageStride = 20;  // words per group of the payload being assembled
constexpr size_t minmax_lds_bytes(int S, bool fine) { return (minmax_table_words(S, fine) + S + kMinmaxBatch * kImageStride + 3) * 4; }

// The indices of the row's values under the pattern whose centroids are at `pair` and whose row of the fine table (ecco_search.h)
// is at `fine`, eight nibbles per lane, first value on top.  per: kFinePer / scale.  Returns the marks of the lane's bins: with
// kFineCrowded in one of its lanes, a row's indices do not hold.  What the kernel takes is VALU issue (92 % of its time): the places
// of two values are formed by four instructions, and an index is its table entry plus the comparison's carry.  Over the uniform
// bins of the full search nearly every wavefront of keys also looked up third candidates: 2 x 131072 groups of keys and values
// at 16 patterns 42.7 -> 37.5 us.
// Every bit pattern of t, NaN included, stays inside the workgroup's LDS: the place is below 1024, the entry below 256, and
// tables and images of at least 2.4 KB follow one another.
__device__ __forceinline__ uint32_t fine_indices(uint32_t fine, uint32_t pair, half2_t s2, half2_t per, const RowValues& v, uint32_t& idx) {
    const uint32_t base = fine - (uint32_t)kFineBins;
    // (in a register, so that sign and constant are joined by one instruction)
    uint32_t least = kFineLeast * 0x10001u;
    asm volatile("" : "+v"(least));
    uint32_t nb[kRowValues], marks = 0;
#pragma unroll
    for (int i = 0; i < kRowValues / 2; ++i) {
        const half2_t c = as_half2((v.x[i] & 0x80008000u) | least);
        const half2_t t = __builtin_elementwise_fma(as_half2(v.x[i]), per, c);
        uint32_t place = __builtin_bit_cast(uint32_t, __builtin_bit_cast(ushort2_t, t) >> 6);
        asm("" : "+v"(place));  // (what is known of its bits would turn a half into a mask and an addition)
        nb[2 * i] = *(const lds_u8*)(size_t)(base + (place & 0xFFFFu));
        nb[2 * i + 1] = *(const lds_u8*)(size_t)(base + (place >> 16));
    }
    idx = 0;
#pragma unroll
    for (int i = 0; i < kRowValues; ++i) {
        const half2_t r = as_half2(lds_word(pair + 4u * nb[i])) * s2;
        const float d0 = distance<0>(v, i, r), d1 = distance<1>(v, i, r);
        idx = (idx << 4) + nb[i] + (d1 < d0 ? 1u : 0u);
        marks |= nb[i];
    }
    return marks;
}

// kStream: the payloads are stored past the caches (ecco_stream.h says when)
template <bool kFine, bool kLong, bool kStream, class Io>
__global__ __launch_bounds__(kMinmaxThreads) void encode_minmax_kernel(Job<Io> j0, Job<Io> j1) {
    extern __shared__ __align__(16) uint32_t smem[];
    const Job<Io>& job = blockIdx.y ? j1 : j0;
    const int S = job.S;
    const Io io = job.io;
    const int lane = threadIdx.x & 63, l = lane & 15, row = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t* ends = smem + minmax_table_words(S, kFine);
    uint32_t* image = ends + S + (wave * kWaveRows + row) * kImageStride;
    const size_t batches = (io.groups() + kMinmaxBatch - 1) / kMinmaxBatch;
    RowValues v, next;
    load_values<kMinmaxBatch>(v, io.values(), io.groups(), blockIdx.x, wave * kWaveRows + row, l);
    const EncTables T = stage_enc_tables<kMinmaxThreads, kFine>(smem, job.dev, S);
    if ((int)threadIdx.x < S) {
        const uint32_t* pair = job.dev + DevLayout{S}.pair() + threadIdx.x * 16;
        ends[threadIdx.x] = __builtin_amdgcn_perm(pair[kK - 1], pair[0], 0x05040100u);  // first and last centroid
    }
    __syncthreads();
    for (size_t b = blockIdx.x; b < batches; b += gridDim.x) {
        const size_t g = b * kMinmaxBatch + wave * kWaveRows + row;
        load_values<kMinmaxBatch>(next, io.values(), io.groups(), b + gridDim.x, wave * kWaveRows + row, l);
        const half2_t ends2 = row_ends(v);
        const uint32_t both = __builtin_bit_cast(uint32_t, ends2) & 0x7FFF7FFFu, smax = max(both & 0xFFFFu, both >> 16);
        const float s = half_bits_f(smax);
        const half2_t s2 = splat_half(smax);
        const uint32_t pattern = select_minmax(ends, 1, S, s2, ends2, l);
        uint32_t idx, marks;
        if (kFine) {
            const uint32_t per = __builtin_bit_cast(unsigned short, (_Float16)(kFinePer * __builtin_amdgcn_rcpf(s)));
            marks = fine_indices(T.fine + (pattern + (pattern & ~3u)) * kFineBins, T.pair + pattern * 64u, s2, splat_half(per), v, idx);
        } else {
            float none;
            set_bins<false>(v, kSearchStep * __builtin_amdgcn_rcpf(s), nullptr, -1);
            marks = rate_pattern<false, true>(T.near + pattern * kSearchBins, T.pair + pattern * 64u, s2, v, -1, none, idx);
        }
        const uint64_t lanes = __builtin_amdgcn_ballot_w64(((marks & (kFine ? kFineCrowded : kNearWide)) != 0u || !(s >= kSearchLeastScale)) && smax != 0u);
        if (lanes != 0ull) {  // rows with crowded bins or a scale too small for the tables
            const uint32_t id = scan_indices(T.pair + pattern * 64u, s2, v, -1);
            idx = row_any(lanes, row) ? id : idx;
        }
        idx = smax == 0u ? 0u : idx;
        uint32_t mw;
        const uint32_t word = pack_row<kLong>(T.enc + pattern * (kK * 4u), image, idx, l, smax, pattern, mw);
        size_t at;
        if (io.place(g, at)) {
            ecco_stream::store<kStream>(io.blocks + at * kBlockWords + l, word);
            if (l == 0) io.meta[at] = mw;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) v.x[i] = next.x[i];
    }
}

// Whether a workgroup per group is the faster way.  For the full search on 256 compute units it takes, in us at 512 / 768 / 1025 / 1537 groups, with up to 16
// patterns 3.7 / 4.3 / 4.8 / 5.9, 32 4.6 / 5.5 / 6.8 / 8.7, 48 5.5 / 6.8 / 8.8 / 11.7, 64 6.3 / 8.1 / 11.1 / 14.6 (a sum per tile of patterns and per
// group that a compute unit gets); the bulk kernel 6.2, 6.7, 7.4 and 7.6 over all of them: the lines cross at about 1700, 1050, 780 and 560 groups, seven, four, three
// and two for each compute unit.  With the min/max selector 2.1 us + 1.2 ns per group and 3.9 us: 1500 groups.
bool few_groups(bool minmax, size_t groups, int S, int cus) {
    constexpr int kMost[] = {7, 4, 3, 2};  // by tiles of 16 patterns
    return groups <= (size_t)cus * (minmax ? 6 : kMost[search_tiles(S) - 1]);
}

// ---- host side -----------------------------------------------------------------------------------------------------------
template <class Io>
int launch_encode(bool minmax, const ecco_model* m0, const Io& io0, const ecco_model* m1, const Io& io1, size_t groups, int jobs, void* stream) {
    const Job<Io> j0{m0->dev, m0->S, io0}, j1{m1->dev, m1->S, io1};
    const int S = std::max(m0->S, m1->S);
    const bool lng = std::max(m0->max_len, m1->max_len) > 8;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const auto run = [&](auto kernel, size_t lds, int batch, int threads, int per_cu) -> int {
        const int rc = allow_lds(kernel, m0->device, lds);
        if (rc != ECCO_OK) return rc;
        const size_t wgs = (groups + batch - 1) / batch;
        const dim3 grid((unsigned)std::min<size_t>(wgs, (size_t)cu_count(m0->device) * per_cu), jobs);
        hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, st, j0, j1);
        ECCO_HIP_CHECK(hipGetLastError());
        return ECCO_OK;
    };
    int rc;
    if (few_groups(minmax, groups * jobs, S, cu_count(m0->device))) {
        const auto few = [&](auto kernel) -> int {
            hipLaunchKernelGGL(kernel, dim3((unsigned)groups, jobs), dim3(kFewThreads), 0, st, j0, j1);
            ECCO_HIP_CHECK(hipGetLastError());
            return ECCO_OK;
        };
        if (minmax) rc = lng ? few(encode_few_kernel<true, true, Io>) : few(encode_few_kernel<true, false, Io>);
        else rc = lng ? few(encode_few_kernel<false, true, Io>) : few(encode_few_kernel<false, false, Io>);
    } else if (minmax) {
        const bool fine = m0->fine_bins && m1->fine_bins;
        const size_t lds = minmax_lds_bytes(S, fine);
        const int per_cu = (int)std::min<size_t>(8, 160 * 1024 / lds);  // at 64 patterns six fit; at 16 eight took 38.8 us for 262144 groups, six 39.8 us
        const auto minmax_run = [&](auto kernel) { return run(kernel, lds, kMinmaxBatch, kMinmaxThreads, per_cu); };
        const auto pick = [&](auto stream_tag) -> int {
            constexpr bool kStream = decltype(stream_tag)::value;
            if (fine) return lng ? minmax_run(encode_minmax_kernel<true, true, kStream, Io>) : minmax_run(encode_minmax_kernel<true, false, kStream, Io>);
            return lng ? minmax_run(encode_minmax_kernel<false, true, kStream, Io>) : minmax_run(encode_minmax_kernel<false, false, kStream, Io>);
        };
        if constexpr (Io::kDense) rc = ecco_stream::encoded(groups * ECCO_BLOCK_BYTES) ? pick(std::true_type{}) : pick(std::false_type{});
        else rc = pick(std::false_type{});
    } else {
        const size_t lds = search_lds_bytes(S);
        switch (search_tiles(S)) {
            case 1: rc = lng ? run(encode_search_kernel<1, true, Io>, lds, kSearchBatch, kSearchThreads, 3) : run(encode_search_kernel<1, false, Io>, lds, kSearchBatch, kSearchThreads, 3); break;
            case 2: rc = lng ? run(encode_search_kernel<2, true, Io>, lds, kSearchBatch, kSearchThreads, 2) : run(encode_search_kernel<2, false, Io>, lds, kSearchBatch, kSearchThreads, 2); break;
            default: rc = lng ? run(encode_search_kernel<4, true, Io>, lds, kSearchBatch, kSearchThreads, 2) : run(encode_search_kernel<4, false, Io>, lds, kSearchBatch, kSearchThreads, 2);
        }
    }
    return rc;
}

int encode_common(bool minmax, const ecco_model* m, const uint16_t* src, size_t n_groups, void* blocks, uint32_t* meta, void* stream) {
    if (!m) return ECCO_EINVAL;
    if (n_groups == 0) return model_ready(m);  // nothing to do; pointers may be null
    if (!src || !blocks || !meta) return ECCO_EINVAL;
    if (!aligned(blocks, 64) || !aligned(src, 4) || !aligned(meta, 4)) return ECCO_EALIGN;
    if (model_ready(m) != ECCO_OK) return ECCO_EINVAL;
    const BulkIo io{reinterpret_cast<const uint32_t*>(src), static_cast<uint32_t*>(blocks), meta, n_groups};
    return launch_encode(minmax, m, io, m, io, n_groups, 1, stream);
}

int kv_append_common(bool minmax, const ecco_model* mk, const ecco_model* mv, const uint16_t* k_new, const uint16_t* v_new,
                     void* k_blocks, uint32_t* k_meta, void* v_blocks, uint32_t* v_meta,
                     const int32_t* seq_len, int B, int H, int T_max, void* stream) {
    if (!mk || !mv || !k_new || !v_new || !k_blocks || !k_meta || !v_blocks || !v_meta || !seq_len) return ECCO_EINVAL;
    if (B <= 0 || H <= 0 || T_max <= 0 || (long long)B * H > 0x7FFFFFFF) return ECCO_ESHAPE;
    if (!aligned(k_blocks, 64) || !aligned(v_blocks, 64) || !aligned(k_new, 4) || !aligned(v_new, 4)) return ECCO_EALIGN;
    if (model_ready(mk) != ECCO_OK || model_ready(mv) != ECCO_OK || mk->device != mv->device) return ECCO_EINVAL;
    const AppendIo k{reinterpret_cast<const uint32_t*>(k_new), static_cast<uint32_t*>(k_blocks), k_meta, seq_len, B * H, H, T_max};
    const AppendIo v{reinterpret_cast<const uint32_t*>(v_new), static_cast<uint32_t*>(v_blocks), v_meta, seq_len, B * H, H, T_max};
    return launch_encode(minmax, mk, k, mv, v, (size_t)B * H, 2, stream);
}

}  // namespace

extern "C" {

int ecco_encode(const ecco_model* m, const uint16_t* src, size_t n_groups, void* blocks, uint32_t* meta, void* stream) {
    return encode_common(false, m, src, n_groups, blocks, meta, stream);
}

int ecco_encode_minmax(const ecco_model* m, const uint16_t* src, size_t n_groups, void* blocks, uint32_t* meta, void* stream) {
    return encode_common(true, m, src, n_groups, blocks, meta, stream);
}

int ecco_kv_append(const ecco_model* mk, const ecco_model* mv, const uint16_t* k_new, const uint16_t* v_new,
                   void* k_blocks, uint32_t* k_meta, void* v_blocks, uint32_t* v_meta,
                   const int32_t* seq_len, int B, int H, int T_max, void* stream) {
    return kv_append_common(false, mk, mv, k_new, v_new, k_blocks, k_meta, v_blocks, v_meta, seq_len, B, H, T_max, stream);
}

int ecco_kv_append_minmax(const ecco_model* mk, const ecco_model* mv, const uint16_t* k_new, const uint16_t* v_new,
                          void* k_blocks, uint32_t* k_meta, void* v_blocks, uint32_t* v_meta,
                          const int32_t* seq_len, int B, int H, int T_max, void* stream) {
    return kv_append_common(true, mk, mv, k_new, v_new, k_blocks, k_meta, v_blocks, v_meta, seq_len, B, H, T_max, stream);
}

}  // extern "C"
