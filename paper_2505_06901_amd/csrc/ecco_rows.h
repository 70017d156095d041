// Device side shared by the encoders of both block formats: a group of 128 values lies in one row of 16 lanes, eight
// consecutive values per lane, so a wavefront holds four groups and everything that is done once per group (extremes,
// scans, sums) is done four groups at a time with cross-lane moves that stay inside a row.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "ecco_search.h"

namespace ecco_rows {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_dword __attribute__((ext_vector_type(4), aligned(4)));  // sixteen bytes on a 4-byte boundary

constexpr int kRowLanes = 16;   // lanes of a group
constexpr int kRowValues = 8;   // values per lane
constexpr int kWaveRows = 4;    // groups per wavefront
// Workgroup of the full search: eight wavefronts, 32 groups at a time, two matrix-core tiles of 16.  (Four wavefronts with
// a pattern tile's whole operands each, 96 registers, ran two workgroups per compute unit, two wavefronts per SIMD, and
// were bound by latency: 79 us for 131072 groups.)
constexpr int kSearchThreads = 512;
constexpr int kSearchWaves = kSearchThreads / 64;
constexpr int kSearchBatch = kSearchWaves * kWaveRows;
constexpr int kHistStride = ecco::kSearchBins + 4;            // words per group of the histogram (skewed over the banks)

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp(uint32_t v) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kCtrl, 0xF, 0xF, true); }
template <int kCtrl>
__device__ __forceinline__ float dpp(float v) { return __builtin_bit_cast(float, dpp<kCtrl>(__builtin_bit_cast(uint32_t, v))); }

template <int kCtrl>
__device__ __forceinline__ half2_t dpp(half2_t v) { return __builtin_bit_cast(half2_t, dpp<kCtrl>(__builtin_bit_cast(uint32_t, v))); }

// a commutative operation over the 16 lanes of a row; every lane of the row returns the result.  As a sum this is the
// balanced tree over lanes l and l ^ 1, then ^ 2, ^ 4, ^ 8: once the quads agree, mirroring is the same as the xor.
template <class T, class Op>
__device__ __forceinline__ T row_all(T t, Op op) {
    t = op(t, dpp<0xB1>(t));   // quad_perm [1,0,3,2]
    t = op(t, dpp<0x4E>(t));   // quad_perm [2,3,0,1]
    t = op(t, dpp<0x141>(t));  // row_half_mirror
    t = op(t, dpp<0x140>(t));  // row_mirror
    return t;
}
__device__ __forceinline__ uint32_t row_max(uint32_t v) { return row_all(v, [](uint32_t a, uint32_t b) { return max(a, b); }); }
__device__ __forceinline__ uint32_t row_min(uint32_t v) { return row_all(v, [](uint32_t a, uint32_t b) { return min(a, b); }); }
// least of non-negative FP32 values (their bits are ordered like whole numbers, and those fuse with the cross-lane moves)
__device__ __forceinline__ float row_min_pos(float v) { return __builtin_bit_cast(float, row_min(__builtin_bit_cast(uint32_t, v))); }
// sum over the lanes of the row up to and including this one
__device__ __forceinline__ uint32_t row_scan(uint32_t v) {
    v += dpp<0x111>(v);  // row_shr 1, 2, 4, 8; zeros come in
    v += dpp<0x112>(v);
    v += dpp<0x114>(v);
    v += dpp<0x118>(v);
    return v;
}
template <int kLane>
__device__ __forceinline__ uint32_t row_lane(uint32_t v) { return dpp<0x150 + kLane>(v); }  // row_newbcast

__device__ __forceinline__ void wave_fence() {  // orders the LDS accesses of one wavefront
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ half2_t as_half2(uint32_t v) { return __builtin_bit_cast(half2_t, v); }
__device__ __forceinline__ float half_bits_f(uint32_t bits) { return (float)__builtin_bit_cast(_Float16, (unsigned short)bits); }
__device__ __forceinline__ half2_t splat_half(uint32_t bits) { return as_half2(bits | (bits << 16)); }

// the eight values of a lane (FP16 pairs) and the bins they fall in, a byte each
struct RowValues {
    uint32_t x[4];
    uint32_t bins[2];
    __device__ __forceinline__ uint32_t bin(int i) const { return (bins[i >> 2] >> (8 * (i & 3))) & 255u; }
};
__device__ __forceinline__ _Float16 value(const RowValues& v, int i) { return as_half2(v.x[i >> 1])[i & 1]; }
// the values of group `local` of batch b (the last group's beyond the end)
template <int kBatch>
__device__ __forceinline__ void load_values(RowValues& v, const uint32_t* src, size_t groups, size_t b, int local, int l) {
    const size_t first = min(b * kBatch, groups - 1);  // uniform
    const int last = (int)min(groups - 1 - first, (size_t)(kBatch - 1));
    const u32x4_dword t = *reinterpret_cast<const u32x4_dword*>(src + first * (kRowLanes * 4) + (min(local, last) * kRowLanes + l) * 4);
    v.x[0] = t.x; v.x[1] = t.y; v.x[2] = t.z; v.x[3] = t.w;
}

// the largest magnitude of the lane's values, as FP16 bits
__device__ __forceinline__ uint32_t lane_absmax(const RowValues& v) {
    ushort2_t m = __builtin_bit_cast(ushort2_t, v.x[0] & 0x7FFF7FFFu);
#pragma unroll
    for (int i = 1; i < 4; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(ushort2_t, v.x[i] & 0x7FFF7FFFu));
    return max((uint32_t)m.x, (uint32_t)m.y);
}
// Bins of the lane's values for axis units `per` = step / scale per unit of x.  Adding 2^23 + 32768 leaves
// rint(x * per) + 32768 in the low 16 bits (q).  hist: this group's row of the histogram; a word counts the bin's values in its
// upper half and sums their places q & 255 in its lower half (kHist).
template <bool kHist>
__device__ __forceinline__ void set_bins(RowValues& v, float per, uint32_t* hist, int skip) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = __builtin_bit_cast(uint32_t, fmaf((float)value(v, 4 * h + i), per, 8421376.0f));
        v.bins[h] = __builtin_amdgcn_perm(q[1], q[0], 0x0C0C0501u) | __builtin_amdgcn_perm(q[3], q[2], 0x05010C0Cu);  // byte 1 of each
        if (kHist) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t one = 65536u | (q[i] & 255u);
                atomicAdd(&hist[(q[i] >> 8) & 255u], 4 * h + i == skip ? 0u : one);
            }
        }
    }
}

// x - r in FP32, rounded once, of the kX-th half of x and the kR-th half of r: one mixed-precision instruction (written
// out, the compiler turns the product with 1 into two conversions and a subtraction)
template <int kX, int kR>
__device__ __forceinline__ float half_diff(uint32_t x, uint32_t r) {
    float d;
    if (kX == 0 && kR == 0) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(x), "v"(r));
    if (kX == 1 && kR == 0) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(x), "v"(r));
    if (kX == 0 && kR == 1) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,1] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(x), "v"(r));
    if (kX == 1 && kR == 1) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(x), "v"(r));
    return d;
}
// the lane's i-th value less the kR-th half of r, and its distance to it
template <int kR>
__device__ __forceinline__ float difference(const RowValues& v, int i, half2_t r) {
    const uint32_t x = v.x[i >> 1], rb = __builtin_bit_cast(uint32_t, r);
    return (i & 1) ? half_diff<1, kR>(x, rb) : half_diff<0, kR>(x, rb);
}
template <int kR>
__device__ __forceinline__ float distance(const RowValues& v, int i, half2_t r) { return fabsf(difference<kR>(v, i, r)); }
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) uint8_t lds_u8;
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(size_t)(const lds_u8*)p; }
__device__ __forceinline__ uint32_t lds_word(uint32_t address) { return *(const lds_u32*)(size_t)address; }

// sum of the squares of the row's 128 distances, in FP32 by the balanced tree over value pairs (i, i ^ 1), (.., i ^ 2), ...;
// the value whose place is `skip` counts as zero
__device__ __forceinline__ float tree_sum(const float (&d)[kRowValues], int skip) {
    float q[kRowValues / 2];
#pragma unroll
    for (int i = 0; i < kRowValues / 2; ++i) {
        const float a = __fmul_rn(d[2 * i], d[2 * i]), b = __fmul_rn(d[2 * i + 1], d[2 * i + 1]);
        q[i] = __fadd_rn(2 * i == skip ? 0.0f : a, 2 * i + 1 == skip ? 0.0f : b);
    }
    return row_all(__fadd_rn(__fadd_rn(q[0], q[1]), __fadd_rn(q[2], q[3])), [](float a, float b) { return __fadd_rn(a, b); });
}

// The row's values under one pattern: every value's index (the lowest of the nearest reconstructed centroids
// fp16(c * s)), eight nibbles per lane, first value on top; (kIdx); and the group's squared error (kSse, by tree_sum).  near, pair: the
// pattern's rows of the tables in LDS (pair as an LDS address, a multiple of 64).  A value whose place is `skip` counts as
// without error, with index 15.  Returns the marks of the lane's bins: with kNearWide (more than three candidates) in one of its
// lanes, a row's results do not hold.
template <bool kSse, bool kIdx, int kAtOnce = 4>
__device__ __forceinline__ uint32_t rate_pattern(const uint8_t* near, uint32_t pair, half2_t s2, const RowValues& v, int skip, float& sse, uint32_t& idx) {
    uint32_t k[kRowValues], marks = 0;
    float d[kRowValues];
    // kAtOnce values at a time: with the indices, all eight in flight need 24 more registers than three workgroups per compute unit leave
#pragma unroll
    for (int h = 0; h < kRowValues; h += kAtOnce) {
        uint32_t nb[kAtOnce];
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i) nb[i] = near[v.bin(h + i)];
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i) {
            const half2_t r = as_half2(lds_word((nb[i] & 0x3Cu) | pair)) * s2;
            if (kIdx) {
                const float d0 = distance<0>(v, h + i, r), d1 = distance<1>(v, h + i, r);
                const bool up = d1 < d0;
                k[h + i] = (nb[i] >> 2) + (up ? 1u : 0u);
                d[h + i] = up ? d1 : d0;
            } else {
                const float d0 = difference<0>(v, h + i, r), d1 = difference<1>(v, h + i, r);
                asm("v_min_f32 %0, |%1|, |%2|" : "=v"(d[h + i]) : "v"(d0), "v"(d1));
            }
            marks |= nb[i];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if (__builtin_amdgcn_ballot_w64((marks & ecco::kNearTwo) != 0u) != 0ull) {
        // the table addresses are formed again here: kept from above they would take eight registers through the search
        uint32_t base = lds_address(near);
        asm volatile("" : "+v"(base));
#pragma unroll
        for (int i = 0; i < kRowValues; ++i) {
            const uint32_t nb = *(const lds_u8*)(size_t)(base + v.bin(i));
            if (nb & ecco::kNearTwo) {
                const half2_t r = as_half2(lds_word(((nb & 0x3Cu) | pair) + 4u)) * s2;
                const float d1 = distance<0>(v, i, r), d2 = distance<1>(v, i, r);
                if (d2 < d1) {
                    if (kIdx) k[i] = (nb >> 2) + 2u;
                    d[i] = d2;
                }
            }
        }
    }
    idx = 0;
    if (kIdx)
#pragma unroll
        for (int i = 0; i < kRowValues; ++i) idx = (idx << 4) | (i == skip ? 15u : k[i]);
    if (kSse) {
        sse = tree_sum(d, skip);
    }
    return marks;
}

// ---- value by value: groups for which the table of nearest centroids does not hold --------------------------------------
// Scales below kSearchLeastScale, and groups that one large value presses into bins with many centroids, where most
// patterns tend to be left over from the bounds as well.  Bound by the vector instructions (24 per value and pattern).  With
// a compare and two masked moves per centroid and value inside the ratings by the table instead, four groups at a time, and
// with all patterns rated at every small scale, 131072 groups under 64 patterns took 3.1 ms at scales of 2^-12 (0.11 ms here,
// 0.61 ms at 2^-20, where all patterns are left), 3.1 ms when all zero (0.06 ms), 1.8 ms with one value 100 times as large as
// the rest (0.38 ms), 3.6 ms in the self-contained format (0.68 ms); all patterns value by value without the bounds: 0.52 and
// 0.61 ms.

// A rating by the table takes 500 to 1000 cycles for the four rows of a wavefront, by how many third candidates have to be looked
// at; value by value it is 160 for one row, and about 3000 to begin with.  So a wavefront goes on that way where the bounds
// have told hardly any patterns apart, which is looked at after this many ratings (ahead of them where the patterns are dealt out).
constexpr int kLookAfter = 4;
__device__ __forceinline__ bool most_left(uint64_t left, int S) { return 4 * (__builtin_popcountll(left) + kLookAfter) > 3 * S; }
// whether `lanes` (a ballot) holds a lane of row `row`
__device__ __forceinline__ bool row_any(uint64_t lanes, int row) {
    const uint32_t half = (row & 2) ? (uint32_t)(lanes >> 32) : (uint32_t)lanes;
    return ((half >> (16 * (row & 1))) & 0xFFFFu) != 0u;
}

// The indices of the row's values under the pattern with centroids at `pair`, compared with all of them.  The distance
// falls (weakly) with k up to its least value and rises (weakly) after it, so the lowest nearest index is the last k at which
// it strictly drops.
__device__ __forceinline__ uint32_t scan_indices(uint32_t pair, half2_t s2, const RowValues& v, int skip) {
    uint32_t k[kRowValues];
    float last[kRowValues];
#pragma unroll
    for (int i = 0; i < kRowValues; ++i) {
        k[i] = 0;
        last[i] = __builtin_inff();
    }
#pragma unroll 1
    for (uint32_t c = 0; c < 16u; c += 2u) {
        const half2_t r = as_half2(lds_word(pair + 4u * c)) * s2;
#pragma unroll
        for (int i = 0; i < kRowValues; ++i) {
            const float a = distance<0>(v, i, r), b = distance<1>(v, i, r);
            k[i] = a < last[i] ? c : k[i];
            k[i] = b < a ? c + 1u : k[i];
            last[i] = b;
        }
    }
    uint32_t idx = 0;
#pragma unroll
    for (int i = 0; i < kRowValues; ++i) idx = (idx << 4) | (i == skip ? 15u : k[i]);
    return idx;
}

// Four sums over the 32 lanes of each half of the wavefront at once, in the balanced tree (lanes l and l ^ 1, then ^ 2, ^ 4, ^ 8,
// ^ 16): at the first two levels a lane keeps the entries that match its own lane bit and sends the others to its partner.
// Lane l returns its half's total of entry l & 3.
__device__ __forceinline__ float half_sum4(const float (&q)[4], int lane) {
    const bool b0 = lane & 1, b1 = lane & 2;
    float a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = __fadd_rn(b0 ? q[2 * i + 1] : q[2 * i], dpp<0xB1>(b0 ? q[2 * i] : q[2 * i + 1]));
    float t = __fadd_rn(b1 ? a[1] : a[0], dpp<0x4E>(b1 ? a[0] : a[1]));
    const auto swizzled = [](float v, auto pattern) { return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), decltype(pattern)::value)); };
    t = __fadd_rn(t, swizzled(t, std::integral_constant<int, 0x101F>{}));     // lane ^ 4
    t = __fadd_rn(t, dpp<0x128>(t));                                          // row_ror 8: lane ^ 8
    return __fadd_rn(t, swizzled(t, std::integral_constant<int, 0x401F>{}));  // lane ^ 16
}
// the least over the wavefront
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
    v = row_min(v);
    const auto of = [&](int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
    return min(min(of(0), of(16)), min(of(32), of(48)));
}

// Rates the rows' patterns `later` and takes the best of them into (best, pattern), the lowest pattern on a tie; won: whether
// it did.  One group after the other, four values per lane, a pattern per half of the wavefront: the reconstructed centroids
// come from LDS as FP32, where a difference is a two-operand FP32 instruction, issued in 2.7 cycles (4.4 for the
// mixed-precision one of half_diff).  pairs: the patterns' (centroid k, centroid k + 1) words in LDS; recon: 128 words of LDS
// of the wavefront; at_skip: place of the group's value that counts as without error (128 or more: none).
__device__ __forceinline__ void scan_patterns(float* recon, const uint32_t* pairs, const RowValues& v, uint32_t smax, uint32_t at_skip, uint64_t later,
                                              int lane, float& best, uint32_t& pattern, bool& won) {
    const uint64_t rows = __builtin_amdgcn_ballot_w64(later != 0ull);
    won = false;
#pragma unroll 1
    for (int g = 0; g < kWaveRows; ++g) {
        if (((rows >> (16 * g)) & 1ull) == 0ull) continue;
        asm volatile("" : "+v"(lane));  // what is derived from the lane is formed here, not kept through the search
        const auto of_row = [&](uint32_t t) { return (uint32_t)__builtin_amdgcn_readlane((int)t, 16 * g); };
        uint64_t todo = ((uint64_t)of_row((uint32_t)(later >> 32)) << 32) | of_row((uint32_t)later);
        const _Float16 s = __builtin_bit_cast(_Float16, (unsigned short)of_row(smax));
        const uint32_t skip = of_row(at_skip);
        // values 4 m .. 4 m + 3 of the group for lane m of either half: two words of the row's lane m / 2
        const int m = lane & 31, from = 4 * (16 * g + (m >> 1));
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)v.x[i]);
        const half2_t xa = as_half2((m & 1) ? w[2] : w[0]), xb = as_half2((m & 1) ? w[3] : w[1]);
        const float x[4] = {(float)xa[0], (float)xa[1], (float)xb[0], (float)xb[1]};
        const uint32_t zero = skip - 4u * (uint32_t)m;  // which of the four counts as zero, if one of 0 .. 3
        float mine = __builtin_inff();  // lane l: the least so far among its half's entries l & 3
        uint32_t mine_p = pattern;
        while (todo != 0ull) {
            // eight patterns, one for each half and entry (the last one again where there are fewer): their reconstructed centroids
            uint32_t entry_p = 0;
            int entries = 0, at = lane;
            asm volatile("" : "+v"(at));  // as above
            const uint32_t k = at & 15;
            float* own = recon + (at >> 5) * 16;
            wave_fence();
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (todo != 0ull) {  // uniform
                    const uint32_t p0 = (uint32_t)__builtin_ctzll(todo);
                    todo &= todo - 1ull;
                    const uint32_t p1 = todo != 0ull ? (uint32_t)__builtin_ctzll(todo) : p0;
                    todo &= todo - 1ull;
                    const uint32_t p = at < 32 ? p0 : p1;
                    entry_p = (at & 3) == e ? p : entry_p;
                    own[e * 32 + k] = (float)(as_half2(pairs[p * 16u + k])[0] * s);
                    entries = e + 1;
                }
            }
            wave_fence();
            float q[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                q[e] = __builtin_inff();
                if (e < entries) {  // uniform
                    const float4_t* r4 = reinterpret_cast<const float4_t*>(own + e * 32);
                    float d[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) d[i] = __builtin_inff();
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float4_t r = r4[c];
#pragma unroll
                        for (int j = 0; j < 4; j += 2)
#pragma unroll
                            for (int i = 0; i < 4; ++i) d[i] = fminf(fminf(d[i], fabsf(__fsub_rn(x[i], r[j]))), fabsf(__fsub_rn(x[i], r[j + 1])));
                    }
                    float sq[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) sq[i] = zero == (uint32_t)i ? 0.0f : __fmul_rn(d[i], d[i]);
                    __builtin_amdgcn_sched_barrier(0);  // one pattern's centroids at a time in registers
                    q[e] = __fadd_rn(__fadd_rn(sq[0], sq[1]), __fadd_rn(sq[2], sq[3]));
                }
            }
            const float t = half_sum4(q, lane);
            if (t < mine) {  // strict <: an earlier pattern keeps a tie
                mine = t;
                mine_p = entry_p;
            }
        }
        const uint32_t least = wave_min(__builtin_bit_cast(uint32_t, mine));
        const uint32_t win = wave_min(__builtin_bit_cast(uint32_t, mine) == least ? mine_p : 0xFFFFu);
        const float sse = __builtin_bit_cast(float, least);
        if ((lane >> 4) == g && (sse < best || (sse == best && win < pattern))) {
            best = sse;
            pattern = win;
            won = true;
        }
    }
    wave_fence();
}

// ---- the patterns left over from the bounds ----------------------------------------------------------------------------
// Rates the patterns `left` of the wavefront's four groups (a bit each; one alone has won and is not looked at) and returns each row's
// best; `later` receives those that the table of nearest centroids does not serve.  A group has 1.3 to 2.1 patterns left on average
// and the most of four groups 1.9 to 3.6, the most of a workgroup's 3.2 to 6, for which all others would wait at the next barrier: so the
// patterns of the four groups are dealt out to the four rows of lanes, one after the other, whosever they are (1.5 to 2.1 rounds).
// The values, bins and scales wait in LDS for this, with a list of (group, pattern); the least error of a group, the lowest
// pattern on a tie, is kept by an atomic minimum.  at: kDealWords words of LDS of the wavefront.  131072 groups, 64 patterns: 63.9 -> 60.3
// us, self-contained blocks encoded and decoded 102.0 -> 99.3 us; 8192 groups 9.7 -> 8.4 us.
constexpr int kDealWords = 64 * 4 + 64 * 2 + kWaveRows * 2 + kWaveRows * 4 + kWaveRows * 64;
static_assert(kDealWords <= kWaveRows * kHistStride, "over the wavefront's part of the histogram");
template <bool kSkip, int kAtOnce>
__device__ __forceinline__ uint32_t rate_left(uint32_t* at, const uint8_t* near, uint32_t pair, RowValues& v, uint32_t smax, int skip, uint64_t left, int S, int lane,
                                              float& least, uint64_t& later) {
    asm volatile("" : "+v"(lane));  // what is derived from the lane is formed here, not kept through the search
    const int row = lane >> 4, l = lane & 15;
    uint4* values = reinterpret_cast<uint4*>(at);
    uint2* bins = reinterpret_cast<uint2*>(at + 256);
    uint2* about = reinterpret_cast<uint2*>(at + 384);                        // per group: scale, place that counts as without error
    unsigned long long* best = reinterpret_cast<unsigned long long*>(at + 392);  // per group: (error, pattern)
    unsigned long long* wide = best + kWaveRows;                              // per group: patterns for a comparison value by value
    uint32_t* list = at + 408;
    uint32_t pattern = left != 0 ? (uint32_t)__builtin_ctzll(left) : 0u;
    least = __builtin_inff();
    if ((left & (left - 1ull)) == 0ull) left = 0;
    // hardly any told apart in one of the groups: value by value is the faster way (kLookAfter)
    const int count = __builtin_popcountll(left);
    const bool most = __builtin_amdgcn_ballot_w64(count > kLookAfter && 4 * count > 3 * S) != 0ull && count > kLookAfter;
    later = most ? left : 0ull;
    left = most ? 0ull : left;
    if (__builtin_amdgcn_ballot_w64(left != 0ull) == 0ull) return pattern;
    wave_fence();
    values[lane] = make_uint4(v.x[0], v.x[1], v.x[2], v.x[3]);
    bins[lane] = make_uint2(v.bins[0], v.bins[1]);
    if (l == 0) {
        about[row].x = smax;
        best[row] = ~0ull;
        wide[row] = 0ull;
    }
    if (kSkip && skip >= 0) about[row].y = (uint32_t)(8 * l + skip);
    uint32_t total = 0;
#pragma unroll
    for (int g = 0; g < kWaveRows; ++g) {  // lane p writes group g's pattern p
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)left, 16 * g), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(left >> 32), 16 * g);
        const uint32_t to = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, total));
        const uint64_t m = ((uint64_t)hi << 32) | lo;
        if ((m >> lane) & 1ull) list[to] = ((uint32_t)g << 8) | (uint32_t)lane;
        total += (uint32_t)__builtin_popcountll(m);
    }
    wave_fence();
    for (uint32_t i = 0; i < total; i += kWaveRows) {  // uniform; a row that has none left repeats the last one
        const uint32_t item = list[min(i + (uint32_t)row, total - 1u)], g = item >> 8, p = item & 0xFFu;
        const uint4 x = values[g * kRowLanes + l];
        const uint2 b = bins[g * kRowLanes + l], a = about[g];
        RowValues w;
        w.x[0] = x.x; w.x[1] = x.y; w.x[2] = x.z; w.x[3] = x.w;
        w.bins[0] = b.x; w.bins[1] = b.y;
        float sse;
        uint32_t none;
        const uint32_t marks = rate_pattern<true, false, kAtOnce>(near + p * ecco::kSearchBins, pair + p * 64u, splat_half(a.x), w,
                                                                  kSkip ? (int)a.y - 8 * l : -1, sse, none);
        const uint64_t lanes = __builtin_amdgcn_ballot_w64((marks & ecco::kNearWide) != 0u);
        const bool served = lanes == 0ull || !row_any(lanes, row);
        if (l == 0) {
            if (served) atomicMin(&best[g], ((unsigned long long)__builtin_bit_cast(uint32_t, sse) << 32) | p);
            else atomicOr(&wide[g], 1ull << p);
        }
    }
    wave_fence();
    const unsigned long long found = best[row];
    later |= wide[row];
    // read again: kept, they would take six registers through the ratings
    const uint4 x = values[lane];
    const uint2 b = bins[lane];
    v.x[0] = x.x; v.x[1] = x.y; v.x[2] = x.z; v.x[3] = x.w;
    v.bins[0] = b.x; v.bins[1] = b.y;
    wave_fence();
    if (found != ~0ull) {
        least = __builtin_bit_cast(float, (uint32_t)(found >> 32));
        pattern = (uint32_t)found;
    }
    return pattern;
}

// Priority of a wavefront's instructions on its SIMD in the phases of a full search.  The workgroups of a compute unit start together and would
// stay in step: all wait for table reads in the ratings, all meet at the barriers of the bounds.  With the ratings ahead of the histogram
// and that ahead of the bounds, whose waits at barriers cost nobody else anything, one workgroup's ratings fill the other's waits: 131072
// groups, 64 patterns 60.2 -> 54.5 us, 16 patterns 43.9 -> 39.9 us, self-contained blocks encoded and decoded 99.4 -> 91.2 us.  (Ratings in front and
// all else alike 56.3 us, histogram in front 58.7 us; packing like the ratings 55.0 us.)  With three workgroups per compute unit (up to
// 16 patterns) the histogram goes with the ratings: behind them, the last of one to two batches per workgroup waits (32768 groups 12.9 us, 13.2 us).
constexpr int kPriorityBounds = 0, kPriorityPack = 1, kPriorityRate = 2;
constexpr int priority_hist(bool three) { return three ? 2 : 1; }

// ---- bounds on every pattern's error, and the patterns that can be the best ------------------------------------------
// Workgroup-wide LDS of the bounds: histogram, partial sums of the matrix product, the pattern tiles' least upper bounds,
// the groups' slack, the patterns left per group.  kOver: the partial sums lie over the histogram, at the price of a barrier,
// so that one more workgroup fits a compute unit.
struct SearchLds {
    uint32_t* hist;   // [kSearchBatch][kHistStride]
    float4_t* part;   // [wavefront (and tile of groups)][sum, error][64]
    float* least;     // [4][kSearchBatch]
    float* slack;     // [kSearchBatch]: what a group's small scale adds to the errors (set_slack)
    uint32_t* spare;  // [kSearchBatch]: a word per group for the caller
    uint16_t* left;   // [kSearchBatch][4]
};
// one tile of patterns per 16; the wavefronts share the tiles evenly, each over its own part of the bins
constexpr int search_parts(int tiles) { return tiles == 1 ? 8 : tiles == 2 ? 4 : 2; }
static_assert(kSearchWaves * 4 * 64 * 4 <= kSearchBatch * kHistStride, "the partial sums fit over the histogram");
constexpr int search_part_words(int tiles) { return kSearchWaves * (search_parts(tiles) == 2 ? 1 : 2) * 2 * 64 * 4; }
template <bool kOver>
constexpr int search_lds_words(int tiles) { return kSearchBatch * kHistStride + (kOver ? 0 : search_part_words(tiles)) + 6 * kSearchBatch + kSearchBatch * 2; }
template <bool kOver>
__device__ __forceinline__ SearchLds search_lds(uint32_t* base, int tiles) {
    SearchLds s;
    s.hist = base;
    s.part = reinterpret_cast<float4_t*>(kOver ? base : base + kSearchBatch * kHistStride);
    s.least = reinterpret_cast<float*>(base + kSearchBatch * kHistStride + (kOver ? 0 : search_part_words(tiles)));
    s.slack = s.least + 4 * kSearchBatch;
    s.spare = reinterpret_cast<uint32_t*>(s.slack + kSearchBatch);
    s.left = reinterpret_cast<uint16_t*>(s.spare + kSearchBatch);
    return s;
}

// A wavefront's operands of the matrix product; they stay in registers for as long as the workgroup lives.
template <int kTiles>
struct Coefs {
    static constexpr int kParts = search_parts(kTiles);
    static constexpr int kBlocks = ecco::kSearchBlocks / kParts;
    uint4 w[kBlocks * 3];
    __device__ __forceinline__ void load(const uint32_t* __restrict__ coef, int wave, int tiles, int lane) {
        const int tile = min(wave / kParts, tiles - 1);
        const uint4* src = reinterpret_cast<const uint4*>(coef) + ((size_t)(tile * ecco::kSearchBlocks + (wave % kParts) * kBlocks) * 3) * 64 + lane;
#pragma unroll
        for (int i = 0; i < kBlocks * 3; ++i) w[i] = src[i * 64];
    }
};

// this wavefront's four rows of the histogram, to "no values"
__device__ __forceinline__ void clear_hist(uint32_t* rows, int lane) {
    uint32_t zero = 0u;  // formed here: a constant in four registers would be kept through the search
    asm volatile("" : "+v"(zero));
    const uint4 none = make_uint4(zero, zero, zero, zero);
    constexpr int kPieces = kWaveRows * kHistStride / 4;
#pragma unroll
    for (int i = 0; i < kPieces / 64; ++i) reinterpret_cast<uint4*>(rows)[i * 64 + lane] = none;
    if (lane < kPieces % 64) reinterpret_cast<uint4*>(rows)[kPieces / 64 * 64 + lane] = none;
}
// sums and counts to FP16 (m, n) pairs, in place
__device__ __forceinline__ void convert_hist(uint32_t* rows, int lane) {
#pragma unroll
    for (int r = 0; r < kWaveRows; ++r) {
        uint4* at = reinterpret_cast<uint4*>(rows + r * kHistStride) + lane;
        uint4 v = *at;
        uint32_t* w = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t m, n;
            asm("v_cvt_f16_u16_e32 %0, %1" : "=v"(m) : "v"(w[i]));
            asm("v_cvt_f16_u16_sdwa %0, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1" : "=v"(n) : "v"(w[i]));
            w[i] = m | (n << 16);
        }
        *at = v;
    }
}

// The tables' errors cover the rounding of reconstructed centroids for scales of at least kSearchLeastScale.  Below, that rounding
// (to a multiple of 2^-24) moves every distance by up to d = 2^-25 / s more, the root of the squared error by sqrt(128) d:
// this is sqrt(128) d in the root of the tables' unit, with a margin, for the row's group (at `own`, zero to begin with).
// Written only by wavefronts that hold such a group, or held one in their last batch (set).
__device__ __forceinline__ void set_slack(float* own, float s, int l, bool& set) {
    constexpr float kUnit = 1.02f * 362.04f * 0x1p-25f;  // sqrt(128 kSearchCoefScale) 2^-25
    static_assert(ecco::kSearchCoefScale == 1024.0f, "sqrt(128 x 1024) = 362.04");
    const bool small = s < ecco::kSearchLeastScale;
    const bool any = __builtin_amdgcn_ballot_w64(small) != 0ull;
    if (any || set) {
        if (l == 0) *own = small && s > 0.0f ? kUnit * __builtin_amdgcn_rcpf(s) : 0.0f;
        set = any;
    }
}

// For the batch's converted histogram: the patterns of this wavefront's group (wave, row) that can have the least error,
// one bit each.  Called by all wavefronts of the workgroup together (barriers inside); the histogram is free afterwards.
template <int kTiles, bool kOver>
__device__ __forceinline__ uint64_t patterns_left(const SearchLds& L, const Coefs<kTiles>& C, int tiles, int wave, int lane) {
    constexpr int kParts = Coefs<kTiles>::kParts, kBlocks = Coefs<kTiles>::kBlocks;
    const int tile = wave / kParts, part = wave % kParts;
    float4_t sum[2], err[2];  // of groups 0..15 and 16..31
    __syncthreads();
    __builtin_amdgcn_s_setprio(kPriorityBounds);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        sum[m] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
        err[m] = sum[m];
        // row l % 16 of the A operand; bins 4 (l / 16) .. + 3 of each 16
        const uint4* a = reinterpret_cast<const uint4*>(L.hist + (16 * m + (lane & 15)) * kHistStride + part * kBlocks * 32 + 4 * (lane >> 4));
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) {
            const uint4 a0 = a[j * 8], a1 = a[j * 8 + 4];
            // the counts alone: the upper halves of the eight words
            const uint4 n = make_uint4(__builtin_amdgcn_perm(a0.y, a0.x, 0x07060302u), __builtin_amdgcn_perm(a0.w, a0.z, 0x07060302u),
                                       __builtin_amdgcn_perm(a1.y, a1.x, 0x07060302u), __builtin_amdgcn_perm(a1.w, a1.z, 0x07060302u));
            sum[m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a0), __builtin_bit_cast(half8_t, C.w[3 * j]), sum[m], 0, 0, 0);
            err[m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, n), __builtin_bit_cast(half8_t, C.w[3 * j + 2]), err[m], 0, 0, 0);
            sum[m] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a1), __builtin_bit_cast(half8_t, C.w[3 * j + 1]), sum[m], 0, 0, 0);
        }
    }
    // (read here, so that the barrier covers the wait)
    int at_lane = lane;  // taken afresh: the address is formed here, not kept through the search
    asm volatile("" : "+v"(at_lane));
    const uint4 bits = *reinterpret_cast<const uint4*>(L.slack + 16 * min(part, 1) + 4 * (at_lane >> 4));
    if (kOver) __syncthreads();
    // parts 0 and 1 of a tile of patterns add up the parts for groups 0..15 and 16..31
    float4_t s, e;
    if (kParts == 2) {
        L.part[(wave * 2) * 64 + lane] = part ? sum[0] : sum[1];
        L.part[(wave * 2 + 1) * 64 + lane] = part ? err[0] : err[1];
        __syncthreads();
        s = (part ? sum[1] : sum[0]) + L.part[((wave ^ 1) * 2) * 64 + lane];
        e = (part ? err[1] : err[0]) + L.part[((wave ^ 1) * 2 + 1) * 64 + lane];
    } else {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            L.part[((wave * 2 + m) * 2) * 64 + lane] = sum[m];
            L.part[((wave * 2 + m) * 2 + 1) * 64 + lane] = err[m];
        }
        __syncthreads();
        const float4_t* at = L.part + (tile * kParts * 4 + min(part, 1) * 2) * 64 + lane;
        s = at[0];
        e = at[64];
#pragma unroll
        for (int q = 1; q < kParts; ++q) {
            s += at[q * 256];
            e += at[q * 256 + 64];
        }
    }
    // lane l, register j: group 16 part + 4 (l / 16) + j of the batch, pattern 16 tile + l % 16
    const bool mine = part < 2;
    if (__builtin_amdgcn_ballot_w64((bits.x | bits.y | bits.z | bits.w) != 0u) != 0ull) {
        const float4_t slack = __builtin_bit_cast(float4_t, bits);
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] += slack[j] * (2.0f * __builtin_amdgcn_sqrtf(fmaxf(s[j] + e[j] + 3.0f, 0.0f)) + slack[j]);
    }
    float least[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        // the FP32 sums that decide differ from the true ones by less than 2^-18 of the error, what all patterns share included
        e[j] += fabsf(s[j]) * 0x1p-16f + 0x1p-12f;
        s[j] += 16.0f;  // the bound with what is shared left out can be below zero, by less than 3
        least[j] = row_min_pos(s[j] + e[j]);
    }
    if (kTiles > 1) {
        if (mine && (lane & 15) == 0)
#pragma unroll
            for (int j = 0; j < 4; ++j) L.least[tile * kSearchBatch + 16 * part + 4 * (lane >> 4) + j] = tile < tiles ? least[j] : __builtin_inff();
        __syncthreads();
        const float* at = L.least + 16 * min(part, 1) + 4 * (lane >> 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            least[j] = fminf(at[j], at[kSearchBatch + j]);
            if (kTiles > 2) least[j] = fminf(least[j], fminf(at[2 * kSearchBatch + j], at[3 * kSearchBatch + j]));
        }
    }
    uint64_t left[4];  // register j: 16 bits for each of the groups j, 4 + j, 8 + j, 12 + j
#pragma unroll
    for (int j = 0; j < 4; ++j) left[j] = __builtin_amdgcn_ballot_w64(s[j] - e[j] <= least[j]);
    if (mine && lane < 16) {  // lane g writes group g = 4 r + j
        const int j = lane & 3;
        const uint64_t m = j == 0 ? left[0] : j == 1 ? left[1] : j == 2 ? left[2] : left[3];
        L.left[(16 * part + lane) * 4 + tile] = tile < tiles ? (uint16_t)(m >> (16 * (lane >> 2))) : (uint16_t)0;
    }
    __syncthreads();
    const uint64_t m = *reinterpret_cast<const uint64_t*>(L.left + (wave * kWaveRows + (lane >> 4)) * 4);
    return kTiles == 1 ? m & 0xFFFFull : kTiles == 2 ? m & 0xFFFFFFFFull : m;  // tiles that do not exist are not written
}

}  // namespace ecco_rows
