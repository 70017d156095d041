// Encoder of the self-contained 4x block (include/ecco_paper_block.h) for gfx950.
//
// The search for the pattern of least squared error is the two-step one of ecco_search.h / ecco_rows.h: bounds for all
// patterns from a matrix product of the group's histogram, exact FP32 errors for the patterns that are left.  (Rating all
// patterns value by value took 0.62 ms for 131072 groups at S = 64, vector instructions throughout.)  A group lies in a row
// of 16 lanes, eight values per lane.  The element of largest magnitude takes index 15 and no error; the codebook is the
// one of least total length (the four lengths of an index are the bytes of one word, summed together); the stream is cut
// at bit 512; if it ends before, the largest remaining magnitudes follow as 15-bit entries: one row maximum per entry,
// kept by the lane of that number, and all entries are converted and written at once.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ecco_pb_launch.h"
#include "ecco_rows.h"

namespace {

using namespace ecco_pb;
using namespace ecco_rows;

// tables in LDS, in words per pattern: near [64], pair [16], codes of the four books [4][16] 16-bit (code << 8 | length), lengths [16]
constexpr int kTableWords = ecco::kSearchBins / 4 + 16 + kBooks * kSym / 2 + kSym;
constexpr int kFp8Words = 128;
constexpr size_t table_words(int S) { return (size_t)S * kTableWords + kFp8Words + ((S + 3) & ~3); }
size_t encode_lds_bytes(int S) { return (table_words(S) + search_lds_words<true>(ecco::search_tiles(S))) * 4; }

__device__ __forceinline__ void copy_words(uint32_t* dst, const uint32_t* __restrict__ src, int words) {  // words % 4 == 0, 16-byte aligned
    for (int i = threadIdx.x; i < words / 4; i += kSearchThreads) reinterpret_cast<uint4*>(dst)[i] = reinterpret_cast<const uint4*>(src)[i];
}

// v to the format's 8-bit float: nearest, ties to the even code, saturating at +-480
__device__ __forceinline__ uint32_t fp8_round(float v) {
    const uint32_t sign = (__float_as_uint(v) >> 24) & 0x80u;
    const float a = fabsf(v);
    uint32_t code;
    if (a < 0.015625f) {
        code = (uint32_t)rintf(a * 512.0f);  // below 2^-6 the values are multiples of 2^-9; 8 is the smallest normal number
    } else {
        const uint32_t b = __float_as_uint(a);
        const uint32_t r = b + 0x7FFFFu + ((b >> 20) & 1u);  // to three mantissa bits, ties to even
        const int e = (int)(r >> 23) - 120;
        code = e > 15 ? 127u : (((uint32_t)e << 3) | ((r >> 20) & 7u));
    }
    return sign | code;
}

// ORs the low `nbits` (1..32) of `value` into the block image at stream bit `at`, most significant bit first; bits at or
// beyond 512 are dropped (the cut)
__device__ __forceinline__ void put_bits(uint32_t* image, uint32_t at, uint32_t value, uint32_t nbits) {
    const uint64_t v = (uint64_t)value << (64u - nbits - (at & 31u));
    const uint32_t wi = at >> 5;
    if (wi < (uint32_t)kBlockWords) atomicOr(&image[wi], (uint32_t)(v >> 32));
    if (wi + 1 < (uint32_t)kBlockWords && (uint32_t)v != 0u) atomicOr(&image[wi + 1], (uint32_t)v);
}

template <int kTiles>
__global__ __launch_bounds__(kSearchThreads) __attribute__((amdgpu_waves_per_eu(4)))
void pb_encode_kernel(const uint32_t* __restrict__ dev, int S, float inv_tscale, const uint32_t* __restrict__ src, size_t n_groups,
                      uint32_t* __restrict__ blocks) {
    extern __shared__ __align__(16) uint32_t smem[];
    const DevLayout D{S};
    const int tiles = ecco::search_tiles(S);
    const int lane0 = threadIdx.x & 63, l0 = lane0 & 15, row0 = lane0 >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint8_t* near = reinterpret_cast<const uint8_t*>(smem);
    uint32_t* pair_at = smem + S * (ecco::kSearchBins / 4);
    uint32_t* codes_at = pair_at + S * 16;
    uint32_t* lens = codes_at + S * (kBooks * kSym / 2);
    uint32_t* fp8_at = lens + S * kSym;
    uint32_t* kpenc = fp8_at + kFp8Words;
    const uint32_t pair = lds_address(pair_at);
    const uint16_t* codes = reinterpret_cast<const uint16_t*>(codes_at);
    const uint16_t* fp8 = reinterpret_cast<const uint16_t*>(fp8_at);
    const SearchLds L = search_lds<true>(smem + table_words(S), kTiles);

    const size_t batches = (n_groups + kSearchBatch - 1) / kSearchBatch;
    RowValues v;
    load_values<kSearchBatch>(v, src, n_groups, blockIdx.x, wave * kWaveRows + row0, l0);
    Coefs<kTiles> C;
    C.load(dev + D.coef(), wave, tiles, lane0);
    copy_words(smem, dev + D.near(), S * kTableWords);  // near, pair, codes, lengths follow each other
    copy_words(fp8_at, dev + D.fp8(), kFp8Words);
    copy_words(kpenc, dev + D.kpenc(), (S + 3) & ~3);
    bool slack_set = false;
    if ((threadIdx.x & 15) == 0) L.slack[threadIdx.x >> 4] = 0.0f;
    __syncthreads();

    for (size_t b = blockIdx.x; b < batches; b += gridDim.x) {
        // the lane taken afresh for each batch: what is derived from it would otherwise take registers through the search
        int at = threadIdx.x & 63;
        asm volatile("" : "+v"(at));
        const int lane = at, l = lane & 15, row = lane >> 4;
        uint32_t* hist = L.hist + (wave * kWaveRows + row) * kHistStride;
        __builtin_amdgcn_s_setprio(priority_hist(false));
        // the element of largest magnitude, first position on ties: the least (position, value) of those that have it
        const uint32_t mag = row_max(lane_absmax(v));
        uint32_t first = 0xFFFFFFFFu;
#pragma unroll
        for (int i = kRowValues - 1; i >= 0; --i) {
            const uint32_t bits = (i & 1) ? v.x[i >> 1] >> 16 : v.x[i >> 1] & 0xFFFFu;
            if ((bits & 0x7FFFu) == mag) first = ((uint32_t)i << 16) | bits;
        }
        if (first != 0xFFFFFFFFu) first += (uint32_t)l << 19;
        const uint32_t top = row_min(first);
        const uint32_t at_top = top >> 16;                       // its position
        const int skip = (int)(at_top >> 3) == l ? (int)(at_top & 7u) : -1;
        const uint32_t s8 = fp8_round(half_bits_f(top & 0xFFFFu) * inv_tscale);
        const uint32_t smag = fp8[s8] & 0x7FFFu;
        const float s = half_bits_f(smag);
        const half2_t s2 = splat_half(smag);
        set_slack(L.slack + wave * kWaveRows + row, s, l, slack_set);
        clear_hist(L.hist + wave * kWaveRows * kHistStride, lane);
        wave_fence();
        set_bins<true>(v, kSearchStep * __builtin_amdgcn_rcpf(s), hist, skip);
        wave_fence();
        convert_hist(L.hist + wave * kWaveRows * kHistStride, lane);
        uint64_t left = patterns_left<kTiles, true>(L, C, tiles, wave, lane0);
        __builtin_amdgcn_s_setprio(kPriorityRate);
        // What the table of nearest centroids does not serve is rated value by value (scan_patterns): from the start scales too
        // small for it, and all patterns where the scale was rounded so far that values lie beyond the bins (which reach 1.09
        // scales).  Of scale 0 all patterns are alike: the first wins with index 0.
        const bool beyond = !(half_bits_f(mag) <= 1.08f * s);
        // the scale's code waits in LDS: the search has no register left for it
        if (l == 0) L.spare[wave * kWaveRows + row] = s8;
        uint64_t later = 0;
        if (beyond || !(s >= ecco::kSearchLeastScale)) {
            later = s == 0.0f ? 0ull : !beyond ? left : S == 64 ? ~0ull : (1ull << S) - 1ull;
            left = 0;
        }
        float best;
        uint64_t crowded;
        uint32_t pattern = rate_left<true, 8>(L.hist + wave * kWaveRows * kHistStride, near, pair, v, smag, skip, left, S, lane, best, crowded);
        later |= crowded;
        bool won = false;  // by the comparison value by value
        if (__builtin_amdgcn_ballot_w64(later != 0) != 0ull)
            scan_patterns(reinterpret_cast<float*>(L.hist + wave * kWaveRows * kHistStride), pair_at, v, __builtin_bit_cast(uint32_t, s2) & 0xFFFFu,
                          top >> 16, later, lane, best, pattern, won);
        int skip_again = skip;  // its comparisons are formed here, not kept through the search
        asm volatile("" : "+v"(skip_again));
        // passed by where no row of the wavefront takes them from the table: 131072 all-zero groups took 74.5 us with them
        uint32_t idx = 0, marks = 0;
        if (__builtin_amdgcn_ballot_w64(!won && s != 0.0f) != 0ull) {
            float none;
            marks = rate_pattern<false, true>(near + pattern * ecco::kSearchBins, pair + pattern * 64u, s2, v, skip_again, none, idx);
        }
        const uint64_t scan = __builtin_amdgcn_ballot_w64((won || (marks & ecco::kNearWide) != 0u) && s != 0.0f);
        if (scan != 0ull) {
            const uint32_t id = scan_indices(pair + pattern * 64u, s2, v, skip_again);
            idx = row_any(scan, row) ? id : idx;
        }
        if (s == 0.0f) idx = skip_again < 0 ? 0u : 15u << (28 - 4 * skip_again);

        __builtin_amdgcn_s_setprio(kPriorityPack);
        // the codebook of least total length, lowest on ties
        uint32_t sum = 0;  // four bytes, at most 8 x 8 each
#pragma unroll
        for (int i = 0; i < kRowValues; ++i) sum += lens[pattern * kSym + ((idx >> (28 - 4 * i)) & 15u)];
        const auto add = [](uint32_t a, uint32_t c) { return a + c; };
        const uint32_t even = row_all(sum & 0x00FF00FFu, add), odd = row_all((sum >> 8) & 0x00FF00FFu, add);
        uint32_t book = 0, total = even & 0xFFFFu;
        if ((odd & 0xFFFFu) < total) { total = odd & 0xFFFFu; book = 1; }
        if ((even >> 16) < total) { total = even >> 16; book = 2; }
        if ((odd >> 16) < total) { total = odd >> 16; book = 3; }

        // header, then the codes at their positions
        // taken afresh: what is derived from the lane's place and from the scale is then formed here, not kept through the search
        int at_lane = lane;
        uint32_t top_again = top;
        asm volatile("" : "+v"(at_lane), "+v"(top_again));
        const int place = at_lane & 15;
        const int top_place = (int)(top_again >> 19) == place ? (int)((top_again >> 16) & 7u) : -1;
        uint32_t* image = L.hist + (wave * kWaveRows + (at_lane >> 4)) * kHistStride;
        const uint32_t kp = kpenc[pattern], base = 10u + (kp >> 16), end = base + total;
        image[place] = place == 0 ? (L.spare[wave * kWaveRows + (at_lane >> 4)] << 24) | (book << 22) | ((kp & 0xFFFFu) << (22u - (kp >> 16))) : 0u;
        uint32_t bits[2], n[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bits[h] = 0;
            n[h] = 0;
#pragma unroll
            for (int i = 4 * h; i < 4 * h + 4; ++i) {
                const uint32_t e = codes[(pattern * kBooks + book) * kSym + ((idx >> (28 - 4 * i)) & 15u)];
                bits[h] = (bits[h] << (e & 31u)) | (e >> 8);
                n[h] += e;
            }
            n[h] &= 0xFFu;
        }
        const uint32_t upto = base + row_scan(n[0] + n[1]);
        wave_fence();
        put_bits(image, upto - n[1] - n[0], bits[0], n[0]);
        put_bits(image, upto - n[1], bits[1], n[1]);

        // room left: the largest remaining magnitudes, lower position first, as (position, 8-bit float) entries
        const uint32_t slots = end <= (uint32_t)kBlockBits ? ((uint32_t)kBlockBits - end) / kOutlierBits : 0u;
        if (__builtin_amdgcn_ballot_w64(slots != 0u) != 0ull) {
            const uint32_t from_end = 127u - 8u * (uint32_t)place;
            uint32_t key[kRowValues];  // magnitude, 127 - position, sign: all different
#pragma unroll
            for (int i = 0; i < kRowValues; ++i) {
                const uint32_t x = (i & 1) ? v.x[i >> 1] >> 16 : v.x[i >> 1] & 0xFFFFu;
                key[i] = i == top_place ? 0u : ((x & 0x7FFFu) << 8) | ((from_end - i) << 1) | (x >> 15) | 0x1000000u;
            }
            uint32_t entry = 0, last = 0xFFFFFFFFu;  // lane j keeps entry j
            for (uint32_t j = 0; __builtin_amdgcn_ballot_w64(j < slots) != 0ull; ++j) {
                uint32_t most = 0;
#pragma unroll
                for (int i = 0; i < kRowValues; ++i) most = max(most, key[i] < last ? key[i] : 0u);
                last = row_max(most);
                if ((uint32_t)place == j) entry = last;
            }
            if ((uint32_t)place < slots && entry != 0u) {
                const uint32_t x = ((entry >> 8) & 0x7FFFu) | ((entry & 1u) << 15);
                put_bits(image, end + place * kOutlierBits, ((127u - ((entry >> 1) & 127u)) << 8) | fp8_round(half_bits_f(x) * inv_tscale), kOutlierBits);
            }
        }
        load_values<kSearchBatch>(v, src, n_groups, b + gridDim.x, wave * kWaveRows + row, l);
        wave_fence();
        // the batch's words in the order of the threads
        if (b * kSearchBatch + (uint32_t)(wave * kWaveRows + row) < n_groups) (blocks + b * (kSearchBatch * kBlockWords))[threadIdx.x] = image[place];
        wave_fence();
    }
}

}  // namespace

extern "C" int ecco_pb_encode(const ecco_pb_model* m, const uint16_t* src, size_t n_groups, void* blocks, void* stream) {
    if (!m) return ECCO_EINVAL;
    if (n_groups == 0) return model_ready(m);
    if (!src || !blocks) return ECCO_EINVAL;
    if (!aligned(src, 4) || !aligned(blocks, 64)) return ECCO_EALIGN;
    if (model_ready(m) != ECCO_OK) return ECCO_EINVAL;
    float inv_tscale = 1.0f;  // 2^-texp, exact
    for (int i = 0; i < (m->texp < 0 ? -m->texp : m->texp); ++i) inv_tscale *= m->texp < 0 ? 2.0f : 0.5f;
    const size_t wgs = (n_groups + kSearchBatch - 1) / kSearchBatch;
    const int grid = (int)std::min<size_t>(wgs, (size_t)ecco::cu_count(m->device) * 2);
    const size_t lds = encode_lds_bytes(m->S);
    const auto run = [&](auto kernel) -> int {
        const int rc = ecco::allow_lds(kernel, m->device, lds);
        if (rc != ECCO_OK) return rc;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kSearchThreads), lds, static_cast<hipStream_t>(stream), m->dev, m->S,
                           inv_tscale, reinterpret_cast<const uint32_t*>(src), n_groups, static_cast<uint32_t*>(blocks));
        ECCO_HIP_CHECK(hipGetLastError());
        return ECCO_OK;
    };
    switch (ecco::search_tiles(m->S)) {
        case 1: return run(pb_encode_kernel<1>);
        case 2: return run(pb_encode_kernel<2>);
        default: return run(pb_encode_kernel<4>);
    }
}
