// Decoder of the self-contained 4x block (include/ecco_paper_block.h) for gfx950, alone and fused into the matrix-vector product.
//
// Two steps per 64 blocks of a wavefront.  (1) The block is one code stream of 128 values behind a variable-length header,
// so a lane owns a whole block and walks it: an 8-bit peek into a byte table per (pattern, codebook) -- 4 x S tables of 256
// bytes, 64 KB for S = 64 -- gives the index and the length; only the 4-bit indices are kept, in LDS.  (2) The values are
// formed with a block per row of 16 lanes, eight values per lane: a row's centroid reads fall into one pattern's 32 bytes,
// the activations come and the decoded values leave in whole lines, and the padded entries (known only when the stream has
// been walked to its end, at most 16) are taken up by the row's lanes side by side.
// What bounds it: step 1 is a serial chain of 128 dependent table reads per lane, and the LDS holds eight wavefronts beside
// the 64 KB of tables.  Doing everything in step 1 (a centroid read, presence and sign tests per value, a loop over the
// padded entries as long as the wavefront's longest list) took twice as long: 29.3 us for the product over 4096 x 4096,
// 21.4 us for the decode.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "ecco_pb_launch.h"

namespace {

using namespace ecco_pb;

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) uint8_t lds_u8;

constexpr int kSlot = kBlockWords + 1;    // LDS words per staged block; the last one is a zero pad
constexpr int kUnit = 64;                 // blocks per wavefront pass, one per lane
constexpr int kPayWords = kUnit * kSlot + 4;
constexpr int kIdxStride = 17;            // words per block of the index image: values 8 w .. 8 w + 3 in the upper nibbles of word w, the next four in the lower ones
constexpr int kInfoWords = 2 * kUnit;     // per block: where its centroids are, values present, padded entries, scale; where its stream ends
constexpr int kRows = 4;                  // blocks per wavefront in step 2
constexpr int kPair = 2;                  // blocks per row at a time: their table reads are in flight together
constexpr int kRowWords = kPair * kRows * kGroup / 2;  // decoded values of the blocks in hand, where padded entries are put in
constexpr int kWaveWords = kInfoWords + kPayWords + kUnit * kIdxStride;  // private LDS of a wavefront, then (decoder only) kRowWords
// the header takes at most 18 bits and a code at most 8: value i ends at or before bit 18 + 8 (i + 1), inside the block for i < 61
constexpr int kAlwaysPresent = (kBlockBits - 18) / kMaxLen;
constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// words % 4 == 0, 16-byte aligned; eight loads in flight per thread
__device__ __forceinline__ void stage_words(uint32_t* dst, const uint32_t* __restrict__ src, int words) {
    const uint4* s = reinterpret_cast<const uint4*>(src);
    uint4* d = reinterpret_cast<uint4*>(dst);
    const int n = words >> 2;
    for (int i = threadIdx.x; i < n; i += 8 * kThreads) {
        uint4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = s[min(i + j * kThreads, n - 1)];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (i + j * kThreads < n) d[i + j * kThreads] = v[j];
    }
}

// LDS of the tables, in words: those of the model, then its centroids once more with index 15 standing for -1 instead of 1
// (a block with a negative scale uses these)
constexpr size_t table_words(int S) { return DevLayout{S}.decode_words() + (size_t)S * 8; }
inline size_t lds_bytes(int S, int wave_words) { return (table_words(S) + (size_t)kWaves * wave_words) * 4; }

struct Tables {
    const uint8_t* lut;
    const uint16_t* kplut;
    const uint16_t* fp8;
    uint32_t cent;           // LDS address
    uint32_t minus;          // from a pattern's centroids to those with -1
};
__device__ __forceinline__ Tables stage_tables(uint32_t* smem, const uint32_t* __restrict__ dev, int S) {
    const DevLayout D{S};
    stage_words(smem, dev, (int)D.decode_words());
    for (int i = threadIdx.x; i < S * 8; i += kThreads) {
        uint32_t c = dev[D.cent() + i];
        if ((i & 7) == 7) c ^= 0x80000000u;
        smem[D.decode_words() + i] = c;
    }
    Tables t;
    t.lut = reinterpret_cast<const uint8_t*>(smem + D.lut());
    t.kplut = reinterpret_cast<const uint16_t*>(smem + D.kplut());
    t.fp8 = reinterpret_cast<const uint16_t*>(smem + D.fp8());
    t.cent = (uint32_t)(size_t)(const lds_u8*)reinterpret_cast<const uint8_t*>(smem + D.cent());
    t.minus = (uint32_t)(D.decode_words() - D.cent()) * 4;
    return t;
}
__device__ __forceinline__ uint32_t lds_half(uint32_t address) { return *(const lds_u16*)(size_t)address; }

struct PieceLoad {
    uint4 v[4];
};
// the `count` blocks at `first` (1..64); slots beyond them hold a copy of the last one
__device__ __forceinline__ PieceLoad load_pieces(const uint4* __restrict__ first, int count, int lane) {
    PieceLoad L;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int q = lane + 64 * r;  // piece q of the pass: block q / 4, part q % 4
        L.v[r] = first[min(q >> 2, count - 1) * 4 + (q & 3)];
    }
    return L;
}
__device__ __forceinline__ void store_pieces(uint32_t* pay, const PieceLoad& L, int lane) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int q = lane + 64 * r;
        uint32_t* d = pay + (q >> 2) * kSlot + (q & 3) * 4;
        d[0] = L.v[r].x; d[1] = L.v[r].y; d[2] = L.v[r].z; d[3] = L.v[r].w;
    }
}

// A wavefront's private LDS.
struct WaveLds {
    uint32_t* rows;  // decoder: values of the blocks in hand
    uint32_t* pay;   // payloads, kSlot words per block
    uint32_t* idx;   // indices, kIdxStride words per block
    uint2* info;     // per block: x = offset of its centroids | values present << 16 | padded entries << 24;  y = |scale| (FP16 bits) | end of the stream << 16
};
__device__ __forceinline__ WaveLds wave_lds(uint32_t* base) {
    WaveLds w;
    w.info = reinterpret_cast<uint2*>(base);
    w.pay = base + kInfoWords;
    w.idx = w.pay + kPayWords;
    w.rows = w.idx + kUnit * kIdxStride;
    return w;
}

// Step 1: walks the block staged in this lane's slot and leaves its indices and its info word in LDS.  Values are taken in
// runs of four out of a 64-bit window (at least 33 valid bits); the words of the next run's window are requested before the
// run, so that the dependent chain holds only the table reads.  A value is present iff its code ends inside the block; the
// position stops at bit 512, where the window is zero.
__device__ __forceinline__ void walk_block(const WaveLds& L, const Tables& T, int lane) {
    const uint32_t* w = L.pay + lane * kSlot;
    const uint32_t first = w[0];
    const uint32_t kpe = T.kplut[(first >> 14) & 0xFFu], p = kpe >> 8;
    const uint32_t sv = T.fp8[first >> 24];  // the signed scale, FP16 bits
    const uint8_t* tab = T.lut + (p * kBooks + ((first >> 22) & 3u)) * 256u;
    uint32_t fetch = 10u + (kpe & 0xFFu);    // where the next run is fetched from; stops at 512
    uint32_t reach = fetch;                   // where the codes read so far end; keeps counting past 512
    uint32_t present = 0;
    uint32_t wi = 0, w0 = first, w1 = w[1], w2 = w[2];
    uint32_t* out = L.idx + lane * kIdxStride;
#pragma unroll
    for (int i0 = 0; i0 < kGroup; i0 += 8) {
        uint32_t packed[2];  // four table bytes each
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
            uint64_t win = (((uint64_t)w0 << 32) | (uint64_t)w1) << (fetch & 31u);
            uint32_t e[4], len[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                e[j] = tab[(uint32_t)(win >> 56)];
                len[j] = e[j] & 15u;
                win <<= len[j];
            }
            packed[h >> 2] = __builtin_amdgcn_perm(e[1], e[0], 0x0C0C0400u) | __builtin_amdgcn_perm(e[3], e[2], 0x04000C0Cu);
            const uint32_t used = (len[0] + len[1]) + (len[2] + len[3]);
            if (i0 + h + 3 >= kAlwaysPresent) {
                // all four, or, in the run that crosses the end, those that end inside
                const bool whole = reach + used <= (uint32_t)kBlockBits;
                present += whole ? 4u : 0u;
                if (!whole && reach <= (uint32_t)kBlockBits) {
                    uint32_t at = reach;
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        at += len[j];
                        present += at <= (uint32_t)kBlockBits ? 1u : 0u;
                    }
                }
            } else {
                present += 4u;
            }
            reach += used;
            if (i0 + h + 4 < kGroup) {
                fetch = min(fetch + used, (uint32_t)kBlockBits);
                const uint32_t nwi = fetch >> 5;  // wi or wi + 1
                const bool adv = nwi != wi;
                w0 = adv ? w1 : w0;
                w1 = adv ? w2 : w1;
                w2 = w[nwi + 2u];  // used one run later at the earliest; past the pad it is never looked at
                wi = nwi;
            }
        }
        out[i0 >> 3] = (packed[0] & 0xF0F0F0F0u) | ((packed[1] >> 4) & 0x0F0F0F0Fu);
    }
    const uint32_t entries = reach <= (uint32_t)kBlockBits ? ((uint32_t)kBlockBits - reach) / kOutlierBits : 0u;
    L.info[lane] = make_uint2((p * 32u + ((sv & 0x8000u) ? T.minus : 0u)) | (present << 16) | (entries << 24), (sv & 0x7FFFu) | (min(reach, 0xFFFFu) << 16));
}

// Step 2, common part: block `blk` of the pass, lane l of its row.
struct RowBlock {
    uint32_t cent;       // LDS address of its centroids
    uint32_t c[8];       // the lane's eight centroids, FP16 bits; 0 where the value is absent
    int present;         // how many of the lane's values are present (may be negative or beyond 8)
    uint32_t entries;    // padded entries of the block
    uint32_t end;        // where they start
    uint32_t scale;      // FP16 bits
};
__device__ __forceinline__ RowBlock row_block(const WaveLds& L, const Tables& T, int blk, int l) {
    const uint2 i = L.info[blk];
    const uint32_t nibbles = L.idx[blk * kIdxStride + l];
    RowBlock r;
    r.cent = T.cent + (i.x & 0xFFFFu);
    r.present = (int)((i.x >> 16) & 0xFFu) - 8 * l;
    r.entries = i.x >> 24;
    r.scale = i.y & 0xFFFFu;
    r.end = i.y >> 16;
    // twice the indices, a byte each (values 0..3 and 4..7): a byte is then one addition away from its address
    const uint32_t twice[2] = {(nibbles >> 3) & 0x1E1E1E1Eu, (nibbles << 1) & 0x1E1E1E1Eu};
#pragma unroll
    for (int k = 0; k < 8; ++k) r.c[k] = lds_half(r.cent + ((twice[k >> 2] >> (8 * (k & 3))) & 0xFFu));
    return r;
}
// Takes out the absent values of the blocks in hand.  Most cut streams lose a value or two, so the first four of a lane
// are looked at only where one of the wavefront's lanes has lost more.
template <int kBlocks>
__device__ __forceinline__ void drop_absent(RowBlock (&r)[kBlocks]) {
    int least = r[0].present;
#pragma unroll
    for (int q = 1; q < kBlocks; ++q) least = min(least, r[q].present);
    if (__builtin_amdgcn_ballot_w64(least < 8) == 0ull) return;
#pragma unroll
    for (int q = 0; q < kBlocks; ++q)
#pragma unroll
        for (int k = 4; k < 8; ++k) r[q].c[k] = k < r[q].present ? r[q].c[k] : 0u;
    if (__builtin_amdgcn_ballot_w64(least < 4) == 0ull) return;
#pragma unroll
    for (int q = 0; q < kBlocks; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) r[q].c[k] = k < r[q].present ? r[q].c[k] : 0u;
}

// The padded entry of this lane (entry l of the block), if there is one and no later entry has the same position: a
// sequential reader of the block ends up with the last one.
struct Entry {
    bool valid;
    uint32_t pos, value;  // position in the block; FP16 bits
};
template <int kShift>
__device__ __forceinline__ bool later_has(uint32_t key) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)key, 0x100 + kShift, 0xF, 0xF, true) == key;  // row_shl: from lane l + kShift, 0 beyond the row
}
__device__ __forceinline__ Entry row_entry(const WaveLds& L, const Tables& T, const RowBlock& r, int blk, int l) {
    const uint32_t* w = L.pay + blk * kSlot;
    const uint32_t at = min(r.end + (uint32_t)l * kOutlierBits, (uint32_t)kBlockBits - 1u), wi = at >> 5;
    const uint64_t win = (((uint64_t)w[wi] << 32) | (uint64_t)w[wi + 1]) << (at & 31u);
    const uint32_t code = (uint32_t)(win >> 49);   // 7-bit position, 8-bit float
    Entry e;
    e.valid = (uint32_t)l < r.entries;
    e.pos = code >> 8;
    e.value = T.fp8[code & 0xFFu];
    const uint32_t key = e.valid ? e.pos + 1u : 0xFFFFu;
    if (__builtin_amdgcn_ballot_w64(r.entries > 1u) != 0ull) {
        bool dup = later_has<1>(key) || later_has<2>(key) || later_has<3>(key);
        if (__builtin_amdgcn_ballot_w64(r.entries > 4u) != 0ull) {
            dup = dup || later_has<4>(key) || later_has<5>(key) || later_has<6>(key) || later_has<7>(key) || later_has<8>(key) || later_has<9>(key);
            dup = dup || later_has<10>(key) || later_has<11>(key) || later_has<12>(key) || later_has<13>(key) || later_has<14>(key) || later_has<15>(key);
        }
        e.valid = e.valid && !dup;
    }
    return e;
}

// grid x 8 wavefronts, each `unit` consecutive blocks at a time (a multiple of four, at most 64): small inputs are spread
// over all wavefronts of the chip, since a chain takes as long for one lane as for 64
__global__ __launch_bounds__(kThreads) void pb_decode_kernel(const uint32_t* __restrict__ dev, int S, const uint4* __restrict__ blocks, size_t n_groups,
                                                             int unit, uint4* __restrict__ dst) {
    extern __shared__ __align__(16) uint32_t smem[];
    const int lane = threadIdx.x & 63, l = lane & 15, row = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const WaveLds L = wave_lds(smem + table_words(S) + wave * (kWaveWords + kRowWords));
    const size_t n_units = (n_groups + unit - 1) / unit, step = (size_t)gridDim.x * kWaves;
    size_t u = (size_t)blockIdx.x * kWaves + wave;
    const auto load = [&](size_t v) {
        const size_t first = min(v * unit, n_groups - 1);
        return load_pieces(blocks + first * 4, (int)min(n_groups - first, (size_t)unit), lane);
    };
    PieceLoad pre = load(u);
    const Tables T = stage_tables(smem, dev, S);
    L.pay[lane * kSlot + kBlockWords] = 0u;
    if (lane < 4) L.pay[kUnit * kSlot + lane] = 0u;
    __syncthreads();

    for (; u < n_units; u += step) {
        wave_lds_fence();
        store_pieces(L.pay, pre, lane);
        wave_lds_fence();
        pre = load(u + step);
        walk_block(L, T, lane);
        wave_lds_fence();
        const int count = (int)min(n_groups - u * unit, (size_t)unit);
        uint4* out = dst + u * unit * (kGroup / 8);
        for (int b0 = 0; b0 < count; b0 += kPair * kRows) {
            RowBlock r[kPair];
#pragma unroll
            for (int q = 0; q < kPair; ++q) r[q] = row_block(L, T, b0 + q * kRows + row, l);
            drop_absent(r);
            uint32_t entries = 0;
#pragma unroll
            for (int q = 0; q < kPair; ++q) {
                const half2_t s2 = __builtin_bit_cast(half2_t, r[q].scale | (r[q].scale << 16));
#pragma unroll
                for (int i = 0; i < 4; ++i)  // each product rounds once
                    r[q].c[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, r[q].c[2 * i] | (r[q].c[2 * i + 1] << 16)) * s2);
                entries |= r[q].entries;
            }
            if (__builtin_amdgcn_ballot_w64(entries != 0u) != 0ull) {  // through LDS, where each entry's lane puts its value in
                wave_lds_fence();
#pragma unroll
                for (int q = 0; q < kPair; ++q) {
                    const Entry e = row_entry(L, T, r[q], b0 + q * kRows + row, l);
                    uint32_t* at = L.rows + (q * kRows + row) * (kGroup / 2);
                    reinterpret_cast<uint4*>(at)[l] = make_uint4(r[q].c[0], r[q].c[1], r[q].c[2], r[q].c[3]);
                    wave_lds_fence();
                    if (e.valid) reinterpret_cast<uint16_t*>(at)[e.pos] = (uint16_t)e.value;
                }
                wave_lds_fence();
#pragma unroll
                for (int q = 0; q < kPair; ++q) {
                    const uint4 t = reinterpret_cast<const uint4*>(L.rows + (q * kRows + row) * (kGroup / 2))[l];
                    r[q].c[0] = t.x; r[q].c[1] = t.y; r[q].c[2] = t.z; r[q].c[3] = t.w;
                }
            }
#pragma unroll
            for (int q = 0; q < kPair; ++q) {
                const int blk = b0 + q * kRows + row;
                if (blk < count) out[blk * (kGroup / 8) + l] = make_uint4(r[q].c[0], r[q].c[1], r[q].c[2], r[q].c[3]);
            }
        }
    }
}

// ---- decode fused into the matrix-vector product --------------------------------------------------------------------
// y = W x without writing W: a workgroup owns a band of rows (its blocks are consecutive in memory); per-block sums go to
// LDS, and each row's blocks are added in a fixed tree.  A padded entry takes centroid * x at its position back and adds its
// own value (times x) instead.
constexpr int kPartFloats = 1536;        // per-block sums of a band: band rows x column groups
inline size_t gemv_lds_bytes(int S) { return lds_bytes(S, kWaveWords) + kPartFloats * 4; }

template <int kCtrl>
__device__ __forceinline__ float dpp_add(float t) {
    return __fadd_rn(t, __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, t), kCtrl, 0xF, 0xF, true)));
}
// FP32 sum over a row of 16 lanes in the balanced tree
__device__ __forceinline__ float row_sum(float t) {
    t = dpp_add<0xB1>(t);    // quad_perm [1,0,3,2]
    t = dpp_add<0x4E>(t);    // quad_perm [2,3,0,1]
    t = dpp_add<0x141>(t);   // row_half_mirror
    return dpp_add<0x140>(t);  // row_mirror
}
__device__ __forceinline__ float wave_sum(float t) {
    t = row_sum(t);
    const auto lane_of = [&](int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, t), l)); };
    return __fadd_rn(__fadd_rn(lane_of(0), lane_of(16)), __fadd_rn(lane_of(32), lane_of(48)));
}
__device__ __forceinline__ float half_f(uint32_t bits) { return (float)__builtin_bit_cast(_Float16, (unsigned short)bits); }

__global__ __launch_bounds__(kThreads) void pb_gemv_kernel(const uint32_t* __restrict__ dev, int S, const uint4* __restrict__ blocks, int rows, int gpr, int band,
                                                           int unit, const uint4* __restrict__ x, float* __restrict__ y) {
    extern __shared__ __align__(16) uint32_t smem[];
    const int lane = threadIdx.x & 63, l = lane & 15, row = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const WaveLds L = wave_lds(smem + table_words(S) + wave * kWaveWords);
    float* part = reinterpret_cast<float*>(smem + table_words(S) + kWaves * kWaveWords);

    const int r0 = blockIdx.x * band, nrows = min(band, rows - r0);
    const uint4* first = blocks + (size_t)r0 * gpr * 4;   // first block of the band
    const int n_blocks = nrows * gpr;                     // <= kPartFloats
    const auto load = [&](int at) {
        at = min(at, n_blocks - 1);
        return load_pieces(first + (size_t)at * 4, min(n_blocks - at, unit), lane);
    };
    int at = wave * unit;
    PieceLoad pre = load(at);
    const Tables T = stage_tables(smem, dev, S);
    L.pay[lane * kSlot + kBlockWords] = 0u;
    if (lane < 4) L.pay[kUnit * kSlot + lane] = 0u;
    __syncthreads();

    const int four = kRows % gpr;
    for (; at < n_blocks; at += kWaves * unit) {
        const int count = min(n_blocks - at, unit);
        wave_lds_fence();
        store_pieces(L.pay, pre, lane);
        wave_lds_fence();
        // the activations of the pass, requested ahead of the walk: eight of each block's column group per lane
        uint4 xs[kUnit / kRows];
        int cg[kUnit / kRows];
        cg[0] = (at + row) % gpr;
#pragma unroll
        for (int i = 1; i < kUnit / kRows; ++i) {
            cg[i] = cg[i - 1] + four;
            cg[i] -= cg[i] >= gpr ? gpr : 0;
        }
#pragma unroll
        for (int i = 0; i < kUnit / kRows; ++i)
            if (i * kRows < count) xs[i] = x[(size_t)cg[i] * 16 + l];
        pre = load(at + kWaves * unit);
        walk_block(L, T, lane);
        wave_lds_fence();
#pragma unroll
        for (int i0 = 0; i0 < kUnit / kRows; i0 += kPair) {
            if (i0 * kRows >= count) break;
            RowBlock r[kPair];
#pragma unroll
            for (int q = 0; q < kPair; ++q) r[q] = row_block(L, T, (i0 + q) * kRows + row, l);
            drop_absent(r);
            float acc[kPair], extra[kPair];
            uint32_t entries = 0;
#pragma unroll
            for (int q = 0; q < kPair; ++q) {
                const uint32_t xw[4] = {xs[i0 + q].x, xs[i0 + q].y, xs[i0 + q].z, xs[i0 + q].w};
                acc[q] = 0.0f;
                extra[q] = 0.0f;
#pragma unroll
                for (int k = 0; k < 8; ++k) acc[q] = fmaf(half_f(r[q].c[k]), half_f(k & 1 ? xw[k >> 1] >> 16 : xw[k >> 1] & 0xFFFFu), acc[q]);
                entries |= r[q].entries;
            }
            if (__builtin_amdgcn_ballot_w64(entries != 0u) != 0ull) {
#pragma unroll
                for (int q = 0; q < kPair; ++q) {
                    const int blk = (i0 + q) * kRows + row;
                    const Entry e = row_entry(L, T, r[q], blk, l);
                    if (e.valid) {
                        const float xi = half_f(reinterpret_cast<const uint16_t*>(x)[(size_t)cg[i0 + q] * kGroup + e.pos]);
                        const uint32_t k = (L.idx[blk * kIdxStride + (e.pos >> 3)] >> (8u * (e.pos & 3u) + ((e.pos & 4u) ? 0u : 4u))) & 15u;
                        acc[q] = fmaf(-half_f(lds_half(r[q].cent + k * 2u)), xi, acc[q]);
                        extra[q] = half_f(e.value) * xi;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < kPair; ++q) {
                const int blk = (i0 + q) * kRows + row;
                const float t = row_sum(fmaf(acc[q], half_f(r[q].scale), extra[q]));
                if (l == 0 && blk < count) part[at + blk] = t;
            }
        }
    }
    __syncthreads();
    // row sums: the blocks of a row in a fixed order (lane-strided partial sums, then the wavefront tree)
    for (int r = wave; r < nrows; r += kWaves) {
        float sum = 0.0f;
        for (int c = lane; c < gpr; c += 64) sum += part[r * gpr + c];
        sum = wave_sum(sum);
        if (lane == 0) y[r0 + r] = sum;
    }
}

// blocks a wavefront takes at a time when n are dealt to `waves` wavefronts
inline int unit_of(size_t n, size_t waves) { return (int)std::min<size_t>(kUnit, ((n + waves - 1) / waves + kRows - 1) / kRows * kRows); }

}  // namespace

extern "C" {

int ecco_pb_decode_gemv(const ecco_pb_model* m, const void* blocks, int rows, int cols, const uint16_t* x, float* y, void* stream) {
    if (!m || !blocks || !x || !y) return ECCO_EINVAL;
    if (rows <= 0 || cols <= 0 || cols % kGroup != 0 || cols > 65536) return ECCO_ESHAPE;
    if (!aligned(blocks, 64) || !aligned(x, 16) || !aligned(y, 4)) return ECCO_EALIGN;
    if (model_ready(m) != ECCO_OK) return ECCO_EINVAL;
    const int gpr = cols / kGroup, cus = ecco::cu_count(m->device);
    // a band of rows per workgroup: about one band per compute unit, at most kPartFloats blocks
    const int band = std::min(std::max(1, (rows + cus - 1) / cus), std::max(1, kPartFloats / gpr));
    const int grid = (rows + band - 1) / band;
    const size_t lds = gemv_lds_bytes(m->S);
    const int rc = ecco::allow_lds(pb_gemv_kernel, m->device, lds);
    if (rc != ECCO_OK) return rc;
    hipLaunchKernelGGL(pb_gemv_kernel, dim3(grid), dim3(kThreads), lds, static_cast<hipStream_t>(stream), m->dev, m->S, static_cast<const uint4*>(blocks), rows, gpr,
                       band, unit_of((size_t)band * gpr, kWaves), reinterpret_cast<const uint4*>(x), y);
    ECCO_HIP_CHECK(hipGetLastError());
    return ECCO_OK;
}

int ecco_pb_decode(const ecco_pb_model* m, const void* blocks, size_t n_groups, uint16_t* dst, void* stream) {
    if (!m) return ECCO_EINVAL;
    if (n_groups == 0) return model_ready(m);
    if (!blocks || !dst) return ECCO_EINVAL;
    if (n_groups >= ((size_t)1 << 31)) return ECCO_ESHAPE;
    if (!aligned(blocks, 64) || !aligned(dst, 16)) return ECCO_EALIGN;
    if (model_ready(m) != ECCO_OK) return ECCO_EINVAL;
    const size_t lds = lds_bytes(m->S, kWaveWords + kRowWords);
    const int rc = ecco::allow_lds(pb_decode_kernel, m->device, lds);
    if (rc != ECCO_OK) return rc;
    const size_t cus = (size_t)ecco::cu_count(m->device);
    const int unit = unit_of(n_groups, cus * kWaves);
    const size_t units = (n_groups + unit - 1) / unit;
    const int grid = (int)std::min<size_t>((units + kWaves - 1) / kWaves, cus);
    hipLaunchKernelGGL(pb_decode_kernel, dim3(grid), dim3(kThreads), lds, static_cast<hipStream_t>(stream), m->dev, m->S, static_cast<const uint4*>(blocks), n_groups,
                       unit, reinterpret_cast<uint4*>(dst));
    ECCO_HIP_CHECK(hipGetLastError());
    return ECCO_OK;
}

}  // extern "C"
