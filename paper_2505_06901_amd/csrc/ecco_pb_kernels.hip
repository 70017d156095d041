// Decoder of the self-contained 4x block (include/ecco_paper_block.h) for gfx950, alone and fused into the matrix-vector product.
//
// Two steps per 64 blocks of a wavefront.  (1) The block is one code stream of 128 values behind a variable-length header,
// so a lane owns a whole block and walks it: an 8-bit peek into a byte table per (pattern, codebook) -- 4 x S tables of 256
// bytes, 64 KB for S = 64 -- gives the index and the length; only the 4-bit indices are kept.  (2) The values are formed with
// a block per row of 16 lanes, eight values per lane: a row's centroid reads fall into one pattern's 32 bytes, and the
// activations come and the decoded values leave in whole lines.  (With the lanes of a matrix-core operand, 16 blocks at a time, the
// reads of one instruction fall into 16 patterns' tables and cost twice as much: 16.8 us where this takes 15.7.)  The padded entries
// are few (one block in ten has any) and are taken up a block per lane, not by the rows.
// What bounds it: step 1 is a serial chain of 128 table reads per lane, about 82 cycles each when nothing else is in the way (56 of the
// read, 8.5 for each of the three dependent instructions; 97 while the window was rebuilt on the chain); step 2 the vector instructions.  Product
// over 4096 x 4096, one pass per wavefront, by events around replayed graphs, before that: 4.6 us launch, tables and payload, 6 us walk, 2 us
// padded entries, 3 us values, 15.6 us together; 18.1 us with the entries taken up by the rows and the index image beside the payload.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "ecco_pb_launch.h"
#include "ecco_stream.h"

namespace {

using namespace ecco_pb;

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) uint8_t lds_u8;

constexpr int kSlot = kBlockWords + 1;    // LDS words per staged block; the last one is a zero pad
constexpr int kUnit = 64;                 // blocks per wavefront pass, one per lane
constexpr int kPayWords = kUnit * kSlot + 4;
constexpr int kInfoWords = 2 * kUnit;     // per block: where its centroids are and how many values are present; scale
constexpr int kIdxWords = kGroup / 8;     // words per block of the index image: values 8 w .. 8 w + 3 in the upper nibbles of word w, the next four in the lower ones
constexpr int kRows = 4;                  // blocks per wavefront in step 2
constexpr int kPair = 2;                  // decoder: blocks per row at a time, so that their table reads are in flight together
// the header takes at most 18 bits and a code at most 8: value i ends at or before bit 18 + 8 (i + 1), inside the block for i < 61
constexpr int kAlwaysPresent = (kBlockBits - 18) / kMaxLen;
constexpr int kDecodeThreads = 512;
constexpr int kGemvThreads = 1024;

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of the tables, in words: those of the model, then its centroids once more with index 15 standing for -1 instead of 1
// (a block with a negative scale uses these)
constexpr size_t table_words(int S) { return DevLayout{S}.decode_words() + (size_t)S * 8; }

struct Tables {
    const uint8_t* lut;
    const uint16_t* kplut;
    const uint16_t* fp8;
    uint32_t cent;           // LDS address
    uint32_t minus;          // from a pattern's centroids to those with -1
};
// Copies the tables to LDS; `prefetch` issues the loads of the first unit.  Loads return in issue order and a wait names how many
// may still be outstanding: every thread requests its pieces of the tables first, on one straight path (indices clamped), and
// the payload behind them, so that the copy does not wait for the payload.  The caller synchronises afterwards.
template <int kThreads, class Prefetch>
__device__ __forceinline__ Tables stage_tables(uint32_t* smem, const uint32_t* __restrict__ dev, int S, Prefetch&& prefetch) {
    const DevLayout D{S};
    constexpr int kMaxPieces = (int)(DevLayout{kMaxS}.decode_words() / 4);
    constexpr int kEach = (kMaxPieces + kThreads - 1) / kThreads;
    static_assert(kMaxS * 8 <= kDecodeThreads && kMaxS * 8 <= kGemvThreads, "a word of the second centroids per thread");
    const uint4* s = reinterpret_cast<const uint4*>(dev);
    uint4* d = reinterpret_cast<uint4*>(smem);
    const int n = (int)(D.decode_words() / 4), tid = threadIdx.x;
    const uint32_t c = dev[D.cent() + min(tid, S * 8 - 1)];
    uint4 v[kEach];
#pragma unroll
    for (int j = 0; j < kEach; ++j) v[j] = s[min(tid + j * kThreads, n - 1)];
    __builtin_amdgcn_sched_barrier(0);
    prefetch();
    __builtin_amdgcn_sched_barrier(0);
    if (tid < S * 8) smem[D.decode_words() + tid] = (tid & 7) == 7 ? c ^ 0x80000000u : c;
#pragma unroll
    for (int j = 0; j < kEach; ++j)
        if (tid + j * kThreads < n) d[tid + j * kThreads] = v[j];
    Tables t;
    t.lut = reinterpret_cast<const uint8_t*>(smem + D.lut());
    t.kplut = reinterpret_cast<const uint16_t*>(smem + D.kplut());
    t.fp8 = reinterpret_cast<const uint16_t*>(smem + D.fp8());
    t.cent = (uint32_t)(size_t)(const lds_u8*)reinterpret_cast<const uint8_t*>(smem + D.cent());
    t.minus = (uint32_t)(D.decode_words() - D.cent()) * 4;
    return t;
}
__device__ __forceinline__ uint32_t lds_half(uint32_t address) { return *(const lds_u16*)(size_t)address; }
__device__ __forceinline__ float half_f(uint32_t bits) { return (float)__builtin_bit_cast(_Float16, (unsigned short)bits); }

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

// What the walk of a block leaves in its lane.
struct Walked {
    uint32_t cent;     // offset of the block's centroids
    uint32_t scale;    // |scale|, FP16 bits
    uint32_t present;  // values present
    uint32_t entries;  // padded entries
    uint32_t end;      // where they start
};
// Step 1: walks the block staged in this lane's slot; put(i, word) receives the indices of values 8 i .. 8 i + 7.  Values are taken
// in runs of four out of a 64-bit window whose upper half is whole again when a run ends (it consumes at most 32 bits); the lower
// half is then filled from the words that follow, in the shadow of the next run's first table read, so that the dependent chain
// holds only the table reads, a mask, a shift and an addition each (whole window rebuilt: seven more dependent instructions per run; 4096 x 4096
// 14.0 -> 13.7 us).  A value is present iff its code ends inside the block; from its end on the stream is zero.
template <class Put>
__device__ __forceinline__ Walked walk_block(const uint32_t* w, const Tables& T, Put&& put) {
    const uint32_t first = w[0];
    const uint32_t kpe = T.kplut[(first >> 14) & 0xFFu], p = kpe >> 8;
    const uint32_t sv = T.fp8[first >> 24];  // the signed scale, FP16 bits
    const uint8_t* tab = T.lut + (p * kBooks + ((first >> 22) & 3u)) * 256u;
    uint32_t reach = 10u + (kpe & 0xFFu);     // where the codes read so far end; below 32 to begin with
    // the window's bits 0..31 are carried along, bits 32..63 come from the words w1, w2; `next` is the first of them, negated
    int32_t next = -1;
    uint32_t w1 = w[1], w2 = w[2], w3 = w[3];
    uint64_t win = ((((uint64_t)first << 32) | (uint64_t)w1) << reach) & 0xFFFFFFFF00000000ull;
    win |= __builtin_amdgcn_alignbit(w1, w2, 0u - reach);
    // of the last run that starts inside the block: how many came before it, where it starts, its table bytes
    uint32_t runs = 0, last_start = 0, last_run = 0;
#pragma unroll
    for (int i0 = 0; i0 < kGroup; i0 += 8) {
        uint32_t packed[2];  // four table bytes each
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
            uint32_t e[4], len[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                e[j] = tab[(uint32_t)(win >> 56)];
                len[j] = e[j] & 15u;
                win <<= len[j];
            }
            packed[h >> 2] = __builtin_amdgcn_perm(e[1], e[0], 0x0C0C0400u) | __builtin_amdgcn_perm(e[3], e[2], 0x04000C0Cu);
            if (i0 + h + 3 >= kAlwaysPresent) {
                const bool inside = reach <= (uint32_t)kBlockBits;
                runs += inside ? 1u : 0u;
                last_start = inside ? reach : last_start;
                last_run = inside ? packed[h >> 2] : last_run;
            }
            const uint32_t used = (len[0] + len[1]) + (len[2] + len[3]);
            reach += used;
            if (i0 + h + 4 < kGroup) {
                const int32_t now = -(int32_t)reach >> 5;  // next or next - 1
                const bool adv = now != next;
                w1 = adv ? w2 : w1;
                w2 = adv ? w3 : w2;
                w3 = w[min(2u - (uint32_t)now, (uint32_t)kBlockWords)];  // used one run later at the earliest; from the pad on zero
                win = (win & 0xFFFFFFFF00000000ull) | (uint64_t)__builtin_amdgcn_alignbit(w1, w2, 0u - reach);
                next = now;
            }
        }
        uint32_t word = (packed[0] & 0xF0F0F0F0u) | ((packed[1] >> 4) & 0x0F0F0F0Fu);
        // finished here: left to the compiler, these are formed after the walk and its 128 table bytes stay in registers
        asm volatile("" : "+v"(word), "+v"(reach), "+v"(runs), "+v"(last_start), "+v"(last_run));
        put(i0 >> 3, word);
    }
    Walked r;
    r.cent = p * 32u + ((sv & 0x8000u) ? T.minus : 0u);
    r.scale = sv & 0x7FFFu;
    r.end = reach;
    r.entries = reach <= (uint32_t)kBlockBits ? ((uint32_t)kBlockBits - reach) / kOutlierBits : 0u;
    constexpr int kSure = kAlwaysPresent / 4 * 4;  // values before the runs that were counted
    r.present = kSure - 4u + 4u * runs;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        last_start += (last_run >> (8 * j)) & 15u;
        r.present += last_start <= (uint32_t)kBlockBits ? 1u : 0u;
    }
    return r;
}

// Padded entry j (< 16) of the block staged at w: position << 8 | 8-bit float.
__device__ __forceinline__ uint32_t entry_code(const uint32_t* w, uint32_t end, uint32_t j) {
    const uint32_t at = min(end + j * kOutlierBits, (uint32_t)kBlockBits - 1u), wi = at >> 5;
    return (uint32_t)(((((uint64_t)w[wi] << 32) | (uint64_t)w[wi + 1]) << (at & 31u)) >> 49);
}

// Step 2, common part: the lane's eight centroids (FP16 bits) for the indices `nibbles`, 0 where the value is absent.
struct RowBlock {
    uint32_t c[8];
    int present;         // how many of the lane's values are present (may be negative or beyond 8)
    uint32_t scale;      // as the info word has it
};
__device__ __forceinline__ RowBlock row_block(const Tables& T, uint2 info, uint32_t nibbles, int l) {
    RowBlock r;
    const uint32_t cent = T.cent + (info.x & 0xFFFFu);
    r.present = (int)(info.x >> 16) - 8 * l;
    r.scale = info.y;
    // twice the indices, a byte each (values 0..3 and 4..7): a byte is then one addition away from its address
    // (passed through an empty asm statement: the compiler would take each byte out of the indices by a shift and a mask of its own)
    uint32_t twice[2] = {(nibbles >> 3) & 0x1E1E1E1Eu, (nibbles << 1) & 0x1E1E1E1Eu};
    asm("" : "+v"(twice[0]), "+v"(twice[1]));
#pragma unroll
    for (int k = 0; k < 8; ++k) r.c[k] = lds_half(cent + ((twice[k >> 2] >> (8 * (k & 3))) & 0xFFu));
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

// ---- decode ------------------------------------------------------------------------------------------------------------
// grid x 8 wavefronts, each `unit` consecutive blocks at a time (a multiple of four, at most 64): small inputs are spread
// over all wavefronts of the chip, since a chain takes as long for one lane as for 64
constexpr int kDecodeWaves = kDecodeThreads / 64;
constexpr int kDecodeIdxStride = kIdxWords + 1;
// padded entries of a lane whose reads are in flight together: a read takes longer than a whole store, and one block with many
// entries holds its wavefront up (1000 groups, 16 patterns: one at a time 10.3 us, so 9.7 us; 131072 mostly-zero groups 20.7, 20.4 us)
constexpr uint32_t kEntriesAtOnce = 4;
constexpr int kDecodeWaveWords = kInfoWords + kPayWords + kUnit * kDecodeIdxStride;  // private LDS of a wavefront
inline size_t decode_lds_bytes(int S) { return (table_words(S) + (size_t)kDecodeWaves * kDecodeWaveWords) * 4; }

// kStores: how the values are stored (ecco_stream.h says when and why)
using ecco_stream::Stores;
template <Stores kStores>
__global__ __launch_bounds__(kDecodeThreads) void pb_decode_kernel(const uint32_t* __restrict__ dev, int S, const uint4* __restrict__ blocks, size_t n_groups,
                                                                   int unit, uint4* __restrict__ dst) {
    extern __shared__ __align__(16) uint32_t smem[];
    const int lane = threadIdx.x & 63, l = lane & 15, row = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint2* info = reinterpret_cast<uint2*>(smem + table_words(S) + wave * kDecodeWaveWords);
    uint32_t* pay = reinterpret_cast<uint32_t*>(info) + kInfoWords;
    uint32_t* idx = pay + kPayWords;
    const size_t n_units = (n_groups + unit - 1) / unit, step = (size_t)gridDim.x * kDecodeWaves;
    size_t u = (size_t)blockIdx.x * kDecodeWaves + wave;
    const auto load = [&](size_t v) {
        const size_t first = min(v * unit, n_groups - 1);
        return load_pieces(blocks + first * 4, (int)min(n_groups - first, (size_t)unit), lane);
    };
    PieceLoad pre;
    const Tables T = stage_tables<kDecodeThreads>(smem, dev, S, [&] { pre = load(u); });
    pay[lane * kSlot + kBlockWords] = 0u;
    __syncthreads();

    for (; u < n_units; u += step) {
        wave_lds_fence();
        store_pieces(pay, pre, lane);
        wave_lds_fence();
        pre = load(u + step);
        const uint32_t* own = pay + lane * kSlot;
        const Walked b = walk_block(own, T, [&](int i, uint32_t word) { idx[lane * kDecodeIdxStride + i] = word; });
        info[lane] = make_uint2(b.cent | (b.present << 16), b.scale);
        wave_lds_fence();
        const int count = (int)min(n_groups - u * unit, (size_t)unit);
        uint4* out = dst + u * unit * (kGroup / 8);
#pragma unroll 1
        for (int b0 = 0; b0 < count; b0 += kPair * kRows) {
            RowBlock r[kPair];
#pragma unroll
            for (int q = 0; q < kPair; ++q) {
                const int blk = b0 + q * kRows + row;
                r[q] = row_block(T, info[blk], idx[blk * kDecodeIdxStride + l], l);
            }
            drop_absent(r);
#pragma unroll
            for (int q = 0; q < kPair; ++q) {
                const half2_t s2 = __builtin_bit_cast(half2_t, r[q].scale | (r[q].scale << 16));
                uint32_t v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)  // each product rounds once
                    v[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, r[q].c[2 * i] | (r[q].c[2 * i + 1] << 16)) * s2);
                const int blk = b0 + q * kRows + row;
                const uint4 v4 = make_uint4(v[0], v[1], v[2], v[3]);
                if constexpr (kStores == Stores::kThrough) ecco_stream::store_through(out, (uint32_t)count * (kGroup * 2), (uint32_t)(blk * (kGroup * 2) + l * 16), v4);
                else if (blk < count) ecco_stream::store<kStores == Stores::kPast>(out + blk * (kGroup / 8) + l, v4);
            }
        }
        // The padded entries, a block per lane again, over the values just written, in the order of the stream: a later one at the
        // same position wins.  (A wavefront's stores to one address arrive in the order they were issued, those that are written
        // through or past the caches among them: that says where a line is kept, and the fence keeps the compiler from exchanging them.)
        wave_lds_fence();
        uint16_t* values = reinterpret_cast<uint16_t*>(out) + lane * kGroup;
        const uint32_t entries = lane < count ? b.entries : 0u;
        for (uint32_t j0 = 0; __builtin_amdgcn_ballot_w64(j0 < entries) != 0ull; j0 += kEntriesAtOnce) {
            uint32_t code[kEntriesAtOnce];
            uint16_t value[kEntriesAtOnce];
#pragma unroll
            for (uint32_t j = 0; j < kEntriesAtOnce; ++j) code[j] = entry_code(own, b.end, j0 + j);
#pragma unroll
            for (uint32_t j = 0; j < kEntriesAtOnce; ++j) value[j] = T.fp8[code[j] & 0xFFu];
#pragma unroll
            for (uint32_t j = 0; j < kEntriesAtOnce; ++j)
                if (j0 + j < entries) values[code[j] >> 8] = value[j];
        }
    }
}

// ---- decode fused into the matrix-vector product --------------------------------------------------------------------
// y = W x without writing W: a workgroup owns a band of rows (its blocks are consecutive in memory) and takes it in chunks
// of whole rows; per-block sums go to LDS, and each row's blocks are added in a fixed tree.  A padded entry takes
// centroid * x at its position back and adds its own value (times x) instead; this is done right after the walk, a block per lane,
// when the indices still lie in registers.  They then take the payload's place in LDS, so that sixteen wavefronts fit beside 64
// patterns' tables (eight with a place of their own): 4096 x 28672 takes 57.5 us, 121 us with eight.
constexpr int kGemvWaves = kGemvThreads / 64;
constexpr int kGemvWaveWords = kInfoWords + kPayWords;  // private LDS of a wavefront
// per-block sums of a chunk (rows x column groups) that fit the LDS: one workgroup takes a compute unit's wavefronts, nothing else needs it
constexpr int gemv_part_floats(int S) { return (int)(160 * 1024 / 4 - table_words(S) - kGemvWaves * kGemvWaveWords); }
static_assert(gemv_part_floats(kMaxS) >= 65536 / kGroup, "the sums of a row fit");

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
// Four sums over a row of 16 lanes at once, in the same tree: at the first two levels a lane keeps the sums that match its own
// lane bit and sends the others to its partner.  Lane l returns sum l & 3.
__device__ __forceinline__ float row_sum4(const float (&q)[4], int l) {
    const bool b0 = l & 1, b1 = l & 2;
    const auto moved = [](float v, auto ctrl) { return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), decltype(ctrl)::value, 0xF, 0xF, true)); };
    float a[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = __fadd_rn(b0 ? q[2 * i + 1] : q[2 * i], moved(b0 ? q[2 * i] : q[2 * i + 1], std::integral_constant<int, 0xB1>{}));
    float t = __fadd_rn(b1 ? a[1] : a[0], moved(b1 ? a[0] : a[1], std::integral_constant<int, 0x4E>{}));
    t = dpp_add<0x124>(t);     // row_ror 4
    return dpp_add<0x128>(t);  // row_ror 8
}
__device__ __forceinline__ float wave_sum(float t) {
    t = row_sum(t);
    const auto lane_of = [&](int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, t), l)); };
    return __fadd_rn(__fadd_rn(lane_of(0), lane_of(16)), __fadd_rn(lane_of(32), lane_of(48)));
}

__global__ __launch_bounds__(kGemvThreads) void pb_gemv_kernel(const uint32_t* __restrict__ dev, int S, const uint4* __restrict__ blocks, int rows, int gpr, int band,
                                                               int chunk, int unit, const uint4* __restrict__ x, float* __restrict__ y) {
    extern __shared__ __align__(16) uint32_t smem[];
    const int lane = threadIdx.x & 63, l = lane & 15, row = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint2* info = reinterpret_cast<uint2*>(smem + table_words(S) + wave * kGemvWaveWords);
    uint32_t* pay = reinterpret_cast<uint32_t*>(info) + kInfoWords;
    float* part = reinterpret_cast<float*>(smem + table_words(S) + kGemvWaves * kGemvWaveWords);

    const int band0 = blockIdx.x * band, band1 = min(rows, band0 + band);
    PieceLoad pre;
    const auto load = [&](const uint4* first, int n_blocks, int at) {
        at = min(at, n_blocks - 1);
        pre = load_pieces(first + (size_t)at * 4, min(n_blocks - at, unit), lane);
    };
    const Tables T = stage_tables<kGemvThreads>(smem, dev, S, [&] { load(blocks + (size_t)band0 * gpr * 4, min(chunk, band1 - band0) * gpr, wave * unit); });
    pay[lane * kSlot + kBlockWords] = 0u;
    __syncthreads();

    constexpr int kAhead = 4;
    const uint32_t four = (uint32_t)(kRows % gpr) * (kGroup * 2), x_end = (uint32_t)gpr * (kGroup * 2);  // bytes
    for (int r0 = band0; r0 < band1; r0 += chunk) {
        const int nrows = min(chunk, band1 - r0), n_blocks = nrows * gpr;
        const uint4* first = blocks + (size_t)r0 * gpr * 4;   // first block of the chunk
        for (int at = wave * unit; at < n_blocks; at += kGemvWaves * unit) {
            const int count = min(n_blocks - at, unit);
            wave_lds_fence();
            store_pieces(pay, pre, lane);
            wave_lds_fence();
            if (at + kGemvWaves * unit < n_blocks) load(first, n_blocks, at + kGemvWaves * unit);
            else if (r0 + chunk < band1) load(first + (size_t)chunk * gpr * 4, min(chunk, band1 - r0 - chunk) * gpr, wave * unit);
            uint32_t* own = pay + lane * kSlot;
            uint32_t k[kIdxWords];
            // The walk has priority over the entries and values of other wavefronts, which fill the waits of its chain (4096 x 28672 56.0 ->
            // 53.2 us, 4096 x 4096 14.5 -> 14.4 us with 64 patterns, 15.1 -> 14.9 us with 16; 11008 x 4096 26.5 -> 26.6 us).
            __builtin_amdgcn_s_setprio(1);
            const Walked b = walk_block(own, T, [&](int i, uint32_t word) { k[i] = word; });
            __builtin_amdgcn_s_setprio(0);
            info[lane] = make_uint2(b.cent | (b.present << 16), __builtin_bit_cast(uint32_t, half_f(b.scale)));
            // The padded entries, last one first: an earlier one at the same position does not count.  Of the last two (few blocks have
            // more) only the codes are taken here; what they stand for follows when the indices lie in LDS, where a value's is one
            // read (out of registers it is a tree of 15 selections), and the products with their activations at the end of the pass.
            const uint32_t entries = lane < count ? b.entries : 0u;
            const uint16_t* xb = reinterpret_cast<const uint16_t*>(x) + (size_t)((uint32_t)(at + min(lane, count - 1)) % (uint32_t)gpr) * kGroup;
            const auto place = [](uint32_t pos) { return 8u * (pos & 3u) + ((pos & 4u) ? 0u : 4u); };  // of a value's index in its word
            const auto adds = [&](uint32_t code, uint32_t i) {  // what an entry adds to the value of index i
                return fmaf(-half_f(lds_half(T.cent + b.cent + i * 2u)), half_f(b.scale), half_f(T.fp8[code & 0xFFu]));
            };
            const auto index_of = [&](uint32_t pos) {  // out of registers
                uint32_t t[kIdxWords];  // word pos / 8 of the indices
#pragma unroll
                for (int i = 0; i < kIdxWords; ++i) t[i] = k[i];
#pragma unroll
                for (int n = kIdxWords / 2; n != 0; n >>= 1) {
                    // masks, not conditions: of these the compiler makes a loop over the lanes with an indexed register
                    uint32_t upper = (pos & (8u * n)) ? 0xFFFFFFFFu : 0u;
                    asm("" : "+v"(upper));
#pragma unroll
                    for (int i = 0; i < n; ++i) t[i] = (t[i] & ~upper) | (t[i + n] & upper);
                }
                return (t[0] >> place(pos)) & 15u;
            };
            float add = 0.0f;
            uint32_t code[2] = {0u, 0u}, last_x[2] = {0u, 0u};  // of the last two; FP16 bits of their activations
            const bool any = __builtin_amdgcn_ballot_w64(entries != 0u) != 0ull;
            if (any) {
#pragma unroll
                for (uint32_t q = 0; q < 2; ++q) {  // (of a block without: some position, and not used)
                    code[q] = entry_code(own, b.end, entries - 1u - q);
                    last_x[q] = xb[code[q] >> 8];
                }
                if (__builtin_amdgcn_ballot_w64(entries > 2u) != 0ull) {
                    uint64_t seen[2] = {0ull, 0ull};
                    const auto see = [&](uint32_t p) {  // whether p was there before
                        const uint64_t bit = 1ull << (p & 63u);
                        const bool high = p >= 64u, again = ((high ? seen[1] : seen[0]) & bit) != 0ull;
                        seen[0] |= high ? 0ull : bit;
                        seen[1] |= high ? bit : 0ull;
                        return again;
                    };
                    see(code[0] >> 8);
                    see(code[1] >> 8);
                    for (uint32_t j = 2; __builtin_amdgcn_ballot_w64(j < entries) != 0ull; ++j)
                        if (j < entries) {
                            const uint32_t c = entry_code(own, b.end, entries - 1u - j), p = c >> 8;
                            const float d = adds(c, index_of(p)), xv = half_f(xb[p]);
                            if (!see(p)) add = fmaf(d, xv, add);
                        }
                }
            }
            wave_lds_fence();
#pragma unroll
            for (int i = 0; i < kIdxWords; ++i) own[i] = k[i];
            wave_lds_fence();
            float last[2] = {0.0f, 0.0f};
            if (any) {
#pragma unroll
                for (uint32_t q = 0; q < 2; ++q) last[q] = adds(code[q], (own[code[q] >> 11] >> place(code[q] >> 8)) & 15u);
                last[0] = entries > 0u ? last[0] : 0.0f;
                last[1] = entries > 1u && (code[0] ^ code[1]) > 0xFFu ? last[1] : 0.0f;  // not at the same position
            }
            // sixteen blocks at a time, four per row of lanes: eight activations of each block's column group per lane, those of the
            // next sixteen requested while these are multiplied
            uint4 xs[kAhead];
            uint32_t x_at = (uint32_t)((at + row) % gpr) * 256u + (uint32_t)l * 16u;  // byte offset into x
            const auto load_x = [&](uint4& to) {
                to = *reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned char*>(x) + x_at);
                x_at += four;
                x_at = min(x_at, x_at - x_end);  // past the row's end (before it the difference wraps round)
            };
#pragma unroll
            for (int q = 0; q < kAhead; ++q) load_x(xs[q]);
#pragma unroll 1
            for (int i0 = 0; i0 < count; i0 += kAhead * kRows) {
                uint2 in[kAhead];
                uint32_t nibbles[kAhead];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    in[q] = info[i0 + q * kRows + row];
                    nibbles[q] = pay[(i0 + q * kRows + row) * kSlot + l];
                }
                RowBlock r[kAhead];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) r[q] = row_block(T, in[q], nibbles[q], l);
                drop_absent(r);
                float t[kAhead] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int i = 0; i < 8; ++i)  // the four sums side by side: each is a chain of eight multiply-adds
#pragma unroll
                    for (int q = 0; q < kAhead; ++q) {
                        const uint32_t xw[4] = {xs[q].x, xs[q].y, xs[q].z, xs[q].w};
                        t[q] = fmaf(half_f(r[q].c[i]), half_f(i & 1 ? xw[i >> 1] >> 16 : xw[i >> 1] & 0xFFFFu), t[q]);
                    }
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    t[q] *= __builtin_bit_cast(float, r[q].scale);
                    load_x(xs[q]);
                }
                const float sum = row_sum4(t, l);  // of block i0 + 4 (l % 4) + row
                const int blk = i0 + (l & 3) * kRows + row;
                if (l < kAhead && blk < count) part[at + blk] = sum;
            }
            // (an entry that does not count adds nothing, also where the activation read for it is infinite)
#pragma unroll
            for (int q = 1; q >= 0; --q) add = last[q] != 0.0f ? fmaf(last[q], half_f(last_x[q]), add) : add;
            wave_lds_fence();
            if (entries != 0u) part[at + lane] += add;
        }
        __syncthreads();
        // row sums: the blocks of a row in a fixed order (lane-strided partial sums, then the wavefront tree)
        for (int r = wave; r < nrows; r += kGemvWaves) {
            float sum = 0.0f;
            for (int c = lane; c < gpr; c += 64) sum += part[r * gpr + c];
            sum = wave_sum(sum);
            if (lane == 0) y[r0 + r] = sum;
        }
        if (r0 + chunk < band1) __syncthreads();
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
    // a band of rows per workgroup and a workgroup per compute unit; the band in chunks whose sums fit the LDS
    const int band = (rows + cus - 1) / cus, grid = (rows + band - 1) / band;
    const int most = std::min(band, gemv_part_floats(m->S) / gpr), chunks = (band + most - 1) / most, chunk = (band + chunks - 1) / chunks;
    // as few wavefronts as hold the blocks 64 at a time, but four (one per SIMD): a chain takes as long for one lane as for 64, and
    // longer the more wavefronts read tables beside it (512 blocks per workgroup: 15.3 us on eight, 16.9 us on sixteen; 40 blocks: 10.4 us on
    // four, 11.1 us on two, 12.5 us on ten; by events around replayed graphs)
    const size_t waves = std::min<size_t>(kGemvWaves, std::max<size_t>(4, ((size_t)chunk * gpr + kUnit - 1) / kUnit));
    const size_t lds = (table_words(m->S) + (size_t)kGemvWaves * kGemvWaveWords + (size_t)chunk * gpr) * 4;
    const int rc = ecco::allow_lds(pb_gemv_kernel, m->device, lds);
    if (rc != ECCO_OK) return rc;
    hipLaunchKernelGGL(pb_gemv_kernel, dim3(grid), dim3(kGemvThreads), lds, static_cast<hipStream_t>(stream), m->dev, m->S, static_cast<const uint4*>(blocks), rows, gpr,
                       band, chunk, unit_of((size_t)chunk * gpr, waves), reinterpret_cast<const uint4*>(x), y);
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
    const size_t lds = decode_lds_bytes(m->S);
    const Stores stores = ecco_stream::self_contained(dst, n_groups * kGroup * 2);
    const auto kernel = stores == Stores::kPast ? pb_decode_kernel<Stores::kPast> : stores == Stores::kThrough ? pb_decode_kernel<Stores::kThrough> : pb_decode_kernel<Stores::kCached>;
    const int rc = ecco::allow_lds(kernel, m->device, lds);
    if (rc != ECCO_OK) return rc;
    const size_t cus = (size_t)ecco::cu_count(m->device);
    const int unit = unit_of(n_groups, cus * kDecodeWaves);
    const size_t units = (n_groups + unit - 1) / unit;
    const int grid = (int)std::min<size_t>((units + kDecodeWaves - 1) / kDecodeWaves, cus);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kDecodeThreads), lds, static_cast<hipStream_t>(stream), m->dev, m->S, static_cast<const uint4*>(blocks), n_groups,
                       unit, reinterpret_cast<uint4*>(dst));
    ECCO_HIP_CHECK(hipGetLastError());
    return ECCO_OK;
}

}  // extern "C"
