// HIP kernels (gfx950) and GPU entry points of libecco.
//
// Decoder design.  A Huffman stream is serial, so the unit of parallelism is the half block: the
// meta word says where the code of value 64 begins, hence every block offers two independent
// chains of 64 values.  One lane owns one chain.  All lanes of a wavefront sit at the same value
// position (whatever their bit positions), which makes the position-dependent operand of the
// consumer -- the activation x[i] in the fused GEMV, the query q[i] in attention -- a register with
// a static index.  Per value a lane does: peek 8 bits of its 64-bit window, one LDS table read that
// returns code length, index and the centroid as FP16, the consumer's multiply-add, one 64-bit
// shift; every four values the window's lower half is filled anew from LDS.  Raw-mode
// blocks run the same instructions against a 16-entry table with a 4-bit peek.  All kernels work
// in units of 32 blocks per wavefront: 2 KB of payload fetched with coalesced 16-byte loads one
// unit ahead, kept in a per-wavefront LDS buffer with a 17-word stride per block (word 16 is a
// zero pad), so the per-lane window reads hit distinct banks and wavefronts never wait for each
// other inside the decode.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "ecco_launch.h"
#include "ecco_plan.h"
#include "ecco_stream.h"

using namespace ecco;

namespace {

constexpr int kHalf = kGroup / 2;         // values per chain

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float half_bits_f(uint32_t bits) { return __half2float(__ushort_as_half((unsigned short)bits)); }

// orders the LDS accesses of one wavefront (private buffers need no workgroup barrier)
__device__ inline void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- LDS tables -------------------------------------------------------------------------------------
struct Tables {
    const uint32_t* lut;      // [S][256]
    const uint32_t* rawlut;   // [S][16]
    const uint32_t* longtab;  // [S][16]
    const __half* cent;       // [S][16]
};
__host__ __device__ constexpr size_t table_words(int S) { return (size_t)S * (kPeekEntries + kK + kK + kK / 2); }  // LDS words of a model's decode tables

// copies `words` (a multiple of 4; both sides 16-byte aligned) from global memory to LDS with all
// threads of the workgroup, four 16-byte loads in flight per thread
__device__ inline void stage_vec(uint32_t* dst, const uint32_t* __restrict__ src, int words) {
    const uint4* s = reinterpret_cast<const uint4*>(src);
    uint4* d = reinterpret_cast<uint4*>(dst);
    const int n = words >> 2, step = blockDim.x;
    for (int i = threadIdx.x; i < n; i += 4 * step) {
        uint4 v0, v1, v2, v3;
        const int i1 = i + step, i2 = i + 2 * step, i3 = i + 3 * step;
        v0 = s[i];
        if (i1 < n) v1 = s[i1];
        if (i2 < n) v2 = s[i2];
        if (i3 < n) v3 = s[i3];
        d[i] = v0;
        if (i1 < n) d[i1] = v1;
        if (i2 < n) d[i2] = v2;
        if (i3 < n) d[i3] = v3;
    }
}

// The thread's index, taken afresh: in a kernel that stages tables in every span, what is derived from it is then formed there and
// does not take registers through the decode loops.
__device__ __forceinline__ int fresh_thread() {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid;
}
// A model's size, likewise: what the staging of a model with long codes derives from it (masks, addresses) would otherwise be formed
// once for all spans and take scalar registers throughout
__device__ __forceinline__ int fresh_size(int S) {
    asm volatile("" : "+s"(S));
    return S;
}

// Building the decode tables of a model in LDS from the compact tables in global memory.  Item
// (p, k) is index k of pattern p: its code of length l <= 8 is the prefix of 2^(8-l) consecutive
// 8-bit peeks, which all get the entry (centroid, index, length); a longer code marks its single
// 8-bit prefix with 0.  The two global loads of an item are split from the LDS writes so that a
// kernel can issue them first, put its payload loads behind them, and build the tables while the
// payload is still on its way.
struct TableItem {
    uint32_t enc, cent;
};
__device__ __forceinline__ TableItem load_table_item(const uint32_t* __restrict__ dev, int S, int t) {
    const DevLayout D{S};
    TableItem it;
    it.enc = dev[D.enc() + t];
    it.cent = reinterpret_cast<const uint16_t*>(dev + D.cent())[t];
    return it;
}
__device__ __forceinline__ void build_table_item(uint32_t* base, int S, int t, TableItem it) {
    uint32_t* lut = base;
    uint32_t* rawlut = lut + S * kPeekEntries;
    const uint32_t code = it.enc & 0xFFFFu, len = it.enc >> 16, k = (uint32_t)t & (kK - 1);
    const uint32_t value = (it.cent << 16) | (k << 8);
    rawlut[t] = value | 4u;
    uint32_t* row = lut + (t / kK) * kPeekEntries;
    if (len > (uint32_t)kPeekBits) {
        row[code >> (len - kPeekBits)] = 0u;  // several long codes may share this prefix: same value
    } else {
        const uint32_t entry = value | len, n = 1u << (kPeekBits - len);
        uint32_t* dst = row + (code << (kPeekBits - len));
        if (n >= 4) {
            // neighbouring items start their runs at different offsets: all rows begin on the same LDS
            // bank and equal-length codes are a multiple of the run length apart, so without the
            // rotation the 64 items of a wavefront would write to a handful of banks at a time
            const uint4 v = make_uint4(entry, entry, entry, entry);
            const uint32_t rot = ((uint32_t)t + ((uint32_t)t >> 4) + (code >> 2)) * 4u;
            for (uint32_t j = 0; j < n; j += 4) *reinterpret_cast<uint4*>(dst + ((j + rot) & (n - 1))) = v;
        } else {
            for (uint32_t j = 0; j < n; ++j) dst[j] = entry;
        }
    }
}
__device__ __forceinline__ Tables table_pointers(uint32_t* base, int S) {
    Tables tb;
    tb.lut = base;
    tb.rawlut = base + S * kPeekEntries;
    tb.longtab = base + S * (kPeekEntries + kK);
    tb.cent = reinterpret_cast<const __half*>(base + S * (kPeekEntries + 2 * kK));
    return tb;
}
// The whole job for a workgroup of at least S * 16 / 2 threads, with a payload prefetch in its shadow: every
// thread first requests its (up to) two table items, then the loads of its first unit, then
// builds the tables.  Loads return in issue order and a wait names how many may still be outstanding, so with
// the items requested first -- the same loads on one straight path in every thread, indices clamped, threads
// beyond the items repeating the last one -- the build does not wait for the payload.  The lists of the long
// codes and the centroids are copied only for a model that needs them (behind the payload, then).  The caller
// synchronises afterwards.
struct TableItems {
    TableItem item[2];
};
__device__ __forceinline__ TableItems load_table_items(const uint32_t* __restrict__ dev, int S) {
    const int n = S * kK, tid = fresh_thread();
    TableItems t;
    t.item[0] = load_table_item(dev, S, min(tid, n - 1));
    t.item[1] = load_table_item(dev, S, min(tid + (int)blockDim.x, n - 1));
    __builtin_amdgcn_sched_barrier(0);
    return t;
}
template <bool kLong>
__device__ __forceinline__ void build_tables(uint32_t* base, const uint32_t* __restrict__ dev, int S, const TableItems& t) {
    __builtin_amdgcn_sched_barrier(0);
    const int n = S * kK, tid = fresh_thread();
    build_table_item(base, S, min(tid, n - 1), t.item[0]);
    build_table_item(base, S, min(tid + (int)blockDim.x, n - 1), t.item[1]);
    if (kLong) {
        const DevLayout D{S};
        stage_vec(base + S * (kPeekEntries + kK), dev + D.longtab(), S * kK);
        stage_vec(base + S * (kPeekEntries + 2 * kK), dev + D.cent(), S * kK / 2);
    }
}

// what one lane needs to decode one chain
struct Lane {
    const uint32_t* lut;      // this lane's table (Huffman: 256 entries, raw: 16)
    uint32_t shift;           // 32 - peek width
    const uint32_t* longtab;  // pattern's canonical list (codes longer than the peek)
    const __half* cent;       // pattern's centroids
    float scale;
    uint32_t second_start;    // stream bit where value 64 begins
};
__device__ __forceinline__ Lane lane_setup(const Tables& T, uint32_t meta, int S) {
    Lane L;
    uint32_t p = (meta >> 16) & 0x3Fu;
    p = p < (uint32_t)S ? p : (uint32_t)(S - 1);
    const bool raw = (meta >> 22) & 1u;
    L.lut = raw ? T.rawlut + p * kK : T.lut + p * kPeekEntries;
    L.shift = raw ? 28u : (uint32_t)(32 - kPeekBits);
    L.longtab = T.longtab + p * kK;
    L.cent = T.cent + p * kK;
    L.scale = half_bits_f(meta & 0xFFFFu);
    L.second_start = raw ? 4u * kHalf : (meta >> 23);
    return L;
}

typedef __attribute__((address_space(3))) uint32_t lds_u32;  // a 32-bit word in LDS, addressed as such
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 global_u4;   // sixteen bytes in global memory

// Priority of a wavefront's instructions on its SIMD while it decodes (0 otherwise), in the batch-1 product and the plain attention:
// wavefronts that store and request units, add up or meet at barriers then do so in the gaps of the others' table reads.  8192 x 28672
// 64.9 -> 63.5 us, attention over 16 x 32 sequences and heads of 1000 tokens 66.3 -> 64.4 us (64 patterns), 48.1 -> 46.3 us (16).  The batched
// product (11008 x 4096, batch 8: 18.0 -> 18.5 us), the standalone decoder (131072 groups 12.65 -> 12.87 us) and the grouped-query
// attention (1024 tokens 20.6 -> 20.9 us) lose by it and go without.
constexpr int kPriorityDecode = 1;

// ---- the chain decoder ----------------------------------------------------------------------------------
// Decodes kCount values starting at stream bit `start` of the staged block `w` (16 words and a zero word), calling sink(i, entry)
// with the table entry of each (length, index, centroid).  Values are taken in runs of 4 (2 when the model has codes longer than
// 8 bits: kLong) out of a left-aligned 64-bit window, so there is no refill test and no branch inside a run.  A run consumes at
// most 32 bits: its upper half is whole again when the run ends, and only the lower half is filled anew, from the words that
// follow.  The next run's first table read and shift need the upper half alone, so the refill passes in the shadow of that read and the
// dependent chain holds the table reads, a shift and two address instructions each.  (With the whole window rebuilt at the end of a
// run, seven more dependent instructions per run: 8192 x 28672 64.1 -> 63.2 us, 4096 x 4096 7.55 -> 7.50 us, batch 8 over 11008 x 4096 18.4 -> 18.3 us,
// append and attention over 8 x 32 sequences and heads of 4096 tokens 92.1 -> 91.0 us.  A shift of either half by v_alignbit, with 32 - length
// in the table, costs an instruction per value: 65.0, 7.65, 19.5 and 94.1 us.)  The word after next is requested a run ahead: a run
// moves by one word at most.  From the block's end on every word is the zero word: arbitrary bytes decode without touching other memory.
// kWhole: the whole window is rebuilt with every run, the position clamped to 512, where its upper half is the zero word and its lower half
// is never looked at (two words behind the zero word have to be readable).  An instruction less where there is a run for every two values: the batched
// product of long codes, bound by its vector instructions and not by the chain (8192 x 28672, batch 8 107.2 -> 104.0 us, 1000 x 28672 56.8 -> 55.3 us).
template <bool kLong, int kCount, bool kWhole = false, class Sink>
__device__ __forceinline__ void decode_chain(const uint32_t* w, uint32_t start, const Lane& L, Sink&& sink) {
    constexpr int kRun = kLong ? 2 : 4;
    static_assert(kCount % kRun == 0, "chain length");
    static_assert(kRun * (kLong ? kMaxLen : kPeekBits) <= 32, "a run stays inside two words");
    // Otherwise the lower half of the window comes from the words w1 and w2, w1 being the first that begins at the position or behind it: with
    // the position counted down from 0, the position itself is the shift count, also on a word's border.
    int32_t down = -(int32_t)start;  // start <= 511
    int32_t next = down >> 5;        // index of w1, negated
    const auto word = [&](int32_t i) { return w[min((uint32_t)i, (uint32_t)kBlockWords)]; };
    [[maybe_unused]] uint32_t pos = start, w0, w1, w2, w3;
    uint32_t wi = start >> 5;
    uint64_t win;
    if constexpr (kWhole) {
        w0 = w[wi], w1 = w[wi + 1], w2 = w[wi + 2];
        win = (((uint64_t)w0 << 32) | (uint64_t)w1) << (start & 31u);
    } else {
        w1 = word(-next), w2 = word(1 - next), w3 = word(2 - next);
        win = ((((uint64_t)w[wi] << 32) | (uint64_t)w[wi + 1]) << (start & 31u)) & 0xFFFFFFFF00000000ull;
        win |= __builtin_amdgcn_alignbit(w1, w2, (uint32_t)down);
    }
#pragma unroll
    for (int i0 = 0; i0 < kCount; i0 += kRun) {
        uint32_t used = 0;  // sum of the run's entries; its low byte is the number of bits consumed (at most 4 x 8 or 2 x 12)
#pragma unroll
        for (int j = 0; j < kRun; ++j) {
            uint32_t e = L.lut[(uint32_t)(win >> 32) >> L.shift];
            if (kLong) {
                if ((e & 0xFFu) == 0u) {
                    // code longer than the peek: rank of the next 12 bits among the left-aligned canonical codes
                    const uint32_t v = (uint32_t)(win >> 32) >> (32 - kMaxLen);
                    // the list is read here, on the rare path, not held in 16 registers throughout: its LDS byte address
                    // passes through an empty asm statement (a pointer passed through one would come back without its
                    // address space, and the reads below would become flat loads instead of LDS reads)
                    uint32_t lt_at = (uint32_t)(size_t)(const lds_u32*)L.longtab;
                    asm volatile("" : "+v"(lt_at));
                    const lds_u32* lt = (const lds_u32*)(size_t)lt_at;
                    int rank = 0;
                    for (int q = 1; q < kK; ++q) rank += ((lt[q] & 0xFFFu) <= v) ? 1 : 0;
                    const uint32_t t = lt[rank];
                    const uint32_t idx = (t >> 12) & 15u;
                    e = ((uint32_t)__half_as_ushort(L.cent[idx]) << 16) | (idx << 8) | (t >> 16);
                }
            }
            sink(i0 + j, e);
            used += e;
            win <<= (e & 0xFFu);
        }
        if constexpr (kWhole) {
            if (i0 + kRun == kCount) break;
            pos = min(pos + (used & 0xFFu), (uint32_t)(kBlockWords * 32));
            const uint32_t now = pos >> 5;  // wi or wi + 1
            const bool adv = now != wi;
            w0 = adv ? w1 : w0;
            w1 = adv ? w2 : w1;
            w2 = w[now + 2];  // used one run later at the earliest
            win = (((uint64_t)w0 << 32) | (uint64_t)w1) << (pos & 31u);
            wi = now;
        } else if (i0 + kRun < kCount) {
            down -= (int32_t)(used & 0xFFu);
            const int32_t now = down >> 5;  // next or next - 1
            const bool adv = now != next;
            w1 = adv ? w2 : w1;
            w2 = adv ? w3 : w2;
            w3 = word(2 - now);  // used one run later at the earliest
            win = (win & 0xFFFFFFFF00000000ull) | (uint64_t)__builtin_amdgcn_alignbit(w1, w2, (uint32_t)down);
            next = now;
        }
    }
}

// ---- payload staging ------------------------------------------------------------------------------------

constexpr int kGemvThreads = 1024;

// ---- ecco_decode_gemv, batch 1 ----------------------------------------------------------------------------
// A workgroup (one per compute unit) owns a band of R consecutive rows; its work is cut into units
// of one row x 32 column groups: 32 blocks, a contiguous 2 KB of payload, 64 chains -- one
// wavefront.  Lane l of the wavefront decodes chain l / 32 of block l % 32.  After the decode tables
// and x are in LDS (one workgroup barrier), the 16 wavefronts run on their own: each fetches the
// payload of its next unit into registers, decodes the current one out of a private 2 KB LDS
// buffer, adds the 64 lane sums with a wavefront reduction and goes on, without any further
// workgroup barrier, so a wavefront starts decoding as soon as its own bytes have arrived and the
// loads of one unit overlap the decode of the one before.  Units of a wavefront stay in one column
// tile as long as possible (a contiguous run of units when the row has several column tiles), and the
// lane keeps the 64 activations of its chain in registers across those units, so a value costs one
// mixed-precision FMA.  Rows are never split over workgroups:
// partial sums of a row's column tiles meet in LDS and are added in a fixed order.
constexpr int kWaves = kGemvThreads / 64;
constexpr int kXGroupWords = kGroup / 2 + 4;           // words per column group of x in LDS (skewed against bank conflicts)
constexpr int kXLdsGroups = 128;                       // x is staged in LDS up to this many column groups, read from L2 beyond
constexpr int kMaxBandRows = 128;
constexpr int kMaxColTiles = 65536 / kGroup / kUnitBlocks;
inline size_t gemv_lds_bytes(int S, int gpr) {
    const size_t xwords = gpr <= kXLdsGroups ? (size_t)gpr * kXGroupWords : 0;
    return (table_words(S) + (size_t)kWaves * kUnitWords + (size_t)kMaxBandRows * kMaxColTiles + xwords) * 4;
}

template <int kCtrl>
__device__ __forceinline__ float dpp_mov(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), kCtrl, 0xF, 0xF, true));
}
__device__ __forceinline__ float read_lane(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
// sum over the 64 lanes of a wavefront in a fixed order, on the VALU (cross-lane moves inside rows of
// 16 lanes, then the four row sums through scalar registers); every lane returns the total
__device__ __forceinline__ float wave_sum(float t) {
    t += dpp_mov<0xB1>(t);   // quad_perm [1,0,3,2]
    t += dpp_mov<0x4E>(t);   // quad_perm [2,3,0,1]
    t += dpp_mov<0x141>(t);  // row_half_mirror
    t += dpp_mov<0x140>(t);  // row_mirror
    return (read_lane(t, 0) + read_lane(t, 16)) + (read_lane(t, 32) + read_lane(t, 48));
}

// the same walk for any associative, commutative, exact operation (minimum, maximum): the order does not matter
template <class T, class Op>
__device__ __forceinline__ T wave_all(T v, Op op) {
    float t = __builtin_bit_cast(float, v);
    const auto f = [&](float a, float b) { return __builtin_bit_cast(float, op(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b))); };
    t = f(t, dpp_mov<0xB1>(t));
    t = f(t, dpp_mov<0x4E>(t));
    t = f(t, dpp_mov<0x141>(t));
    t = f(t, dpp_mov<0x140>(t));
    return __builtin_bit_cast(T, f(f(read_lane(t, 0), read_lane(t, 16)), f(read_lane(t, 32), read_lane(t, 48))));
}

struct UnitLoad {
    uint4 v0, v1;
    uint32_t meta;
};
// the payload pieces of this lane for unit (row, ct) and the meta word of the unit's block `slot` (the one it decodes).
// Block indices are clamped into the row, so every lane issues the same loads and a slot past the row end holds a copy of
// the row's last block: it decodes to finite values, which the caller drops.  Nothing here uses the loaded
// data, so the loads stay in flight while the previous unit is decoded.
__device__ __forceinline__ UnitLoad load_unit(const uint4* __restrict__ blocks, const uint32_t* __restrict__ meta,
                                              int row, int gpr, int ct, int lane, int slot) {
    UnitLoad u;
    const size_t row_base = (size_t)row * gpr;
    const int g0 = ct * kUnitBlocks + (lane >> 2), g1 = g0 + 16;
    u.v0 = blocks[(row_base + min(g0, gpr - 1)) * 4 + (lane & 3)];
    u.v1 = blocks[(row_base + min(g1, gpr - 1)) * 4 + (lane & 3)];
    u.meta = meta[row_base + min(ct * kUnitBlocks + slot, gpr - 1)];
    return u;
}
__device__ __forceinline__ UnitLoad load_unit(const uint4* __restrict__ blocks, const uint32_t* __restrict__ meta,
                                              int row, int gpr, int ct, int lane) {
    return load_unit(blocks, meta, row, gpr, ct, lane, lane & (kUnitBlocks - 1));
}
// Lane l writes pieces of blocks l / 4 and l / 4 + 16; the chains are then read by other lanes (lane b and b + 32
// read block b).  The exchange goes through the wavefront's private buffer without a workgroup barrier, so it is
// fenced on both sides at wavefront scope: the reads of the previous unit come before these writes, and these
// writes before the reads that follow.
__device__ __forceinline__ void store_unit(uint32_t* wbuf, const UnitLoad& u, int lane) {
    wave_lds_fence();
    uint32_t* d = wbuf + (lane >> 2) * kStride + (lane & 3) * 4;
    d[0] = u.v0.x; d[1] = u.v0.y; d[2] = u.v0.z; d[3] = u.v0.w;
    d += 16 * kStride;
    d[0] = u.v1.x; d[1] = u.v1.y; d[2] = u.v1.z; d[3] = u.v1.w;
    wave_lds_fence();
}

template <bool kLong>
__global__ __launch_bounds__(kGemvThreads) void gemv_kernel(const uint32_t* __restrict__ dev, int S,
                                                            const uint4* __restrict__ blocks, const uint32_t* __restrict__ meta,
                                                            int rows, int gpr, int band,
                                                            const uint32_t* __restrict__ x, float* __restrict__ y) {
    extern __shared__ __align__(16) uint32_t smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = blockIdx.x * band;
    const int band_rows = min(band, rows - row0);
    const int col_tiles = (gpr + kUnitBlocks - 1) / kUnitBlocks;
    const int units = band_rows * col_tiles;  // unit u = (column tile u / band_rows, row u % band_rows)
    const bool x_in_lds = gpr <= kXLdsGroups;
    uint32_t* wbuf = smem + table_words(S) + wave * kUnitWords;
    float* part = reinterpret_cast<float*>(smem + table_words(S) + kWaves * kUnitWords);
    uint32_t* xt = reinterpret_cast<uint32_t*>(part + kMaxBandRows * kMaxColTiles);
    const uint4* x4 = reinterpret_cast<const uint4*>(x);

    // Loads in the order they are needed: table item, x, then the first unit's payload (from HBM).  Loads
    // return in issue order and a wait names how many may still be outstanding, so every thread issues the
    // same loads on one straight path (indices clamped instead of branches around them): only then can the
    // wait for the table item leave the payload in flight while the tables are built.
    // (The scheduling barriers keep the compiler from issuing them in another order.)
    const int ti = min(tid, S * kK - 1);  // threads beyond the items repeat the last one: same values to the same words
    const TableItem item = load_table_item(dev, S, ti);
    __builtin_amdgcn_sched_barrier(0);
    static_assert(ECCO_MAX_S * kK <= kGemvThreads, "one table item per thread");
    static_assert(kXLdsGroups * 16 == 2 * kGemvThreads, "two x pieces per thread");
    const uint4 xp0 = x4[min(tid, gpr * 16 - 1)];
    const uint4 xp1 = x4[min(tid + kGemvThreads, gpr * 16 - 1)];
    __builtin_amdgcn_sched_barrier(0);
    // With several column tiles a wavefront takes a contiguous run of units (column tile by column tile, row by
    // row; runs differ by one unit at most), so it changes its column tile -- and fetches 64 activations per
    // lane -- as rarely as possible.  With one column tile there is nothing to keep, and the wavefronts stride
    // through the rows together, so that the workgroup reads one contiguous stretch of memory at a time.
    const bool runs = col_tiles > 1;
    const int u_step = runs ? 1 : kWaves;
    int u = runs ? wave * units / kWaves : wave;
    const int u_end = runs ? (wave + 1) * units / kWaves : units;
    const int u_first = min(u, units - 1);  // a wavefront without work loads the band's last unit and drops it
    UnitLoad pre = load_unit(blocks, meta, row0 + u_first % band_rows, gpr, u_first / band_rows, lane);
    __builtin_amdgcn_sched_barrier(0);
    build_table_item(smem, S, ti, item);
    if (kLong) {
        const DevLayout D{S};
        for (int i = tid; i < S * kK; i += kGemvThreads) smem[S * (kPeekEntries + kK) + i] = dev[D.longtab() + i];
        for (int i = tid; i < S * kK / 2; i += kGemvThreads) smem[S * (kPeekEntries + 2 * kK) + i] = dev[D.cent() + i];
    }
    if (x_in_lds) {
        const int i0 = tid, i1 = tid + kGemvThreads;
        if (i0 < gpr * 16) *reinterpret_cast<uint4*>(xt + (i0 >> 4) * kXGroupWords + (i0 & 15) * 4) = xp0;
        if (i1 < gpr * 16) *reinterpret_cast<uint4*>(xt + (i1 >> 4) * kXGroupWords + (i1 & 15) * 4) = xp1;
    }
    if (lane < kUnitBlocks) wbuf[lane * kStride + kBlockWords] = 0u;  // zero pads of the private buffer
    const Tables T = table_pointers(smem, S);
    __syncthreads();

    const int blk = lane & (kUnitBlocks - 1), half = lane >> 5;
    uint32_t xs[kHalf / 2];
    int cur_ct = -1;
    for (; u < u_end; u += u_step) {
        const int ct = u / band_rows, r = u - ct * band_rows;
        store_unit(wbuf, pre, lane);
        const uint32_t mw = pre.meta;
        const int cg = ct * kUnitBlocks + blk;
        if (ct != cur_ct) {  // the activations of this lane's chain: 64 FP16 = 8 x 16 bytes
            cur_ct = ct;
            const int cgx = min(cg, gpr - 1);
            if (x_in_lds) {
                const uint4* src = reinterpret_cast<const uint4*>(xt + cgx * kXGroupWords + half * (kHalf / 2));
#pragma unroll
                for (int j = 0; j < kHalf / 8; ++j) {
                    const uint4 v = src[j];
                    xs[4 * j] = v.x; xs[4 * j + 1] = v.y; xs[4 * j + 2] = v.z; xs[4 * j + 3] = v.w;
                }
            } else {
                const uint4* src = x4 + (size_t)cgx * 16 + half * 8;
#pragma unroll
                for (int j = 0; j < kHalf / 8; ++j) {
                    const uint4 v = src[j];
                    xs[4 * j] = v.x; xs[4 * j + 1] = v.y; xs[4 * j + 2] = v.z; xs[4 * j + 3] = v.w;
                }
            }
        }
        // the next unit's payload is requested after the activations: loads return in issue order, and the
        // activations (from cache) must not queue behind a fetch from HBM
        const int un = u + u_step;
        if (un < u_end) pre = load_unit(blocks, meta, row0 + un % band_rows, gpr, un / band_rows, lane);
        const Lane L = lane_setup(T, mw, S);
        float acc = 0.0f;
        __builtin_amdgcn_s_setprio(kPriorityDecode);
        decode_chain<kLong, kHalf>(wbuf + blk * kStride, half ? L.second_start : 0u, L, [&](int i, uint32_t e) {
            const uint32_t xp = xs[i >> 1];
            const float xv = half_bits_f((i & 1) ? (xp >> 16) : (xp & 0xFFFFu));
            acc = fmaf(half_bits_f(e >> 16), xv, acc);
            // pins the running sum every four values: otherwise the multiply-adds are sunk below the whole
            // chain and all 64 table entries stay in registers
            if ((i & 3) == 3) asm volatile("" : "+v"(acc));
        });
        __builtin_amdgcn_s_setprio(0);
        const float t = wave_sum(cg < gpr ? acc * L.scale : 0.0f);
        if (lane == 0) {
            if (col_tiles == 1) y[row0 + r] = t;
            else part[r * col_tiles + ct] = t;
        }
    }
    if (col_tiles > 1) {
        __syncthreads();
        if (tid < band_rows) {
            // four reads in flight at a time (indices clamped, the surplus not added): same order of additions
            float sum = 0.0f;
            for (int ct0 = 0; ct0 < col_tiles; ct0 += 4) {
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = part[tid * col_tiles + min(ct0 + j, col_tiles - 1)];
#pragma unroll
                for (int j = 0; j < 4; ++j) sum += ct0 + j < col_tiles ? v[j] : 0.0f;
            }
            y[row0 + tid] = sum;
        }
    }
}

// ---- ecco_decode / ecco_decode_indices ---------------------------------------------------------------
// The streaming scheme of the batch-1 GEMV on a linear array of blocks: a unit is 32 consecutive
// groups, lane l decodes chain l / 32 of block l % 32, a workgroup takes a contiguous range of units
// and its wavefronts stride through it.  A lane ends up with 128 contiguous output bytes, 16 at a
// time; written directly, one store instruction would touch 64 different lines with 16 bytes each,
// and the L2 request rate, not bandwidth, would bound the kernel (measured: 13 of 21 us on the
// 4096 x 4096 matrix).  So the FP16 values pass through a per-wavefront LDS image, 32 values per
// chain at a time, and are read back so that adjacent lanes hold adjacent 16-byte pieces: four lanes
// write the 64 contiguous bytes a segment gets per pass.  The image is swizzled (piece c of segment
// s sits at 4 s + (c ^ (s / 4) % 4)) so that the transposed reads are conflict-free.  The 4 KB image
// lies over the wavefront's 2.2 KB payload buffer, which is dead once both chains are decoded (the
// values wait in registers meanwhile), so sixteen wavefronts fit 160 KB of LDS next to the S = 64
// tables; the zero words that bound each block's stream are rewritten with every unit.
constexpr int kDecWaves = 16;
struct DecCfg {
    static constexpr int kLinePieces = kHalf / 8;                  // 16-byte pieces of a chain's 128 output bytes
    static constexpr int kImageWords = 32 * kLinePieces * 4;       // 32 lines at a time
    static constexpr int kWaveWords = kImageWords > kUnitWords ? kImageWords : kUnitWords;  // private LDS of a wavefront: payload, then image
};
inline size_t decode_lds_bytes(int S) { return (table_words(S) + (size_t)kDecWaves * DecCfg::kWaveWords) * 4; }

// kThrough: the values are written through (ecco_stream.h says when and why)
template <bool kLong, bool kIndices, bool kThrough>
__global__ __launch_bounds__(kDecWaves * 64) void decode_kernel(const uint32_t* __restrict__ dev, int S,
                                                              const uint4* __restrict__ blocks, const uint32_t* __restrict__ meta,
                                                              int n_groups, int units_per_wg, void* __restrict__ dst) {
    using Cfg = DecCfg;
    extern __shared__ __align__(16) uint32_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t* wbuf = smem + table_words(S) + wave * Cfg::kWaveWords;
    uint4* image = reinterpret_cast<uint4*>(wbuf);
    const int total_units = (n_groups + kUnitBlocks - 1) / kUnitBlocks;
    const int u_end = min(total_units, (int)(blockIdx.x + 1) * units_per_wg);
    int u = blockIdx.x * units_per_wg + wave;
    // table item first, then the first unit's payload, the same loads in every thread, and the tables are built
    // while the payload is on its way (see gemv_kernel)
    static_assert(ECCO_MAX_S * kK <= kDecWaves * 64, "one table item per thread");
    const int ti = min(tid, S * kK - 1);
    const TableItem item = load_table_item(dev, S, ti);
    __builtin_amdgcn_sched_barrier(0);
    UnitLoad pre = load_unit(blocks, meta, 0, n_groups, min(u, u_end - 1), lane);
    __builtin_amdgcn_sched_barrier(0);
    build_table_item(smem, S, ti, item);
    if (kLong) {
        const DevLayout D{S};
        for (int i = tid; i < S * kK; i += kDecWaves * 64) smem[S * (kPeekEntries + kK) + i] = dev[D.longtab() + i];
        for (int i = tid; i < S * kK / 2; i += kDecWaves * 64) smem[S * (kPeekEntries + 2 * kK) + i] = dev[D.cent() + i];
    }
    const Tables T = table_pointers(smem, S);
    __syncthreads();

    const int blk = lane & (kUnitBlocks - 1), half = lane >> 5;  // block of the unit and chain of this lane
    for (; u < u_end; u += kDecWaves) {
        store_unit(wbuf, pre, lane);  // fenced: the previous unit's image has been read
        if (lane < kUnitBlocks) wbuf[lane * kStride + kBlockWords] = 0u;  // zero pads of the payload buffer (the image lay over them)
        wave_lds_fence();
        const uint32_t mw = pre.meta;
        if (u + kDecWaves < u_end) pre = load_unit(blocks, meta, 0, n_groups, u + kDecWaves, lane);
        const Lane L = lane_setup(T, mw, S);
        const int g = u * kUnitBlocks + blk;
        const uint32_t* w = wbuf + blk * kStride;
        const uint32_t start = half ? L.second_start : 0u;
        if (kIndices) {
            uint4* out = reinterpret_cast<uint4*>(static_cast<uint8_t*>(dst) + (size_t)g * kGroup + half * kHalf);
            uint32_t acc[4] = {0, 0, 0, 0};
            decode_chain<kLong, kHalf>(w, start, L, [&](int i, uint32_t e) {
                acc[(i >> 2) & 3] |= ((e >> 8) & 15u) << (8 * (i & 3));
                if ((i & 15) == 15) {
                    if (g < n_groups) out[i >> 4] = make_uint4(acc[0], acc[1], acc[2], acc[3]);
                    acc[0] = acc[1] = acc[2] = acc[3] = 0;
                }
            });
        } else {
            uint8_t* obase = static_cast<uint8_t*>(dst) + (size_t)u * kUnitBlocks * kGroup * 2;  // the unit's 8 KB of output
            const _Float16 sh = __builtin_bit_cast(_Float16, (unsigned short)(mw & 0xFFFFu));
            const half2_t s2 = {sh, sh};
            uint32_t vals[kHalf / 2];  // the chain's 64 values = one 128-byte line of output
            uint32_t pk = 0;
            decode_chain<kLong, kHalf>(w, start, L, [&](int i, uint32_t e) {
                if ((i & 1) == 0) {
                    pk = e >> 16;
                    return;
                }
                // fp16(centroid * scale) for two values: the packed FP16 product rounds once, like the FP32 rule
                vals[i >> 1] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, pk | (e & 0xFFFF0000u)) * s2);
                if ((i & 7) == 7) asm volatile("" : "+v"(vals[i >> 1]));  // finished here, not gathered at the end of the chain
            });
            // Write-out in whole 128-byte lines: a store instruction that leaves half a line for later costs a second
            // write of that line.  First the 32 lanes with the first chains put their lines into the image (32 rows of
            // eight 16-byte pieces, piece k of row r at column k ^ (r & 7)) and all 64 lanes store them, eight lanes per
            // line; then the same for the second chains.
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                wave_lds_fence();
                if (half == h) {
#pragma unroll
                    for (int k = 0; k < Cfg::kLinePieces; ++k)
                        image[blk * Cfg::kLinePieces + (k ^ (blk & 7))] = make_uint4(vals[4 * k], vals[4 * k + 1], vals[4 * k + 2], vals[4 * k + 3]);
                }
                wave_lds_fence();
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = (lane >> 3) + 8 * r, part = lane & 7;
                    const uint4 v = image[row * Cfg::kLinePieces + (part ^ (row & 7))];
                    if constexpr (kThrough)
                        ecco_stream::store_through(obase, (uint32_t)min(n_groups - u * kUnitBlocks, kUnitBlocks) * (kGroup * 2), row * (kGroup * 2) + h * (kHalf * 2) + part * 16, v);
                    else if (u * kUnitBlocks + row < n_groups)
                        *reinterpret_cast<uint4*>(obase + row * (kGroup * 2) + h * (kHalf * 2) + part * 16) = v;
                }
            }
        }
    }
}

// ---- ecco_decode_gemv, batch 2..16: MFMA ------------------------------------------------------------------
// The streaming scheme of the batch-1 kernel with the multiply-adds on the matrix cores.  A unit is
// 16 rows x 2 column groups (32 blocks, 16 runs of 128 contiguous bytes): lane l decodes, for row
// l % 16, chain (l / 16) % 2 of column group l / 32.  Eight decoded values of the lane are exactly
// its A operand of v_mfma_f32_16x16x32_f16 (row l % 16, k slice l / 16); the B operand of the lane
// is eight activations of batch row l % 16 at the columns of the chain of slice l / 16, which it
// holds in registers for the unit (zeros past the batch); the 16 x 16 FP32 accumulator (rows x
// batch) stays in registers over all units of a 16-row block.  The weights enter as
// fp16(centroid * scale) -- packed FP16 multiplies, which round exactly like the
// FP32-multiply-then-round rule -- so no per-row scaling of the accumulator is needed.  A workgroup
// owns whole 16-row blocks (all their column groups), so nothing is split over workgroups: per row
// block the 16 wavefronts add their accumulators through LDS in a fixed order.
constexpr int kMmaRows = 16;
constexpr int kMaxBatch = 16;
typedef float float4_t __attribute__((ext_vector_type(4)));
constexpr int kRbChunk = 3;  // row blocks whose per-wavefront sums wait in LDS for one common reduction
static_assert((table_words(ECCO_MAX_S) + (size_t)(kGemvThreads / 64) * (32 * kStride + 4) + (size_t)kRbChunk * (kGemvThreads / 64) * 16 * 16) * 4 <= 160 * 1024, "the batched kernel's LDS fits a compute unit");
inline size_t gemm_lds_bytes(int S) { return (table_words(S) + (size_t)kWaves * kUnitWords + (size_t)kRbChunk * kWaves * kMmaRows * kMaxBatch) * 4; }

// this lane's payload pieces and meta word of unit (rb, u): block (r, c) of the unit -- row 16 rb + r,
// column group 2 u + c -- goes to slot 2 r + c.  Indices are clamped into the matrix (see load_unit).
__device__ __forceinline__ UnitLoad load_unit16(const uint4* __restrict__ blocks, const uint32_t* __restrict__ meta,
                                                int rows, int gpr, int rb, int u, int lane) {
    UnitLoad t;
    const int slot = lane >> 2, c = slot & 1;
    const int cg = min(2 * u + c, gpr - 1);
    const int r0 = min(rb * kMmaRows + (slot >> 1), rows - 1), r1 = min(rb * kMmaRows + 8 + (slot >> 1), rows - 1);
    t.v0 = blocks[((size_t)r0 * gpr + cg) * 4 + (lane & 3)];
    t.v1 = blocks[((size_t)r1 * gpr + cg) * 4 + (lane & 3)];
    const int mr = min(rb * kMmaRows + (lane & 15), rows - 1), mc = min(2 * u + (lane >> 5), gpr - 1);
    t.meta = meta[(size_t)mr * gpr + mc];
    return t;
}

template <bool kLong>
__global__ __launch_bounds__(kGemvThreads) void gemm_kernel(const uint32_t* __restrict__ dev, int S,
                                                            const uint4* __restrict__ blocks, const uint32_t* __restrict__ meta,
                                                            int rows, int gpr, int rb_per_wg, int batch,
                                                            const uint16_t* __restrict__ x, float* __restrict__ y) {
    // (one more register than the allocation the body ends in: none of its 64-bit shifts may have its amount in the last one, see build.py)
    asm volatile("" ::: "v97");
    extern __shared__ __align__(16) uint32_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t* wbuf = smem + table_words(S) + wave * kUnitWords;
    float* part = reinterpret_cast<float*>(smem + table_words(S) + kWaves * kUnitWords);  // [row block of the chunk][wavefront][batch 16][row 16]
    const int total_rb = (rows + kMmaRows - 1) / kMmaRows;
    const int rb0 = blockIdx.x * rb_per_wg, rb1 = min(total_rb, rb0 + rb_per_wg);
    const int upr = (gpr + 1) / 2;  // units per row block
    const size_t cols = (size_t)gpr * kGroup;

    TableItem item{0u, 0u};
    if (tid < S * kK) item = load_table_item(dev, S, tid);
    UnitLoad pre;
    if (wave < upr) pre = load_unit16(blocks, meta, rows, gpr, rb0, wave, lane);
    if (tid < S * kK) build_table_item(smem, S, tid, item);
    if (kLong) {
        const DevLayout D{S};
        for (int i = tid; i < S * kK; i += kGemvThreads) smem[S * (kPeekEntries + kK) + i] = dev[D.longtab() + i];
        for (int i = tid; i < S * kK / 2; i += kGemvThreads) smem[S * (kPeekEntries + 2 * kK) + i] = dev[D.cent() + i];
    }
    if (lane < kUnitBlocks) wbuf[lane * kStride + kBlockWords] = 0u;
    if (kLong && lane < 2) wbuf[kUnitBlocks * kStride + lane] = 0u;  // read behind the last slot's zero word, though not used
    const Tables T = table_pointers(smem, S);
    __syncthreads();

    const int r = lane & 15, c = lane >> 5, half = (lane >> 4) & 1;  // this lane's chain: row r, column group 2 u + c, chain `half`
    const int n = lane & 15;                                          // its batch row in B and its column in the accumulator
    uint4 bx[kHalf / 8];  // B: 64 activations of batch row n at this chain's columns
    for (int c0 = rb0; c0 < rb1; c0 += kRbChunk) {
        const int nrb = min(kRbChunk, rb1 - c0);
        for (int u = wave; u < upr; u += kWaves) {
            const int cg = 2 * u + c;
            for (int k = 0; k < nrb; ++k) {
                store_unit(wbuf, pre, lane);
                uint32_t mw = pre.meta;
                // the meta word is taken here, ahead of the activation loads: a wait for it placed behind them
                // would have to wait for them as well (they sit under a condition, so their number is not known)
                asm volatile("" : "+v"(mw));
                if (k == 0) {
#pragma unroll
                    for (int j = 0; j < kHalf / 8; ++j) bx[j] = make_uint4(0, 0, 0, 0);
                    if (n < batch && cg < gpr) {
                        const uint4* src = reinterpret_cast<const uint4*>(x + (size_t)n * cols + (size_t)cg * kGroup + half * kHalf);
#pragma unroll
                        for (int j = 0; j < kHalf / 8; ++j) bx[j] = src[j];
                    }
                }
                // the next unit's payload is requested after the activations (loads return in issue order):
                // the next row block of the chunk at the same columns, else the wavefront's next columns,
                // else the first unit of the next chunk
                int un = u, rbn = c0 + k + 1;
                if (k + 1 == nrb) {
                    un = u + kWaves;
                    rbn = c0;
                    if (un >= upr) {
                        un = wave;
                        rbn = c0 + kRbChunk;
                    }
                }
                if (rbn >= rb1) {  // nothing follows: the unit in hand is requested again (from cache) and dropped, so that
                    rbn = c0 + k;  // the same loads are in flight on every path and the waits for the activations
                    un = u;        // below can leave them outstanding
                }
                pre = load_unit16(blocks, meta, rows, gpr, rbn, un, lane);
                const Lane L = lane_setup(T, mw, S);
                const _Float16 sh = __builtin_bit_cast(_Float16, (unsigned short)(mw & 0xFFFFu));
                const half2_t s2 = {sh, sh};
                uint32_t pk[4] = {0, 0, 0, 0};
                float4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
                decode_chain<kLong, kHalf, kLong>(wbuf + (2 * r + c) * kStride, half ? L.second_start : 0u, L, [&](int i, uint32_t e) {
                    if ((i & 1) == 0) {
                        pk[(i >> 1) & 3] = e >> 16;
                        return;
                    }
                    pk[(i >> 1) & 3] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, pk[(i >> 1) & 3] | (e & 0xFFFF0000u)) * s2);
                    if ((i & 7) != 7) return;
                    const uint4 av = make_uint4(pk[0], pk[1], pk[2], pk[3]);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, av), __builtin_bit_cast(half8_t, bx[i >> 3]), acc, 0, 0, 0);
                });
                // accumulator layout of the 16 x 16 tile: register j of lane l is row 4 * (l / 16) + j, column l % 16.
                // The wavefront's sums of a row block live in its own slice of LDS: the first unit stores, later ones add.
                float4_t* slot = reinterpret_cast<float4_t*>(part + (k * kWaves + wave) * (kMmaRows * kMaxBatch) + n * kMmaRows + 4 * (lane >> 4));
                if (u != wave) acc += *slot;
                *slot = acc;
            }
        }
        if (wave >= upr) {  // a wavefront without units contributes zeros
            const float4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int k = 0; k < nrb; ++k) reinterpret_cast<float4_t*>(part + (k * kWaves + wave) * (kMmaRows * kMaxBatch))[lane] = zero;
        }
        __syncthreads();
        if (tid < kMmaRows * kMaxBatch) {
            // the thread index is taken afresh: addresses derived from it are then formed here and not kept in
            // registers across the decode loop above, which has none to spare
            int t = tid;
            asm volatile("" : "+v"(t));
            const int b = t >> 4;
            for (int k = 0; k < nrb; ++k) {
                // a fixed number of reads, all in flight at once (a loop with a run-time bound waits for one after the other)
                float sum = 0.0f;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) sum += part[(k * kWaves + w) * (kMmaRows * kMaxBatch) + t];
                const int row = (c0 + k) * kMmaRows + (t & 15);
                if (b < batch && row < rows) y[(size_t)b * rows + row] = sum;
            }
        }
        __syncthreads();
    }
}

// ---- single-query attention over compressed K / V ----------------------------------------------------
// One workgroup per (sequence, head).  The cache of a head is a band of T blocks, so the kernel reuses the streaming scheme of the batch-1 GEMV: a
// unit is 32 consecutive tokens (2 KB of payload), lane l of a wavefront decodes chain l / 32 of token l % 32, units are prefetched into registers
// and decoded out of the wavefront's private LDS buffer.  The sequence is walked in spans whose scores fit LDS.  Per span a wavefront takes its units
// twice.  With the K tables it forms the scores q.K_t / sqrt(128) (the lane keeps the 64 query elements of its chain in registers), which wait in
// LDS; with the V tables every lane adds p_t * V_t of its chain into 64 private FP32 accumulators (a static register per value position, nothing
// shared).  The softmax is the wavefront's own: p_t is relative to the largest score of its units, and maxima, denominators and outputs of the
// wavefronts meet at the end of the span, once.  (A maximum and a denominator common to the workgroup took four more barriers and a loop over the
// scores between the passes.)  Where both models' tables fit they are built together, and a wavefront passes from K to V on its own; otherwise the V
// tables replace those of K in between, behind a barrier.  The decoding is bound by the table reads; what is fixed per span (builds, sums, waits at
// barriers) is what this form cuts.  Append and attention, 8 x 32 sequences and heads, 64 patterns: 4096 tokens 95.4 -> 91.9 us, 512 tokens 26.8 ->
// 24.7 us; 16 patterns: 4096 tokens 89.5 -> 84.7 us, 512 tokens 22.5 -> 20.5 us.  K and V enter as fp16(centroid * scale), formed two at a time by a
// packed FP16 multiply, which rounds exactly like the FP32-multiply-then-round rule.
template <bool kLongK, bool kLongV, int kWaves>
__global__ __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(kWaves == 12 ? 3 : 4))) void kv_attend_kernel(
    const uint32_t* __restrict__ dev_k, int Sk, const uint32_t* __restrict__ dev_v, int Sv, const uint16_t* __restrict__ q,
    const uint4* __restrict__ k_blocks, const uint32_t* __restrict__ k_meta, const uint4* __restrict__ v_blocks, const uint32_t* __restrict__ v_meta,
    const int32_t* __restrict__ seq_len, int H, int T_max, int table_words, int both, int span_max, float* __restrict__ out) {
    static_assert(2 * kWaves * 64 >= kMaxS * kK, "load_table_items: two table items per thread cover every model");
    // (one more register than the allocation the body ends in: none of its 64-bit shifts may have its amount in the last one, see build.py)
    asm volatile("" ::: "v113");
    extern __shared__ __align__(16) uint32_t smem[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t* wbuf = smem + table_words + wave * kUnitWords;
    float* state = reinterpret_cast<float*>(smem + table_words + kWaves * kUnitWords);  // per wavefront: its maximum, and its denominator
    float* scores = state + 2 * kWaves;
    uint32_t* v_tables = smem + (both ? decode_table_words(Sk, kLongK) : 0);

    const int bh = blockIdx.x;
    const int T = min(seq_len[bh / H], T_max);
    float my_out = 0.0f;  // threads 0..127: output element `tid`, not yet divided by the denominator
    float run_max = -INFINITY, run_den = 0.0f;
    const float inv_sqrt_d = 0.08838834764831845f;  // 1 / sqrt(128)
    for (int s0 = 0; s0 < T; s0 += span_max) {
        const int span = min(span_max, T - s0);
        const int units = (span + kUnitBlocks - 1) / kUnitBlocks, unit0 = s0 / kUnitBlocks;
        // ---- scores of the span
        __syncthreads();
        UnitLoad pre;
        float wave_max;  // uniform
        {
            const int lane = fresh_thread() & 63, blk = lane & (kUnitBlocks - 1), half = lane >> 5;
            if (lane < kUnitBlocks) wbuf[lane * kStride + kBlockWords] = 0u;  // zero pads of the private buffer (the sums lay over it)
            int u = wave;
            const auto load_k = [&](int at) { pre = load_unit(k_blocks, k_meta, bh, T_max, unit0 + min(at, units - 1), lane); };
            if (!both) {
                const TableItems items = load_table_items(dev_k, kLongK ? fresh_size(Sk) : Sk);
                load_k(u);
                build_tables<kLongK>(smem, dev_k, kLongK ? fresh_size(Sk) : Sk, items);
            } else if (s0 == 0) {  // both models' items, then the payload, then both builds
                const TableItems k_items = load_table_items(dev_k, kLongK ? fresh_size(Sk) : Sk), v_items = load_table_items(dev_v, kLongV ? fresh_size(Sv) : Sv);
                load_k(u);
                build_tables<kLongK>(smem, dev_k, kLongK ? fresh_size(Sk) : Sk, k_items);
                build_tables<kLongV>(v_tables, dev_v, kLongV ? fresh_size(Sv) : Sv, v_items);
            } else {
                load_k(u);
            }
            const Tables TK = table_pointers(smem, Sk);
            __syncthreads();
            // the query elements of this lane's chain, FP16 pairs: reloaded per span (from cache) rather than kept alive across the V
            // pass; the pointer that comes back from the empty asm statement is given its address space again, or its loads would be
            // flat loads.  (Requested ahead of the build, behind the payload: 4 sequences and heads of 64 tokens 13.71 -> 13.94 us, 256
            // of 4096 no difference.)
            uint32_t qx[kHalf / 2];
            const uint4* qgen = reinterpret_cast<const uint4*>(q + (size_t)bh * kGroup + half * kHalf);
            asm volatile("" : "+v"(qgen));
            const global_u4* qsrc = (const global_u4*)qgen;
#pragma unroll
            for (int j = 0; j < kHalf / 8; ++j) {
                const u32x4 v = qsrc[j];
                qx[4 * j] = v.x; qx[4 * j + 1] = v.y; qx[4 * j + 2] = v.z; qx[4 * j + 3] = v.w;
            }
            float my_max = -INFINITY;
            for (; u < units; u += kWaves) {
                store_unit(wbuf, pre, lane);
                const uint32_t mw = pre.meta;
                if (u + kWaves < units) load_k(u + kWaves);
                // the query stays packed: without this the conversions to FP32 are hoisted out of the loop and
                // occupy 64 registers instead of 32
#pragma unroll
                for (int j = 0; j < kHalf / 2; ++j) asm volatile("" : "+v"(qx[j]));
                const Lane L = lane_setup(TK, mw, Sk);
                const _Float16 sh = __builtin_bit_cast(_Float16, (unsigned short)(mw & 0xFFFFu));
                const half2_t s2 = {sh, sh};
                uint32_t pk = 0;
                float acc = 0.0f;
                __builtin_amdgcn_s_setprio(kPriorityDecode);
                decode_chain<kLongK, kHalf>(wbuf + blk * kStride, half ? L.second_start : 0u, L, [&](int i, uint32_t e) {
                    if ((i & 1) == 0) {
                        pk = e >> 16;
                    } else {
                        const half2_t w2 = __builtin_bit_cast(half2_t, pk | (e & 0xFFFF0000u)) * s2;
                        const half2_t q2 = __builtin_bit_cast(half2_t, qx[i >> 1]);
                        acc = fmaf((float)w2[0], (float)q2[0], acc);
                        acc = fmaf((float)w2[1], (float)q2[1], acc);
                        if ((i & 3) == 3) asm volatile("" : "+v"(acc));  // keeps the multiply-adds next to their table reads
                    }
                });
                __builtin_amdgcn_s_setprio(0);
                acc += __shfl_xor(acc, 32);
                const int t = u * kUnitBlocks + blk;
                const float sc = t < span ? acc * inv_sqrt_d : -INFINITY;
                if (half == 0) scores[t] = sc;  // for this wavefront alone
                my_max = fmaxf(my_max, sc);
            }
            wave_max = wave_all(my_max, [](float a, float b) { return fmaxf(a, b); });
        }
        // ---- weighted sum of V over the span
        {
            const int lane = fresh_thread() & 63, blk = lane & (kUnitBlocks - 1), half = lane >> 5;
            int u = wave;
            const auto load_v = [&](int at) { pre = load_unit(v_blocks, v_meta, bh, T_max, unit0 + min(at, units - 1), lane); };
            if (both) {
                load_v(u);
            } else {
                const TableItems items = load_table_items(dev_v, kLongV ? fresh_size(Sv) : Sv);
                load_v(u);
                __syncthreads();
                build_tables<kLongV>(v_tables, dev_v, kLongV ? fresh_size(Sv) : Sv, items);
                __syncthreads();
            }
            const Tables TV = table_pointers(v_tables, Sv);
            const float base = wave_max == -INFINITY ? 0.0f : wave_max;  // (a wavefront without units, or without a score above -inf)
            float den = 0.0f;
            float o[kHalf];
#pragma unroll
            for (int i = 0; i < kHalf; ++i) o[i] = 0.0f;
            for (; u < units; u += kWaves) {
                store_unit(wbuf, pre, lane);
                // a slot past the sequence end may hold anything (the cache behind seq_len need not be initialised):
                // its scale is taken as 0, so that its values are zeros and not, say, NaN times a zero weight
                const uint32_t mw = (u * kUnitBlocks + blk < span) ? pre.meta : (pre.meta & 0xFFFF0000u);
                if (u + kWaves < units) load_v(u + kWaves);
                const Lane L = lane_setup(TV, mw, Sv);
                const _Float16 sh = __builtin_bit_cast(_Float16, (unsigned short)(mw & 0xFFFFu));
                const half2_t s2 = {sh, sh};
                const float p = __expf(scores[u * kUnitBlocks + blk] - base);  // 0 for the tokens past the span
                den += p;
                uint32_t pk = 0;
                __builtin_amdgcn_s_setprio(kPriorityDecode);
                decode_chain<kLongV, kHalf>(wbuf + blk * kStride, half ? L.second_start : 0u, L, [&](int i, uint32_t e) {
                    if ((i & 1) == 0) {
                        pk = e >> 16;
                    } else {
                        const half2_t w2 = __builtin_bit_cast(half2_t, pk | (e & 0xFFFF0000u)) * s2;
                        o[i - 1] = fmaf(p, (float)w2[0], o[i - 1]);
                        o[i] = fmaf(p, (float)w2[1], o[i]);
                        if ((i & 3) == 3) asm volatile("" : "+v"(o[i - 3]), "+v"(o[i - 2]), "+v"(o[i - 1]), "+v"(o[i]));  // as above
                    }
                });
                __builtin_amdgcn_s_setprio(0);
            }
            // The span's sums over the rows of 16 lanes (rows 0 and 1 hold values 0..63, rows 2 and 3 values 64..127).  At the first two
            // levels a lane keeps the values that match its own lane bit and sends the others to its partner, so that lane l of a row ends
            // with the row's totals of values 4 j + l % 4; the first four lanes put them over the wavefront's payload buffer.  (A tree per
            // value and a store of its first lane: 256 additions and 64 stores, this way 144 instructions and 4 stores.)
            const int ln = fresh_thread() & 63;
            const bool b0 = ln & 1, b1 = ln & 2;
            float a[kHalf / 4];
#pragma unroll
            for (int j = 0; j < kHalf / 4; ++j) {
                float t[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const float x = o[4 * j + 2 * i], y = o[4 * j + 2 * i + 1];
                    t[i] = (b0 ? y : x) + dpp_mov<0xB1>(b0 ? x : y);  // quad_perm [1,0,3,2]
                }
                float r = (b1 ? t[1] : t[0]) + dpp_mov<0x4E>(b1 ? t[0] : t[1]);  // quad_perm [2,3,0,1]
                r += dpp_mov<0x124>(r);       // row_ror 4
                a[j] = r + dpp_mov<0x128>(r);  // row_ror 8
            }
            den = 0.5f * wave_sum(den);  // both halves hold the tokens' weights
            wave_lds_fence();
            if ((ln & 15) < 4) {
                float4_t* to = reinterpret_cast<float4_t*>(wbuf) + (ln >> 4) * (kHalf / 4) + (ln & 3) * 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) to[j] = float4_t{a[4 * j], a[4 * j + 1], a[4 * j + 2], a[4 * j + 3]};
            }
            if (ln == 0) {
                state[wave] = wave_max;
                state[kWaves + wave] = den;
            }
        }
        __syncthreads();
        if (tid < kGroup) {
            const int i = tid & (kHalf - 1);
            const float* rows = reinterpret_cast<const float*>(smem + table_words) + (tid >> 6) * kGroup + (i & 3) * 16 + (i >> 2);
            float most = run_max;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) most = fmaxf(most, state[w]);
            const float rescale = run_max == -INFINITY ? 0.0f : __expf(run_max - most);
            float v = 0.0f, d = 0.0f;
#pragma unroll 4
            for (int w = 0; w < kWaves; ++w) {
                const float part = state[w] == -INFINITY ? 0.0f : __expf(state[w] - most);
                v += part * (rows[w * kUnitWords] + rows[w * kUnitWords + kHalf]);
                d += part * state[kWaves + w];
            }
            my_out = my_out * rescale + v;
            run_den = run_den * rescale + d;
            run_max = most;
        }
    }
    if (tid < kGroup) out[(size_t)bh * kGroup + tid] = T > 0 ? my_out / run_den : 0.0f;
}

// ---- grouped-query attention over compressed K / V, split over the tokens ---------------------------------
// Several query heads share one key/value head (Section 5.3: with grouped-query attention the batched matrix-vector products become small matrix
// products).  One workgroup per (sequence, key/value head, token range) decodes every K and V block of its range once and serves all grp = Hq / Hkv
// query heads of the group with it, on the matrix cores, in 16 x 16 tiles (v_mfma_f32_16x16x32_f16): a lane's four accumulator registers per tile
// leave room for three wavefronts per SIMD, four where workgroups share a compute unit, where 32 x 32 tiles, half of whose columns no group of at
// most 16 heads can use, left two. A unit is 32 tokens; lane l decodes chain (l / 16) % 2 of token l % 16 + 16 (l / 32).
//   scores  S[token][head] = sum_dim K[token][dim] q[head][dim]: eight decoded values of a lane are its A operand (row
//           l % 16, k slice l / 16).  Slices 0 and 1 belong to tokens 0..15, slices 2 and 3 to tokens 16..31; with up to
//           eight heads, B holds the queries in columns 0..7 for the former and in columns 8..15 for the latter (zeros
//           elsewhere), so one product gives 32 tokens x 8 heads.  With more heads (kWide) there are two products, the
//           other tokens' rows of A zeroed.
//   output  O[dim][head] = sum_token V[token][dim] P[head][token]: here the reduction runs over the tokens, so the
//           decoded values have to be turned: every 8 values the wavefront writes a 16 dims x 32 tokens FP16 tile
//           to its private LDS buffer (neighbouring lanes first swap halves so that each writes two tokens of one
//           dimension), reads it back as an A operand (row = dimension, eight tokens per lane) and multiplies with
//           the probabilities; the eight 16 x 16 accumulator tiles (32 registers) live across the spans.
// The sequence is walked in spans whose scores fit LDS; per span a wavefront takes its units twice, with the K and with the V tables. The softmax is
// the wavefront's own: scores become probabilities, relative to the largest score that the wavefront has met, when they are read as B operands,
// each as two FP16 numbers (the rounded value and the rest, 22 bits together), and the accumulators of a lane -- all of one head -- are rescaled from
// span to span.  Up to eight heads leave columns 8..15 of the product free for the rests, more take a second product.  (With one FP16 number and a
// denominator of the rounded values the error against 64 bits followed the number of wavefronts, each of which holds its own largest probability
// exactly: 8 x 8 heads in groups of 4, 4096 tokens, 2.2e-5 to 3.1e-5 with 12 wavefronts, 2.2e-5 to 3.0e-5 with 16; 4e-7 to 5e-7 so. With append and
// merge 31.7 us either way; a second product there 31.8 us, and 1 to 3 % at short ranges.)  Maxima,
// denominators and outputs of the wavefronts meet once, at the end.  If both models' tables fit they are built once, and that is the only barrier
// until then (8 x 8 heads in groups of 4, 16 patterns, append, attention and merge: 4096 tokens 34.9 us with a softmax of the workgroup between the
// passes, 33.3 us so; groups of 8, 1024 tokens 19.1 -> 17.9 us); otherwise the V tables replace the K tables in every span.  With one range per
// sequence the result is normalised and written; otherwise (maximum, denominator, unnormalised output) of the range go to the caller's workspace and
// kv_attend_combine_kernel merges them.

// grid: (B * Hkv, n_splits).  The partial result of a split and query head is at
// index (sequence * Hq + query head) * n_splits + split of the workspace: 128 outputs each, then (maximum, denominator) pairs.
struct GqaArgs {
    const uint32_t* dev_k;
    const uint32_t* dev_v;
    const uint16_t* q;
    const uint4* k_blocks;
    const uint32_t* k_meta;
    const uint4* v_blocks;
    const uint32_t* v_meta;
    const int32_t* seq_len;
    float* out;
    float* ws;
    int Sk, Sv, B, Hq, Hkv, T_max, table_words, both, span, step;
};

template <bool kLongK, bool kLongV, bool kWide, int kWaves>
__global__ __launch_bounds__(kWaves * 64) void kv_attend_gqa_kernel(GqaArgs args) {
    constexpr int kThreads = kWaves * 64;
    static_assert(2 * kThreads >= kMaxS * kK, "load_table_items: two table items per thread cover every model");
    constexpr int kOutputs = (kGqaMaxGroup * kGroup + kThreads - 1) / kThreads;  // output elements per thread
    // (one more register than the allocation the body ends in: none of its 64-bit shifts may have its amount in the last one, see build.py)
    asm volatile("" ::: "v121");
    const int Sk = args.Sk, Sv = args.Sv, B = args.B, Hq = args.Hq, Hkv = args.Hkv, T_max = args.T_max, both = args.both, table_words = args.table_words;
    extern __shared__ __align__(16) uint32_t smem[];
    const int grp = Hq / Hkv, sstride = gqa_score_stride(args.span), n_splits = gridDim.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float* state = reinterpret_cast<float*>(smem);  // [wavefront][16] maxima, [wavefront][16] denominators
    uint32_t* k_tables = smem + gqa_state_words(kWaves);
    uint32_t* wbuf = k_tables + table_words + wave * kUnitWords;
    uint32_t* tile = k_tables + table_words + kWaves * kUnitWords + wave * kTileWords;
    float* scores = reinterpret_cast<float*>(k_tables + table_words + kWaves * (kUnitWords + kTileWords));  // [grp][sstride]
    uint32_t* v_tables = k_tables + (both ? decode_table_words(Sk, kLongK) : 0);
    if (lane < kUnitBlocks) wbuf[lane * kStride + kBlockWords] = 0u;

    const int b = blockIdx.x / Hkv, hkv = blockIdx.x - b * Hkv, split = blockIdx.y, bkv = blockIdx.x;
    const int T = max(0, min(args.seq_len[b], T_max));
    const int per_range = ((T + kUnitBlocks - 1) / kUnitBlocks + n_splits - 1) / n_splits;
    const int t_begin = min(T, split * per_range * kUnitBlocks), t_end = min(T, (split + 1) * per_range * kUnitBlocks);
    const int span_max = t_end - t_begin <= args.span ? args.span : args.step;  // a range that one span holds is not cut
    // the lane's place in a unit, formed in either pass: kept, what is derived from it would take registers through both
    struct Place {
        int lane, n, slice, half, tok;  // n: matrix-core row or column; slice: k slice; half: chain of the lane's token `tok` of the unit
        __device__ Place() : lane(fresh_thread() & 63), n(lane & 15), slice(lane >> 4), half(slice & 1), tok(n + 16 * (lane >> 5)) {}
    };
    const float inv_sqrt_d = 0.08838834764831845f;  // 1 / sqrt(128)
    float4_t o[8];  // tile j: row r is dimension 64 (r / 8) + 8 j + r % 8, column the head
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
    float run_max = -INFINITY, run_den = 0.0f;  // of this wavefront and of head l % 16; the denominator of the lane's tokens

    for (int s0 = t_begin; s0 < t_end; s0 += span_max) {
        const int span = min(span_max, t_end - s0);
        const int units = (span + kUnitBlocks - 1) / kUnitBlocks, unit0 = s0 / kUnitBlocks;  // s0 is a multiple of 32
        // ---- scores of the span, all query heads of the group
        UnitLoad pre;
        float mx = -INFINITY;
        {
        const Place P;
        const int lane = P.lane, n = P.n, slice = P.slice, half = P.half, tok = P.tok;
        const int head = kWide ? n : n & 7;                             // head of this lane's column
        const bool head_ok = head < grp, b_ok = head_ok && (kWide || (n >> 3) == (lane >> 5));
        const size_t q_row = ((size_t)b * Hq + (size_t)hkv * grp + (head_ok ? head : 0)) * kGroup;
        int u = wave;
        const auto load_k = [&](int at) { pre = load_unit(args.k_blocks, args.k_meta, bkv, T_max, unit0 + min(at, units - 1), lane, tok); };
        uint4 bq[kHalf / 8];  // B operands: the query of this lane's head, dimensions 64 * half + 8j .. + 7
        // requested behind the payload, so that it arrives during the builds; reloaded per span rather than kept alive across the V
        // phase (the pointer passes through an empty asm statement and is given its address space again)
        const auto load_q = [&] {
            const uint4* qgen = reinterpret_cast<const uint4*>(args.q + q_row + half * kHalf);
            asm volatile("" : "+v"(qgen));
            const global_u4* qsrc = (const global_u4*)qgen;
#pragma unroll
            for (int j = 0; j < kHalf / 8; ++j) {
                const u32x4 v = qsrc[j];
                bq[j] = make_uint4(v.x, v.y, v.z, v.w);
            }
        };
        if (!both) {
            const TableItems items = load_table_items(args.dev_k, kLongK ? fresh_size(Sk) : Sk);
            load_k(u);
            load_q();
            __syncthreads();  // the V tables of the span before have been read
            build_tables<kLongK>(k_tables, args.dev_k, kLongK ? fresh_size(Sk) : Sk, items);
            __syncthreads();
        } else if (s0 == t_begin) {  // both models' items, then the payload, then both builds
            const TableItems k_items = load_table_items(args.dev_k, kLongK ? fresh_size(Sk) : Sk), v_items = load_table_items(args.dev_v, kLongV ? fresh_size(Sv) : Sv);
            load_k(u);
            load_q();
            build_tables<kLongK>(k_tables, args.dev_k, kLongK ? fresh_size(Sk) : Sk, k_items);
            build_tables<kLongV>(v_tables, args.dev_v, kLongV ? fresh_size(Sv) : Sv, v_items);
            __syncthreads();
        } else {
            load_k(u);
            load_q();
        }
        const Tables TK = table_pointers(k_tables, Sk);
        {
#pragma unroll
            for (int j = 0; j < kHalf / 8; ++j) bq[j] = b_ok ? bq[j] : make_uint4(0u, 0u, 0u, 0u);
            for (; u < units; u += kWaves) {
                store_unit(wbuf, pre, lane);
                // a slot past the range may hold anything: scale 0, so that its values are zeros (tokens m and 16 + m share a row
                // of the product, and NaN * 0 would poison it)
                const uint32_t mw = (u * kUnitBlocks + tok < span) ? pre.meta : (pre.meta & 0xFFFF0000u);
                if (u + kWaves < units) load_k(u + kWaves);
                const Lane L = lane_setup(TK, mw, Sk);
                const _Float16 sh16 = __builtin_bit_cast(_Float16, (unsigned short)(mw & 0xFFFFu));
                const half2_t s2 = {sh16, sh16};
                uint32_t pk[4];
                float4_t acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
                decode_chain<kLongK, kHalf>(wbuf + tok * kStride, half ? L.second_start : 0u, L, [&](int i, uint32_t e) {
                    if ((i & 1) == 0) {
                        pk[(i >> 1) & 3] = e >> 16;
                        return;
                    }
                    pk[(i >> 1) & 3] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, pk[(i >> 1) & 3] | (e & 0xFFFF0000u)) * s2);
                    if ((i & 7) != 7) return;
                    const half8_t bv = __builtin_bit_cast(half8_t, bq[i >> 3]);
                    if (kWide) {
                        const bool low = lane < 32;
                        const uint4 a0 = make_uint4(low ? pk[0] : 0u, low ? pk[1] : 0u, low ? pk[2] : 0u, low ? pk[3] : 0u);
                        const uint4 a1 = make_uint4(low ? 0u : pk[0], low ? 0u : pk[1], low ? 0u : pk[2], low ? 0u : pk[3]);
                        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a0), bv, acc[0], 0, 0, 0);
                        acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a1), bv, acc[1], 0, 0, 0);
                    } else {
                        const uint4 av = make_uint4(pk[0], pk[1], pk[2], pk[3]);
                        acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, av), bv, acc[0], 0, 0, 0);
                    }
                });
                // accumulator layout of the 16 x 16 tile: register i of lane l is row 4 * (l / 16) + i, column l % 16
#pragma unroll
                for (int w = 0; w < (kWide ? 2 : 1); ++w) {
                    const int t0 = u * kUnitBlocks + 4 * slice + (kWide ? 16 * w : 16 * (n >> 3));
                    float4_t v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        v[i] = t0 + i < span ? acc[w][i] * inv_sqrt_d : -INFINITY;
                        mx = fmaxf(mx, v[i]);
                    }
                    if (head_ok) *reinterpret_cast<float4_t*>(scores + head * sstride + t0) = v;  // for this wavefront alone
                }
            }
            // the wavefront's maximum per head: over the lanes of the column
            if (!kWide) mx = fmaxf(mx, __shfl_xor(mx, 8));
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
        }
        }
        // ---- weighted sum of V over the span
        const Place P;
        const int lane = P.lane, n = P.n, slice = P.slice, half = P.half, tok = P.tok;
        const uint32_t swap_sel = (lane & 1) ? 0x03020706u : 0x05040100u;  // odd lanes keep the high halves, even lanes the low halves
        int u = wave;
        const auto load_v = [&](int at) { pre = load_unit(args.v_blocks, args.v_meta, bkv, T_max, unit0 + min(at, units - 1), lane, tok); };
        if (both) {
            load_v(u);
        } else {
            const TableItems items = load_table_items(args.dev_v, kLongV ? fresh_size(Sv) : Sv);
            load_v(u);
            __syncthreads();
            build_tables<kLongV>(v_tables, args.dev_v, kLongV ? fresh_size(Sv) : Sv, items);
            __syncthreads();
        }
        const Tables TV = table_pointers(v_tables, Sv);
        {
            const float before = run_max;
            run_max = fmaxf(before, mx);
            const float base = run_max == -INFINITY ? 0.0f : run_max;  // (a wavefront without units, or without a score above -inf)
            if (s0 != t_begin) {  // every accumulator of a lane belongs to head l % 16
                const float alpha = before == -INFINITY ? 0.0f : __expf(before - base);
                run_den *= alpha;
#pragma unroll
                for (int j = 0; j < 8; ++j) o[j] *= alpha;
            }
            const int head = kWide ? n : n & 7;
            const float* score = scores + min(head, grp - 1) * sstride + 8 * slice;
            for (; u < units; u += kWaves) {
                store_unit(wbuf, pre, lane);
                const uint32_t mw = (u * kUnitBlocks + tok < span) ? pre.meta : (pre.meta & 0xFFFF0000u);
                if (u + kWaves < units) load_v(u + kWaves);
                const Lane L = lane_setup(TV, mw, Sv);
                const _Float16 sh16 = __builtin_bit_cast(_Float16, (unsigned short)(mw & 0xFFFFu));
                const half2_t s2 = {sh16, sh16};
                // B operand: probabilities of head l % 16 for tokens 8 * (l / 16) .. + 7 of the unit; 0 for the tokens past the span. What an
                // FP16 probability leaves of the FP32 one is the operand of a product of its own, or with up to eight heads of columns 8..15.
                // (A block without a finite scale: its infinities must meet no rest of 0 or below, which would make NaN of them.)
                const bool no_rest = __ballot((mw & 0x7C00u) == 0x7C00u) != 0;
                const float taken = no_rest || (!kWide && n < 8) ? 0.0f : 1.0f;
                half8_t pb, rest;
                {
                    const float4_t s[2] = {reinterpret_cast<const float4_t*>(score + u * kUnitBlocks)[0], reinterpret_cast<const float4_t*>(score + u * kUnitBlocks)[1]};
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float p = head < grp ? __expf(s[i >> 2][i & 3] - base) : 0.0f;
                        pb[i] = (_Float16)p;
                        rest[i] = (_Float16)fmaf(-taken, (float)pb[i], p);
                        run_den += p;
                    }
                    if (!kWide) pb = rest;
                }
                uint32_t pk[4];
                decode_chain<kLongV, kHalf>(wbuf + tok * kStride, half ? L.second_start : 0u, L, [&](int i, uint32_t e) {
                    if ((i & 1) == 0) {
                        pk[(i >> 1) & 3] = e >> 16;
                        return;
                    }
                    pk[(i >> 1) & 3] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, pk[(i >> 1) & 3] | (e & 0xFFFF0000u)) * s2);
                    if ((i & 7) != 7) return;
                    // 8 values of this lane's token -> rows 8 * half + r of the tile (dimension 64 * half + 8 * (i / 8) + r);
                    // an even lane takes dimension 2 r2 of its own and its neighbour's token, the odd neighbour dimension 2 r2 + 1
                    wave_lds_fence();
#pragma unroll
                    for (int r2 = 0; r2 < 4; ++r2) {
                        const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)pk[r2], 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
                        tile[(8 * half + 2 * r2 + (lane & 1)) * kTileStride + (tok >> 1)] = __builtin_amdgcn_perm(other, pk[r2], swap_sel);
                    }
                    wave_lds_fence();
                    const uint4 a0 = *reinterpret_cast<const uint4*>(tile + n * kTileStride + 4 * slice);
                    o[i >> 3] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a0), pb, o[i >> 3], 0, 0, 0);
                    if (kWide) o[i >> 3] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a0), rest, o[i >> 3], 0, 0, 0);
                });
            }
        }
    }
    // ---- sum over the wavefronts; everything in LDS but the state is dead behind the first barrier
    const Place P;
    const int n = P.n, slice = P.slice;
    float *out = args.out, *ws = args.ws;
    const size_t first_head = (size_t)b * Hq + (size_t)hkv * grp;
    const size_t part = first_head * n_splits + split, total = (size_t)B * Hq * n_splits;  // of the group's first head
    run_den += __shfl_xor(run_den, 16);
    run_den += __shfl_xor(run_den, 32);
    if (lane < 16) state[wave * kGqaMaxGroup + lane] = run_max;
    __syncthreads();
    float most = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) most = fmaxf(most, state[w * kGqaMaxGroup + n]);
    const float mine = run_max == -INFINITY ? 0.0f : __expf(run_max - most);
    if (lane < 16) state[(kWaves + wave) * kGqaMaxGroup + lane] = run_den * mine;
    float* red = reinterpret_cast<float*>(k_tables);  // [wavefront][8 tiles][4 slices][16 lanes][4]
    if (!kWide) {  // what the rests contributed
#pragma unroll
        for (int j = 0; j < 8; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float here = o[j][i];
                o[j][i] = here + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, here), 0x128, 0xF, 0xF, true));  // row_ror:8
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) *reinterpret_cast<float4_t*>(red + (wave * 8 + j) * kRedTile + slice * kRedRow + n * 4) = o[j] * mine;
    __syncthreads();
    const auto denominator = [&](int g) {
        float den = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) den += state[(kWaves + w) * kGqaMaxGroup + g];
        return den;
    };
    if (n_splits > 1 && tid < grp) {  // (the first wavefront's lane of head `tid` holds that head's maximum)
        const size_t at = total * kGroup + (part + (size_t)tid * n_splits) * 2;
        ws[at] = most;
        ws[at + 1] = denominator(tid);
    }
#pragma unroll
    for (int k = 0; k < kOutputs; ++k) {
        const int e = tid + k * kThreads, g = e / kGroup, dim = e % kGroup;
        if (g < grp) {
            const int row = 8 * (dim >> 6) + (dim & 7);
            const float* at = red + ((dim & 63) >> 3) * kRedTile + (row >> 2) * kRedRow + g * 4 + (row & 3);
            float sum = 0.0f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) sum += at[w * 8 * kRedTile];
            if (n_splits == 1) {
                const float den = denominator(g);
                out[(first_head + g) * kGroup + dim] = den > 0.0f ? sum / den : 0.0f;
            } else {
                ws[(part + (size_t)g * n_splits) * kGroup + dim] = sum;
            }
        }
    }
}

// merges the token ranges of one (sequence, query head): grid B * Hq, 128 threads
__global__ __launch_bounds__(kGroup) void kv_attend_combine_kernel(const float* __restrict__ ws, int n_heads, int n_splits, float* __restrict__ out) {
    const size_t bh = blockIdx.x;
    const float* ml = ws + (size_t)n_heads * n_splits * kGroup + bh * n_splits * 2;
    const float* part = ws + bh * n_splits * kGroup + threadIdx.x;
    // Sixteen splits at a time (four or eight where there are no more) with all their loads in flight together, indices
    // clamped; the additions run in split order.  An empty split (maximum -inf, zeros) gets weight 0, also when every
    // split is empty (mx = -inf).  The kernel is bound by the latency of the partial results, which come from memory: up to
    // sixteen splits the maximum is formed from the values in hand and not in a round trip of its own.
    float num = 0.0f, den = 0.0f;
    const auto batch = [&](auto count, int s0, float mx) {
        constexpr int kCount = decltype(count)::value;
        float m[kCount], d[kCount], v[kCount];
#pragma unroll
        for (int j = 0; j < kCount; ++j) {
            const int sj = min(s0 + j, n_splits - 1);
            m[j] = ml[2 * sj];
            d[j] = ml[2 * sj + 1];
            v[j] = part[(size_t)sj * kGroup];
        }
        if (s0 == 0 && n_splits <= kCount) {
            mx = m[0];
#pragma unroll
            for (int j = 1; j < kCount; ++j) mx = fmaxf(mx, m[j]);
        }
#pragma unroll
        for (int j = 0; j < kCount; ++j) {
            if (s0 + j < n_splits) {  // uniform
                const float w = m[j] == -INFINITY ? 0.0f : __expf(m[j] - mx);
                num += w * v[j];
                den += w * d[j];
            }
        }
    };
    if (n_splits <= 4) batch(std::integral_constant<int, 4>{}, 0, 0.0f);
    else if (n_splits <= 8) batch(std::integral_constant<int, 8>{}, 0, 0.0f);
    else if (n_splits <= 16) batch(std::integral_constant<int, 16>{}, 0, 0.0f);
    else {
        // the largest of the splits' maxima: a few splits per lane and a wavefront maximum (exact whatever the order),
        // instead of a chain of n_splits dependent loads
        float mx = -INFINITY;
        for (int s = threadIdx.x & 63; s < n_splits; s += 64) mx = fmaxf(mx, ml[2 * s]);
        mx = wave_all(mx, [](float a, float b) { return fmaxf(a, b); });
        for (int s0 = 0; s0 < n_splits; s0 += 16) batch(std::integral_constant<int, 16>{}, s0, mx);
    }
    out[bh * kGroup + threadIdx.x] = den > 0.0f ? num / den : 0.0f;
}

// ---- device scratch of the entry point that allocates nothing -----------------------------------------------
// ecco_kv_attend_gqa_noalloc keeps the token splits' partial results here instead of in a caller's workspace.
// Each GPU the library runs on holds its own copy of the array, at its own address, until the process ends.  In host
// code the array's name is only a handle: the address kernels can use comes from hipGetSymbolAddress, asked once
// per device with that device current, and is what every launch and every host call is given.
static __device__ __align__(256) float scratch[ECCO_GQA_SCRATCH_BYTES / sizeof(float)];

constexpr int kMaxDevices = 16;
std::mutex scratch_lock;
float* scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each device, once asked

// The address of `scratch` on `device`, which must be the current device.  nullptr if the runtime refuses.
float* scratch_on_current_device(int device) {
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> hold(scratch_lock);
    if (!scratch_ptr[device]) {
        float* p = nullptr;
        if (hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        scratch_ptr[device] = p;
    }
    return scratch_ptr[device];
}

// ---- host side -----------------------------------------------------------------------------------------
}  // namespace

namespace ecco {
// compute units of a device, asked once per device (atomics: host threads may race to fill the cache, with the same value)
int cu_count(int device) {
    static std::atomic<int> cached[16];
    if (device < 0 || device >= 16) return 256;
    int n = cached[device].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || n <= 0) n = 256;
        cached[device].store(n, std::memory_order_relaxed);
    }
    return n;
}

// A kernel that needs more than 64 KB of LDS has to be told so; the attribute belongs to the kernel (on the
// current device), not to a launch, so it is set the first time a kernel is launched on a device -- to the most
// any launch can ask for -- and remembered (a short list under a mutex: host threads may enter together).
int allow_lds_once(const void* kernel, int device, size_t bytes) {
    if (bytes <= 64 * 1024) return ECCO_OK;
    static std::mutex lock;
    static std::vector<std::pair<const void*, int>> done;
    std::lock_guard<std::mutex> hold(lock);
    for (const auto& d : done)
        if (d.first == kernel && d.second == device) return ECCO_OK;
    ECCO_HIP_CHECK(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    done.emplace_back(kernel, device);
    return ECCO_OK;
}

// Called by ecco_model_to_device with `device` current: asks for the scratch array's address on that device, so that
// the entry point that allocates nothing finds it ready (also under stream capture).
int init_device_scratch(int device) { return scratch_on_current_device(device) ? ECCO_OK : ECCO_EHIP; }
}  // namespace ecco

extern "C" {

static int decode_common(const ecco_model* m, const void* blocks, const uint32_t* meta, size_t n_groups, void* dst,
                         void* stream, bool indices) {
    if (!m) return ECCO_EINVAL;
    if (n_groups == 0) return model_ready(m);  // nothing to do; pointers may be null
    if (!blocks || !meta || !dst) return ECCO_EINVAL;
    if (n_groups > (size_t)0x7FFFFFFF - kUnitBlocks) return ECCO_ESHAPE;
    if (!aligned(blocks, 64) || !aligned(dst, 16) || !aligned(meta, 4)) return ECCO_EALIGN;
    if (model_ready(m) != ECCO_OK) return ECCO_EINVAL;
    const int units = (int)((n_groups + kUnitBlocks - 1) / kUnitBlocks);
    const int cus = cu_count(m->device);
    const int units_per_wg = std::max(1, (units + cus - 1) / cus);  // small inputs: few units on many compute units (a wavefront's chain is the floor)
    const int grid = (units + units_per_wg - 1) / units_per_wg;
    const size_t lds = decode_lds_bytes(m->S);
    const bool lng = m->max_len > kPeekBits;
    const int dev_id = m->device;
    auto launch = [&](auto kernel) -> int {
        int rc = allow_lds(kernel, dev_id, lds);
        if (rc != ECCO_OK) return rc;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kDecWaves * 64), lds, static_cast<hipStream_t>(stream), m->dev, m->S,
                           static_cast<const uint4*>(blocks), meta, (int)n_groups, units_per_wg, dst);
        ECCO_HIP_CHECK(hipGetLastError());
        return ECCO_OK;
    };
    if (indices) return lng ? launch(decode_kernel<true, true, false>) : launch(decode_kernel<false, true, false>);
    if (ecco_stream::weights(dst, n_groups * kGroup * 2) == ecco_stream::Stores::kThrough) return lng ? launch(decode_kernel<true, false, true>) : launch(decode_kernel<false, false, true>);
    return lng ? launch(decode_kernel<true, false, false>) : launch(decode_kernel<false, false, false>);
}

int ecco_decode(const ecco_model* m, const void* blocks, const uint32_t* meta, size_t n_groups, uint16_t* dst, void* stream) {
    return decode_common(m, blocks, meta, n_groups, dst, stream, false);
}

int ecco_decode_indices(const ecco_model* m, const void* blocks, const uint32_t* meta, size_t n_groups, uint8_t* idx, void* stream) {
    return decode_common(m, blocks, meta, n_groups, idx, stream, true);
}

int ecco_decode_gemv(const ecco_model* m, const void* blocks, const uint32_t* meta, int rows, int cols,
                     const uint16_t* x, int batch, float* y, void* stream) {
    if (!m || !blocks || !meta || !x || !y) return ECCO_EINVAL;
    if (rows <= 0 || cols <= 0 || cols % kGroup != 0 || cols > 65536 || batch < 1 || batch > 16) return ECCO_ESHAPE;
    if (!aligned(blocks, 64) || !aligned(x, 16) || !aligned(y, 4) || !aligned(meta, 4)) return ECCO_EALIGN;
    if (model_ready(m) != ECCO_OK) return ECCO_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int gpr = cols / kGroup;
    const int cus = cu_count(m->device);
    const bool lng = m->max_len > kPeekBits;
    if (batch == 1) {
        // one band of rows per workgroup, one workgroup per compute unit where the matrix allows it
        const int band = std::min(kMaxBandRows, std::max(1, (rows + cus - 1) / cus));
        const size_t lds = gemv_lds_bytes(m->S, gpr);
        int rc = lng ? allow_lds(gemv_kernel<true>, m->device, lds) : allow_lds(gemv_kernel<false>, m->device, lds);
        if (rc != ECCO_OK) return rc;
        const uint32_t* xb = reinterpret_cast<const uint32_t*>(x);
        const int grid = (rows + band - 1) / band;
        if (lng)
            hipLaunchKernelGGL(gemv_kernel<true>, dim3(grid), dim3(kGemvThreads), lds, st, m->dev, m->S,
                               static_cast<const uint4*>(blocks), meta, rows, gpr, band, xb, y);
        else
            hipLaunchKernelGGL(gemv_kernel<false>, dim3(grid), dim3(kGemvThreads), lds, st, m->dev, m->S,
                               static_cast<const uint4*>(blocks), meta, rows, gpr, band, xb, y);
    } else {
        // whole 16-row blocks per workgroup, one workgroup per compute unit where the matrix allows it
        const int total_rb = (rows + kMmaRows - 1) / kMmaRows;
        const int rb_per_wg = std::max(1, (total_rb + cus - 1) / cus);
        const int grid = (total_rb + rb_per_wg - 1) / rb_per_wg;
        const size_t glds = gemm_lds_bytes(m->S);
        int rc = lng ? allow_lds(gemm_kernel<true>, m->device, glds) : allow_lds(gemm_kernel<false>, m->device, glds);
        if (rc != ECCO_OK) return rc;
        if (lng)
            hipLaunchKernelGGL(gemm_kernel<true>, dim3(grid), dim3(kGemvThreads), glds, st, m->dev, m->S,
                               static_cast<const uint4*>(blocks), meta, rows, gpr, rb_per_wg, batch, x, y);
        else
            hipLaunchKernelGGL(gemm_kernel<false>, dim3(grid), dim3(kGemvThreads), glds, st, m->dev, m->S,
                               static_cast<const uint4*>(blocks), meta, rows, gpr, rb_per_wg, batch, x, y);
    }
    ECCO_HIP_CHECK(hipGetLastError());
    return ECCO_OK;
}

int ecco_kv_attend_gqa_splits(int device, int B, int Hkv, int tokens) {
    if (B <= 0 || Hkv <= 0 || tokens <= 0) return ECCO_ESHAPE;
    const long long heads = (long long)B * Hkv;
    const long long by_units = std::max<long long>(1, cu_count(device) / heads);  // a workgroup for every compute unit
    const long long by_tokens = ((long long)tokens + 255) / 256;                  // but at least 256 tokens per split
    return (int)std::min<long long>(std::min(by_units, by_tokens), 256);
}

size_t ecco_kv_attend_gqa_workspace(int B, int Hq, int n_splits) {
    if (B <= 0 || Hq <= 0 || n_splits <= 1) return 0;
    return (size_t)B * Hq * n_splits * (kGroup + 2) * sizeof(float);
}

// argument checks shared by the two grouped-query entry points (everything but the workspace)
static int gqa_check(const ecco_model* mk, const ecco_model* mv, const uint16_t* q,
                     const void* k_blocks, const uint32_t* k_meta, const void* v_blocks, const uint32_t* v_meta,
                     const int32_t* seq_len, int B, int Hq, int Hkv, int T_max, int n_splits, const float* out) {
    if (!mk || !mv || !q || !k_blocks || !k_meta || !v_blocks || !v_meta || !seq_len || !out) return ECCO_EINVAL;
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || T_max <= 0 || Hq % Hkv != 0 || Hq / Hkv > kGqaMaxGroup) return ECCO_ESHAPE;
    if (n_splits < 1 || n_splits > 256 || (long long)B * Hkv > 0x7FFFFFFF || (long long)B * Hq > 0x7FFFFFFF) return ECCO_ESHAPE;
    return ECCO_OK;
}

// the two launches: the attention kernel over (sequence, key/value head, split), then the merge of the splits
static int gqa_launch(const ecco_model* mk, const ecco_model* mv, const uint16_t* q,
                      const void* k_blocks, const uint32_t* k_meta, const void* v_blocks, const uint32_t* v_meta,
                      const int32_t* seq_len, int B, int Hq, int Hkv, int T_max, int n_splits, float* workspace,
                      float* out, void* stream) {
    const bool lk = mk->max_len > kPeekBits, lv = mv->max_len > kPeekBits;
    const int units = ((T_max - 1) / kUnitBlocks + n_splits) / n_splits;  // of a range: ceil(ceil(T_max / 32) / n_splits)
    const GqaPlan plan = gqa_plan(mk->S, lk, mv->S, lv, Hq / Hkv, (size_t)B * Hkv * n_splits, units, cu_count(mk->device));
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int dev_id = mk->device;
    auto launch = [&](auto kernel) -> int {
        int rc = allow_lds(kernel, dev_id, plan.lds);
        if (rc != ECCO_OK) return rc;
        hipLaunchKernelGGL(kernel, dim3(B * Hkv, n_splits), dim3(plan.waves * 64), plan.lds, st,
                           GqaArgs{mk->dev, mv->dev, q, static_cast<const uint4*>(k_blocks), k_meta, static_cast<const uint4*>(v_blocks), v_meta, seq_len,
                                   out, workspace, mk->S, mv->S, B, Hq, Hkv, T_max, plan.table_words, plan.both, plan.span, plan.step});
        ECCO_HIP_CHECK(hipGetLastError());
        return ECCO_OK;
    };
    const auto pick = [&](auto wide) -> int {
        constexpr bool kWide = decltype(wide)::value;
        if (lk) return lv ? launch(kv_attend_gqa_kernel<true, true, kWide, 12>) : launch(kv_attend_gqa_kernel<true, false, kWide, 12>);
        if (lv) return launch(kv_attend_gqa_kernel<false, true, kWide, 12>);
        return plan.waves == 8 ? launch(kv_attend_gqa_kernel<false, false, kWide, 8>) : launch(kv_attend_gqa_kernel<false, false, kWide, 12>);
    };
    const int rc = Hq / Hkv > 8 ? pick(std::true_type{}) : pick(std::false_type{});
    if (rc != ECCO_OK || n_splits == 1) return rc;
    hipLaunchKernelGGL(kv_attend_combine_kernel, dim3(B * Hq), dim3(kGroup), 0, st, workspace, B * Hq, n_splits, out);
    ECCO_HIP_CHECK(hipGetLastError());
    return ECCO_OK;
}

int ecco_kv_attend_gqa(const ecco_model* mk, const ecco_model* mv, const uint16_t* q,
                       const void* k_blocks, const uint32_t* k_meta, const void* v_blocks, const uint32_t* v_meta,
                       const int32_t* seq_len, int B, int Hq, int Hkv, int T_max, int n_splits, void* workspace,
                       float* out, void* stream) {
    const int rc = gqa_check(mk, mv, q, k_blocks, k_meta, v_blocks, v_meta, seq_len, B, Hq, Hkv, T_max, n_splits, out);
    if (rc != ECCO_OK) return rc;
    if (n_splits > 1 && !workspace) return ECCO_EINVAL;
    if (!aligned(k_blocks, 64) || !aligned(v_blocks, 64) || !aligned(q, 16) || !aligned(out, 4) || !aligned(workspace, 16)) return ECCO_EALIGN;
    if (model_ready(mk) != ECCO_OK || model_ready(mv) != ECCO_OK || mk->device != mv->device) return ECCO_EINVAL;
    return gqa_launch(mk, mv, q, k_blocks, k_meta, v_blocks, v_meta, seq_len, B, Hq, Hkv, T_max, n_splits,
                      static_cast<float*>(workspace), out, stream);
}

int ecco_kv_attend_gqa_noalloc(const ecco_model* mk, const ecco_model* mv, const uint16_t* q,
                               const void* k_blocks, const uint32_t* k_meta, const void* v_blocks, const uint32_t* v_meta,
                               const int32_t* seq_len, int B, int Hq, int Hkv, int T_max, int n_splits,
                               float* out, void* stream) {
    const int rc = gqa_check(mk, mv, q, k_blocks, k_meta, v_blocks, v_meta, seq_len, B, Hq, Hkv, T_max, n_splits, out);
    if (rc != ECCO_OK) return rc;
    // the partial results of the splits must fit the static array
    if (n_splits > 1 && ecco_kv_attend_gqa_workspace(B, Hq, n_splits) > (size_t)ECCO_GQA_SCRATCH_BYTES) return ECCO_ESHAPE;
    if (!aligned(k_blocks, 64) || !aligned(v_blocks, 64) || !aligned(q, 16) || !aligned(out, 4)) return ECCO_EALIGN;
    if (model_ready(mk) != ECCO_OK || model_ready(mv) != ECCO_OK || mk->device != mv->device) return ECCO_EINVAL;
    float* ws = nullptr;
    if (n_splits > 1) {
        // this device's copy of the array: asked for when the model was uploaded; looked up here otherwise, which
        // needs the model's device to be the current one
        {
            std::lock_guard<std::mutex> hold(scratch_lock);
            ws = mk->device < kMaxDevices ? scratch_ptr[mk->device] : nullptr;
        }
        if (!ws) {
            int cur = -1;
            if (hipGetDevice(&cur) != hipSuccess || cur != mk->device) return ECCO_EINVAL;
            ws = scratch_on_current_device(cur);
            if (!ws) return ECCO_EHIP;
        }
    }
    return gqa_launch(mk, mv, q, k_blocks, k_meta, v_blocks, v_meta, seq_len, B, Hq, Hkv, T_max, n_splits, ws, out, stream);
}

int ecco_kv_attend(const ecco_model* mk, const ecco_model* mv, const uint16_t* q,
                   const void* k_blocks, const uint32_t* k_meta, const void* v_blocks, const uint32_t* v_meta,
                   const int32_t* seq_len, int B, int H, int T_max, float* out, void* stream) {
    if (!mk || !mv || !q || !k_blocks || !k_meta || !v_blocks || !v_meta || !seq_len || !out) return ECCO_EINVAL;
    if (B <= 0 || H <= 0 || T_max <= 0 || (long long)B * H > 0x7FFFFFFF) return ECCO_ESHAPE;
    if (!aligned(k_blocks, 64) || !aligned(v_blocks, 64) || !aligned(q, 16) || !aligned(out, 4)) return ECCO_EALIGN;
    if (model_ready(mk) != ECCO_OK || model_ready(mv) != ECCO_OK || mk->device != mv->device) return ECCO_EINVAL;
    const bool lk = mk->max_len > kPeekBits, lv = mv->max_len > kPeekBits;
    const int dev_id = mk->device;
    const AttnPlan plan = attn_plan(mk->S, lk, mv->S, lv, (size_t)B * H, T_max, cu_count(dev_id));
    auto launch = [&](auto kernel) -> int {
        int rc = allow_lds(kernel, dev_id, plan.lds);
        if (rc != ECCO_OK) return rc;
        hipLaunchKernelGGL(kernel, dim3(B * H), dim3(plan.waves * 64), plan.lds, static_cast<hipStream_t>(stream), mk->dev, mk->S, mv->dev,
                           mv->S, q, static_cast<const uint4*>(k_blocks), k_meta, static_cast<const uint4*>(v_blocks), v_meta,
                           seq_len, H, T_max, plan.table_words, plan.both, plan.span, out);
        ECCO_HIP_CHECK(hipGetLastError());
        return ECCO_OK;
    };
    if (lk) return lv ? launch(kv_attend_kernel<true, true, 12>) : launch(kv_attend_kernel<true, false, 12>);
    if (lv) return launch(kv_attend_kernel<false, true, 12>);
    return plan.waves == 8 ? launch(kv_attend_kernel<false, false, 8>) : plan.waves == 12 ? launch(kv_attend_kernel<false, false, 12>) : launch(kv_attend_kernel<false, false, 16>);
}

}  // extern "C"
