// Decoder of the self-contained 4x block (include/ecco_paper_block.h) for gfx950.
//
// Decoder: the block has one code stream of 128 values behind a variable-length header, so a lane owns a whole
// block: 64 blocks (4 KB) per wavefront pass, loaded with 16-byte pieces on consecutive addresses into a private
// LDS buffer (17-word slots) one pass ahead, decoded in lockstep (value i of 64 blocks at a time) with an 8-bit
// peek into a byte table per (pattern, codebook) -- 4 x S tables of 256 bytes, 64 KB for S = 64 -- and a second
// small table for the centroid.  Values past the cut (code ends beyond bit 512) become zeros; the lane keeps
// counting bits, so the test stays true once it fails.  Decoded values leave through a private LDS image, 32 per
// lane at a time, as 64-byte pieces (four lanes per block).  The padded entries are only known when the stream
// has been walked to its end: the lane then overwrites those positions in global memory, after the wavefront's
// earlier stores have completed.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "ecco_pb_launch.h"

namespace {

using namespace ecco_pb;

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int kSlot = kBlockWords + 1;    // LDS words per staged block; the last one is a zero pad
constexpr int kUnit = 64;                 // blocks per wavefront pass, one per lane
constexpr int kPayWords = kUnit * kSlot + 4;
constexpr int kPassValues = 32;           // values per lane between two write-outs
constexpr int kImgWords = 32 * 32;        // the write-out image: 32 lines of 128 bytes
// the header takes at most 18 bits and a code at most 8: value i ends at or before bit 18 + 8 (i + 1), inside the block for i <= 60
constexpr int kAlwaysPresent = (kBlockBits - 18) / kMaxLen;
constexpr int kDecThreads = 512;
constexpr int kDecWaves = kDecThreads / 64;

__device__ inline void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline void stage_words(uint32_t* dst, const uint32_t* __restrict__ src, int words) {  // words % 4 == 0, 16-byte aligned
    const uint4* s = reinterpret_cast<const uint4*>(src);
    uint4* d = reinterpret_cast<uint4*>(dst);
    for (int i = threadIdx.x; i < (words >> 2); i += blockDim.x) d[i] = s[i];
}

inline size_t dec_lds_bytes(int S) { return (DevLayout{S}.decode_words() + (size_t)kDecWaves * (kPayWords + kImgWords)) * 4; }

struct PieceLoad {
    uint4 v[4];
};
__device__ __forceinline__ PieceLoad load_pieces(const uint4* __restrict__ blocks, size_t g0, size_t n_groups, int lane) {
    PieceLoad L;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int q = lane + 64 * r;  // piece q of the pass: block q / 4, part q % 4
        const size_t g = min(g0 + (size_t)(q >> 2), n_groups - 1);
        L.v[r] = blocks[g * 4 + (q & 3)];
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

__global__ __launch_bounds__(kDecThreads) void pb_decode_kernel(const uint32_t* __restrict__ dev, int S,
                                                               const uint4* __restrict__ blocks, size_t n_groups,
                                                               uint16_t* __restrict__ dst) {
    extern __shared__ __align__(16) uint32_t smem[];
    const DevLayout D{S};
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint8_t* lut = reinterpret_cast<const uint8_t*>(smem + D.lut());
    const uint16_t* kplut = reinterpret_cast<const uint16_t*>(smem + D.kplut());
    const uint16_t* cent = reinterpret_cast<const uint16_t*>(smem + D.cent());
    const uint16_t* fp8 = reinterpret_cast<const uint16_t*>(smem + D.fp8());
    uint32_t* pay = smem + D.decode_words() + wave * (kPayWords + kImgWords);
    uint32_t* img = pay + kPayWords;

    const size_t n_units = (n_groups + kUnit - 1) / kUnit;
    const size_t first = (size_t)blockIdx.x * kDecWaves + wave, step = (size_t)gridDim.x * kDecWaves;
    PieceLoad pre;
    if (first < n_units) pre = load_pieces(blocks, first * kUnit, n_groups, lane);
    stage_words(smem, dev, (int)D.decode_words());
    pay[lane * kSlot + kBlockWords] = 0u;
    if (lane < 4) pay[kUnit * kSlot + lane] = 0u;
    __syncthreads();

    for (size_t u = first; u < n_units; u += step) {
        const size_t g0 = u * kUnit;
        wave_lds_fence();
        store_pieces(pay, pre, lane);
        wave_lds_fence();
        if (u + step < n_units) pre = load_pieces(blocks, (u + step) * kUnit, n_groups, lane);
        const uint32_t* w = pay + lane * kSlot;
        const uint32_t w0 = w[0];
        const uint32_t kpe = kplut[(w0 >> 14) & 0xFFu];
        const uint32_t p = kpe >> 8;
        const uint32_t sv = fp8[w0 >> 24];                 // the signed scale, FP16 bits
        const __half sabs = __ushort_as_half((unsigned short)(sv & 0x7FFFu));
        const uint8_t* tab = lut + (p * kBooks + ((w0 >> 22) & 3u)) * 256u;
        const uint16_t* cp = cent + p * 16u;
        uint32_t fetch = 10u + (kpe & 0xFFu);              // where the next run is fetched from; stops at 512
        uint32_t reach = fetch;                             // where the codes read so far end; keeps counting past 512
#pragma unroll 1
        for (int pp = 0; pp < kGroup / (2 * kPassValues); ++pp) {
            // 64 values per lane = one 128-byte line of output, kept in registers until the line is complete: a store
            // instruction that leaves half a line for later costs a second write of that line
            uint32_t packed[kPassValues];
#pragma unroll
            for (int i0 = 0; i0 < 2 * kPassValues; i0 += 4) {
                const uint32_t wi = fetch >> 5;
                uint64_t win = (((uint64_t)w[wi] << 32) | (uint64_t)w[wi + 1]) << (fetch & 31u);
                uint32_t used = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t e = tab[(uint32_t)(win >> 56)];
                    const uint32_t len = e & 15u;
                    reach += len;
                    used += len;
                    win <<= len;
                    const __half prod = __hmul(__ushort_as_half(cp[e >> 4]), sabs);   // one rounding: fp16(c * |s|)
                    uint32_t val = e >= 0xF0u ? sv : (uint32_t)__half_as_ushort(prod);
                    val = reach <= (uint32_t)kBlockBits ? val : 0u;                     // a code that ends beyond the block is absent
                    const int i = i0 + j;
                    if (i & 1) packed[i >> 1] |= val << 16; else packed[i >> 1] = val;
                }
                fetch = min(fetch + used, (uint32_t)kBlockBits);
            }
            // write-out: the lines of lanes 0..31, then of lanes 32..63, through the image (32 rows of eight 16-byte
            // pieces, piece k of row r at column k ^ (r & 7)); every store instruction carries whole lines, 8 lanes each
            uint4* image = reinterpret_cast<uint4*>(img);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                wave_lds_fence();
                if ((lane >> 5) == h) {
                    const int row = lane & 31;
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        image[row * 8 + (k ^ (row & 7))] = make_uint4(packed[4 * k], packed[4 * k + 1], packed[4 * k + 2], packed[4 * k + 3]);
                }
                wave_lds_fence();
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = (lane >> 3) + 8 * r, part = lane & 7;
                    const uint4 v = image[row * 8 + (part ^ (row & 7))];
                    const size_t b = g0 + 32 * h + row;
                    if (b < n_groups) reinterpret_cast<uint4*>(dst)[b * 16 + pp * 8 + part] = v;
                }
            }
        }
        // padded entries: only if all 128 values were present
        if (reach <= (uint32_t)kBlockBits && g0 + lane < n_groups) {
            const uint32_t n_out = ((uint32_t)kBlockBits - reach) / kOutlierBits;
            if (__builtin_amdgcn_ballot_w64(n_out > 0) != 0ull) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores above have landed
            for (uint32_t j = 0; j < n_out; ++j) {
                const uint32_t at = reach + j * kOutlierBits, wi = at >> 5;
                const uint64_t win = (((uint64_t)w[wi] << 32) | (uint64_t)w[wi + 1]) << (at & 31u);
                const uint32_t entry = (uint32_t)(win >> 49);   // 7-bit position, 8-bit float
                dst[(g0 + lane) * kGroup + (entry >> 8)] = fp8[entry & 0xFFu];
            }
        }
    }
}

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kCtrl, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }
// an associative, commutative, exact operation over the 64 lanes (cross-lane moves inside rows of 16, then the four
// row results through scalar registers); every lane returns the result
template <class Op>
__device__ __forceinline__ uint32_t wave_all_u32(uint32_t t, Op op) {
    t = op(t, dpp_u32<0xB1>(t));   // quad_perm [1,0,3,2]
    t = op(t, dpp_u32<0x4E>(t));   // quad_perm [2,3,0,1]
    t = op(t, dpp_u32<0x141>(t));  // row_half_mirror
    t = op(t, dpp_u32<0x140>(t));  // row_mirror
    return op(op(lane_u32(t, 0), lane_u32(t, 16)), op(lane_u32(t, 32), lane_u32(t, 48)));
}
// FP32 sum in the balanced tree: aligned blocks of 2, 4, 8, 16 lanes, then (row 0 + row 1) + (row 2 + row 3)
__device__ __forceinline__ float wave_tree_sum(float t) {
    const auto f = [](float v) { return __builtin_bit_cast(uint32_t, v); };
    const auto g = [](uint32_t v) { return __builtin_bit_cast(float, v); };
    t = __fadd_rn(t, g(dpp_u32<0xB1>(f(t))));
    t = __fadd_rn(t, g(dpp_u32<0x4E>(f(t))));
    t = __fadd_rn(t, g(dpp_u32<0x141>(f(t))));
    t = __fadd_rn(t, g(dpp_u32<0x140>(f(t))));
    return __fadd_rn(__fadd_rn(g(lane_u32(f(t), 0)), g(lane_u32(f(t), 16))), __fadd_rn(g(lane_u32(f(t), 32)), g(lane_u32(f(t), 48))));
}

// ---- decode fused into the matrix-vector product --------------------------------------------------------------------
// y = W x without writing W: a workgroup owns a band of rows (its blocks are consecutive in memory); a wavefront
// takes 64 consecutive blocks of the band at a time, one per lane, exactly as the decoder does.  The lane keeps the
// 128 activations of its block's column group in 64 registers and adds centroid * x for every value that is present
// (index 15 counts as +-1); the sum is multiplied by |scale| at the end.  The 128 indices are kept as nibbles in 16
// registers: when padded entries follow, the lane takes back centroid * x at their positions and adds the entries'
// own values (times x) instead -- from the last entry to the first, each position once, which is what a sequential
// reader of the block ends up with.  Per-block sums go to LDS, and each row's blocks are added in a fixed tree.
constexpr int kGvThreads = 512;
constexpr int kGvWaves = kGvThreads / 64;
constexpr int kGvPartFloats = 2048;      // per-block sums of a band: band rows x column groups
constexpr int kGvXMaxCols = 8192;        // activations are staged in LDS up to this many columns, read through L2 beyond
constexpr int kNibStride = 17;           // words per lane of the index store (16 + 1)

inline size_t gv_lds_bytes(int S, int cols) {
    return (DevLayout{S}.decode_words() + (size_t)kGvWaves * (kPayWords + 64 * kNibStride) + kGvPartFloats +
            (cols <= kGvXMaxCols ? cols / 2 : 0)) * 4;
}

template <bool kXLds>
__global__ __launch_bounds__(kGvThreads) void pb_gemv_kernel(const uint32_t* __restrict__ dev, int S,
                                                             const uint4* __restrict__ blocks, int rows, int gpr, int band,
                                                             const uint4* __restrict__ x, float* __restrict__ y) {
    extern __shared__ __align__(16) uint32_t smem[];
    const DevLayout D{S};
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint8_t* lut = reinterpret_cast<const uint8_t*>(smem + D.lut());
    const uint16_t* kplut = reinterpret_cast<const uint16_t*>(smem + D.kplut());
    const uint16_t* cent = reinterpret_cast<const uint16_t*>(smem + D.cent());
    const uint16_t* fp8 = reinterpret_cast<const uint16_t*>(smem + D.fp8());
    uint32_t* pay = smem + D.decode_words() + wave * (kPayWords + 64 * kNibStride);
    uint32_t* nibs = pay + kPayWords + lane * kNibStride;
    float* part = reinterpret_cast<float*>(smem + D.decode_words() + kGvWaves * (kPayWords + 64 * kNibStride));
    uint32_t* xl = reinterpret_cast<uint32_t*>(part + kGvPartFloats);

    const int r0 = blockIdx.x * band, nrows = min(band, rows - r0);
    const size_t base = (size_t)r0 * gpr;                 // first block of the band
    const int n_blocks = nrows * gpr;                     // <= kGvPartFloats
    const int n_units = (n_blocks + kUnit - 1) / kUnit;
    PieceLoad pre;
    if (wave < n_units) pre = load_pieces(blocks + base * 4, (size_t)wave * kUnit, (size_t)n_blocks, lane);
    stage_words(smem, dev, (int)D.decode_words());
    if (kXLds)
        for (int i = threadIdx.x; i < gpr * 16; i += kGvThreads) reinterpret_cast<uint4*>(xl)[i] = x[i];
    pay[lane * kSlot + kBlockWords] = 0u;
    if (lane < 4) pay[kUnit * kSlot + lane] = 0u;
    __syncthreads();

    for (int u = wave; u < n_units; u += kGvWaves) {
        wave_lds_fence();
        store_pieces(pay, pre, lane);
        wave_lds_fence();
        if (u + kGvWaves < n_units) pre = load_pieces(blocks + base * 4, (size_t)(u + kGvWaves) * kUnit, (size_t)n_blocks, lane);
        const int bl = u * kUnit + lane;                  // block of the band; slots past the band hold a copy of its last block
        const int cg = min(bl, n_blocks - 1) % gpr;       // its column group
        const uint4* xsrc = kXLds ? reinterpret_cast<const uint4*>(xl) + cg * 16 : x + (size_t)cg * 16;
        uint32_t xs[kGroup / 4];  // the activations of half a column group at a time
        const uint32_t* w = pay + lane * kSlot;
        const uint32_t w0 = w[0];
        const uint32_t kpe = kplut[(w0 >> 14) & 0xFFu];
        const uint32_t p = kpe >> 8;
        const uint32_t sv = fp8[w0 >> 24];
        const uint8_t* tab = lut + (p * kBooks + ((w0 >> 22) & 3u)) * 256u;
        const uint16_t* cp = cent + p * 16u;
        uint32_t fetch = 10u + (kpe & 0xFFu), reach = fetch;
        float acc = 0.0f;
        uint32_t nib[kGroup / 8];
#pragma unroll
        for (int i0 = 0; i0 < kGroup; i0 += 4) {
            if ((i0 & 63) == 0) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint4 v = xsrc[(i0 >> 6) * 8 + k];
                    xs[4 * k] = v.x; xs[4 * k + 1] = v.y; xs[4 * k + 2] = v.z; xs[4 * k + 3] = v.w;
                }
            }
            const uint32_t wi = fetch >> 5;
            uint64_t win = (((uint64_t)w[wi] << 32) | (uint64_t)w[wi + 1]) << (fetch & 31u);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = i0 + j;
                const uint32_t e = tab[(uint32_t)(win >> 56)];
                const uint32_t len = e & 15u, idx = e >> 4;
                reach += len;
                win <<= len;
                // FP16 operands go straight into mixed-precision multiply-adds: the activations stay packed in their
                // registers (converted ahead of time they would need 128)
                const half2_t x2 = __builtin_bit_cast(half2_t, xs[(i & 63) >> 1]);
                const _Float16 xh = (i & 1) ? x2[1] : x2[0];
                uint32_t cb = cp[idx], keep = idx;
                if (i >= kAlwaysPresent) {  // only these values can lie beyond the cut: they then count as zero and as index 0
                    const bool present = reach <= (uint32_t)kBlockBits;
                    cb = present ? cb : 0u;
                    keep = present ? idx : 0u;
                }
                acc = fmaf((float)__builtin_bit_cast(_Float16, (unsigned short)cb), (float)xh, acc);
                nib[i >> 3] = (i & 7) ? ((nib[i >> 3] << 4) | keep) : keep;
                if ((i & 3) == 3) asm volatile("" : "+v"(acc), "+v"(nib[i >> 3]), "+v"(xs[(i & 63) >> 1]));  // keeps the arithmetic next to its table reads
            }
            fetch = min(reach, (uint32_t)kBlockBits);
        }
        const uint16_t* xh16 = kXLds ? reinterpret_cast<const uint16_t*>(xl) + cg * kGroup : reinterpret_cast<const uint16_t*>(x) + (size_t)cg * kGroup;
        if (sv & 0x8000u) {
            // index 15 was added as +1 times its activation; the scale is negative, so it is -1: find the positions with
            // index 15 (all four bits of the nibble set; an absent value was recorded as index 0, unless it really is
            // index 0 ... which is not 15 either) and take twice their activations back
#pragma unroll
            for (int k = 0; k < kGroup / 8; ++k) {
                uint32_t hit = nib[k] & (nib[k] >> 1) & (nib[k] >> 2) & (nib[k] >> 3) & 0x11111111u;
                while (hit) {
                    const uint32_t b = 31u - (uint32_t)__builtin_clz(hit);   // bit 4 * (7 - position in the register)
                    hit &= ~(1u << b);
                    const uint32_t pos = 8u * k + (7u - (b >> 2));
                    acc = fmaf(-2.0f, __half2float(__ushort_as_half(xh16[pos])), acc);
                }
            }
        }
        float extra = 0.0f;  // padded entries: absolute values, not multiples of the scale
        const uint32_t n_out = reach <= (uint32_t)kBlockBits ? ((uint32_t)kBlockBits - reach) / kOutlierBits : 0u;
        if (__builtin_amdgcn_ballot_w64(n_out > 0u) != 0ull) {
#pragma unroll
            for (int k = 0; k < kGroup / 8; ++k) nibs[k] = nib[k];
            const uint16_t* xh = xh16;
            uint64_t seen_lo = 0, seen_hi = 0;
            for (int j = (int)n_out - 1; j >= 0; --j) {
                const uint32_t at = reach + (uint32_t)j * kOutlierBits, wi = at >> 5;
                const uint64_t win = (((uint64_t)w[wi] << 32) | (uint64_t)w[wi + 1]) << (at & 31u);
                const uint32_t entry = (uint32_t)(win >> 49), pos = entry >> 8;
                const uint64_t bit = 1ull << (pos & 63u);
                const bool dup = ((pos < 64u ? seen_lo : seen_hi) & bit) != 0ull;
                if (pos < 64u) seen_lo |= bit; else seen_hi |= bit;
                if (dup) continue;  // a later entry for this position has been applied already
                const uint32_t idx = (nibs[pos >> 3] >> (4u * (7u - (pos & 7u)))) & 15u;
                const float xi = __half2float(__ushort_as_half(xh[pos]));
                float c = __half2float(__ushort_as_half(cp[idx]));
                if (idx == 15u && (sv & 0x8000u)) c = -c;
                acc = fmaf(-c, xi, acc);
                extra = fmaf(__half2float(__ushort_as_half(fp8[entry & 0xFFu])), xi, extra);
            }
        }
        if (bl < n_blocks) part[bl] = fmaf(acc, __half2float(__ushort_as_half((unsigned short)(sv & 0x7FFFu))), extra);
    }
    __syncthreads();
    // row sums: the blocks of a row in a fixed order (lane-strided partial sums, then the wavefront tree)
    for (int r = wave; r < nrows; r += kGvWaves) {
        float sum = 0.0f;
        for (int c = lane; c < gpr; c += 64) sum += part[r * gpr + c];
        sum = wave_tree_sum(sum);
        if (lane == 0) y[r0 + r] = sum;
    }
}

}  // namespace

extern "C" {

int ecco_pb_decode_gemv(const ecco_pb_model* m, const void* blocks, int rows, int cols, const uint16_t* x, float* y, void* stream) {
    if (!m || !blocks || !x || !y) return ECCO_EINVAL;
    if (rows <= 0 || cols <= 0 || cols % kGroup != 0 || cols > 65536) return ECCO_ESHAPE;
    if (!aligned(blocks, 64) || !aligned(x, 16) || !aligned(y, 4)) return ECCO_EALIGN;
    if (model_ready(m) != ECCO_OK) return ECCO_EINVAL;
    const int gpr = cols / kGroup;
    // a band of rows per workgroup: about one band per compute unit, at most kGvPartFloats blocks
    int band = std::max(1, (rows + 255) / 256);
    band = std::min(band, std::max(1, kGvPartFloats / gpr));
    const int grid = (rows + band - 1) / band;
    const size_t lds = gv_lds_bytes(m->S, cols);
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto launch = [&](auto kernel) -> int {
        const int rc = ecco::allow_lds(kernel, m->device, lds);
        if (rc != ECCO_OK) return rc;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kGvThreads), lds, st, m->dev, m->S, static_cast<const uint4*>(blocks), rows, gpr, band,
                           reinterpret_cast<const uint4*>(x), y);
        ECCO_HIP_CHECK(hipGetLastError());
        return ECCO_OK;
    };
    return cols <= kGvXMaxCols ? launch(pb_gemv_kernel<true>) : launch(pb_gemv_kernel<false>);
}

int ecco_pb_decode(const ecco_pb_model* m, const void* blocks, size_t n_groups, uint16_t* dst, void* stream) {
    if (!m) return ECCO_EINVAL;
    if (n_groups == 0) return model_ready(m);
    if (!blocks || !dst) return ECCO_EINVAL;
    if (n_groups >= ((size_t)1 << 31)) return ECCO_ESHAPE;
    if (!aligned(blocks, 64) || !aligned(dst, 16)) return ECCO_EALIGN;
    if (model_ready(m) != ECCO_OK) return ECCO_EINVAL;
    const size_t lds = dec_lds_bytes(m->S);
    const int rc = ecco::allow_lds(pb_decode_kernel, m->device, lds);
    if (rc != ECCO_OK) return rc;
    const size_t units = (n_groups + kUnit - 1) / kUnit;
    const int grid = (int)std::min<size_t>((units + kDecWaves - 1) / kDecWaves, 1024);
    hipLaunchKernelGGL(pb_decode_kernel, dim3(grid), dim3(kDecThreads), lds, static_cast<hipStream_t>(stream), m->dev, m->S,
                       static_cast<const uint4*>(blocks), n_groups, dst);
    ECCO_HIP_CHECK(hipGetLastError());
    return ECCO_OK;
}

}  // extern "C"
