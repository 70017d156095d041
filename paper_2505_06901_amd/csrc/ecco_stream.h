// Outputs that are written through, and outputs and inputs that pass the caches by (non-temporal accesses), for gfx950, by sizes.
//
// What a kernel stores the ordinary way stays in the L2 (4 MB for each of eight dies) and is written back when the kernel ends; the last-level
// cache (256 MB) then holds it for a reader.  Whole lines that are stored once can be written through as they are produced (a store of
// device scope): the kernel does not end with the write-back, and the reader finds them where it did before.  Past the caches the kernel is done sooner
// still, but a reader finds its lines in memory: that is for outputs that the last-level cache would not hold anyway.  The lines are drawn
// where the kernel and what reads its output behind it take no longer together than with ordinary stores (where one such reader loses, it
// is said).  All times in us, graphs of several launches, each replayed once untimed: a graph that follows another writes back what that
// one has left dirty.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace ecco_stream {

constexpr size_t kMiB = (size_t)1 << 20;
// Outputs of the decoders may begin in the middle of a 128-byte line; a store of part of a line is better left to the cache.
inline bool whole_lines(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 127u) == 0; }

enum class Stores { kCached, kThrough, kPast };

// Decoder of two-chain blocks: written through from 4 to 96 MiB of FP16.  Ordinary -> through, into one buffer used again and again, alone / with a
// plain reader / with products of 16 and 512 rows behind it: 32768 groups 7.6 -> 6.9 / 13.2 -> 12.6 / 18.0 -> 17.2, 25.4 -> 24.7; 131072 13.1 -> 11.6
// / 28.9 -> 28.0 / 26.7 -> 25.6, 41.3 -> 40.3; 352256 23.4 -> 22.3 / 38.6 -> 37.8 / 40.9 -> 40.1, 76.3 -> 75.4; not taken: 4096 5.7 -> 5.7, 524288
// 42.0 -> 43.2 / 63.9 -> 64.8 / 64.8 -> 65.7, 103 -> 103.  Past the caches every product loses up to 256 MiB (352256 25.9 / 40.7 / 46.0, 81.2), and
// beyond, a step of other kernels between two decodings (0.436 -> 0.450 ms for 448 MiB).
inline Stores weights(const void* to, size_t bytes) { return whole_lines(to) && bytes >= 4 * kMiB && bytes <= 96 * kMiB ? Stores::kThrough : Stores::kCached; }

// Decoder of self-contained blocks: written through below 400 MiB, past the caches from there on.  Ordinary -> through, as above: 4096 groups 9.7 ->
// 9.8, 32768 11.8 -> 10.8 / 17.2 -> 16.1 / 22.0 -> 20.5, 30.6 -> 29.1; 131072 18.2 -> 15.5 / 30.3 -> 30.2 / 31.3 -> 30.2, 46.5 -> 44.8; 352256 38.0
// -> 34.5 / 54.8 -> 51.3 / 55.4 -> 53.6, 87.8 -> 85.4; 1048576 96.6 -> 91.6 / 141 -> 137 / 159 -> 156, 221 -> 219.  Ordinary -> past: 1835008 157 ->
// 144 / 276 -> 235 / 288 -> 269, 368 -> 349, but 131072 18.2 -> 16.4 / 30.3 -> 30.6 / 31.3 -> 34.1, 46.5 -> 48.5.
inline Stores self_contained(const void* to, size_t bytes) {
    return !whole_lines(to) || bytes < 4 * kMiB ? Stores::kCached : bytes < 400 * kMiB ? Stores::kThrough : Stores::kPast;
}

// Activation decoder and the FP16 input of the activation encoder: past the caches from 192 MiB on.  Together they are what the last-level cache
// would hold little of, and the blocks stay in it.  Ordinary -> past, over several buffers (in brackets into one), decoder with a product of 256
// columns behind it / encoder and decoder / with a product behind / with a writer in front and a plain reader behind: 1572864 groups 133 -> 123 (127
// -> 116) / 129 -> 99 / 198 -> 172 / 215 -> 206; 2097152 158 -> 154 (160 -> 143) / 156 -> 132 / 237 -> 224 / 286 -> 278; encoder alone 59 -> 56, 78
// -> 72, 176 -> 160 for 4194304.  A program that only decodes and reads once over loses: 87 -> 89 (81 -> 88), 115 -> 118 (113 -> 114).  Not taken:
// 1048576 100 -> 88 (79 -> 88) / 78 -> 69 / 139 -> 122 / 147 -> 138, reader 59 -> 60 (56 -> 59); 700000 64 -> 72 (62 -> 71) / 49 -> 48 / 85 -> 96 /
// 98 -> 97; 262144 30 -> 34 (34 -> 39) / 23 -> 21 / 40 -> 43 / 38 -> 38.  Written through as the weights are, readers of up to 64 MiB lose 5 to 16 %
// where one buffer is used again and again, and nothing gains more than 5 %.
inline bool activations(const void* to, size_t bytes) { return bytes >= 192 * kMiB && whole_lines(to); }
constexpr bool encoder_input(size_t bytes) { return bytes >= 192 * kMiB; }

// Blocks of the min/max encoder: from 8 to 16 MiB.  Alone / with a plain reader / with the decoder behind it, 16 patterns: 131072 groups 18.5 -> 18.1
// / 21.0 -> 20.6 / 30.6 -> 30.2, 262144 32.6 -> 31.7 / 34.9 -> 35.1 / 50.7 -> 50.2; not taken: 65536 11.3 -> 10.9 / 13.4 -> 13.4 / 19.2 -> 19.4,
// 524288 60.5 -> 60.9 / 63.7 -> 63.8 / 91.0 -> 97.0.  The full search gains 1 % and goes without.
constexpr bool encoded(size_t bytes) { return bytes >= 8 * kMiB && bytes <= 16 * kMiB; }

typedef uint32_t word4_t __attribute__((ext_vector_type(4)));

// to[0] = v, sixteen bytes, past the caches if kStream
template <bool kStream>
__device__ __forceinline__ void store(uint4* to, uint4 v) {
    if constexpr (kStream) __builtin_nontemporal_store(word4_t{v.x, v.y, v.z, v.w}, reinterpret_cast<word4_t*>(to));
    else *to = v;
}
// Sixteen bytes at byte `at` of the `bytes` behind `base` (both the same for the wavefront's lanes) that are written through to memory; nothing is
// stored beyond them.  The descriptor's last word says raw 32-bit elements, the operand 16 device scope (sc1).
__device__ __forceinline__ void store_through(void* base, uint32_t bytes, uint32_t at, uint4 v) {
    const auto r = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(word4_t{v.x, v.y, v.z, v.w}, r, (int)at, 0, 16);
}
template <bool kStream>
__device__ __forceinline__ void store(uint32_t* to, uint32_t v) {
    if constexpr (kStream) __builtin_nontemporal_store(v, to);
    else *to = v;
}
template <bool kStream>
__device__ __forceinline__ uint4 load(const uint4* from) {
    if constexpr (!kStream) return *from;
    const word4_t v = __builtin_nontemporal_load(reinterpret_cast<const word4_t*>(from));
    return make_uint4(v.x, v.y, v.z, v.w);
}

}  // namespace ecco_stream
