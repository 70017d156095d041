// Outputs and inputs that pass the caches by (non-temporal accesses), for gfx950, and from which size on.
//
// What a kernel stores the ordinary way stays in the L2 (4 MB for each of eight dies) and is written back when the kernel ends, and it takes the
// place of other data in the last-level cache (256 MB).  Whole lines that are stored once can go to memory as they are produced, and the
// kernel is done sooner; but a reader that follows then finds them in memory instead of a cache.  So the lines are drawn where the
// kernel and what reads its output behind it take no longer together than before (where one such reader loses, it is said).  All
// times in us, ordinary -> streamed, graphs of several launches, each replayed once untimed: a graph that follows another writes back
// what that one has left dirty.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace ecco_stream {

constexpr size_t kMiB = (size_t)1 << 20;
// Outputs of the decoders may begin in the middle of a 128-byte line; a store of part of a line is better left to the cache.
inline bool whole_lines(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 127u) == 0; }

// Decoder of self-contained blocks: from 400 MiB of FP16 on.  Alone / with a plain reader / with products of 16 and 512 rows behind it, into one buffer used again
// and again: 1835008 groups 157 -> 152 / 276 -> 238 / 273 -> 267, 368 -> 356.  What the cache holds is better left there: 131072
// 18.5 -> 16.8 / 32.6 -> 32.3 / 31.8 -> 35.0, 46.4 -> 48.1; 352256 38.5 -> 36.9 / 53.9 -> 55.1 / 55.8 -> 60.9, 87.5 -> 91.4; 1048576 95.3 -> 90.2 / 136 -> 139 /
// 155 -> 157, 207 -> 204.
inline bool decoded(const void* to, size_t bytes) { return whole_lines(to) && bytes >= 400 * kMiB; }

// Activation decoder: from 256 MiB of FP16 on.  Alone / with a plain reader / with a product of 256 columns behind it, into one buffer used again and again:
// 2097152 groups 72.7 -> 69.4 / 111 -> 114 / 152 -> 144, over several buffers 74.9 -> 63.1 / 115 -> 119 / 154 -> 152, 3145728 113 -> 108 / 194 -> 177 / 233 ->
// 233; encoded and decoded 157 -> 138 and 236 -> 226, with a writer in front and a plain reader behind, and the encoder's input streamed as well, 286 -> 278 and 460 ->
// 429.  (A program that only decodes and reads 256 MiB loses 3 %.)  Below, readers lose: one buffer, 262144 11.0 -> 10.2 / 20.0 -> 22.7 / 35.5 -> 40.7, 524288
// 17.3 -> 17.0 / 29.4 -> 30.3 / 54.4 -> 56.0, 1048576 34.2 -> 31.2 / 56.1 -> 59.2 / 78.5 -> 86.2.
inline bool activations(const void* to, size_t bytes) { return bytes >= 256 * kMiB && whole_lines(to); }

// Activation encoder's input: from 256 MiB on, so that it does not take the place of the blocks.  Alone / with a writer of the input in front / and a
// reader of the blocks behind: 2097152 groups 77.9 -> 72.0 / 174 -> 171 / 195 -> 188, 4194304 176 -> 160 / 386 -> 361 / 423 -> 393.  Below, it depends on what is beside it:
// 524288 21.5 -> 21.3 / 38.5 -> 39.6 / 45.2 -> 46.4; 786432 30.7 -> 30.8 / 69.6 -> 56.6 / 76.9 -> 67.7, but with the decoder and a product behind 92.7 -> 111;
// 1048576 40.3 -> 39.4 / 89.7 -> 81.6 / 99.0 -> 99.5.
constexpr bool encoder_input(size_t bytes) { return bytes >= 256 * kMiB; }

// Blocks of the min/max encoder: from 8 to 16 MiB.  Alone / with a plain reader / with the decoder behind it, 16 patterns: 131072 groups 18.5 -> 18.1 / 21.0 -> 20.6 /
// 30.6 -> 30.2, 262144 32.6 -> 31.7 / 34.9 -> 35.1 / 50.7 -> 50.2; not taken: 65536 11.3 -> 10.9 / 13.4 -> 13.4 / 19.2 -> 19.4, 524288 60.5 -> 60.9 / 63.7 -> 63.8 /
// 91.0 -> 97.0.  The full search gains 1 % and goes without.
constexpr bool encoded(size_t bytes) { return bytes >= 8 * kMiB && bytes <= 16 * kMiB; }

typedef uint32_t word4_t __attribute__((ext_vector_type(4)));

// to[0] = v, sixteen bytes, past the caches if kStream
template <bool kStream>
__device__ __forceinline__ void store(uint4* to, uint4 v) {
    if constexpr (kStream) __builtin_nontemporal_store(word4_t{v.x, v.y, v.z, v.w}, reinterpret_cast<word4_t*>(to));
    else *to = v;
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
