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

// Activation decoder: from 8 MiB of FP16 on.  65536 groups 4.5 -> 3.4 (7.8 -> 7.7), 131072 7.7 -> 5.4 (12.2 -> 11.8), 262144 12.7 -> 9.3 (18.4 -> 19.0),
// 524288 21.9 -> 17.1 (31.2 -> 33.3), 1048576 39.6 -> 32.8 (59.8 -> 61.3), 2097152 76.1 -> 64.7 (117 -> 117).  Between 32 and 128 MiB the
// reader alone loses by it, but the codec's blocks stay in the cache: encoded and decoded 524288 groups 41.3 -> 38.1, 1048576 80.4 -> 69.8,
// and with a writer of the input and a reader of the output around them 76.7 -> 71.7 and 148 -> 139.
inline bool activations(const void* to, size_t bytes) { return bytes >= 8 * kMiB && whole_lines(to); }

// Activation encoder's input: from 64 MiB on, so that it does not take the place of the blocks.  32768 groups 3.55 -> 3.85 and 262144
// 13.0 -> 13.2 (not taken), 524288 22.2 -> 22.1, 1048576 41.5 -> 40.7, 1572864 61.3 -> 58.4, 2097152 81.3 -> 73.7; with a writer of the input in
// front 22.7 -> 23.4 at 262144, then 41.2 -> 41.2, 92.8 -> 84.9, 133 -> 130, 176 -> 168.  (Writer, encoder, decoder and reader of 524288 groups take
// 79.3 if only the decoder streams.)
constexpr bool encoder_input(size_t bytes) { return bytes >= 64 * kMiB; }

// Blocks of the min/max encoder: from 4 MiB on.  16384 groups 4.9 -> 4.9 (7.3 -> 7.5), 65536 11.1 -> 10.6 (13.7 -> 13.6), 131072
// 18.4 -> 17.6 (21.7 -> 21.3), 524288 62.1 -> 60.8 (68.2 -> 68.1).  The full search gains 1 % and goes without.
constexpr bool encoded(size_t bytes) { return bytes >= 4 * kMiB; }

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
