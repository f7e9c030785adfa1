// HIP kernels of libhzp for CDNA4 (gfx950) and their launchers.
//
// Every kernel here streams: each byte is read once and written once, there is no reuse and
// no contraction, so the bound is HBM bandwidth (26+2R bytes per element for the fused update
// with bf16 gradients, against about 30 fp32 operations).  The design therefore is
//   - every load/store instruction of a wavefront covers one contiguous run of memory;
//   - single-wavefront workgroups, dispatched in address order, with a few loads in flight each and a
//     cap on how many are resident: a small, coherent front of requests serves the memory
//     controllers better than as many requests as the chip can hold;
//   - everything a wavefront needs to ask for its data (pointers, lengths, scalars) arrives in one
//     round of scalar loads;
//   - non-temporal loads, and stores that are written through to memory with the streaming
//     hint: nothing is touched twice, so no line should be kept;
//   - many layers per launch: shards of one layer are only a few MB, so the per-layer
//     pointers travel in the kernel-argument block and one grid covers all of them;
//   - consecutive workgroups take consecutive tiles (neighbouring ones in pairs in the fused update).
//     The hardware deals workgroups to the 8 XCDs round-robin; with no reuse there is nothing for an
//     XCD-local L2 to keep, the tiles of any window of workgroups still spread over all memory
//     channels, and a remap that gives each XCD its own contiguous eighth measured 5 % slower.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <memory>
#include <type_traits>
#include <utility>
#include <vector>

#include "hzp_internal.hpp"

namespace hzp {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
typedef uint64_t u64x4 __attribute__((ext_vector_type(4)));
// Same vector with element alignment only, for sources that follow an unaligned destination.
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

template <class T>
__device__ __forceinline__ T ld_stream(const T *p)
{
    return __builtin_nontemporal_load(p);
}

// Vector `idx` of a stream whose base address is uniform: base + 32-bit byte offset in global memory, so
// that the access uses a scalar base register and one VGPR offset.  Callers keep streams below 4 GiB.
template <class T>
__device__ __forceinline__ T ld_stream(uint64_t base, uint32_t idx)
{
    typedef const __attribute__((address_space(1))) char *bytes;
    typedef const __attribute__((address_space(1))) T *vectors;
    return __builtin_nontemporal_load((vectors)((bytes)base + idx * (uint32_t)sizeof(T)));
}

// Streaming store with write-through to memory: system scope plus the non-temporal hint.  Measured
// on MI355X, the many concurrent write streams of the fused update drain 1-4 % faster with these
// cache-policy bits than with the non-temporal hint alone.  The compiler has no source-level way
// to ask for this combination on a 16-byte store, hence the instruction is written out.  The
// trailing s_nop keeps the two wait states this hardware generation needs between a store of more
// than 8 bytes and an overwrite of its data registers (the compiler cannot see inside the asm to
// add them; with one wait state the first dword of some lanes was stored from the next value
// when the store pipeline was under pressure).
__device__ __forceinline__ void st_writethrough(uint64_t base, uint32_t byte_off, f32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, %2 sc0 sc1 nt\n\ts_nop 1" ::"v"(byte_off), "v"(v), "s"(base) : "memory");
}
// The same store for a full 64-bit address in a VGPR pair (copy kernels, whose lanes compute their
// own destination).
__device__ __forceinline__ void st_writethrough(u32x4 *dst, u32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1 nt\n\ts_nop 1" ::"v"(dst), "v"(v) : "memory");
}
__device__ __forceinline__ void st_writethrough(uint64_t base, uint32_t byte_off, u32x2 v)
{
    asm volatile("global_store_dwordx2 %0, %1, %2 sc0 sc1 nt" ::"v"(byte_off), "v"(v), "s"(base) : "memory");
}

// bf16 pair packed in one 32-bit word (element 0 in the low half) -> two fp32 values.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Two fp32 -> packed bf16 pair (first value in the low half), round to nearest even, NaN stays a
// quiet NaN: gfx950's packed conversion instruction.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 x = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

// ---------------------------------------------------------------------------------------
// Work decomposition of the element-wise kernels.
//
// A workgroup is ONE wavefront and owns one group of 256 consecutive elements, a quad of 4 to a
// lane, so every load or store of the wavefront covers one contiguous run (1 KiB of an fp32 stream,
// 512 B of a bf16 stream).  The contributions are requested a few at a time (a chunk) and added as
// they come, and unused LDS caps the resident wavefronts: with 15-19 concurrent streams what decides
// is how many bytes are in flight per CU, and at what spread of addresses, not how many loads one
// wavefront can have outstanding.  About 32-50 KiB in flight per CU serve the memory best; below
// that latency shows, above it the requests queue in an order the memory controllers serve badly.
// Measured on MI355X, 100 M elements, all R + 3 loads of a 512-element group up front against
// chunks on 256-element groups: R = 8 bf16 6.68 -> 6.78 TB/s, R = 16 6.24 -> 6.72, fp32 R = 8
// 6.37 -> 6.73, R = 1 fp32 6.67 -> 6.79.
// Shards are multiples of 8 elements, so a quad is never split; lanes past the end of a segment
// read its last quad again and store nothing.
// ---------------------------------------------------------------------------------------
constexpr int kWave = 64;
// The runtime copies a launch's arguments into memory that another of its threads gives back, a thousand launches at a time.  Where copies
// are longer than this the two threads wait for each other.  Calls in a row, blocks of 24 / 96 / 104 / 112 / 120 / 128 / 256 / 816 / 3616
// bytes, us a launch: in a C++ program of nothing else 2.7 / 2.8 / 2.85 / 2.85 / 3.45 / 3.5 / 3.6 / 3.7 / 3.9, with PyTorch loaded - / 2.80
// / 2.81 / 2.78 / 3.25-3.6 / 3.55 / 3.65 / 3.9 / -.  (Of this runtime with this C library; longer blocks work as well.)
constexpr size_t kFewBytes = 112;
constexpr uint32_t kGroupQuads = 64;        // quads per group (256 elements)

// Dynamic LDS that leaves room for `waves` single-wavefront workgroups per CU, or the next smaller number that there is: a CU's 160 KiB
// are given out in 128 units of 1280 bytes (so 13 are 12, 15 are 14, 17 are 16, 19 and 20 are 18, 22 to 24 are 21, 26 to 31 are 25).
constexpr unsigned lds_for(unsigned waves) { return waves ? (128u / (waves + 1) + 1) * 1280u : 0u; }

constexpr uint32_t kReduceChunk = 4;
// A launch of so few groups that all wavefronts are resident at once lasts as long as one wavefront, whose chunks follow
// each other: there, more than 8 contributions are requested up to 16 at a time (chunks of 4 / 16, us a call: 64 k elements, R = 32:
// reduction 6.1 / 4.2, update 6.5 / 4.4; 512 k 7.9 / 7.7 and 10.8 / 10.1, fp32 R = 32 at 512 k 12.4 / 12.9 and 14.8 / 15.3; the update of
// several segments, 0.15 M elements, R = 16 / 32: 5.8 -> 5.1 and 7.3 -> 5.3; with R <= 8 no difference).
constexpr uint32_t kFewGroups = 2048;
constexpr uint32_t few_chunk(uint32_t R, uint32_t chunk) { return R > 8 ? 16u : chunk; }
// Most contributions one wavefront of the update has in flight, by the launch's class (fused_class).
//   kLarge: few large chunks beat many small ones (a wavefront waits once for each), with so many fewer wavefronts that a CU has about
//   50 KiB in flight (fused_lds).  Chunks of at most 4 / 6 / 8, each with the best number of wavefronts, mean over 9 to 105 M
//   elements against chunks of 4 with 9 or 11: bf16 R = 10 .995 / .981 / .982, R = 14 .996 / .979 / .974, R = 16 .996 / .986 / .979,
//   R = 20 .996 / .985 / .979, R = 24 .999 / .991 / .988, R = 28 .997 / .990 / .989, R = 32 .997 / .996 / .991.
//   fp32 with chunks of at most 3 / 4 / 6, over 1.5 to 71 M: R = 4 .989 / .978 / -, R = 8 .993 / .973 / -, R = 12 .982 / .980 / .975,
//   R = 16 .996 / .983 / .983, R = 24 .991 / .992 / 1.004, R = 32 .997 / .998 / 1.019.
//   kMid: in shorter launches large chunks read too many streams side by side, and where no cap holds the wavefronts back they ask for
//   too much (bf16 R = 12 / 24 of 0.66 M elements 7.6 / 9.9 us, with chunks of 8 7.9 / 10.2; fp32 R = 4 6.1, with chunks of 4 6.4).
//   kFew: all resident, and so few that latency counts.
enum ChunkClass { kFew, kMid, kLarge };
constexpr uint32_t fused_most(bool g32, uint32_t R, ChunkClass c)
{
    const uint32_t mid = g32 ? 3u : 4u;
    if (c == kFew) return few_chunk(R, mid);
    if (c == kMid || (g32 && R > 16)) return mid;
    return g32 || R <= 4 ? 4u : R <= 8 ? R : 8u;
}

// Contributions in the largest chunk: R spread evenly over the fewest chunks of at most `most`.
constexpr uint32_t chunk_of(uint32_t R, uint32_t most)
{
    const uint32_t chunks = (R + most - 1) / most;
    return (R + chunks - 1) / chunks;
}
// (a kernel is made for the chunk and not for the most, so that classes that come to the same share one)
constexpr uint32_t fused_chunk(bool g32, uint32_t R, ChunkClass c) { return chunk_of(R, fused_most(g32, R, c)); }

// Four gradient elements of one contribution, widened to fp32 on access.
template <bool G32>
struct GradQuad;
template <>
struct GradQuad<false> {
    u32x2 w;
    __device__ __forceinline__ void load(uint64_t base, uint32_t quad) { w = ld_stream<u32x2>(base, quad); }
    __device__ __forceinline__ float get(int e) const
    {
        const uint32_t word = w[e >> 1];
        return (e & 1) ? bf16_hi(word) : bf16_lo(word);
    }
};
template <>
struct GradQuad<true> {
    f32x4 a;
    __device__ __forceinline__ void load(uint64_t base, uint32_t quad) { a = ld_stream<f32x4>(base, quad); }
    __device__ __forceinline__ float get(int e) const { return a[e]; }
};

// Pins uniform values: they are read (from the arguments) no later than here, and not where they are used, with
// nothing to hide the read behind.
template <class T>
__device__ __forceinline__ void pin(T &x)
{
    asm volatile("" : "+s"(x));
}
template <class T, class... Rest>
__device__ __forceinline__ void pin(T &x, Rest &...rest)
{
    pin(x);
    pin(rest...);
}

// Address `d` units of 16 bytes from another.
__device__ __forceinline__ uint64_t at_distance(uint64_t base, int32_t d) { return base + (int64_t)d * 16; }

// So many wait states (a multiple of 8) between the requests before and behind it.
template <uint32_t STATES>
__device__ __forceinline__ void gap()
{
    static_assert(STATES % 8 == 0, "whole s_nop 7");
    if constexpr (STATES > 0) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (uint32_t k = 0; k < STATES / 8; ++k) asm volatile("s_nop 7");
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Left-to-right fp32 sum of R contributions, ((g0 + g1) + g2) + ..., at most `MOST` of them in flight, for
// Q quads; slice(r) + shift is contribution r, and `at` holds the first chunk's pointers.  meanwhile() runs when the first chunk
// is requested.  Where the chunks are not all of one size the larger ones are the first (LARGER_FIRST) or the last.  GAP wait states
// lie between any two contributions' requests.
template <uint32_t R, uint32_t MOST, bool G32, int Q, bool LARGER_FIRST, uint32_t GAP, class Slice, class Meanwhile>
__device__ __forceinline__ void sum_contributions(uint64_t (&at)[MOST], Slice slice, int64_t shift,
                                                  const uint32_t (&quad)[Q], float (&s)[Q][4], Meanwhile meanwhile)
{
    constexpr uint32_t C = chunk_of(R, MOST), CHUNKS = (R + C - 1) / C, UP = LARGER_FIRST ? CHUNKS - 1 : 0;
#pragma unroll
    for (uint32_t k = 0; k < CHUNKS; ++k) {
        const uint32_t base = (k * R + UP) / CHUNKS, end = ((k + 1) * R + UP) / CHUNKS, next = ((k + 2) * R + UP) / CHUNKS;
        GradQuad<G32> g[C][Q];
#pragma unroll
        for (uint32_t c = 0; c < C; ++c)
            if (base + c < end) {
#pragma unroll
                for (int q = 0; q < Q; ++q) g[c][q].load(at[c] + shift, quad[q]);
                gap<GAP>();
            }
#pragma unroll
        for (uint32_t c = 0; c < C; ++c)
            if (k + 1 < CHUNKS && end + c < next) at[c] = slice(end + c);
        __builtin_amdgcn_sched_barrier(0);      // the whole chunk is requested (and the next one's pointers) before its first add,
        if (base == 0) meanwhile();
#pragma unroll
        for (uint32_t c = 0; c < C; ++c)
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (base + c < end) s[q][e] = base + c ? s[q][e] + g[c][q].get(e) : g[c][q].get(e);
        // and the next chunk only behind its last: the sum is pinned here, or the adds sink to the sum's use
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(s[q][e]));
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ---------------------------------------------------------------------------------------
// Standalone reduction (bit-exact with the scalar definition: fixed order, no contraction).
// ---------------------------------------------------------------------------------------
// Argument blocks hold as many pointers as the kernel reads (kFewBytes).
template <uint32_t N>
struct Pointers {
    uint64_t g[N];
};
template <uint32_t R>
struct ReduceArgs {
    uint64_t out;
    uint32_t nquad;                     // 4-element quads in the slice
    float scale;
    Pointers<R> all;
};
static_assert(sizeof(ReduceArgs<12>) == kFewBytes, "up to 12 contributions");
// Pointer `r` of those behind the leading arguments, of which there may be none.
__device__ __forceinline__ uint64_t behind(uint32_t) { return 0; }
template <uint32_t N>
__device__ __forceinline__ uint64_t behind(uint32_t r, const Pointers<N> &p) { return p.g[r]; }

// The forms of a launch: contributions in flight (chunk), quads per lane, and whether the sum that is accumulated onto is requested
// behind the contributions instead of ahead of them.
enum ReduceForm { kReducePlain, kReduceFew, kReduceNarrow };
constexpr uint32_t reduce_chunk(uint32_t R, ReduceForm form)
{
    return form == kReducePlain ? kReduceChunk : form == kReduceFew ? few_chunk(R, kReduceChunk) : 2u;
}
// Quads per lane: with a single bf16 contribution one quad is 512 B of reads to a wavefront, too little even at full
// occupancy (25 M elements: 5.89 TB/s; with two quads 6.22).
constexpr int reduce_quads(uint32_t R, bool g32, ReduceForm form) { return form == kReduceNarrow || (R == 1 && !g32) ? 2 : 1; }

template <uint32_t R, bool G32, bool ACC, ReduceForm FORM, uint32_t CHUNK, class Slice>
__device__ __forceinline__ void reduce(uint64_t out, uint32_t nquad, float scale, uint64_t (&at)[CHUNK], Slice slice)
{
#pragma clang fp contract(off)
    constexpr int Q = reduce_quads(R, G32, FORM);
    // (in chunks of 2 a first chunk of one loses: fp32 R = 9 / 13 of 1.5 M elements 10.3 / 13.8 us, 10.0 / 13.5 with the larger ones first; in longer
    // chunks it gains: R = 5 / 10 accumulating of 7.4 M 33.0 / 55.7, 33.5 / 56.8)
    constexpr bool LATE = FORM == kReduceNarrow;
    uint32_t q0[Q], quad[Q];
    f32x4 t[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        q0[q] = (blockIdx.x * Q + q) * kGroupQuads + threadIdx.x;
        quad[q] = q0[q] < nquad ? q0[q] : nquad - 1;
        if (ACC && !LATE) t[q] = ld_stream<f32x4>(out, quad[q]);
    }
    float s[Q][4];
    sum_contributions<R, CHUNK, G32, Q, LATE, 0>(at, slice, 0, quad, s, [] {});
#pragma unroll
    for (int q = 0; q < Q; ++q)
        if (ACC && LATE) t[q] = ld_stream<f32x4>(out, quad[q]);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = scale * s[q][e];
            t[q][e] = ACC ? t[q][e] + x : x;
        }
        if (q0[q] < nquad) st_writethrough(out, quad[q] * 16u, t[q]);
    }
}

// What the first requests need, the first four pointers and the output (o[1]: number of quads, scale), is in scalar registers when a
// wavefront starts: leading arguments that are no structs arrive there (the build asks for 14 words; vectors, because the host spends 15 ns
// on every argument).  With all of it read from the argument block, us: bf16 R = 4 / 8 of 2.1 M elements 5.8 / 8.2 (here 5.5 / 8.1), R = 32
// of 0.5 M 7.4 (6.9), R = 8 of 25 M 76.6 (75.8); fp32 R = 4 accumulating, 1 / 6.3 M 6.0 / 25.1 (5.8 / 25.0).
// REST is Pointers<R - 4>, or nothing.
template <uint32_t R, bool G32, bool ACC, ReduceForm FORM, class... REST>
__global__ __launch_bounds__(kWave) void reduce_kernel(const u64x4 g, const u64x2 o, const REST... rest)
{
    constexpr uint32_t CHUNK = reduce_chunk(R, FORM);
    uint64_t at[CHUNK];
#pragma unroll
    for (uint32_t c = 0; c < CHUNK; ++c) at[c] = c >= R ? 0 : c < 4 ? g[c] : behind(c - 4, rest...);
    reduce<R, G32, ACC, FORM>(o[0], (uint32_t)o[1], __uint_as_float((uint32_t)(o[1] >> 32)), at,
                              [&](uint32_t r) { return r < 4 ? g[r] : behind(r - 4, rest...); });
}

// The same with all of it read from the argument block in one round of scalar loads, for the launches of reduce_from_block().
template <uint32_t R, bool G32, bool ACC, ReduceForm FORM>
__global__ __launch_bounds__(kWave) void reduce_block_kernel(const ReduceArgs<R> a)
{
    constexpr uint32_t CHUNK = reduce_chunk(R, FORM);
    uint64_t out = a.out, at[CHUNK];
    uint32_t nquad = a.nquad;
    float scale = a.scale;
#pragma unroll
    for (uint32_t c = 0; c < CHUNK; ++c) at[c] = c < R ? a.all.g[c] : 0;
    pin(out, at[0], at[1], at[CHUNK > 2 ? 2 : 0], at[CHUNK > 2 ? 3 : 0], nquad, scale);
    reduce<R, G32, ACC, FORM>(out, nquad, scale, at, [&](uint32_t r) { return a.all.g[r]; });
}

// Short launches of more contributions than kFewBytes holds pointers of, where these lie at equal distances.
// o: output, number of quads and scale; g: the first contribution, the distance from one to the next.
constexpr uint32_t kReduceEvenLeast = 13;
template <uint32_t R, bool G32, bool ACC>
__global__ __launch_bounds__(kWave) void reduce_even_kernel(const u64x2 o, const u64x2 g)
{
    constexpr uint32_t CHUNK = reduce_chunk(R, kReduceFew);
    uint64_t at[CHUNK];
#pragma unroll
    for (uint32_t c = 0; c < CHUNK; ++c) at[c] = c < R ? g[0] + c * g[1] : 0;
    reduce<R, G32, ACC, kReduceFew>(o[0], (uint32_t)o[1], __uint_as_float((uint32_t)(o[1] >> 32)), at,
                                    [&](uint32_t r) { return g[0] + r * g[1]; });
}

// ---------------------------------------------------------------------------------------
// Fused reduce + scale + AdamW + cast over many shard segments.
// ---------------------------------------------------------------------------------------
// What one launch covers travels in the argument block: `segments` runs of elements, each with its R + 4
// pointers (master, m, v, parameter output or null, R contributions) followed by a record.  A call of many
// small segments that lie at the same distances from each other in all streams (the layers of an arena)
// can share one set of pointers; a record then gives the segment's distance from the first.
//   word 0: groups up to and including the segment (2-D grid: the segment's own), number of quads
//   word 1: decay multiplier; where the launch looks decay up: first entry and number of entries
//   word 2 (launches that look decay up): bucket position of the segment's first element
//   last word (launches with one set of pointers): distance in quads, and the output's own
constexpr uint32_t kPlainRecord = 2;        // words of a record with pointers of its own and no look-up
constexpr uint32_t kTableWords = 480;       // 3840 bytes: 34 segments at R = 8 with pointers of their own
struct FusedArgs {
    uint32_t segments;
    uint32_t stride, ptr_stride;            // words from a segment's record / pointers to the next one's (0: shared)
    uint32_t dist;                          // where the distance stands in a record (0: no distance)
    uint32_t grid2d;                        // 1: grid is (groups, segments)
    uint32_t lookup;                        // 1: decay multipliers come from the tables
    const uint64_t *run_off;                // device: bucket positions where the decay multiplier changes
    const float *run_wd;                    // device: the multiplier from there on
    const AdamScalars *scalars_dev;         // device, or null: `scalars` are the step's
    AdamScalars scalars;
    uint64_t word[kTableWords];
};
static_assert(sizeof(FusedArgs) <= 4096, "kernel arguments");
// The same for one segment with pointers of its own and one multiplier, whose leading arguments (FusedLead) are in scalar registers when a
// wavefront starts: all that its first requests need, up to two contributions.  The block is a tenth of the other,
// which the host has to write to device memory (kFewBytes).
struct FusedOneArgs {
    uint64_t out;
    AdamScalars scalars;
    uint64_t g[HZP_MAX_REPLICAS];
    static constexpr size_t kScalars = 8;       // where the scalars lie behind the leading arguments
    __device__ __forceinline__ uint64_t output() const { return out; }
    __device__ __forceinline__ uint64_t contribution(uint32_t r) const { return g[r]; }
};
static_assert(offsetof(FusedOneArgs, scalars) == FusedOneArgs::kScalars, "argument block");
struct FusedLead {
    u64x4 p;                                // master, m, v, the first contribution
    u64x2 w;                                // the second, the step's scalars in device memory (or null: they are in the block)
    uint64_t size;                          // number of quads, decay multiplier
};
constexpr uint32_t kLeadBytes = 56;         // of the argument block; the struct follows
static_assert(sizeof(u64x4) + sizeof(u64x2) + sizeof(uint64_t) == kLeadBytes && alignof(FusedOneArgs) == 8, "argument block");
// The same for short launches where contributions lie at equal distances, as in the planner's arena or one receive buffer: any number of
// them, within kFewBytes.
struct FusedEvenArgs {
    uint64_t out;
    AdamScalars scalars;
};
static_assert(kLeadBytes + sizeof(FusedEvenArgs) <= kFewBytes && alignof(FusedEvenArgs) == 8, "argument block");
struct FusedEven {                          // what fused_adamw asks of them
    uint64_t out, first, stride;
    static constexpr size_t kScalars = offsetof(FusedEvenArgs, scalars);
    __device__ __forceinline__ uint64_t output() const { return out; }
    __device__ __forceinline__ uint64_t contribution(uint32_t r) const { return first + r * stride; }
};
enum FusedForm { kSearched, kPlain, kOne };

// The decay runs that a group meets, found while the streams arrive: begin() narrows the search to 64
// runs and requests their starts (lane by lane), find() requests the next ones and the first multiplier,
// get() picks the lane's own.  Runs are whole numbers of 8 elements, so a group meets at most 33.
struct DecayRuns {
    const uint64_t *off;
    const float *wd;
    uint32_t lo, end;           // find(): the run that holds the group's first element; the slice's last + 1
    uint64_t start, next;       // lane l: the starts of runs lo + l; lo + 1 + l
    float mult;                 // run lo's multiplier
    __device__ __forceinline__ void begin(uint32_t first, uint32_t n, uint64_t pos)
    {
        const uint32_t lane = threadIdx.x;
        lo = first;
        end = first + n;
        uint32_t left = n;
        while (left > kWave) {                  // 64 pivots a round
            const uint32_t stride = (left + kWave - 1) / kWave;
            const uint32_t mine = lane * stride;
            const bool le = mine < left && off[lo + mine] <= pos;
            const uint32_t step = ((uint32_t)__popcll(__ballot(le)) - 1u) * stride;
            left = left - step < stride ? left - step : stride;
            lo += step;
        }
        start = ~0ull;
        if (lane < left) start = off[lo + lane];
    }
    __device__ __forceinline__ void find(uint64_t pos)
    {
        const uint32_t lane = threadIdx.x;
        lo = __builtin_amdgcn_readfirstlane(lo + (uint32_t)__popcll(__ballot(start <= pos)) - 1u);
        next = ~0ull;
        if (lo + 1 + lane < end) next = off[lo + 1 + lane];
        mult = wd[lo];
    }
    __device__ __forceinline__ float get(uint64_t pos) const
    {
        const uint32_t inside = (uint32_t)__popcll(__ballot(next < pos + 4 * kGroupQuads));
        if (inside == 0) return mult;
        const uint64_t mine = pos + 4 * threadIdx.x;
        uint32_t r = lo;
        for (uint32_t k = 1; k <= inside; ++k)
            if (off[lo + k] <= mine) r = lo + k;
        return wd[r];
    }
};

// PAIRS: each XCD takes two neighbouring groups (workgroups are dealt to the 8 XCDs round-robin, so of every
// 16 consecutive groups workgroups x and x + 8 take groups 2x and 2x + 1).  A bf16 access of a group covers
// 512 B; as pairs an XCD's accesses to a bf16 stream cover 1 KiB, like those to an fp32 stream.  Measured
// with bf16 contributions (R = 4 / 8 / 16, 100 M elements): 6.74 / 6.68 / 6.58 -> 6.77 / 6.78 / 6.72 TB/s;
// quadruples lose again (6.66 / 6.73 / 6.66), and where all streams are fp32 pairs lose 1 % (6.79 -> 6.73).
//
// kPlain: a 2-D grid over segments with pointers of their own and one multiplier each; everything a wavefront needs lies at an
// address that blockIdx gives and arrives in one round of scalar loads.  kOne: a single such segment (a whole arena of equal decay
// is one); what its first requests need is there when it starts (read from the argument block / in registers, us: bf16 R = 4 of
// 0.46 M elements 5.0 / 4.6, R = 1 and 8 of 2.1 M 11.5 / 11.3 and 16.6 / 16.4, fp32 R = 12 of 0.26 M 5.9 / 5.5; from 25 M the same).
// kSearched: a uniform binary search may have to find the segment, three more rounds, which the few resident wavefronts hide badly
// (105 M elements, R = 8, one segment: 6.65 TB/s at the best number of wavefronts, 6.73 with one round).
//
// Where all of one segment's wavefronts are resident they start with their pointers at hand and ask for everything at once, and
// streams that lie at the wrong distance from each other then collide in the memory channels.  A pause between
// requests avoids that (s_nop; where the pointers came from the argument block, the compiler's 64-bit address arithmetic lay there): 8 wait states between any two
// fp32 contributions' where up to 16 go at a time, and HEAD between the state's requests and the contributions' where one or two follow in a launch
// of 12 to 20 wavefronts per CU.  Against the pointers in the argument block, on buffers of one call's size, without / with 8 states: fp32 of 0.2 to 0.3 M elements,
// streams 2, 4, .. 18 MiB apart, R = 9 to 16, 210 sets, mean 1.02 / 0.90, worst 1.72 / 1.10 (R = 14 of 0.26 M, 6 MiB apart, 9.3 us, 5.8 now); 0.08 to 0.5 M,
// R = 9 to 32, .98 / .93, in a larger allocation .95 / .95; bf16, which has none, .95 / .93, but near 2048 groups up to 1.16 / 1.42.  Without / with 96 states, 0.85 to 1.05 M: bf16 R = 1 1.00 / .93, R = 2
// .99 / .90, fp32 R = 1 1.04 / .94, in a larger allocation 1.02 / .94, .98 / .94, .99 / .95.  (Longer launches are capped, and a pause only delays them: 96 states 0 to 1 %
// more, 16 between requests 0 to 2 %.)
template <uint32_t R, bool G32, bool O32, FusedForm FORM, uint32_t CHUNK, uint32_t HEAD, class Args>
__device__ __forceinline__ void fused_adamw(const FusedLead lead, const Args &a)
{
    constexpr bool PAIRS = !G32;
    // Which segment and which group of it?
    uint32_t grp = blockIdx.x;
    const uint64_t *slice = nullptr, *rec = nullptr;        // the contributions' pointers, the segment's record
    int64_t shift = 0, out_shift = 0;           // of the segment against the pointers, in quads
    bool lookup = false;
    DecayRuns runs;
    uint64_t pos = 0;                           // of the group's first element in its bucket
    uint64_t P, M, V, OUT, decay, at[CHUNK], scalars_dev;
    uint32_t groups, nquad;
    AdamScalars h;
    if constexpr (FORM == kOne) {
        P = lead.p[0];
        M = lead.p[1];
        V = lead.p[2];
        OUT = a.output();
        scalars_dev = lead.w[1];
        nquad = (uint32_t)lead.size;
        decay = lead.size >> 32;
        groups = (nquad + kGroupQuads - 1) / kGroupQuads;
#pragma unroll
        for (uint32_t c = 0; c < CHUNK; ++c) at[c] = c >= R ? 0 : c == 0 ? lead.p[3] : c == 1 ? lead.w[0] : a.contribution(c);
    } else {
        const uint64_t *ptr;
        uint32_t before = 0;                    // workgroups of the segments ahead of it
        if constexpr (FORM == kPlain) {
            ptr = a.word + blockIdx.y * (R + 4 + kPlainRecord);
            rec = ptr + R + 4;
        } else {
            uint32_t segments = a.segments, stride = a.stride, ptr_stride = a.ptr_stride, dist = a.dist, grid2d = a.grid2d, look = a.lookup;
            pin(segments, stride, ptr_stride, dist, grid2d, look);
            lookup = look;
            const uint64_t *const records = a.word + R + 4;
            uint32_t seg = blockIdx.y;
            if (!grid2d) {
                uint32_t lo = 0, hi = segments - 1;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (blockIdx.x < (uint32_t)records[mid * stride])
                        hi = mid;
                    else
                        lo = mid + 1;
                }
                seg = lo;
                before = seg ? (uint32_t)records[(seg - 1) * stride] : 0u;
            }
            rec = records + seg * stride;
            ptr = a.word + seg * ptr_stride;
            grp -= before;
            if (dist) {
                const uint64_t d = rec[dist];
                shift = (int32_t)(uint32_t)d;
                out_shift = (int32_t)(uint32_t)(d >> 32);
            }
        }
        slice = ptr + 4;
        uint64_t extent = rec[0];
        P = ptr[0];
        M = ptr[1];
        V = ptr[2];
        OUT = ptr[3];
        decay = rec[1];
#pragma unroll
        for (uint32_t c = 0; c < CHUNK; ++c) at[c] = c < R ? slice[c] : 0;
        h = a.scalars;
        scalars_dev = reinterpret_cast<uint64_t>(a.scalars_dev);
        pin(P, M, V, OUT, extent, decay, at[0], at[CHUNK > 1 ? 1 : 0], at[CHUNK > 2 ? 2 : 0], at[CHUNK > 3 ? 3 : 0], scalars_dev);
        pin(h.lr, h.beta1, h.beta2, h.one_minus_beta1, h.one_minus_beta2, h.eps, h.weight_decay, h.grad_scale, h.inv_bc1, h.inv_bc2);
        groups = (uint32_t)extent - before;
        nquad = (uint32_t)(extent >> 32);
        if (grp >= groups) return;              // of a longer segment of a 2-D grid
    }
    // (ahead of the requests: behind a branch, an offset that was used before it no longer goes with a scalar base)
    if constexpr (FORM == kOne)
        if (!scalars_dev) scalars_dev = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + kLeadBytes + Args::kScalars;
    if (FORM == kOne || scalars_dev) {
        typedef const __attribute__((address_space(4))) float const_float;      // scalar loads
        const_float *c = reinterpret_cast<const_float *>(scalars_dev);
        h = {c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], c[8], c[9]};
    }
    if (PAIRS && grp < (groups & ~15u)) grp = (grp & ~15u) | ((grp & 7u) << 1) | ((grp >> 3) & 1u);
    P += shift * 16;
    M += shift * 16;
    V += shift * 16;

    const uint32_t q0 = grp * kGroupQuads + threadIdx.x;
    const uint32_t quad = q0 < nquad ? q0 : nquad - 1;
    const uint32_t quads[1] = {quad};
    if constexpr (FORM == kSearched) {
        if (lookup) {
            runs.off = a.run_off;
            runs.wd = a.run_wd;
            pos = rec[2] + 4ull * kGroupQuads * grp;
            runs.begin((uint32_t)decay, (uint32_t)(decay >> 32), pos);
        }
    }
    // The states are requested ahead of the contributions: they are needed last and then have the
    // contributions' time to arrive.
    f32x4 p = ld_stream<f32x4>(P, quad);
    f32x4 m = ld_stream<f32x4>(M, quad);
    f32x4 v = ld_stream<f32x4>(V, quad);
    __builtin_amdgcn_sched_barrier(0);
    if (FORM == kSearched && lookup) runs.find(pos);
    float g[1][4];
    gap<HEAD>();
    auto contribution = [&](uint32_t r) {
        if constexpr (FORM == kOne)
            return a.contribution(r);
        else
            return slice[r];
    };
    constexpr uint32_t GAP = FORM == kOne && G32 && CHUNK > 8 ? 8 : 0;
    sum_contributions<R, CHUNK, G32, 1, false, GAP>(at, contribution, shift * (G32 ? 16 : 8), quads, g, [&] {
        if (FORM == kOne)       // needed last, but read by now
            pin(OUT, h.lr, h.beta1, h.beta2, h.one_minus_beta1, h.one_minus_beta2, h.eps, h.weight_decay, h.grad_scale, h.inv_bc1, h.inv_bc2);
    });

    const float wd = h.weight_decay * (FORM == kSearched && lookup ? runs.get(pos) : __uint_as_float((uint32_t)decay));

    // The arithmetic is hardly hidden behind other wavefronts (few are resident by design), so it is
    // kept short: hardware square root and reciprocal (1 ulp each) instead of the correctly
    // rounded expansions.  Their error enters p only through lr*u, far below the tolerance.  Which products are
    // fused into a sum is written out, so that every form gives the same bits.
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma clang fp contract(off)
        const float ge = h.grad_scale * g[0][e];
        const float mn = __builtin_fmaf(h.beta1, m[e], h.one_minus_beta1 * ge);
        const float vn = __builtin_fmaf(h.beta2, v[e], (h.one_minus_beta2 * ge) * ge);
        const float denom = __builtin_amdgcn_sqrtf(vn * h.inv_bc2) + h.eps;
        const float u = (mn * h.inv_bc1) * __builtin_amdgcn_rcpf(denom);
        const float pe = p[e];
        m[e] = mn;
        v[e] = vn;
        p[e] = __builtin_fmaf(-h.lr, __builtin_fmaf(wd, pe, u), pe);
    }
    if (q0 >= nquad) return;
    const bool has_out = OUT != 0;
    OUT += out_shift * (O32 ? 16 : 8);
    st_writethrough(P, quad * 16u, p);
    st_writethrough(M, quad * 16u, m);
    st_writethrough(V, quad * 16u, v);
    if (has_out) {
        if constexpr (O32) {
            st_writethrough(OUT, quad * 16u, p);
        } else {
            u32x2 o;
            o[0] = pack_bf16(p[0], p[1]);
            o[1] = pack_bf16(p[2], p[3]);
            st_writethrough(OUT, quad * 8u, o);
        }
    }
}

template <uint32_t R, bool G32, bool O32, uint32_t CHUNK, uint32_t HEAD>
__global__ __launch_bounds__(kWave) void fused_one_kernel(const u64x4 p, const u64x2 w, const uint64_t size, const FusedOneArgs a)
{
    fused_adamw<R, G32, O32, kOne, CHUNK, HEAD>({p, w, size}, a);
}
// w: distance from one contribution to the next, the step's scalars in device memory.
template <uint32_t R, bool G32, bool O32, uint32_t CHUNK>
__global__ __launch_bounds__(kWave) void fused_even_kernel(const u64x4 p, const u64x2 w, const uint64_t size, const FusedEvenArgs a)
{
    fused_adamw<R, G32, O32, kOne, CHUNK, 0>({p, {p[3] + w[0], w[1]}, size}, FusedEven{a.out, p[3], w[0]});
}
template <uint32_t R, bool G32, bool O32, FusedForm FORM, uint32_t CHUNK>
__global__ __launch_bounds__(kWave) void fused_adamw_kernel(const FusedArgs a)
{
    fused_adamw<R, G32, O32, FORM, CHUNK, 0>({}, a);
}

// ---------------------------------------------------------------------------------------
// Gather: copies of whole pieces (16-byte vectors; everything is aligned).
//
// One wavefront per workgroup, one 16-byte vector per lane: of the shapes measured (1-8 vectors per lane, 64- and
// 256-thread workgroups, with and without an occupancy cap, neighbouring tiles paired per XCD or not) this one copies
// fastest on MI355X (6.8 TB/s on the 8 x 51 MB -> 405 MB layer gather); a plain copy keeps few bytes in flight per
// wavefront and wants every wave slot filled.  A wavefront's piece is given by blockIdx and everything about it
// arrives in one round of scalar loads.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void copy_tile(uint32_t tile, uint64_t src, uint64_t dst, uint32_t nvec)
{
    typedef const __attribute__((address_space(1))) u32x4 *vectors;
    const uint32_t vec = tile * kWave + threadIdx.x;
    if (vec >= nvec) return;
    const u32x4 val = __builtin_nontemporal_load((vectors)src + vec);
    st_writethrough(reinterpret_cast<u32x4 *>(dst) + vec, val);
}

// A list of pieces, of one bucket or of many layers (the post-step gather runs for all layers at once; 34 launches of
// 16 us each leave the memory system idle between them).  grid = (tiles of the longest piece, pieces); a piece that
// already lies in place is left out of the list.
template <int PIECES>
struct CopyListArgs {
    static constexpr int kPieces = PIECES;
    uint64_t src[PIECES], dst[PIECES];
    uint32_t nvec[PIECES];                  // length in 16-byte vectors
};
typedef CopyListArgs<5> CopyLeastArgs;
typedef CopyListArgs<8> CopyFewArgs;
typedef CopyListArgs<64> CopyGroupArgs;
typedef CopyListArgs<192> CopyManyArgs;
static_assert(sizeof(CopyManyArgs) <= 4096 && sizeof(CopyLeastArgs) <= kFewBytes, "kernel arguments");
template <class Args>
__global__ __launch_bounds__(kWave) void copy_list_kernel(const Args a)
{
    uint64_t src = a.src[blockIdx.y], dst = a.dst[blockIdx.y];
    uint32_t nvec = a.nvec[blockIdx.y];
    pin(src, dst, nvec);
    copy_tile(blockIdx.x, src, dst, nvec);
}

// Up to 8 pieces of one bucket: all of one length, each to its place in the bucket.  grid = (tiles of a piece, pieces).
struct CopyBucketArgs {
    static constexpr uint32_t kPieces = 8;
    uint64_t src[kPieces];
    uint64_t dst;
    uint64_t slots;                         // a piece's place in the bucket, 8 bits each
    uint32_t nvec;
};
static_assert(sizeof(CopyBucketArgs) <= kFewBytes && HZP_MAX_GROUP <= 256, "kernel arguments");
__global__ __launch_bounds__(kWave) void copy_bucket_kernel(const CopyBucketArgs a)
{
    uint64_t src = a.src[blockIdx.y], dst = a.dst, slots = a.slots;
    uint32_t nvec = a.nvec;
    pin(src, dst, slots, nvec);
    copy_tile(blockIdx.x, src, dst + (slots >> (8 * blockIdx.y) & 255u) * nvec * 16, nvec);
}

// Layers of one length, at equal distances in every source and in the output (the blocks of a transformer in an arena, or in one buffer per
// source): up to 8 pieces of the first layer and the two distances, in place of a list of pieces or of layers (1.5 to 4 KB).  Lists / so,
// us, calls in a row: 8 layers of 4 pieces of 2 KB 3.5 / 3.25, 16 of 8 3.8 / 3.4, 60 of 2 5.2 / 4.6, 120 of 8 7.7 / 6.25, 300 of 2 12.4 /
// 8.2 (two launches), 32 of 4 of 128 KB 6.0 / 5.6, of 2 MB 78.9 / 78.7; on the device alone .98.
// grid = (tiles of a piece, pieces, layers).
struct CopyStackArgs {
    CopyBucketArgs first;                   // (its output the first layer's)
    uint64_t src_step, dst_step;            // from one layer to the next
};
static_assert(sizeof(CopyStackArgs) <= kFewBytes, "kernel arguments");
__global__ __launch_bounds__(kWave) void copy_stack_kernel(const CopyStackArgs a)
{
    uint64_t src = a.first.src[blockIdx.y], dst = a.first.dst, slots = a.first.slots, src_step = a.src_step, dst_step = a.dst_step;
    uint32_t nvec = a.first.nvec;
    pin(src, dst, slots, src_step, dst_step, nvec);
    copy_tile(blockIdx.x, src + blockIdx.z * src_step, dst + blockIdx.z * dst_step + (slots >> (8 * blockIdx.y) & 255u) * nvec * 16, nvec);
}

// Many layers whose pieces lie at the same distances from the first layer's in every source (the layers of an arena, or
// of one buffer per source): one pointer per source and a record per layer, so that a launch covers 204 layers of up to 64
// pieces instead of 192 pieces.  grid = (tiles of the longest piece, sources, layers).
constexpr int kSharedLayers = 204;
struct CopySharedArgs {
    uint64_t src[HZP_MAX_GROUP];            // the first layer's piece in each source
    uint32_t slot[HZP_MAX_GROUP];           // its position in the layer's output
    struct Layer {
        uint64_t dst;
        int32_t dist;                       // of its pieces from the first layer's, in 16-byte vectors
        uint32_t nvec;
    } layer[kSharedLayers];
};
static_assert(sizeof(CopySharedArgs) <= 4096, "kernel arguments");
__global__ __launch_bounds__(kWave) void copy_shared_kernel(const CopySharedArgs a)
{
    uint64_t src = a.src[blockIdx.y], dst = a.layer[blockIdx.z].dst;
    uint32_t slot = a.slot[blockIdx.y], nvec = a.layer[blockIdx.z].nvec;
    int32_t dist = a.layer[blockIdx.z].dist;
    pin(src, dst, slot, nvec, dist);
    copy_tile(blockIdx.x, src + (int64_t)dist * 16, dst + (uint64_t)slot * nvec * 16, nvec);
}

// The same copy for pieces of different lengths (a ZeRO-3 shard rebuilt from whole and partial
// ZeRO-1 shards when the group sizes do not nest).  One-dimensional grid over the 64-vector tiles
// of all pieces, so no workgroup is launched for nothing; a workgroup counts the pieces that end at or before
// its tile, eight to a scalar load.
// The pieces follow each other in the output.
template <int PIECES>
struct CopyRangesArgs {
    static constexpr int kPieces = PIECES;
    uint64_t dst;
    uint64_t src[PIECES];
    uint32_t tile_end[PIECES];              // running count of tiles up to and including the piece; ~0 behind the last
    uint32_t vec[PIECES + 1];               // vectors ahead of the piece (modulo 2^32 behind the last)
    uint32_t n;
};
typedef CopyRangesArgs<6> CopyRangesFewArgs;
static_assert(sizeof(CopyRangesFewArgs) <= kFewBytes && HZP_MAX_GROUP % 8 == 0, "kernel arguments");
template <class Args>
__global__ __launch_bounds__(kWave) void copy_ranges_kernel(const Args a)
{
    constexpr uint32_t kRound = Args::kPieces < 8 ? Args::kPieces : 8;
    uint32_t s = 0, first = 0;              // the workgroup's piece and its first tile
    for (uint32_t i = 0; i < (Args::kPieces == kRound ? kRound : a.n); i += kRound) {
#pragma unroll
        for (uint32_t k = 0; k < kRound; ++k)
            if (blockIdx.x >= a.tile_end[i + k]) {
                s = i + k + 1;
                first = a.tile_end[i + k];
            }
    }
    uint64_t src = a.src[s], dst = a.dst;
    uint32_t begin = a.vec[s], end = a.vec[s + 1];
    pin(src, dst, begin, end);
    copy_tile(blockIdx.x - first, src, dst + (uint64_t)begin * 16, end - begin);
}

// ---------------------------------------------------------------------------------------
// Gather + unpack: ZeRO-3 shards -> separate, unpadded tensor buffers.
//
// A part is a run of elements that moves from one shard to one tensor.  Sources are 16-byte aligned where a part
// begins; a tensor is only element-aligned, so a part is written as up to 15 bytes of single elements to reach a
// 16-byte boundary of the destination, whole 16-byte vectors (whose source is then read unaligned), single elements.
// The kernel is the plain copy's: one vector per lane, pointers and lengths in the argument block.
//   - Parts of about equal length (the host cuts a few long ones to that end): grid = (tiles of the longest part, parts),
//     one round of scalar loads before a wavefront asks for data.
//   - FLAT, parts of very different lengths: a grid without surplus workgroups over the tiles of all parts; a workgroup
//     counts the parts that end at or before its tile, 64 to a load.
// (Finding the piece of a chunk in device tables took four rounds, and even at full occupancy those bound the rate. MoE
// layer of 199 tensors 6.57 -> 6.75 TB/s, dense layer 6.48 -> 6.75, odd sizes 5.91 -> 6.35, 25 MB layers 4.31 -> 5.28.)
//
// BOTH: the part is also copied to its place in the layer bucket, aligned as the shard is, together with the padding
// behind it in the same shard (`n_bucket` >= n elements, whole vectors).  A part may be padding alone (n = 0).
// Dense layer into bucket and tensors: two kernels 981 us, one 749.
// ---------------------------------------------------------------------------------------
template <int PARTS, bool BOTH, bool FLAT>
struct UnpackListArgs {
    static constexpr int kParts = PARTS;
    static constexpr bool kBoth = BOTH, kFlat = FLAT;
    uint64_t src[PARTS], dst[PARTS];
    uint64_t bucket[BOTH ? PARTS : 1];
    uint32_t n[PARTS];                  // elements
    uint32_t n_bucket[BOTH ? PARTS : 1];
    uint32_t tile_end[FLAT ? (PARTS + kWave - 1) / kWave * kWave : 1];      // running count of tiles; behind the last part ~0
    template <int ES>
    __device__ __forceinline__ void target(uint32_t part, uint64_t &to, uint32_t &count) const { to = dst[part], count = n[part]; }
};
template <int PARTS>
struct UnpackListArgs<PARTS, false, false> {
    static constexpr int kParts = PARTS;
    static constexpr bool kBoth = false, kFlat = false;
    uint64_t src[PARTS], dst[PARTS];
    uint32_t n[PARTS];
    template <int ES>
    __device__ __forceinline__ void target(uint32_t part, uint64_t &to, uint32_t &count) const { to = dst[part], count = n[part]; }
};
// Up to 8 parts of one tensor, which follow each other there.
struct UnpackTensorArgs {
    static constexpr int kParts = 8;
    static constexpr bool kBoth = false, kFlat = false;
    uint64_t src[kParts], dst;
    uint32_t begin[kParts + 1];         // elements of the tensor ahead of the part
    template <int ES>
    __device__ __forceinline__ void target(uint32_t part, uint64_t &to, uint32_t &count) const
    {
        const uint32_t first = begin[part], end = begin[part + 1];
        to = dst + (uint64_t)first * ES, count = end - first;
    }
};
static_assert(sizeof(UnpackTensorArgs) <= kFewBytes, "kernel arguments");
typedef UnpackListArgs<5, false, false> UnpackList5;
typedef UnpackListArgs<8, false, false> UnpackList8;
typedef UnpackListArgs<72, false, false> UnpackList72;
typedef UnpackListArgs<200, false, false> UnpackList200;
typedef UnpackListArgs<64, false, true> UnpackFlat64;
typedef UnpackListArgs<160, false, true> UnpackFlat160;
typedef UnpackListArgs<124, true, false> UnpackBoth124;
typedef UnpackListArgs<64, true, true> UnpackBothFlat64;
typedef UnpackListArgs<108, true, true> UnpackBothFlat108;
static_assert(sizeof(UnpackList200) <= 4096 && sizeof(UnpackFlat160) <= 4096 && sizeof(UnpackBoth124) <= 4096 &&
              sizeof(UnpackBothFlat108) <= 4096 && sizeof(UnpackList5) <= kFewBytes, "kernel arguments");

template <int ES, class Args>   // element size in bytes: 2 or 4
__global__ __launch_bounds__(kWave) void unpack_list_kernel(const Args a)
{
    constexpr uint32_t VE = 16 / ES;    // elements per vector
    typedef typename std::conditional<ES == 2, uint16_t, uint32_t>::type elem_t;
    typedef typename std::conditional<ES == 2, u32x4_a2, u32x4_a4>::type vec_unaligned_t;
    typedef const __attribute__((address_space(1))) vec_unaligned_t *vectors;
    typedef const __attribute__((address_space(1))) elem_t *elements;
    typedef __attribute__((address_space(1))) elem_t *elements_out;
    const uint32_t lane = threadIdx.x;
    uint32_t part = blockIdx.y, tile = blockIdx.x;
    if constexpr (Args::kFlat) {
        part = 0;
#pragma unroll
        for (int k = 0; k < Args::kParts; k += kWave) part += (uint32_t)__popcll(__ballot(a.tile_end[k + lane] <= blockIdx.x));
        part = __builtin_amdgcn_readfirstlane(part);
        tile -= part ? a.tile_end[part - 1] : 0u;
    }
    uint64_t src = a.src[part], dst, bucket = 0;
    uint32_t n, n_bucket = 0;
    a.template target<ES>(part, dst, n);
    if constexpr (Args::kBoth) {
        bucket = a.bucket[part];
        n_bucket = a.n_bucket[part];
    }
    pin(src, dst, bucket, n, n_bucket);
    const uint32_t q = tile * kWave + lane;
    if constexpr (Args::kBoth) {        // source, bucket and tensor are aligned alike
        if (q >= n_bucket / VE) return;
        const u32x4 val = __builtin_nontemporal_load((vectors)src + q);
        st_writethrough(reinterpret_cast<u32x4 *>(bucket) + q, val);
        if (q < n / VE) {
            st_writethrough(reinterpret_cast<u32x4 *>(dst) + q, val);
        } else if (q == n / VE) {       // the tensor's last elements
#pragma unroll
            for (uint32_t e = 0; e < VE - 1; ++e)
                if (e < n % VE) ((elements_out)dst)[q * VE + e] = (elem_t)(ES == 4 ? val[e] : val[e / 2] >> (e % 2 * 16));
        }
    } else {
        uint32_t head = ((16u - (uint32_t)(dst & 15u)) & 15u) / ES;
        if (head > n) head = n;
        const uint32_t nbody = (n - head) / VE, tail0 = head + nbody * VE;
        if (tile == 0) {
            if (lane < head) ((elements_out)dst)[lane] = ((elements)src)[lane];
            if (lane < n - tail0) ((elements_out)dst)[tail0 + lane] = ((elements)src)[tail0 + lane];
        }
        if (q >= nbody) return;
        const u32x4 val = __builtin_nontemporal_load((vectors)(src + head * (uint32_t)ES) + q);
        st_writethrough(reinterpret_cast<u32x4 *>(dst + head * (uint32_t)ES) + q, val);
    }
}

// Tensors that lie in one buffer as they do in the bucket (its parameters are views of a flat buffer of the same alignment): every
// vector's place is known without its tensor, and which of its elements belong to one is looked up while the data arrive, in the plan's
// device table of the tensors' begins and ends.  Up to 8 shards.  grid = (tiles of a shard, shards).
// One round of memory instead of a list's two (three in a flat grid), and a block of 104 bytes whatever the number of tensors.
struct UnpackPlacedArgs {
    static constexpr uint32_t kShards = 8;
    uint64_t src[kShards];
    uint64_t dst;                       // of bucket position 0
    uint64_t bucket;                    // BOTH: the layer bucket
    const u32x2 *span;                  // device: begin and end of each tensor in the bucket, in elements
    uint32_t n;                         // tensors
    uint32_t nvec;                      // vectors of a shard
    uint32_t end;                       // of the last tensor
};
static_assert(sizeof(UnpackPlacedArgs) <= kFewBytes, "kernel arguments");

// The same for up to 64 tensors that lie anywhere on 16 bytes, but no further apart than 32 bits of such units reach (nor the shards): a
// lane finds its tensor's distance with its end.  For 12 tensors the block stays within kFewBytes.
template <uint32_t N>
struct UnpackNearArgs {
    static constexpr uint32_t kTensors = N;
    uint64_t src, dst;                  // the first shard; the first tensor
    const u32x2 *span;
    uint32_t n, nvec;
    int32_t shard[UnpackPlacedArgs::kShards];       // distances from the first one, in 16 bytes
    int32_t tensor[N];
};
typedef UnpackNearArgs<12> UnpackNear12;
typedef UnpackNearArgs<64> UnpackNear64;
static_assert(sizeof(UnpackNear12) <= kFewBytes, "kernel arguments");

constexpr int32_t kNoDistance = INT32_MIN;

// FEW: at most 64 tensors, whose spans are asked for together with the data; else 64 pivots a round lead to the first that a tile meets
// (asking for up to 256 spans at once, four a lane, took as long: 100 tensors of 0.07 MB 2.61 us, with pivots 2.46).  NEAR: lane t's
// `distance` is tensor t's.
template <int ES, bool BOTH, bool FEW, bool NEAR>
__device__ __forceinline__ void unpack_spans(uint64_t src, uint64_t dst, uint64_t bucket, uint64_t table, uint32_t nvec, uint32_t n, uint32_t end,
                                             const int32_t *distances)
{
    constexpr uint32_t VE = 16 / ES, TILE = kWave * VE;         // elements of a vector, of a tile
    typedef typename std::conditional<ES == 2, uint16_t, uint32_t>::type elem_t;
    typedef const __attribute__((address_space(1))) u32x2 *spans;
    typedef __attribute__((address_space(1))) elem_t *elements_out;
    const uint32_t lane = threadIdx.x, vec = blockIdx.x * kWave + lane;
    const uint32_t first = (blockIdx.y * nvec + blockIdx.x * kWave) * VE, mine = first + lane * VE;     // bucket positions
    if (!BOTH && first >= end) return;  // padding behind the last tensor
    const u32x4 val = ld_stream<u32x4>(src, vec < nvec ? vec : nvec - 1);
    // (the bucket's store needs the data alone, so there they are asked for first, 30 tensors of 1.8 MB 3.4 -> 3.2 us; else the spans, 64
    // of 12.8 MB 6.7 -> 6.3)
    if (BOTH) __builtin_amdgcn_sched_barrier(0);
    int32_t distance = 0, away = 0;     // tensor `lane`'s, the one's that the lane's vector belongs to
    if (NEAR) distance = distances[lane < n ? lane : n - 1];
    uint32_t at = 0;                    // no tensor ahead of this one meets the tile
    for (uint32_t left = n; !FEW && left > kWave;) {
        const uint32_t stride = (left + kWave - 1) / kWave, off = lane * stride;
        const bool le = off < left && ((spans)table)[at + off][0] <= first;
        const uint32_t step = ((uint32_t)__popcll(__ballot(le)) - 1u) * stride;
        left = left - step < stride ? left - step : stride;
        at += step;
    }
    uint32_t from = 0, until = 0;       // begin and end of that tensor
    for (;;) {
        const uint32_t here = n - at;   // (64 tensors at a time; a tile meets up to 65)
        const u32x2 span = ((spans)table)[at + (lane < here ? lane : here - 1)];
        const bool is = lane < here && distance != kNoDistance;        // (always; so that the distance is asked for with the span)
        uint32_t ahead = (uint32_t)__popcll(__ballot(is && span[0] <= first));         // begin up to the tile's first element,
        uint32_t met = (uint32_t)__popcll(__ballot(is && span[0] < first + TILE));     // up to its last
        ahead = __builtin_amdgcn_readfirstlane(ahead);
        met = __builtin_amdgcn_readfirstlane(met);
        for (uint32_t k = ahead - (ahead != 0); k < met; ++k) {
            const uint32_t b = __builtin_amdgcn_readlane(span[0], k), e = __builtin_amdgcn_readlane(span[1], k);
            const bool in = mine >= b;
            until = in ? e : until;
            if (NEAR) {
                const int32_t d = (int32_t)__builtin_amdgcn_readlane((uint32_t)distance, k);
                from = in ? b : from;
                away = in ? d : away;
            }
        }
        if (FEW || met < (uint32_t)kWave || here <= (uint32_t)kWave) break;
        at += kWave;
    }
    if (vec >= nvec) return;
    if (BOTH && src != bucket + (uint64_t)(blockIdx.y * nvec) * 16)         // (else it lies in place)
        st_writethrough(bucket, mine * ES, __builtin_bit_cast(f32x4, val));
    if (mine >= until) return;
    const uint64_t to = NEAR ? dst + (int64_t)away * 16 + (uint64_t)(mine - from) * ES : dst + (uint64_t)mine * ES;
    if (until - mine >= VE) {
        if (NEAR)
            st_writethrough(reinterpret_cast<u32x4 *>(to), val);
        else
            st_writethrough(dst, mine * ES, __builtin_bit_cast(f32x4, val));
    } else {                            // the tensor's last elements
#pragma unroll
        for (uint32_t e = 0; e < VE - 1; ++e)
            if (mine + e < until) ((elements_out)to)[e] = (elem_t)(ES == 4 ? val[e] : val[e / 2] >> (e % 2 * 16));
    }
}
template <int ES, bool BOTH, bool FEW>
__global__ __launch_bounds__(kWave) void unpack_placed_kernel(const UnpackPlacedArgs a)
{
    uint64_t src = a.src[blockIdx.y], dst = a.dst, bucket = BOTH ? a.bucket : 0, table = reinterpret_cast<uint64_t>(a.span);
    uint32_t nvec = a.nvec, n = a.n, end = a.end;
    pin(src, dst, bucket, table, nvec, n, end);
    unpack_spans<ES, BOTH, FEW, false>(src, dst, bucket, table, nvec, n, end, nullptr);
}
template <int ES, class Args>
__global__ __launch_bounds__(kWave) void unpack_near_kernel(const Args a)
{
    int32_t shard = a.shard[blockIdx.y];
    uint64_t src = a.src, dst = a.dst, table = reinterpret_cast<uint64_t>(a.span);
    uint32_t nvec = a.nvec, n = a.n;
    pin(shard, src, dst, table, nvec, n);
    unpack_spans<ES, false, true, true>(at_distance(src, shard), dst, 0, table, nvec, n, ~0u, a.tensor);
}

// The same for buckets of very many tensors in short copies: one single-wavefront workgroup per chunk of at most
// kUnpackChunk elements of one piece (a run of one tensor inside one shard), found in the plan's device tables, so that a
// launch covers 400 tensors whatever their sizes.
constexpr int kUnpackTensorCap = 400;
struct UnpackArgs {
    const Piece *pieces;                // device table of the bucket, pieces [0, n_pieces)
    const uint32_t *piece_chunk;        // device: chunk_begin of the same pieces, densely packed
    uint32_t n_pieces;
    uint32_t chunk0, chunk_end;         // chunks handled by this launch
    uint32_t tensor0;
    const void *shard[HZP_MAX_GROUP];
    void *tensor[kUnpackTensorCap];     // tensor[t - tensor0]
};
static_assert(sizeof(UnpackArgs) <= 4096, "kernel arguments");

template <int ES>   // element size in bytes: 2 or 4
__global__ __launch_bounds__(kWave) void unpack_kernel(const UnpackArgs a)
{
    constexpr uint32_t VE = 16 / ES;    // elements per vector
    typedef typename std::conditional<ES == 2, uint16_t, uint32_t>::type elem_t;
    typedef typename std::conditional<ES == 2, u32x4_a2, u32x4_a4>::type vec_unaligned_t;
    const uint32_t lane = threadIdx.x;
    const uint32_t chunk = a.chunk0 + blockIdx.x;
    // Last piece whose chunk_begin <= chunk, by a 64-ary search: every lane probes one pivot and
    // a ballot counts the pivots at or below the chunk.  One round covers 64 pieces, two 4096.
    uint32_t lo = 0, n = a.n_pieces;
    while (n > kWave) {
        const uint32_t stride = (n + kWave - 1) / kWave;
        const uint32_t off = lane * stride;
        const bool le = off < n && a.piece_chunk[lo + off] <= chunk;
        const uint32_t c = (uint32_t)__popcll(__ballot(le));       // >= 1: piece lo is at or below
        const uint32_t step = (c - 1) * stride;
        n = n - step < stride ? n - step : stride;
        lo += step;
    }
    const bool le = lane < n && a.piece_chunk[lo + lane] <= chunk;
    const uint32_t piece = __builtin_amdgcn_readfirstlane(lo + (uint32_t)__popcll(__ballot(le)) - 1u);
    const Piece pc = a.pieces[piece];
    const uint64_t first = (uint64_t)(chunk - pc.chunk_begin) * kUnpackChunk;
    const uint64_t left = pc.len - first;
    const uint32_t n_el = left < kUnpackChunk ? (uint32_t)left : kUnpackChunk;
    const elem_t *src = reinterpret_cast<const elem_t *>(a.shard[pc.shard]) + pc.src_off + first;
    elem_t *dst = reinterpret_cast<elem_t *>(a.tensor[pc.tensor - a.tensor0]) + pc.dst_off + first;

    uint32_t head = (uint32_t)((16u - (uint32_t)(reinterpret_cast<uintptr_t>(dst) & 15u)) & 15u) / ES;
    if (head > n_el) head = n_el;
    const uint32_t nbody = (n_el - head) / VE;
    const uint32_t tail0 = head + nbody * VE;
    if (lane < head) dst[lane] = src[lane];
    if (lane < n_el - tail0) dst[tail0 + lane] = src[tail0 + lane];

    const elem_t *bsrc = src + head;
    u32x4 *bdst = reinterpret_cast<u32x4 *>(dst + head);
    constexpr int U = 4;
    for (uint32_t q0 = 0; q0 < nbody; q0 += kWave * U) {
        u32x4 val[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint32_t q = q0 + i * kWave + lane;
            if (q < nbody) val[i] = __builtin_nontemporal_load(reinterpret_cast<const vec_unaligned_t *>(bsrc + (size_t)q * VE));
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const uint32_t q = q0 + i * kWave + lane;
            if (q < nbody) st_writethrough(bdst + q, val[i]);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Launchers (host).  Arguments were validated by the callers in api.cpp.
// ---------------------------------------------------------------------------------------
template <class T>
struct AsIs {
    typedef T type;
};
// Launches a kernel whose arguments lie at `args`; it reads as many bytes there as its own parameters have.
template <class... P>
static hzp_status_t start_any(const char *who, const void *kernel, dim3 grid, dim3 block, unsigned lds, hipStream_t stream,
                              const P *...args)
{
    void *ptrs[] = {const_cast<void *>(static_cast<const void *>(args))...};
    (void)hipLaunchKernel(kernel, grid, block, ptrs, lds, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(HZP_ERR_HIP, "%s: launch failed: %s", who, hipGetErrorString(e));
    return HZP_OK;
}
// Launches `kernel`.  (The <<<>>> form first pushes the launch shape for a stub that pops it again: 0.1 us more a launch.)
template <class... P>
static hzp_status_t start(const char *who, void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds, hipStream_t stream,
                          const typename AsIs<P>::type &...args)
{
    return start_any(who, reinterpret_cast<const void *>(kernel), grid, block, lds, stream, &args...);
}

// Is the call being captured?  A replay costs the host nothing for each launch, so there the shortest time on the device is all that
// counts.
static bool captured(hipStream_t stream)
{
    if (!stream) return false;          // the null stream cannot be (asking costs 40 ns)
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) != hipSuccess) (void)hipGetLastError();       // (no later launch is to find it)
    return status != hipStreamCaptureStatusNone;
}

// One kernel per number of contributions: the loads of a chunk are then straight-line code (a run-time R
// puts a wait between any two of them), and all of a launch's pointers arrive in one round of scalar loads.
// (the other forms are for more than 8 contributions)
typedef std::array<const void *, HZP_MAX_REPLICAS> KernelOfR;
template <uint32_t R, bool G32, bool ACC, ReduceForm FORM>
static const void *reduce_kernel_of()
{
    if constexpr (R <= 4)
        return reinterpret_cast<const void *>(reduce_kernel<R, G32, ACC, FORM>);
    else
        return reinterpret_cast<const void *>(reduce_kernel<R, G32, ACC, FORM, Pointers<R - 4>>);
}
template <bool G32, bool ACC, ReduceForm FORM, size_t... I>
static KernelOfR reduce_kernels(std::index_sequence<I...>)
{
    return {reduce_kernel_of<I + 1, G32, ACC, I < 8 ? kReducePlain : FORM>()...};
}
template <uint32_t R, bool G32, bool ACC, ReduceForm FORM>
static const void *reduce_block_kernel_of()
{
    if constexpr (R <= 8 && FORM == kReduceNarrow)
        return nullptr;
    else
        return reinterpret_cast<const void *>(reduce_block_kernel<R, G32, ACC, R <= 8 ? kReducePlain : FORM>);
}
template <bool G32, bool ACC, ReduceForm FORM, size_t... I>
static KernelOfR reduce_block_kernels(std::index_sequence<I...>)
{
    return {reduce_block_kernel_of<I + 1, G32, ACC, FORM>()...};
}

typedef void (*ReduceEvenKernel)(u64x2, u64x2);
typedef std::array<ReduceEvenKernel, HZP_MAX_REPLICAS - kReduceEvenLeast + 1> ReduceEvenOfR;
template <bool G32, bool ACC, size_t... I>
static ReduceEvenOfR reduce_even_kernels(std::index_sequence<I...>)
{
    return {reduce_even_kernel<I + kReduceEvenLeast, G32, ACC>...};
}

typedef void (*FusedKernel)(FusedArgs);
typedef void (*FusedOneKernel)(u64x4, u64x2, uint64_t, FusedOneArgs);
template <bool G32, bool O32, FusedForm FORM, ChunkClass CLASS, size_t... I>
static constexpr std::array<FusedKernel, sizeof...(I)> fused_kernels(std::index_sequence<I...>)
{
    return {fused_adamw_kernel<I + 1, G32, O32, FORM, fused_chunk(G32, I + 1, CLASS)>...};
}
template <bool G32, bool O32, ChunkClass CLASS, size_t... I>
static constexpr std::array<FusedOneKernel, sizeof...(I)> fused_one_kernels(std::index_sequence<I...>)
{
    return {fused_one_kernel<I + 1, G32, O32, fused_chunk(G32, I + 1, CLASS), 0>...};
}

// Wavefronts per CU for the reduction, from the bytes that they ask for.  Where several chunks follow each other about 30 KiB per CU, from
// what a wavefront asks for on average; in a short launch (below about 30 us) half as much again, because there filling and draining
// the chip weighs more than the order of the requests.
// Measured at 100 M elements, TB/s with 7 / 8 / 9 / 12 wavefronts: fp32 R = 8 6.83 / 7.00 / 6.84 / 6.61, R = 16 6.92 / 6.79 / 6.61 / 6.49,
// accumulating 6.93 / 6.95 / 6.78 / 6.65 and 6.90 / 6.74 / 6.61 / 6.51; bf16 with 11 / 14 / 16 / 21: R = 6 5.54 / 6.35 / 6.74 /
// 6.72, R = 8 accumulating (11 / 12 / 14 / 16) 6.70 / 6.80 / 6.73 / 6.54, R = 12 6.37 / 6.71 / 6.60 / 6.41,
// R = 16 6.28 / 6.55 / 6.52 / 6.30, R = 32 6.07 / 6.32 / 6.40 / 6.11.
// At 25 M / 6.3 M elements with 25 -> by this rule: bf16 R = 8 6.33 / 6.04 -> 6.59 / 6.05, R = 16 6.31 / 6.10 -> 6.60 / 6.30; fp32 R = 8
// 6.00 / 5.86 -> 6.49 / 6.09.
// Where the contributions fit one chunk a wavefront has all of its bytes in flight: 42 KiB per CU, with fp32 more in short launches (66 KiB
// below 80 MB, 54 below 200 MB), and no more than 21.  With 9 / 12 / 16 / 25, against 25 in launches of up to 256 MB (160 with bf16) and 48 KiB beyond: fp32 R = 4
// accumulating 3.1 M elements 1.02 / .99 / .99 / 1.00, 6.3 M .99 / .98 / .99 / 1.00, 12.6 M .96 / .97 / 1.00 / 1.00, 25 M 1.00 / 1.04 / 1.06 /
// 1.07; R = 2 accumulating (12 / 16 / 21 / 25) 3.1 M 1.02 / .99 / .98 / .98, 12.6 M .97 / .97 / .99 / 1.00; bf16 R = 4 (16 / 18 / 21 / 25) 3.1 M .98 / .96 /
// .95 / .96, 25 M 1.01 / .99 / 1.00 / 1.01, accumulating .99 / .97 / .97 / .98 and .99 / 1.00 / 1.01 / 1.02.
static unsigned reduce_waves(bool g32, uint32_t R, uint64_t n, int accumulate)
{
    if (n <= 256u * 32u * 4u * kGroupQuads) return 0;       // all resident at once
    const uint32_t chunk = chunk_of(R, kReduceChunk), chunks = (R + chunk - 1) / chunk, es = g32 ? 4u : 2u;
    const uint64_t bytes = n * (R * es + 4u);
    const int quads = reduce_quads(R, g32, kReducePlain);
    if (chunks == 1) {
        if (quads > 1 || R * es + (accumulate ? 2u : 0u) <= 4u) return 25;
        const uint64_t moved = bytes + (accumulate ? n * 4 : 0);
        const unsigned kib = !g32 || moved >= 200000000u ? 42 : moved >= 80000000u ? 54 : 66;
        return std::min(21u, kib * 1024u / (R * es * 256u + (accumulate ? 512u : 0u)));
    }
    const bool brief = bytes < (g32 ? 256u << 20 : 160u << 20);
    const unsigned asked = (brief ? chunk * es * 256u : R * es * 256u / chunks) + (accumulate ? 512u : 0u);
    unsigned half_kib;
    if (g32)
        half_kib = brief ? 114 : R > 8 ? (accumulate ? 67 : 62) : accumulate ? 72 : 64;
    else
        half_kib = brief ? 102 : R <= 16 && bytes >= 1000000000u ? (accumulate ? 65 : 60) : 68;
    const unsigned waves = std::min(28u, half_kib * 512u / asked);
    return waves >= 10 && waves <= 12 ? waves - 1 : waves;          // (measured with one fewer)
}

// The form of a launch of `groups` groups.  Where all wavefronts are resident at once there is no cap, and a CU has groups / 256 x chunk
// x 512 B (bf16) or 1 KiB (fp32) in flight; as in long launches, what exceeds 40-48 KiB only queues.  So with more than 8
// contributions: up to 2048 groups 16 at a time (latency counts); up to that limit chunks of 4; above it chunks of 2 on two quads (half as
// many wavefronts, so that they still all fit), to where a capped launch no longer suffers from its uneven last round.
// Chunks of 4 / of 2 on two quads, us: bf16 R = 32 1.05 M elements 11.6 / 13.9, 1.47 M 19.6 / 16.8, 1.8 M 24.1 / 20.6, R = 24 2.36 M
// (capped) 21.5 / 19.9, R = 32 3.1 M (capped) 32.3 / 37.9; fp32 R = 32 0.66 M 14.9 / 14.9, 1.05 M 24.5 / 22.0, 1.8 M 40.4 / 37.2,
// 2.2 M (capped) 44.8 / 48.9; R = 9 (chunks of 3) 1.05 M 8.0 / 8.5, 1.3 M 9.8 / 9.7.
static ReduceForm reduce_form(bool g32, uint32_t R, uint64_t groups)
{
    if (R <= 8) return kReducePlain;
    if (groups <= kFewGroups) return kReduceFew;
    const uint64_t in_flight = groups * chunk_of(R, kReduceChunk) * (g32 ? 4 : 2);      // bytes per CU
    return in_flight > (g32 ? 48u << 10 : 40u << 10) && groups <= (g32 ? 8192u : 10240u) ? kReduceNarrow : kReducePlain;
}

// Launches whose wavefronts read their arguments from the block.
// So short that the launch's own time on the device is all there is (1.9 us in a graph): filling the registers adds 0.15 us to it.  With registers /
// with the block, graph replay: bf16 R = 1 of 16 k / 0.26 / 0.5 M elements 2.02 / 1.88, 2.00 / 1.92, 2.14 / 2.09 us, R = 4 of 64 / 131 / 262 k
// 2.01 / 1.88, 1.99 / 1.90, 2.33 / 2.33, R = 9 of 33 / 66 k 1.99 / 1.89, 1.99 / 1.92; fp32 R = 1 of 0.26 / 0.46 / 0.5 M 2.08 / 2.03, 2.56 / 2.59,
// 2.67 / 2.60.  (An accumulating launch takes longer: even, or up to 2 % less with registers.)
// And bf16 in chunks of 2, whose wavefronts all start at once and ask for more than the memory serves in order; the round of scalar loads
// spreads them and brings the later pointers along (2.1 M elements R = 9 / 13 / 16 / 32 8.95 / 11.3 / 13.1 / 23.0 us, with the block 8.6 /
// 10.9 / 12.7 / 22.6; fp32 1.1 / 2.1 M the other way round, 2 and 0 %).
static bool reduce_from_block(bool g32, uint32_t R, ReduceForm form, uint64_t n, int accumulate)
{
    const uint32_t es = g32 ? 4u : 2u;
    return form == kReduceNarrow ? !g32 : !accumulate && n * R * es <= (R * es <= 4 ? 2u << 20 : 1250000u);
}

// Most bytes one launch of the reduction moves (0.45 / 0.9 ms); with more streams a drift of the XCDs (below) costs more.  285 M elements
// in 1 / 2 / 4 / 8 launches: bf16 R = 16 (10.3 GB) 6.53 / 6.57 / 6.59 / 6.58 TB/s, fp32 R = 16 accumulating (20.6 GB) 6.72 / 6.78 /
// 6.84 / 6.85, bf16 R = 8 (5.7 GB) 6.89 / 6.88 / 6.82 / 6.70, R = 4 (3.4 GB) 6.84 / 6.82 / 6.80 / 6.68.
constexpr uint64_t most_reduce_bytes(uint32_t R) { return R > 8 ? 3000000000ull : 6000000000ull; }

// Longest launch of equally distant contributions by their distance, in groups.  Against pointers (120 to 272 bytes of arguments), R = 13
// to 32, up to 0.2 M elements, accumulating or not, streams 2, 4 .. 18 MiB apart, medians over the distances: calls in a row on an idle
// queue bf16 .86, fp32 .90 (R = 16 of 16 k elements 4.2 -> 3.6 us); behind a long kernel, with the host ahead, .974 and .982 (worst: bf16 R
// = 16 accumulating 0.1 M elements 1.04, fp32 R = 13 of 4 k 1.07); in graphs 1.008 and 1.003 (worst 1.06), so captured ones take pointers.
// Beyond, what starts faster collides in the memory channels (in a row, worst distance: bf16 of 0.46 / 0.52 M elements 1.12, fp32 of 0.26 M
// 1.13).  Contributions at any distances, 13 to 23 of them each by its own from the first, would take .86 in a row too, but 1.05 on average
// and up to 1.19 behind a long kernel: these take pointers.
static uint32_t reduce_even_groups(bool g32) { return g32 ? 384u : 768u; }

// Such a launch; *done is false (and nothing launched) where the distances differ.
static hzp_status_t start_reduce_even(bool g32, uint32_t R, bool accumulate, const uint64_t *g, u64x2 o, dim3 grid, unsigned lds,
                                      hipStream_t stream, bool *done)
{
    constexpr std::make_index_sequence<HZP_MAX_REPLICAS - kReduceEvenLeast + 1> all;
    static const ReduceEvenOfR kernels[2][2] = {{reduce_even_kernels<false, false>(all), reduce_even_kernels<false, true>(all)},
                                                {reduce_even_kernels<true, false>(all), reduce_even_kernels<true, true>(all)}};
    const uint64_t distance = g[1] - g[0];
    *done = true;
    for (uint32_t r = 2; r < R; ++r) *done = *done && g[r] - g[r - 1] == distance;
    if (!*done) return HZP_OK;
    const ReduceEvenKernel kernel = kernels[g32][accumulate][R - kReduceEvenLeast];
    return start("hzp_reduce_shard", kernel, grid, dim3(kWave), lds, stream, o, u64x2{g[0], distance});
}

hzp_status_t launch_reduce(bool g32, const void *const *slices, uint32_t R, uint64_t n, float scale,
                           int accumulate, float *out, hipStream_t stream)
{
    if (n == 0) return HZP_OK;
    const uint32_t es = g32 ? 4u : 2u;
    constexpr std::make_index_sequence<HZP_MAX_REPLICAS> all;
    static const KernelOfR kernels[2][2][3] = {
        {{reduce_kernels<false, false, kReducePlain>(all), reduce_kernels<false, false, kReduceFew>(all), {}},
         {reduce_kernels<false, true, kReducePlain>(all), reduce_kernels<false, true, kReduceFew>(all), {}}},
        {{reduce_kernels<true, false, kReducePlain>(all), reduce_kernels<true, false, kReduceFew>(all), reduce_kernels<true, false, kReduceNarrow>(all)},
         {reduce_kernels<true, true, kReducePlain>(all), reduce_kernels<true, true, kReduceFew>(all), reduce_kernels<true, true, kReduceNarrow>(all)}}};
    static const KernelOfR narrow_block[2] = {reduce_block_kernels<false, false, kReduceNarrow>(all),
                                              reduce_block_kernels<false, true, kReduceNarrow>(all)};
    static const KernelOfR short_block[2] = {reduce_block_kernels<false, false, kReduceFew>(all),
                                             reduce_block_kernels<true, false, kReduceFew>(all)};
    // Launches of about equal length; over a longer one the XCDs drift apart, as in the update below.
    const uint64_t launches = (n * (R * es + (accumulate ? 8u : 4u)) + most_reduce_bytes(R) - 1) / most_reduce_bytes(R);
    constexpr uint64_t kTwoGroups = 8 * kGroupQuads;        // what a wavefront with two quads per lane takes
    const uint64_t most = ((n + launches - 1) / launches + kTwoGroups - 1) / kTwoGroups * kTwoGroups;
    for (uint64_t first = 0; first < n; first += most) {
        const uint64_t here = std::min(n - first, most);
        const uint32_t nquad = (uint32_t)(here / 4);
        const ReduceForm form = reduce_form(g32, R, (nquad + kGroupQuads - 1) / kGroupQuads);
        const uint32_t quads = kGroupQuads * reduce_quads(R, g32, form);        // to a wavefront
        const dim3 grid((nquad + quads - 1) / quads), block(kWave);
        const unsigned lds = lds_for(form == kReduceNarrow ? 0 : reduce_waves(g32, R, here, accumulate));
        ReduceArgs<HZP_MAX_REPLICAS> a;         // a kernel reads its R pointers, and of the first four whatever there is
        a.out = reinterpret_cast<uint64_t>(out + first);
        a.nquad = nquad;
        a.scale = scale;
        uint64_t *const g = a.all.g;
        for (uint32_t r = 0; r < R; ++r) g[r] = reinterpret_cast<uint64_t>(slices[r]) + first * es;
        for (uint32_t r = R; r < 4; ++r) g[r] = 0;
        uint32_t scale_bits;
        std::memcpy(&scale_bits, &scale, sizeof scale_bits);
        const u64x2 o{a.out, nquad | (uint64_t)scale_bits << 32};
        hzp_status_t st = HZP_OK;
        bool done = false;
        if (R >= kReduceEvenLeast && (nquad + kGroupQuads - 1) / kGroupQuads <= reduce_even_groups(g32) && !captured(stream))
            st = start_reduce_even(g32, R, accumulate != 0, g, o, grid, lds, stream, &done);
        if (done) {
        } else if (reduce_from_block(g32, R, form, here, accumulate)) {
            const void *const kernel = form == kReduceNarrow ? narrow_block[accumulate != 0][R - 1] : short_block[g32][R - 1];
            st = start_any("hzp_reduce_shard", kernel, grid, block, lds, stream, &a);
        } else {
            const u64x4 lead{g[0], g[1], g[2], g[3]};
            st = start_any("hzp_reduce_shard", kernels[g32][accumulate != 0][form][R - 1], grid, block, lds, stream, &lead, &o, g + 4);
        }
        if (st != HZP_OK) return st;
    }
    return HZP_OK;
}

// Most groups one launch of the fused update covers (about 150 M elements, 0.6-1.3 ms of work).
// Workgroups go to the 8 XCDs round-robin, so each XCD owns a fixed eighth of the groups of a
// launch; the XCDs do not run at exactly the same speed, and over a long launch they drift apart
// (measured on MI355X: by 5-10 % of the grid after 3 ms), which spreads the addresses in flight and
// leaves the slowest XCD to finish alone.  A launch boundary lines them up again for a few
// microseconds.  Shorter launches lose to the gaps between them: R = 16, 571 M elements, launches of at most 100 / 200 / 300 /
// 400 / 600 / 800 / 1200 k groups and one launch for all 6.35 / 6.42 / 6.44 / 6.45 / 6.46 / 6.46 / 6.45 / 6.42 TB/s.
constexpr uint32_t kMaxGroupsPerLaunch = 600000;

// Segments share one set of pointers where that saves launches and a launch of segments with their own would hold fewer
// groups than this (8 M elements, about 50 us): a wavefront then has to read a record before it can ask for data, which
// costs 2-3 % of the launch, against 2.7 us for one more launch.
constexpr uint64_t kShareGroups = 32768;

// Elements [first, first + n) of segment `seg`, with the decay multiplier they share, or (runs != 0)
// with the table entries that hold theirs.
struct SegRun {
    uint32_t seg;
    uint64_t first, n;
    float wd;
    uint32_t run0, runs;
};

static inline char *out_at(const FusedSegment &f, uint64_t elem, uint32_t osz)
{
    return f.out ? static_cast<char *>(f.out) + elem * osz : nullptr;
}

// Do the elements of run b follow run a's in every stream (so that one segment can cover both)?
static bool follows(const FusedSegment *segs, const SegRun &a, const SegRun &b, uint32_t R, uint32_t gsz, uint32_t osz)
{
    const FusedSegment &f = segs[a.seg], &g = segs[b.seg];
    const uint64_t end = a.first + a.n;
    if (f.master + end != g.master + b.first || f.m + end != g.m + b.first || f.v + end != g.v + b.first) return false;
    if (!f.out != !g.out || out_at(f, end, osz) != out_at(g, b.first, osz)) return false;
    for (uint32_t r = 0; r < R; ++r)
        if (static_cast<const char *>(f.grads[r]) + end * gsz != static_cast<const char *>(g.grads[r]) + b.first * gsz) return false;
    return true;
}

// Distance of run b from run a in quads where it is the same in every stream (the output has its own).
static bool distance(const FusedSegment *segs, const SegRun &a, const SegRun &b, uint32_t R, uint32_t gsz, uint32_t osz,
                     int32_t *quads, int32_t *out_quads)
{
    const FusedSegment &f = segs[a.seg], &g = segs[b.seg];
    auto bytes = [](const void *x, uint64_t xo, const void *y, uint64_t yo) {
        return (int64_t)((reinterpret_cast<uint64_t>(y) + yo) - (reinterpret_cast<uint64_t>(x) + xo));
    };
    const int64_t d = bytes(f.master, a.first * 4, g.master, b.first * 4);     // a multiple of 16
    if (bytes(f.m, a.first * 4, g.m, b.first * 4) != d || bytes(f.v, a.first * 4, g.v, b.first * 4) != d) return false;
    for (uint32_t r = 0; r < R; ++r)
        if (bytes(f.grads[r], a.first * gsz, g.grads[r], b.first * gsz) != d / 4 * (int64_t)gsz) return false;
    int64_t o = 0;
    if (f.out) o = bytes(f.out, a.first * osz, g.out, b.first * osz) / (4 * (int64_t)osz);   // both multiples of 16 bytes
    const int64_t q = d / 16;
    if (q != (int32_t)q || o != (int32_t)o) return false;
    *quads = (int32_t)q;
    *out_quads = (int32_t)o;
    return true;
}

// The call as runs: a bucket's slice has one multiplier (most do) or needs the tables, and slices that follow
// each other in every stream and share the multiplier become one run.
static void list_runs(const hzp_plan_t *plan, const FusedSegment *segs, size_t nseg, uint32_t R, uint32_t gsz, uint32_t osz,
                      std::vector<SegRun> &runs)
{
    runs.reserve(nseg);
    for (size_t s = 0; s < nseg; ++s) {
        const FusedSegment &f = segs[s];
        const uint64_t *off = plan->run_off.data() + f.first_run;
        const uint32_t lo = (uint32_t)(std::upper_bound(off, off + f.n_runs, f.shard_begin) - off) - 1;
        const uint32_t hi = (uint32_t)(std::upper_bound(off + lo, off + f.n_runs, f.shard_begin + f.n - 1) - off);
        SegRun r{(uint32_t)s, 0, f.n, plan->run_wd[f.first_run + lo], f.first_run + lo, hi - lo > 1 ? hi - lo : 0};
        if (!runs.empty() && !r.runs && !runs.back().runs && std::memcmp(&runs.back().wd, &r.wd, sizeof r.wd) == 0 &&
            follows(segs, runs.back(), r, R, gsz, osz))
            runs.back().n += r.n;
        else
            runs.push_back(r);
    }
}

// A launch of so few groups has no cap: at most 20 wavefronts per CU are resident then, and a cap of 14 or 8 would leave a second,
// nearly empty round.  With / without one, us: fp32 0.66 M elements R = 1 / 4 / 16 5.9 / 7.4 / 13.4 and 5.3 / 6.4 / 11.3, 1.05 M
// 7.5 / 9.9 / 17.7 and 7.2 / 9.3 / 17.2, 1.3 M 8.8 / 11.5 / 22.2 and 8.7 / 11.4 / 21.6; bf16 R = 8 / 24 / 32 0.98 M 9.7 / 16.2 / 19.5
// and 9.4 / 14.2 / 16.8, 1.3 M 11.4 / 19.4 / 22.9 and 11.5 / 19.2 / 22.7; beyond, the order of the requests counts (below).
constexpr uint32_t kUncappedGroups = 5120;

// Chunks are small up to 20480 groups (fp32 10240): the streams then lie a few MB apart and partly in the memory-side cache, and what counts is
// how many of them are read side by side (buffers of one call's size, R = 12 / 16 / 24 of 1.8 M elements 17.3 / 20.1 / 24.4 us, with
// chunks of 8 18.5 / 23.9 / 28.3; 4.4 M 38.0 / 46.5 / 54, 41.8 / 46.5 / 54; from 5 M chunks of 8 take 1-4 % less; fp32 R = 4 / 8 of 1.8 M 14.6 /
// 19.9, with chunks of 4 14.9 / 20.2).  One segment whose chunks would be few and not much larger keeps small ones a little longer (small / large
// chunks on buffers of one call's size, against small ones with the pointers in the argument block: bf16 R = 7 5.3 to 7.7 M 1.00 / 1.02, 8.4 M .98 /
// .98; R = 9 / 11 / 12 5.3 to 6.1 M .99-1.00 / 1.01-1.02, 1.04-1.05, 1.02-1.03, 6.7 M .99 / .99, 1.00 / 1.00, 1.00 / 1.00; R = 13 / 16 5.3 M .98 / .96, 1.00 / .98; fp32 R = 4
// 3.6 / 4.6 / 6.1 / 7.2 M .99 / 1.05, .99 / 1.07, .99 / 1.01, .99 / .99; R = 5 / 6 / 8 2.6 to 4.1 M .98-.99 / 1.01-1.02, 1.00 / 1.01-1.03, .98 / 1.00-1.01, 4.6 M .98 /
// 1.00, 1.00 / 1.01, .98 / .96; R = 10 2.8 M .97 / .97.  In a larger allocation the large ones are 1-3 % ahead everywhere.)  Beyond, 6 to 8 bf16 contributions
// go in one chunk up to 65536 groups and in two above (one against two, both with the best number of wavefronts: R = 7 9.1 / 21 / 48 M elements
// 1.00 / 1.00 / 1.005, R = 8 1.00 / 1.00 / 1.00, 105 M 1.01; R = 6 9.1 / 21 / 33 M .98 / .99 / 1.01; several segments of 10 M together R = 6 / 8 .97 / .99).
static ChunkClass fused_class(bool g32, uint32_t R, FusedForm form, uint32_t groups)
{
    // (where wavefronts also read tables, 16 fp32 contributions are too many a little earlier: 32 segments of 0.52 M elements together,
    // R = 16, 10.1 us without and 10.5 with them; 0.38 M 8.6 and 8.4)
    if (groups <= (g32 && form != kOne ? kFewGroups / 4 * 3 : kFewGroups)) return kFew;
    uint32_t small = g32 ? 10240u : 20480u;
    if (form == kOne && g32 && R <= 9) small = R == 4 ? 24576u : 16384u;
    if (form == kOne && !g32 && R > 6 && R <= 12) small = R <= 8 ? 32768u : 24576u;
    if (groups <= small) return kMid;
    return !g32 && R > 5 && R <= 8 && groups > 65536u ? kMid : kLarge;
}

// Longest launch without a cap.  One segment's wavefronts all ask at once (their pointers are there when they start), so where a few streams
// make them ask for much they are capped earlier.  Without / with a cap (bf16 14, fp32 8), against the same with the pointers in the argument block, on
// buffers of one call's size: bf16 R = 5 / 6 / 7 / 8 of 1.25 M elements .98 / .91, 1.00 / .93, .97 / .95, .98 / .96, of 1.1 M .99 / 1.03, .97 / 1.00,
// .97 / .98, .97 / .97; R = 4 / 9 of 1.25 M .96 / .98, .97 / .99; fp32 R = 2 / 3 of 0.72 M .92 / .99, .96 / .92, of 0.79 M 1.07 / .86, 1.44 / .72, of 1.3 M
// 1.10 / .90, 1.03 / .90; R = 1 of 0.92 M 1.01 / 1.02.
static uint32_t uncapped_groups(bool g32, uint32_t R, FusedForm form)
{
    if (form == kOne && g32 && (R == 2 || R == 3)) return 2816u;
    return form == kOne && !g32 && R > 4 && R <= 8 ? 4608u : kUncappedGroups;
}

// Dynamic LDS of a launch, for so many wavefronts per CU:
//   bf16, chunks of 5 to 8: what keeps about 50 KiB in flight, 7 to 10; one more where a wavefront reads pointers or tables before it asks for data.
//   bf16, several chunks of at most 4: 14 up to 32768 groups.  Beyond, R = 6 10, R = 7 and 8 9.
//   bf16, one chunk: R = 1 to 4 11 up to 20480 groups (14 / 12 / 11 / 10 / 9 against the 14 of block arguments, mean over 1.3 to 5.2 M: R = 1 .982 / .977 /
//   .971 / .974 / .983, R = 2 .976 / .975 / .970 / .977 / .985, R = 3 .985 / .971 / .965 / .969 / .975, R = 4 .991 / .982 / .974 / .973 / .985), then 10 and, R = 4, 9;
//   R = 6 to 8 10.  With tables in between 14 up to 32768 groups and 11 beyond.
//   fp32: chunks of 4 6; small chunks 8; of R = 2, 3, 5, 6 and 9 beyond 32768 groups 7 (8 / 7: R = 2 1.8 to 7.2 M elements .99 / 1.02, 8.7 M 1.00 / 1.00;
//   R = 3 1.00 / 1.02, 1.00 / .99; R > 16 stays at 8: R = 24 / 28 of 9 to 21 M .99 / 1.01, 48 to 71 M 1.00 / .99 and .99 / 1.01).  One more with tables, and chunks
//   below 4 9.
// Means over 9 to 105 M elements against chunks of at most 4 and 9 or 11 wavefronts, by wavefronts 6 / 7 / 8 / 9 /
// 10 / 11: bf16 R = 5 1.022 / .996 / .990 / .990 / .988 / .987, R = 10 1.045 / .997 / .984 / .982 / .983 / .984, R = 16 .987 / .979 / .986 /
// .991 / .996 / 1.001, R = 24 .992 / .988 / .996 / .999 / 1.004 / 1.010; R = 8 in two chunks 1.094 / 1.032 / 1.005 / .997 / .998 / 1.000.
// Over 1.5 to 71 M against chunks of 3 and 8 wavefronts, by 4 / 5 / 6 / 7 / 8: fp32 R = 2 1.175 / 1.045 / .990 / .981 / .989, R = 4 1.077 /
// .991 / .978 / .987 / .993, R = 8 1.057 / .978 / .973 / .991 / 1.000, R = 16 1.074 / .991 / .983 / .999 / 1.008; R = 24 in chunks of 3
// 1.230 / 1.094 / 1.022 / .991 / .994.
static unsigned fused_lds(bool g32, uint32_t R, ChunkClass c, FusedForm form, uint32_t groups)
{
    if (groups <= uncapped_groups(g32, R, form)) return 0;
    const uint32_t chunk = fused_chunk(g32, R, c), asked = (chunk * (g32 ? 4u : 2u) + 12u) * 4u * kGroupQuads;
    const bool late = form == kSearched || (form == kPlain && groups <= 32768u);
    if (c == kMid && groups <= 32768u && chunk < R) return lds_for(g32 ? (late ? 9u : 8u) : 14u);
    if (g32 && chunk < 4) return lds_for(late ? 9u : R > 16 || chunk == 1 || groups <= 32768u ? 8u : 7u);
    if (g32) return lds_for(late + (groups <= 16384u ? 7u : 6u));       // (chunks of 4 in so short a launch: several segments, or R > 9)
    if (late && chunk <= 4) return lds_for(groups <= 32768u ? 14u : 11u);
    if (form == kOne && R <= 4 && groups <= 20480u) return lds_for(11u);
    return lds_for(late + (R > 5 && R <= 8 && chunk == R ? 10u : chunk == 4 ? 9u : std::min(10u, 51200u / asked)));
}

// The kernel of a form and class for each R; fp32 contributions with a bf16 output are one, already summed.
template <FusedForm FORM, ChunkClass CLASS>
static FusedKernel fused_kernel(bool g32, bool o32, uint32_t R)
{
    constexpr std::make_index_sequence<HZP_MAX_REPLICAS> all;
    static constexpr auto kernels16 = fused_kernels<false, false, FORM, CLASS>(all);
    static constexpr auto kernels32 = fused_kernels<true, true, FORM, CLASS>(all);
    return !g32 ? kernels16[R - 1] : o32 ? kernels32[R - 1] : fused_adamw_kernel<1, true, false, FORM, fused_chunk(true, 1, CLASS)>;
}
template <ChunkClass CLASS>
static FusedOneKernel fused_one_kernel_of(bool g32, bool o32, uint32_t R)
{
    constexpr std::make_index_sequence<HZP_MAX_REPLICAS> all;
    static constexpr auto kernels16 = fused_one_kernels<false, false, CLASS>(all);
    static constexpr auto kernels32 = fused_one_kernels<true, true, CLASS>(all);
    return !g32 ? kernels16[R - 1] : o32 ? kernels32[R - 1] : fused_one_kernel<1, true, false, fused_chunk(true, 1, CLASS), 0>;
}

template <bool G32, bool O32, size_t... I>
static std::array<const void *, sizeof...(I)> fused_even_kernels(std::index_sequence<I...>)
{
    return {reinterpret_cast<const void *>(fused_even_kernel<I + 1, G32, O32, fused_chunk(G32, I + 1, kFew)>)...};
}

template <FusedForm FORM>
static hzp_status_t start_fused(bool g32, bool o32, uint32_t R, const FusedArgs &a, dim3 grid, uint32_t groups, hipStream_t stream)
{
    const ChunkClass c = fused_class(g32, R, FORM, groups);
    const FusedKernel kernel = c == kFew ? fused_kernel<FORM, kFew>(g32, o32, R) : c == kMid ? fused_kernel<FORM, kMid>(g32, o32, R) : fused_kernel<FORM, kLarge>(g32, o32, R);
    return start("hzp_adamw_shard", kernel, grid, dim3(kWave), fused_lds(g32, R, c, FORM, groups), stream, a);
}

// Longest launch that takes equally distant contributions by their distance.  Against pointers, buffers of one call's size, streams 2, 4 ..
// 18 MiB apart, medians over the distances, bf16 and fp32, up to these lengths: calls in a row on an idle queue .89 and .92 (R = 16 of 16 k
// elements 4.5 -> 3.7 us), behind a long kernel, with the host ahead, .975 and .997 (worst 1.01), in graphs 1.00 and 1.005 (worst 1.02), so
// captured ones take pointers.  Beyond, what starts faster collides in the memory channels; behind a long kernel: bf16 R = 3 / 4 of 0.39 M
// elements 1.01 / 1.09, R = 9 / 12 / 16 of 0.26 M 1.11 / 1.15 / 1.04, fp32 R = 3 of 0.33 / 0.39 M 1.09 / 1.07; fp32 R >= 9 of 0.23 / 0.26 M
// in a row, worst distance, 1.13 / 1.7. (Others, each by its own distance from the first, gained 3 % in a row and lost 3 %, R = 5 14 %,
// behind a long kernel.)
static uint32_t even_groups(bool g32, uint32_t R)
{
    return R > 8 ? 640u : R == 3 || (R == 4 && !g32) ? 1024u : kFewGroups;
}

// One segment with one multiplier: its record and pointers are a.word's first.
static hzp_status_t start_fused_one(bool g32, bool o32, uint32_t R, const FusedArgs &a, uint32_t groups, hipStream_t stream)
{
    const ChunkClass c = fused_class(g32, R, kOne, groups);
    FusedOneKernel kernel = c == kFew ? fused_one_kernel_of<kFew>(g32, o32, R) : c == kMid ? fused_one_kernel_of<kMid>(g32, o32, R) : fused_one_kernel_of<kLarge>(g32, o32, R);
    if (groups > 3072 && groups <= uncapped_groups(g32, R, kOne) && (R == 1 || (R == 2 && !g32)))       // with a pause behind the state's requests
        kernel = R == 2 ? fused_one_kernel<2, false, false, 2, 96> : !g32 ? fused_one_kernel<1, false, false, 1, 96>
                 : o32 ? fused_one_kernel<1, true, true, 1, 96> : fused_one_kernel<1, true, false, 1, 96>;
    const uint64_t *const w = a.word, *const rec = a.word + R + 4;
    const uint64_t size = rec[0] >> 32 | rec[1] << 32;
    bool even = groups <= even_groups(g32, R) && !captured(stream);
    for (uint32_t r = 2; even && r < R; ++r) even = w[4 + r] - w[3 + r] == w[5] - w[4];
    if (even) {
        constexpr std::make_index_sequence<HZP_MAX_REPLICAS> all;
        static const auto kernels16 = fused_even_kernels<false, false>(all), kernels32 = fused_even_kernels<true, true>(all);
        const void *const k = !g32 ? kernels16[R - 1]
                              : o32 ? kernels32[R - 1]
                                    : reinterpret_cast<const void *>(fused_even_kernel<1, true, false, fused_chunk(true, 1, kFew)>);
        const u64x4 p{w[0], w[1], w[2], w[4]};
        const u64x2 far{R > 1 ? w[5] - w[4] : 0, reinterpret_cast<uint64_t>(a.scalars_dev)};
        const FusedEvenArgs rest{w[3], a.scalars};
        return start_any("hzp_adamw_shard", k, dim3(groups), dim3(kWave), 0, stream, &p, &far, &size, &rest);
    }
    FusedOneArgs one;
    one.out = a.word[3];
    one.scalars = a.scalars;
    std::memcpy(one.g, a.word + 4, R * sizeof one.g[0]);
    return start("hzp_adamw_shard", kernel, dim3(groups), dim3(kWave), fused_lds(g32, R, c, kOne, groups), stream, u64x4{w[0], w[1], w[2], w[4]},
                 u64x2{R > 1 ? w[5] : 0, reinterpret_cast<uint64_t>(a.scalars_dev)}, size, one);
}

hzp_status_t launch_fused(const hzp_plan_t *plan, bool g32, bool o32, uint32_t R, const FusedSegment *segs, size_t nseg,
                          const AdamScalars *scalars, const AdamScalars *scalars_dev, hipStream_t stream)
{
    const uint32_t per_seg = R + 4;
    const uint32_t gsz = g32 ? 4u : 2u, osz = o32 ? 4u : 2u;
    constexpr uint64_t kGroupElems = 4ull * kGroupQuads;
    std::vector<SegRun> runs;
    try {
        list_runs(plan, segs, nseg, R, gsz, osz, runs);
    } catch (const std::bad_alloc &) {
        return fail(HZP_ERR_NOMEM, "hzp_adamw_shard: out of host memory");
    }
    bool lookup = false;
    uint64_t groups = 0;
    for (const SegRun &r : runs) {
        lookup = lookup || r.runs;
        groups += (r.n + kGroupElems - 1) / kGroupElems;
    }
    FusedArgs a;                // the words a launch uses are all written below
    if (!plan->uniform_wd) {
        const DeviceTables *tab = nullptr;
        hzp_status_t st = device_tables(plan, &tab);
        if (st != HZP_OK) return st;
        a.run_off = tab->run_off;
        a.run_wd = tab->run_wd;
    }
    a.lookup = lookup;
    a.scalars = scalars ? *scalars : AdamScalars{};
    a.scalars_dev = scalars_dev;
    // Launches of about equal length; a run is cut where a launch is full.
    const uint64_t launches = (groups + kMaxGroupsPerLaunch - 1) / kMaxGroupsPerLaunch;
    const uint64_t most = (groups + launches - 1) / launches;
    size_t next = 0;            // first run not yet launched, and how much of it is done
    uint64_t done = 0;
    const uint32_t rec_own = kPlainRecord + a.lookup, rec_shared = rec_own + 1;
    const size_t cap_own = kTableWords / (per_seg + rec_own), cap_shared = (kTableWords - per_seg) / rec_shared;
    const bool may_share = runs.size() > cap_own && groups * cap_own / runs.size() < kShareGroups;
    SegRun part[kTableWords / 3];
    int32_t dist[kTableWords / 3], out_dist[kTableWords / 3];
    while (next < runs.size()) {
        uint32_t cnt = 0;
        uint64_t total = 0;
        bool same = may_share;
        size_t at = next;
        uint64_t at_done = done;
        while (at < runs.size() && total < most && cnt < (same ? cap_shared : cap_own)) {
            SegRun r = runs[at];
            r.first += at_done;
            r.n = std::min(r.n - at_done, (most - total) * kGroupElems);
            part[cnt] = r;
            if (same && !distance(segs, part[0], r, R, gsz, osz, &dist[cnt], &out_dist[cnt])) {
                if (cnt >= cap_own) break;      // the ones before it share their pointers: launch those
                same = false;
            }
            ++cnt;
            total += (r.n + kGroupElems - 1) / kGroupElems;
            at_done += r.n;
            if (at_done == runs[at].n) {
                ++at;
                at_done = 0;
            }
        }
        const bool shared = same && cnt > cap_own;
        a.segments = cnt;
        a.stride = shared ? rec_shared : per_seg + rec_own;
        a.ptr_stride = shared ? 0 : a.stride;
        a.dist = shared ? rec_shared - 1 : 0;
        uint32_t blocks = 0, longest = 0;
        for (uint32_t c = 0; c < cnt; ++c) {
            const SegRun &r = part[c];
            const FusedSegment &f = segs[r.seg];
            if (c == 0 || !shared) {
                uint64_t *w = a.word + (size_t)c * a.ptr_stride;
                w[0] = reinterpret_cast<uint64_t>(f.master + r.first);
                w[1] = reinterpret_cast<uint64_t>(f.m + r.first);
                w[2] = reinterpret_cast<uint64_t>(f.v + r.first);
                w[3] = reinterpret_cast<uint64_t>(out_at(f, r.first, osz));
                for (uint32_t i = 0; i < R; ++i) w[4 + i] = reinterpret_cast<uint64_t>(f.grads[i]) + r.first * gsz;
            }
            const uint32_t nb = (uint32_t)((r.n + kGroupElems - 1) / kGroupElems);
            blocks += nb;
            longest = std::max(longest, nb);
            uint64_t *w = a.word + per_seg + (size_t)c * a.stride;
            w[0] = blocks | (r.n / 4) << 32;
            if (a.lookup) {
                w[1] = r.run0 | (uint64_t)std::max(r.runs, 1u) << 32;
                w[2] = f.shard_begin + r.first;
            } else {
                uint32_t bits;
                std::memcpy(&bits, &r.wd, sizeof bits);
                w[1] = bits;
            }
            if (shared) w[a.dist] = (uint32_t)dist[c] | (uint64_t)(uint32_t)out_dist[c] << 32;
        }
        // Two-dimensional grid unless the segments differ so much in length that more than an
        // eighth of its workgroups would be surplus.
        a.grid2d = (uint64_t)longest * cnt - blocks <= blocks / 8;
        dim3 grid(blocks);
        if (a.grid2d) {
            uint64_t *w = a.word + per_seg;
            for (uint32_t c = cnt; c-- > 1;) w[(size_t)c * a.stride] -= (uint32_t)w[(size_t)(c - 1) * a.stride];
            grid = dim3(longest, cnt);
        }
        const hzp_status_t st = cnt == 1 && !a.lookup                ? start_fused_one(g32, o32, R, a, blocks, stream)
                                : a.grid2d && !shared && !a.lookup ? start_fused<kPlain>(g32, o32, R, a, grid, blocks, stream)
                                                                   : start_fused<kSearched>(g32, o32, R, a, grid, blocks, stream);
        if (st != HZP_OK) return st;
        for (uint32_t c = 0; c < cnt; ++c) {
            done += part[c].n;
            if (done == runs[next].n) {
                ++next;
                done = 0;
            }
        }
    }
    return HZP_OK;
}

// A piece that has to move.
struct Move {
    uint64_t src, dst, nvec;
};

template <class Args>
static hzp_status_t copy_list(const Move *moves, size_t n, hipStream_t stream, const char *who)
{
    Args a;
    uint64_t longest = 0;
    for (size_t s = 0; s < n; ++s) {
        a.src[s] = moves[s].src;
        a.dst[s] = moves[s].dst;
        a.nvec[s] = (uint32_t)moves[s].nvec;
        longest = std::max(longest, moves[s].nvec);
    }
    const dim3 grid((uint32_t)((longest + kWave - 1) / kWave), (uint32_t)n), block(kWave);
    return start(who, copy_list_kernel<Args>, grid, block, 0, stream, a);
}

// Most tiles of 64 vectors in one launch of a copy of many pieces (600 MB, about 180 us).  Over a longer launch the XCDs drift apart, as in the
// update; shorter ones lose to the gaps.  Post-step gather of 2.95 GB, launches of 100 / 200 / 400 / 600 / 800 / 1200 k tiles and
// one for all: 6.59 / 6.71 / 6.77 / 6.77 / 6.76 / 6.71 / 6.70 TB/s.
constexpr uint64_t kMaxTilesPerLaunch = 600000;

static uint64_t tiles_of(uint64_t nvec) { return (nvec + kWave - 1) / kWave; }

// (a grid holds fewer than 2^32 threads per dimension: one thread per vector, rounded up to whole wavefronts)
constexpr uint64_t kMostVectors = 0xFFFFFFFFull - kWave;

// How many of the next `left` units (`rows` pieces each, tiles_at(i) tiles a piece) one launch takes: at most `most` of them and
// kMaxTilesPerLaunch tiles (or one unit), with no more than an eighth and `each` surplus workgroups after every unit, and `last`
// at the end (else none).
template <class TilesAt>
static size_t take_units(size_t left, size_t most, uint64_t rows, uint64_t each, uint64_t last, TilesAt tiles_at)
{
    size_t cnt = 0;
    uint64_t tiles = 0, longest = 0;
    while (cnt < left && cnt < most) {
        const uint64_t here = tiles_at(cnt) * rows, with = tiles + here, longer = std::max(longest, here);
        if (cnt > 0 && (with > kMaxTilesPerLaunch || longer * (cnt + 1) - with > with / 8 + each)) break;
        tiles = with;
        longest = longer;
        ++cnt;
    }
    return longest * cnt - tiles > tiles / 8 + last ? 0 : cnt;
}

// A grid has the tiles of its longest piece for every piece, and a workgroup with nothing to do costs 0.15 ns, another launch
// 2.5-4 us: all that fit where no more than an eighth and 24 k workgroups are then surplus, otherwise those of about equal length (an
// eighth and 8 k surplus).  48 layers of 3 M elements between an embedding and a head of 26 M, K = 16 / 2: in one launch 65 / 36 us,
// this way, longest first, 23 / 14; 64 layers of 0.1 to 8 M, K = 16 62 -> 33.
constexpr uint64_t kSurplusAll = 24576, kSurplusEven = 8192, kSurplusNone = 2048, kNoLimit = 1ull << 62;
template <class TilesAt>
static size_t units_of_launch(size_t left, size_t most, uint64_t rows, TilesAt tiles_at)
{
    const size_t all = take_units(left, most, rows, kNoLimit, kSurplusAll, tiles_at);
    return all ? all : take_units(left, most, rows, kSurplusEven, kSurplusEven, tiles_at);
}

// One launch, with the smallest block that holds the pieces: up to 5 stay within kFewBytes (as a bucket of up to 8 shards does, which is no
// list); buckets of 64 KiB to 1 MiB from 9 to 64 shards, call after call, 4.75 us with the block of 192, 4.55 with the block of 64.
static hzp_status_t copy_one(const Move *moves, size_t n, hipStream_t stream, const char *who)
{
    if (n <= (size_t)CopyLeastArgs::kPieces) return copy_list<CopyLeastArgs>(moves, n, stream, who);
    if (n <= (size_t)CopyFewArgs::kPieces) return copy_list<CopyFewArgs>(moves, n, stream, who);
    if (n <= (size_t)CopyGroupArgs::kPieces) return copy_list<CopyGroupArgs>(moves, n, stream, who);
    return copy_list<CopyManyArgs>(moves, n, stream, who);
}

// Launches over the pieces of many layers.
static hzp_status_t copy_moves(const Move *moves, size_t n, hipStream_t stream, const char *who)
{
    for (size_t at = 0; at < n;) {
        const size_t cnt = units_of_launch(n - at, CopyManyArgs::kPieces, 1, [&](size_t i) { return tiles_of(moves[at + i].nvec); });
        const hzp_status_t st = copy_one(moves + at, cnt, stream, who);
        if (st != HZP_OK) return st;
        at += cnt;
    }
    return HZP_OK;
}

hzp_status_t launch_concat(const void *const *srcs, uint32_t n_shards, uint64_t bytes_per_shard, void *dst,
                           hipStream_t stream)
{
    if (bytes_per_shard == 0) return HZP_OK;
    const uint64_t nvec = bytes_per_shard / 16;
    if (nvec > kMostVectors) return fail(HZP_ERR_UNSUPPORTED, "hzp_gather_layer: shard of 64 GiB or more");
    const uint64_t to = reinterpret_cast<uint64_t>(dst);
    CopyBucketArgs few;
    few.dst = to;
    few.slots = 0;
    few.nvec = (uint32_t)nvec;
    Move moves[HZP_MAX_GROUP];
    size_t n = 0;
    for (uint32_t s = 0; s < n_shards; ++s) {
        const uint64_t from = reinterpret_cast<uint64_t>(srcs[s]), place = to + s * bytes_per_shard;
        if (from == place) continue;                            // it lies in place
        if (n < few.kPieces) {
            few.src[n] = from;
            few.slots |= (uint64_t)s << (8 * n);
        }
        moves[n++] = {from, place, nvec};
    }
    // (one bucket's pieces stay one launch: cut into launches, 1.7-2.3 GB buckets copy no faster)
    if (n == 0) return HZP_OK;
    if (n > few.kPieces) return copy_one(moves, n, stream, "hzp_gather_layer");
    return start("hzp_gather_layer", copy_bucket_kernel, dim3((uint32_t)tiles_of(nvec), (uint32_t)n), dim3(kWave), 0, stream, few);
}

// Layers whose pieces lie at equal distances, in launches of kSharedLayers; *done is false (and nothing launched) where
// they do not.  Every layer leaves out the same pieces (those that lie in place).
static hzp_status_t copy_shared(const void *const *srcs, uint32_t per_layer, const uint64_t *bytes_per_piece,
                                void *const *dsts, const std::vector<uint32_t> &layers, hipStream_t stream, bool *done)
{
    *done = false;
    if (layers.empty()) return HZP_OK;
    const uint32_t first = layers[0];
    auto piece = [&](uint32_t l, uint32_t k) { return reinterpret_cast<uint64_t>(srcs[(size_t)l * per_layer + k]); };
    auto place = [&](uint32_t l, uint32_t k) { return reinterpret_cast<uint64_t>(dsts[l]) + k * bytes_per_piece[l]; };
    CopySharedArgs a;
    uint32_t n_src = 0;
    for (uint32_t k = 0; k < per_layer; ++k)
        if (piece(first, k) != place(first, k)) {
            a.src[n_src] = piece(first, k);
            a.slot[n_src++] = k;
        }
    if (n_src == 0) return HZP_OK;
    for (uint32_t l : layers) {
        const int64_t d = (int64_t)(piece(l, a.slot[0]) - a.src[0]);
        if (d / 16 != (int32_t)(d / 16)) return HZP_OK;
        for (uint32_t k = 0, i = 0; k < per_layer; ++k) {
            const bool listed = i < n_src && a.slot[i] == k;
            if (listed == (piece(l, k) == place(l, k))) return HZP_OK;
            if (listed && (int64_t)(piece(l, k) - a.src[i++]) != d) return HZP_OK;
        }
    }
    *done = true;
    for (size_t at = 0; at < layers.size();) {
        const size_t cnt = units_of_launch(layers.size() - at, kSharedLayers, n_src,
                                           [&](size_t i) { return tiles_of(bytes_per_piece[layers[at + i]] / 16); });
        uint32_t longest = 0;
        for (size_t i = 0; i < cnt; ++i) {
            const uint32_t l = layers[at + i];
            const int64_t d = (int64_t)(piece(l, a.slot[0]) - a.src[0]);
            longest = std::max(longest, (uint32_t)(bytes_per_piece[l] / 16));
            a.layer[i] = {reinterpret_cast<uint64_t>(dsts[l]), (int32_t)(d / 16), (uint32_t)(bytes_per_piece[l] / 16)};
        }
        const dim3 grid((uint32_t)tiles_of(longest), n_src, (uint32_t)cnt), block(kWave);
        const hzp_status_t st = start("hzp_gather_layers", copy_shared_kernel, grid, block, 0, stream, a);
        if (st != HZP_OK) return st;
        at += cnt;
    }
    return HZP_OK;
}

// Layers of one length at equal distances, in one launch; *done is false (and nothing launched) where they are not, would exceed a launch
// or have more than 8 pieces that move, and where some of a source's pieces lie in place.
static hzp_status_t copy_stack(const void *const *srcs, uint32_t per_layer, const uint64_t *bytes_per_piece, void *const *dsts,
                               const std::vector<uint32_t> &layers, hipStream_t stream, bool *done)
{
    *done = false;
    const size_t n = layers.size();
    const uint64_t bytes = bytes_per_piece[layers[0]], nvec = bytes / 16;
    if (n > 4096 || tiles_of(nvec) * per_layer * n > kMaxTilesPerLaunch) return HZP_OK;     // (a grid has at most 65535 planes)
    auto piece = [&](size_t i, uint32_t k) { return reinterpret_cast<uint64_t>(srcs[(size_t)layers[i] * per_layer + k]); };
    auto place = [&](size_t i) { return reinterpret_cast<uint64_t>(dsts[layers[i]]); };
    uint32_t moving = 0;
    for (uint32_t k = 0; k < per_layer; ++k) moving += piece(0, k) != place(0) + k * bytes;
    if (moving > CopyBucketArgs::kPieces) return HZP_OK;
    CopyStackArgs a;
    a.first.dst = place(0);
    a.first.slots = 0;
    a.first.nvec = (uint32_t)nvec;
    a.src_step = 0;
    a.dst_step = n > 1 ? place(1) - place(0) : 0;
    for (size_t i = 1; i < n; ++i)
        if (bytes_per_piece[layers[i]] != bytes || place(i) - place(i - 1) != a.dst_step) return HZP_OK;
    moving = 0;
    for (uint32_t k = 0; k < per_layer; ++k) {
        const bool still = piece(0, k) == place(0) + k * bytes;
        const uint64_t step = n > 1 ? piece(1, k) - piece(0, k) : 0;
        for (size_t i = 1; i < n; ++i)
            if (piece(i, k) - piece(i - 1, k) != step || (piece(i, k) == place(i) + k * bytes) != still) return HZP_OK;
        if (still) continue;
        if (moving && step != a.src_step) return HZP_OK;
        a.src_step = step;
        a.first.src[moving] = piece(0, k);
        a.first.slots |= (uint64_t)k << (8 * moving++);
    }
    *done = true;
    if (moving == 0) return HZP_OK;
    return start("hzp_gather_layers", copy_stack_kernel, dim3((uint32_t)tiles_of(nvec), moving, (uint32_t)n), dim3(kWave), 0, stream, a);
}

// Sorts layers by the length of their pieces, longest first, equal ones in order.  Mostly they are nearly so (equal layers beside a few
// longer ones), and insertion is enough: 256 small layers between two longer ones in two launches 14.6 us a call with a general sort
// that compares lengths, 11.8 this way, 11.3 unsorted.
static void longest_first(std::vector<uint32_t> &layers, const uint64_t *bytes_per_piece)
{
    const size_t n = layers.size();
    std::vector<uint64_t> keys(n);
    for (size_t i = 0; i < n; ++i) keys[i] = (0xFFFFFFFFull - bytes_per_piece[layers[i]] / 16) << 32 | layers[i];    // (below 2^32 vectors)
    size_t moves_left = 4 * n;
    for (size_t i = 1; i < n && moves_left; ++i) {
        const uint64_t key = keys[i];
        size_t at = i;
        for (; at && keys[at - 1] > key && moves_left; --moves_left, --at) keys[at] = keys[at - 1];
        keys[at] = key;
    }
    if (!moves_left) std::sort(keys.begin(), keys.end());
    for (size_t i = 0; i < n; ++i) layers[i] = (uint32_t)keys[i];
}

hzp_status_t launch_concat_layers(const void *const *srcs, uint32_t per_layer, const uint64_t *bytes_per_piece,
                                  void *const *dsts, uint32_t n_layers, hipStream_t stream)
{
    for (uint32_t l = 0; l < n_layers; ++l)
        if (bytes_per_piece[l] / 16 > kMostVectors) return fail(HZP_ERR_UNSUPPORTED, "hzp_gather_layers: shard of 64 GiB or more");
    std::vector<uint32_t> layers;   // those that hold anything
    try {
        layers.reserve(n_layers);
        for (uint32_t l = 0; l < n_layers; ++l)
            if (bytes_per_piece[l]) layers.push_back(l);
    } catch (const std::bad_alloc &) {
        return fail(HZP_ERR_NOMEM, "hzp_gather_layers: out of host memory");
    }
    if (layers.empty()) return HZP_OK;
    const size_t pieces = layers.size() * per_layer;
    if (pieces > CopyLeastArgs::kPieces) {
        bool done = false;
        const hzp_status_t st = copy_stack(srcs, per_layer, bytes_per_piece, dsts, layers, stream, &done);
        if (st != HZP_OK || done) return st;
    }
    const size_t lists = (pieces + CopyManyArgs::kPieces - 1) / CopyManyArgs::kPieces;
    const bool shared = lists > (layers.size() + kSharedLayers - 1) / kSharedLayers;        // where that saves launches
    // Longest pieces first, so that neighbours differ little; not where the launches as they come have next to no surplus.
    size_t cnt = 1, at = 0;
    for (; cnt && at < layers.size(); at += cnt)
        cnt = take_units(layers.size() - at, shared ? kSharedLayers : layers.size(), per_layer, kNoLimit, kSurplusNone,
                         [&](size_t i) { return tiles_of(bytes_per_piece[layers[at + i]] / 16); });
    const bool ordered = cnt != 0, one_launch = cnt == layers.size();
    Move few[CopyManyArgs::kPieces], *moves = few;
    std::unique_ptr<Move[]> listed;
    try {
        if (!ordered) longest_first(layers, bytes_per_piece);
        if (shared) {
            bool done = false;
            const hzp_status_t st = copy_shared(srcs, per_layer, bytes_per_piece, dsts, layers, stream, &done);
            if (st != HZP_OK || done) return st;
        }
        if (lists > 1) listed.reset(moves = new Move[pieces]);
    } catch (const std::bad_alloc &) {
        return fail(HZP_ERR_NOMEM, "hzp_gather_layers: out of host memory");
    }
    size_t n = 0;                   // the pieces that have to move
    for (uint32_t l : layers) {
        const uint64_t bytes = bytes_per_piece[l];
        for (uint32_t k = 0; k < per_layer; ++k) {
            const uint64_t src = reinterpret_cast<uint64_t>(srcs[(size_t)l * per_layer + k]);
            const uint64_t dst = reinterpret_cast<uint64_t>(dsts[l]) + k * bytes;
            if (src != dst) moves[n++] = {src, dst, bytes / 16};        // else the piece lies in place
        }
    }
    if (one_launch && lists == 1) return n ? copy_one(moves, n, stream, "hzp_gather_layers") : HZP_OK;
    return copy_moves(moves, n, stream, "hzp_gather_layers");
}

template <class Args>
static hzp_status_t copy_ranges(const Move *moves, uint32_t n, void *dst, uint32_t tiles, hipStream_t stream)
{
    Args a;
    std::fill(std::begin(a.tile_end), std::end(a.tile_end), ~0u);
    a.dst = reinterpret_cast<uint64_t>(dst);
    a.n = n;
    uint32_t end = 0, vec = 0;
    for (uint32_t s = 0; s < n; ++s) {
        a.src[s] = moves[s].src;
        a.tile_end[s] = end += (uint32_t)tiles_of(moves[s].nvec);
        a.vec[s] = vec;
        a.vec[s + 1] = vec += (uint32_t)moves[s].nvec;
    }
    return start("hzp_gather_shard", copy_ranges_kernel<Args>, dim3(tiles), dim3(kWave), 0, stream, a);
}

hzp_status_t launch_concat_ranges(const void *const *srcs, const uint64_t *dst_off, const uint64_t *bytes,
                                  uint32_t n, void *dst, hipStream_t stream)
{
    Move moves[HZP_MAX_GROUP];
    uint64_t tiles = 0, total = 0;
    bool uniform = true;
    for (uint32_t s = 0; s < n; ++s) {
        if (bytes[s] / 16 > kMostVectors || dst_off[s] / 16 > 0xFFFFFFFFull)
            return fail(HZP_ERR_UNSUPPORTED, "hzp_gather_shard: shard larger than 64 GiB");
        moves[s] = {reinterpret_cast<uint64_t>(srcs[s]), reinterpret_cast<uint64_t>(dst) + dst_off[s], bytes[s] / 16};
        tiles += tiles_of(moves[s].nvec);
        uniform = uniform && bytes[s] == bytes[0] && dst_off[s] == s * bytes[0];
        total += bytes[s];
    }
    if (total == 0) return HZP_OK;
    if (uniform) return launch_concat(srcs, n, bytes[0], dst, stream);     // equal whole pieces
    if (tiles > 0x7FFFFFFFull) return fail(HZP_ERR_UNSUPPORTED, "hzp_gather_shard: shard too large for one launch");
    if (n <= (uint32_t)CopyRangesFewArgs::kPieces) return copy_ranges<CopyRangesFewArgs>(moves, n, dst, (uint32_t)tiles, stream);
    if (n <= 8) return copy_ranges<CopyRangesArgs<8>>(moves, n, dst, (uint32_t)tiles, stream);
    return copy_ranges<CopyRangesArgs<HZP_MAX_GROUP>>(moves, n, dst, (uint32_t)tiles, stream);
}

// A run of elements to move; with a bucket beside the tensors, its place there and its length with the padding behind it.
struct Part {
    uint64_t src, dst, n, bucket, n_bucket;
    uint64_t length() const { return std::max(n, n_bucket); }
};
constexpr uint64_t kMostInPart = 1ull << 30;        // (a part's length has 32 bits)

// Where the launches find their parts: a list, or the pieces of a bucket and the caller's pointers as they are (short calls
// show the time of a list made first: 100 / 160 small tensors, 4.6 / 4.8 us a call with one, 4.2 / 4.3 without).
struct ListedParts {
    const Part *part;
    uint64_t length(size_t i) const { return part[i].length(); }
    const Part &operator[](size_t i) const { return part[i]; }
    ListedParts from(size_t i) const { return {part + i}; }
};
template <int ES>
struct PieceParts {
    const Piece *piece;
    const void *const *shards;
    void *const *tensors;               // tensors[0] is tensor t_begin's
    uint32_t t_begin;
    uint64_t length(size_t i) const { return piece[i].len; }
    Part operator[](size_t i) const
    {
        const Piece &p = piece[i];
        return {reinterpret_cast<uint64_t>(shards[p.shard]) + p.src_off * ES,
                reinterpret_cast<uint64_t>(tensors[p.tensor - t_begin]) + p.dst_off * ES, p.len, 0, 0};
    }
    PieceParts from(size_t i) const { return {piece + i, shards, tensors, t_begin}; }
};

// Are parts of about equal length, so that a grid with the longest part's tiles for each has few workgroups with nothing to do?
// `tile` elements make a tile.  100 parts of 80 MB, every tenth longer by 5 / 10 / 20 / 40 / 80 %, even / flat grid, us: 27.9 / 29.1, 27.7 /
// 29.1, 25.2 / 26.4, 27.6 / 29.1, 30.2 / 29.2 (surplus 4 / 9 / 18 / 35 / 67 %): the line is a cautious one.
static bool even_parts(size_t n, uint64_t total, uint64_t longest, uint64_t tile)
{
    return longest * n <= total + std::max(total / 16, 256 * tile);
}

// Lists of parts in the argument block, or pieces found in the device tables?  The lists copy 5-20 % faster (2.0-2.3 us on the device
// against 2.6-3.0 for up to 100 short parts), but 200 even or 160 uneven parts fill a launch, and the tables' launch covers 400 tensors.
// So tables where lists take several launches that are not long enough (tables / lists, us): 16 MB a launch of even parts (243 parts of
// 31 MB 13.7 / 14.1, of 63 MB 23.3 / 22.4; 800 of 52 MB 23.9 / 25.6, of 105 MB 40.3 / 39.1), 128 MB of uneven ones (243 parts of 126 MB
// 46.7 / 47.2, of 252 MB 88.8 / 88.8; 800 of 26 MB 16.9 / 28.7, of 210 MB 79.3 / 85.6, of 839 MB 296 / 296), 62 MB of those where the
// longest lies at an odd address (243 parts of 63 MB 27.6 / 27.9, of 126 MB 56.9 / 53.5; 2000 of 1.05 GB 490 / 431).
static bool lists_pay(size_t n, uint64_t total, uint64_t longest, bool odd, uint32_t es)
{
    const bool even = even_parts(n, total, longest, kWave * 16 / es);
    const uint64_t most = even ? UnpackList200::kParts : UnpackFlat160::kParts, launches = (n + most - 1) / most;
    return launches == 1 || total * es >= (even ? 16 : odd ? 62 : 128) * 1000000 * launches;
}

// One launch over parts, cut into runs of at most `cut` elements.
template <class Args, int ES, class Parts>
static hzp_status_t unpack_list(const Parts &parts, size_t n, uint64_t cut, hipStream_t stream, const char *who)
{
    Args a;
    uint32_t cnt = 0, tiles = 0;
    uint64_t longest = 0;
    for (size_t i = 0; i < n; ++i) {
        const Part p = parts[i];
        for (uint64_t at = 0; at < p.length(); at += cut) {
            const uint64_t len = std::min(p.length() - at, cut);
            a.src[cnt] = p.src + at * ES;
            a.dst[cnt] = p.dst + at * ES;
            a.n[cnt] = (uint32_t)(p.n > at ? std::min(p.n - at, cut) : 0);
            if constexpr (Args::kBoth) {
                a.bucket[cnt] = p.bucket + at * ES;
                a.n_bucket[cnt] = (uint32_t)len;
            }
            // (a part with an unaligned destination has fewer whole vectors, never more)
            if constexpr (Args::kFlat) a.tile_end[cnt] = tiles += (uint32_t)std::max<uint64_t>(1, tiles_of(len * ES / 16));
            longest = std::max(longest, len);
            ++cnt;
        }
    }
    dim3 grid((uint32_t)std::max<uint64_t>(1, tiles_of(longest * ES / 16)), cnt);
    if constexpr (Args::kFlat) {
        std::fill(a.tile_end + cnt, std::end(a.tile_end), ~0u);
        grid = dim3(tiles);
    }
    return start(who, unpack_list_kernel<ES, Args>, grid, dim3(kWave), 0, stream, a);
}

// Launches over a list of parts: each takes parts while they fit its table and hold no more than kMaxTilesPerLaunch tiles. The smaller
// blocks save the host what they leave out (5 parts stay within kFewBytes; 4 MB in 24 / 48 / 72 even parts, block of 72 / of 200, us: 4.9 /
// 5.1, 5.1 / 5.4, 5.3 / 5.5).
template <int ES, bool BOTH, class Parts>
static hzp_status_t unpack_parts(const Parts &parts, size_t n, hipStream_t stream, const char *who)
{
    constexpr uint64_t kTile = kWave * 16 / ES;     // elements of a tile
    constexpr size_t cap = BOTH ? UnpackBoth124::kParts : UnpackList200::kParts;
    constexpr size_t cap_flat = BOTH ? UnpackBothFlat108::kParts : UnpackFlat160::kParts;
    for (size_t at = 0; at < n;) {
        const Parts first = parts.from(at);
        size_t cnt = 0;
        uint64_t total = 0, longest = 0;
        auto take = [&](size_t most) {
            cnt = 0;
            total = longest = 0;
            while (at + cnt < n && cnt < most) {
                const uint64_t len = first.length(cnt);
                if (cnt > 0 && (total + len) / kTile > kMaxTilesPerLaunch) break;
                total += len;
                longest = std::max(longest, len);
                ++cnt;
            }
        };
        take(cap);
        const bool even = even_parts(cnt, total, longest, kTile);
        uint64_t cut = 0;           // 0: a flat grid
        if (even) {
            cut = std::min(longest, kMostInPart);       // (a part beyond that is alone: a launch has fewer tiles)
        } else if (cnt <= cap / 9 && total * ES >= 1000000) {       // cut at an eighth more than total / cap, they fill the table
            // (cut / flat, us: 3 to 22 very uneven parts of 20 MB 8.6-9.0 / 8.9-9.3, of 300 MB 94-107 / 97-110; 40 of 300 MB 101 / 105; call
            // after call and on the device alone, 12 of 0.4 MB 4.8 / 4.5 and 2.55 / 2.52, 0.8 MB 4.8 / 4.5 and 2.84 / 2.74, 1.5 MB 4.8 / 4.6
            // and 3.1 / 3.3, 4 MB 4.7 / 4.9 and 4.1 / 4.3)
            cut = (total + (cap - cnt) - 1) / (cap - cnt);
            cut = std::min(longest, (cut + kTile - 1) / kTile * kTile);
        } else if (cnt > cap_flat) {
            take(cap_flat);
        }
        hzp_status_t st;
        if constexpr (BOTH)
            st = cut                   ? unpack_list<UnpackBoth124, ES>(first, cnt, cut, stream, who)
                 : cnt <= 64           ? unpack_list<UnpackBothFlat64, ES>(first, cnt, longest, stream, who)
                                       : unpack_list<UnpackBothFlat108, ES>(first, cnt, longest, stream, who);
        else
            st = !cut                  ? (cnt <= 64 ? unpack_list<UnpackFlat64, ES>(first, cnt, longest, stream, who)
                                                    : unpack_list<UnpackFlat160, ES>(first, cnt, longest, stream, who))
                 : cut < longest || cnt > 72 ? unpack_list<UnpackList200, ES>(first, cnt, cut, stream, who)
                 : cnt <= 5            ? unpack_list<UnpackList5, ES>(first, cnt, cut, stream, who)
                 : cnt <= 8            ? unpack_list<UnpackList8, ES>(first, cnt, cut, stream, who)
                                       : unpack_list<UnpackList72, ES>(first, cnt, cut, stream, who);
        if (st != HZP_OK) return st;
        at += cnt;
    }
    return HZP_OK;
}

// One tensor of below 2^32 elements in up to 8 parts of about equal length.
template <int ES>
static hzp_status_t unpack_tensor(const Piece *pieces, size_t n, const void *const *shards, void *tensor, uint64_t longest,
                                  hipStream_t stream)
{
    UnpackTensorArgs a;
    a.dst = reinterpret_cast<uint64_t>(tensor);
    a.begin[0] = 0;
    for (size_t i = 0; i < n; ++i) {
        a.src[i] = reinterpret_cast<uint64_t>(shards[pieces[i].shard]) + pieces[i].src_off * ES;
        a.begin[i + 1] = (uint32_t)(pieces[i].dst_off + pieces[i].len);
    }
    const dim3 grid((uint32_t)std::max<uint64_t>(1, tiles_of(longest * ES / 16)), (uint32_t)n);
    return start("hzp_gather_layer", unpack_list_kernel<ES, UnpackTensorArgs>, grid, dim3(kWave), 0, stream, a);
}

// What the launches of one unpacking call share.
struct UnpackCall {
    const Piece *pieces;                // device tables that hold the bucket's pieces from entry 0
    const uint32_t *piece_chunk;
    const BucketRec &b;
    const void *const *shards;
    uint32_t n_shards;
    hipStream_t stream;
};

// One launch: tensors [t0, t1), whose pieces are [p0, p1).
static hzp_status_t start_unpack(const UnpackCall &u, void *const *tensors, uint32_t t0, uint32_t t1, size_t p0, size_t p1,
                                 const char *who)
{
    UnpackArgs a;
    a.pieces = u.pieces;
    a.piece_chunk = u.piece_chunk;
    a.n_pieces = (uint32_t)u.b.pieces.size();
    a.chunk0 = u.b.pieces[p0].chunk_begin;
    a.chunk_end = p1 < u.b.pieces.size() ? u.b.pieces[p1].chunk_begin : u.b.n_chunks;
    a.tensor0 = t0;
    for (uint32_t s = 0; s < u.n_shards; ++s) a.shard[s] = u.shards[s];
    for (uint32_t t = t0; t < t1; ++t) a.tensor[t - t0] = tensors[t - t0];
    return start(who, u.b.cls == HZP_CLASS_F32 ? unpack_kernel<4> : unpack_kernel<2>, dim3(a.chunk_end - a.chunk0), dim3(kWave), 0, u.stream, a);
}

// First piece at or behind `from` of a tensor or a later one (pieces are sorted by tensor).
static size_t first_piece(const BucketRec &b, size_t from, uint32_t tensor)
{
    return (size_t)(std::lower_bound(b.pieces.begin() + from, b.pieces.end(), tensor,
                                     [](const Piece &p, uint32_t t) { return p.tensor < t; }) - b.pieces.begin());
}

// Launches of the unpack kernel for tensors [t_begin, t_end) of a bucket.
static hzp_status_t launch_unpack_with(const UnpackCall &u, void *const *tensors, uint32_t t_begin, uint32_t t_end,
                                       const char *who)
{
    // Tensors travel in the argument block, kUnpackTensorCap at a time; pieces are sorted by tensor.
    size_t p0 = first_piece(u.b, 0, t_begin);
    for (uint32_t t0 = t_begin; t0 < t_end; t0 += kUnpackTensorCap) {
        const uint32_t t1 = std::min<uint32_t>(t_end, t0 + kUnpackTensorCap);
        const size_t p1 = first_piece(u.b, p0, t1);
        const hzp_status_t st = start_unpack(u, tensors + (t0 - t_begin), t0, t1, p0, p1, who);
        if (st != HZP_OK) return st;
        p0 = p1;
    }
    return HZP_OK;
}

// Distance of one address from another in units of 16 bytes, where it is a whole number that fits 32 bits (else *fits becomes false).
static int32_t units_apart(uint64_t to, uint64_t from, bool *fits)
{
    const int64_t d = (int64_t)(to - from) / 16;
    *fits = *fits && d == (int32_t)d && d != kNoDistance && (to - from) % 16 == 0;
    return (int32_t)d;
}

// Do all tensors of the bucket lie in one buffer as they do in the bucket?  Then *origin is where position 0 would be.
static bool placed_as_in_bucket(const hzp_plan_t *plan, const BucketRec &b, void *const *tensors, uint32_t es, uint64_t *origin)
{
    auto place = [&](uint32_t t) { return reinterpret_cast<uint64_t>(tensors[t]) - plan->tensors[b.tensor_ids[t]].offset * es; };
    *origin = place(0);
    if (*origin % 16) return false;
    for (uint32_t t = 1; t < b.n_tensors; ++t)
        if (place(t) != *origin) return false;
    return true;
}

// The launches that lists of a bucket's parts take.
struct ListShape {
    bool even;          // one launch of even parts
    size_t launches;
};
static ListShape list_shape(const BucketRec &b, uint32_t es)
{
    const size_t n = b.pieces.size();
    const bool even = n <= (size_t)UnpackList200::kParts && even_parts(n, b.payload, b.longest, kWave * 16 / es);
    return {even, even ? 1 : (n + UnpackFlat160::kParts - 1) / UnpackFlat160::kParts};
}
static bool spans_reach(const BucketRec &b, uint32_t n_shards, uint32_t es)
{
    return n_shards <= UnpackPlacedArgs::kShards && b.P * es < 1ull << 32;      // (kernels address with 32 bits)
}
// Most bytes of a bucket that are written by the bucket's lines of 128 bytes where those are not the tensors' own (a wavefront then writes
// parts of lines).  Lists / so, us: tensors in the bucket's layout, 9 of 18 / 72 / 360 MB 9.0 / 8.6, 27.2 / 27.0, 127 / 128, of 720 MB 249
// / 255; elsewhere, 9 of 7 / 18 / 72 / 360 MB 5.2 / 5.2, 8.6 / 8.6, 26.5 / 27.1, 116 / 123, 64 of 13 / 128 MB 7.6 / 7.2, 45 / 47.
constexpr uint64_t kOffLinesPlaced = 64u << 20, kOffLinesNear = 16u << 20;
// Is the one launch of unpack_placed the better way to write the bucket's tensors?  Lists / placed, us, behind a long kernel (the host is
// ahead, so that the device's time shows) and in a row on an idle queue, 8 shards but where others are named:
//   up to 64 tensors: 6 / 9 / 30 / 64 uneven ones of 0.06-0.1 MB in all 1.78 / 1.80, 1.88 / 1.85, 1.83 / 1.92, 1.86 / 1.98 (in a row 4.4 /
//   4.0), of 0.16 MB 1.88 / 1.86, 1.87 / 1.86, 2.14 / 1.93, 2.26 / 1.99, 9 of 0.5 / 3.6 MB 2.33 / 2.01, 3.34 / 3.09 (3.65 / 3.25), of 18 /
//   360 MB 7.8 / 7.5, 107 / 106; even parts (2 shards), placed by lists: 6 / 9 / 12 / 30 / 64 of 0.2 MB 1.06 / .99 / 1.01 / 1.06 / .98, of
//   0.5 MB 1.00 / 1.01 / 1.03 / 1.01 / 1.12, of 1.2 MB 1.00 / .91 / .91 / .86 / .84 (in a row .89), from 20 MB the same.  (What the
//   shortest lose on the device shows behind a long kernel alone: a launch costs the host longer.)
//   more, where lists are one launch: 100 uneven ones of 0.07 / 0.6 / 2 / 20 MB 2.28 / 2.46 (in a graph), 2.48 / 2.32, 3.02 / 2.57, 9.4 /
//   9.7, even ones of 2 / 20 MB 2.9 / 3.0, 8.3 / 9.3.
//   more, where lists are several launches (or tables), 8 MiB for each: 170 uneven ones of 7 / 15 / 20 / 60 / 120 MB 5.45 / 4.93, 8.26 /
//   8.04, 10.0 / 9.7, 23.1 / 22.6, 41.1 / 41.9; 400 of 8 / 24 / 32 / 80 / 200 MB 5.8 / 5.6, 11.3 / 11.4, 13.9 / 14.3, 29.6 / 29.6, 65.9 /
//   68.4, even ones 5.6 / 4.9, 10.9 / 10.6, 14.6 / 13.2, 28.1 / 28.1, 62.8 / 65.0; 1000 uneven ones of 0.7 / 20 / 56 / 80 / 200 / 400 MB
//   11.6 / 5.2, 18.0 / 11.1, 28.8 / 24.0, 36.9 / 31.9, 79 / 72, 141 / 139.  (So the line is a cautious one for 1000.)
static bool placed_pays(const BucketRec &b, const ListShape &lists, uint32_t es)
{
    const uint64_t bytes = b.P * es;
    if (b.n_tensors <= (uint32_t)kWave) return !lists.even || bytes <= 4u << 20;
    if (lists.even) return false;
    return lists.launches == 1 ? bytes >= 512u << 10 && bytes <= 4u << 20 : bytes <= lists.launches * (8u << 20);
}
// And that of unpack_near?  Up to 12 tensors as above, near by lists: uneven ones, behind a long kernel 6 / 9 / 12 of 0.1 MB 1.11 / 1.12 /
// 1.11, of 0.28 MB 1.11 / 1.00 / .91, of 0.4 MB 1.00 / .90 / .95, of 3.6 MB .94; even parts (2 shards), of 0.2 MB 1.14 / 1.11 / 1.14, of
// 0.56 MB 1.05 / 1.09 / 1.07, of 1.2 MB 1.11 / 1.01 / .99, of 2 MB 1.02 / 1.02 / .96; off the bucket's 128-byte lines .97-1.03 of 0.4 MB,
// .91-.99 of 0.5 MB.  In a row .88-.93 throughout.  So the shortest cost the device 0.1 to 0.3 us and save the host 0.4, and the host takes
// longer than the device for a launch: a program that makes many such calls sees the latter. More, in a block of 320 bytes, only where they
// are uneven and long enough: 64 of 0.05 / 0.76 / 12.8 / 128 MB 4.6 / 4.35, 4.5 / 4.3, 7.3 / 6.6, 41.6 / 39.0 in a row and 2.26 / 2.32,
// 2.50 / 2.45, 7.3 / 6.4, 42.9 / 40.4 in a graph: a cautious line.
// (With the bucket beside them 0.2 us more on the device than lists: 9 of 0.06 MB 2.08 / 2.33.)
static bool near_pays(const BucketRec &b, const ListShape &lists, uint32_t es)
{
    if (b.n_tensors <= UnpackNear12::kTensors) return placed_pays(b, lists, es);
    return b.n_tensors <= UnpackNear64::kTensors && !lists.even && b.P * es >= 1u << 20;
}
// The same with the bucket written too, where lists (`one_pass`) are one launch: 9 uneven / 30 even / 64 even ones of 0.06-0.1 MB 1.81 /
// 1.88, 1.77 / 1.85, 1.80 / 1.95 (in a row 4.5 / 3.9, 4.8 / 3.9, 5.0 / 4.1), 9 / 30 / 64 even ones of 0.5 MB 2.06 / 1.84, 2.03 / 1.93, 1.89
// / 1.86, 9 uneven ones of 4 MB 4.23 / 3.69, 9 of 18 / 360 MB 11.2 / 10.7, 172 / 173; 100 even ones of 0.08 / 2 / 20 MB 2.1 / 2.4, 3.2 /
// 3.1, 11.6 / 12.4 in a graph.  Else there are two passes: 100 uneven ones of 0.6 / 2 / 10 / 40 / 200 MB 4.19 / 2.37, 5.74 / 2.78, 11.1 /
// 7.9, 28.5 / 21.9, 123 / 95, 1000 of 0.7 / 200 MB 16.8 / 4.5, 139 / 105.
static bool placed_pays_both(const BucketRec &b, uint32_t es, bool one_pass)
{
    const uint64_t bytes = b.P * es;
    return !one_pass || (bytes <= 4u << 20 && (b.n_tensors <= (uint32_t)kWave || bytes >= 512u << 10));
}

template <int ES, bool BOTH>
static hzp_status_t unpack_placed(const DeviceTables &tab, const BucketRec &b, const void *const *shards, uint32_t n_shards, uint64_t origin,
                                  void *bucket, hipStream_t stream)
{
    UnpackPlacedArgs a;
    for (uint32_t j = 0; j < n_shards; ++j) a.src[j] = reinterpret_cast<uint64_t>(shards[j]);
    a.dst = origin;
    a.bucket = reinterpret_cast<uint64_t>(bucket);
    a.span = reinterpret_cast<const u32x2 *>(tab.span) + b.tensor_slot;
    a.n = b.n_tensors;
    a.nvec = (uint32_t)(b.S3 * ES / 16);
    a.end = (uint32_t)b.payload_end;
    const auto kernel = b.n_tensors <= (uint32_t)kWave ? unpack_placed_kernel<ES, BOTH, true> : unpack_placed_kernel<ES, BOTH, false>;
    return start("hzp_gather_layer", kernel, dim3((uint32_t)tiles_of(a.nvec), n_shards), dim3(kWave), 0, stream, a);
}

// The same for tensors that lie elsewhere; *done is false (and nothing launched) where they or the shards lie too far apart, or off 16
// bytes.
template <int ES, class Args>
static hzp_status_t unpack_near(const hzp_plan_t *plan, const DeviceTables &tab, const BucketRec &b, const void *const *shards,
                                uint32_t n_shards, void *const *tensors, hipStream_t stream, bool *done)
{
    Args a;
    a.src = reinterpret_cast<uint64_t>(shards[0]);
    a.dst = reinterpret_cast<uint64_t>(tensors[0]);
    a.span = reinterpret_cast<const u32x2 *>(tab.span) + b.tensor_slot;
    a.n = b.n_tensors;
    a.nvec = (uint32_t)(b.S3 * ES / 16);
    bool fits = a.dst % 16 == 0;
    uint64_t off = 0;                   // by how much any tensor's 128-byte lines are not the bucket's
    for (uint32_t j = 0; j < n_shards; ++j) a.shard[j] = units_apart(reinterpret_cast<uint64_t>(shards[j]), a.src, &fits);
    for (uint32_t t = 0; t < b.n_tensors; ++t) {
        a.tensor[t] = units_apart(reinterpret_cast<uint64_t>(tensors[t]), a.dst, &fits);
        off |= reinterpret_cast<uint64_t>(tensors[t]) - plan->tensors[b.tensor_ids[t]].offset * ES;
    }
    if (off % 128 && b.P * ES > kOffLinesNear) fits = false;
    *done = fits;
    if (!fits) return HZP_OK;
    return start("hzp_gather_layer", unpack_near_kernel<ES, Args>, dim3((uint32_t)tiles_of(a.nvec), n_shards), dim3(kWave), 0, stream, a);
}
template <int ES>
static hzp_status_t unpack_near(const hzp_plan_t *plan, const DeviceTables &tab, const BucketRec &b, const void *const *shards,
                                uint32_t n_shards, void *const *tensors, hipStream_t stream, bool *done)
{
    return b.n_tensors <= UnpackNear12::kTensors ? unpack_near<ES, UnpackNear12>(plan, tab, b, shards, n_shards, tensors, stream, done)
                                                 : unpack_near<ES, UnpackNear64>(plan, tab, b, shards, n_shards, tensors, stream, done);
}

// Do lists serve the unpacking of pieces [p0, p1), or the plan's tables?  A graph may be replayed after its plan has been freed where
// nothing of the plan's is read, so captured calls that lists serve take lists and not the spans, which are a table too.
static bool lists_serve(const BucketRec &b, size_t p0, size_t p1, void *const *tensors, uint32_t t_begin, uint32_t es)
{
    const size_t n = p1 - p0;
    if (n <= (size_t)UnpackFlat160::kParts) return true;        // one launch
    uint64_t total = 0;
    size_t longest = p0;
    for (size_t i = p0; i < p1; ++i) {
        total += b.pieces[i].len;
        if (b.pieces[i].len > b.pieces[longest].len) longest = i;
    }
    const Piece &l = b.pieces[longest];
    const bool odd = (reinterpret_cast<uint64_t>(tensors[l.tensor - t_begin]) + l.dst_off * es) & 15u;
    return lists_pay(n, total, l.len, odd, es);
}

hzp_status_t launch_unpack(const hzp_plan_t *plan, const BucketRec &b, const void *const *shards,
                           uint32_t n_shards, void *const *tensors, uint32_t t_begin, uint32_t t_end,
                           hipStream_t stream)
{
    const size_t p0 = first_piece(b, 0, t_begin), p1 = first_piece(b, p0, t_end), n = p1 - p0;
    const uint32_t es = b.cls == HZP_CLASS_F32 ? 4 : 2;
    const DeviceTables *tab = nullptr;
    const hzp_status_t st = device_tables(plan, &tab);
    if (st != HZP_OK) return st;
    if (n > (size_t)UnpackList5::kParts && t_end - t_begin == b.n_tensors && spans_reach(b, n_shards, es)) {
        const ListShape lists = list_shape(b, es);
        auto outlived = [&] { return captured(stream) && lists_serve(b, p0, p1, tensors, t_begin, es); };
        uint64_t origin = 0;
        if (placed_pays(b, lists, es) && placed_as_in_bucket(plan, b, tensors, es, &origin) &&
            (origin % 128 == 0 || b.P * es <= kOffLinesPlaced) && !outlived())
            return es == 4 ? unpack_placed<4, false>(*tab, b, shards, n_shards, origin, nullptr, stream)
                           : unpack_placed<2, false>(*tab, b, shards, n_shards, origin, nullptr, stream);
        if (near_pays(b, lists, es) && !outlived()) {
            bool done = false;
            const hzp_status_t near = es == 4 ? unpack_near<4>(plan, *tab, b, shards, n_shards, tensors, stream, &done)
                                              : unpack_near<2>(plan, *tab, b, shards, n_shards, tensors, stream, &done);
            if (done) return near;
        }
    }
    if (!lists_serve(b, p0, p1, tensors, t_begin, es)) {
        const UnpackCall u{tab->pieces + b.piece_slot, tab->piece_chunk + b.piece_slot, b, shards, n_shards, stream};
        return launch_unpack_with(u, tensors, t_begin, t_end, "hzp_gather_layer");
    }
    const Piece *const piece = b.pieces.data() + p0;
    if (t_end - t_begin == 1 && n <= (size_t)UnpackTensorArgs::kParts) {
        uint64_t total = 0, longest = 0;
        for (size_t i = 0; i < n; ++i) {
            total += piece[i].len;
            longest = std::max(longest, piece[i].len);
        }
        const uint64_t tile = kWave * 16 / es;
        // (what unpack_parts puts into one uncut launch)
        if (total / tile <= kMaxTilesPerLaunch && even_parts(n, total, longest, tile))
            return es == 4 ? unpack_tensor<4>(piece, n, shards, tensors[0], longest, stream)
                           : unpack_tensor<2>(piece, n, shards, tensors[0], longest, stream);
    }
    return es == 4 ? unpack_parts<4, false>(PieceParts<4>{piece, shards, tensors, t_begin}, n, stream, "hzp_gather_layer")
                   : unpack_parts<2, false>(PieceParts<2>{piece, shards, tensors, t_begin}, n, stream, "hzp_gather_layer");
}

hzp_status_t launch_unpack_both(const hzp_plan_t *plan, const BucketRec &b, const void *const *shards, uint32_t n_shards,
                                void *bucket, void *const *tensors, hipStream_t stream)
{
    const uint32_t es = b.cls == HZP_CLASS_F32 ? 4 : 2;
    const uint64_t out = reinterpret_cast<uint64_t>(bucket);
    // One pass serves both outputs where what is aligned in the shard is aligned in the tensor too and no shard lies in
    // place; not for so many small tensors that it would take more launches than the two passes.  One pass / two, us: 60 and 100 tensors
    // of 128 KB 5.9 / 9.2 and 8.5 / 11.9, of 2 MB 58.9 / 75.8 and 98 / 125; several launches: 200 tensors of 32 KB 10.7 / 10.0, of 128 KB
    // 17.8 / 19.2, of 2 MB 193 / 246: the line at 2 MB (bf16) is a cautious one.
    bool one_pass = b.pieces.size() + n_shards <= (size_t)UnpackBothFlat108::kParts || b.P / b.pieces.size() >= (1u << 20);
    for (uint32_t t = 0; t < b.n_tensors; ++t) one_pass = one_pass && (reinterpret_cast<uint64_t>(tensors[t]) & 15u) == 0;
    for (uint32_t j = 0; j < n_shards; ++j) one_pass = one_pass && reinterpret_cast<uint64_t>(shards[j]) != out + j * b.S3 * es;
    const DeviceTables *tab = nullptr;
    hzp_status_t st = device_tables(plan, &tab);
    if (st != HZP_OK) return st;
    uint64_t origin = 0;
    if (spans_reach(b, n_shards, es) && placed_pays_both(b, es, one_pass) && placed_as_in_bucket(plan, b, tensors, es, &origin) &&
        !(captured(stream) && (one_pass || lists_serve(b, 0, b.pieces.size(), tensors, 0, es))))
        return es == 4 ? unpack_placed<4, true>(*tab, b, shards, n_shards, origin, bucket, stream)
                       : unpack_placed<2, true>(*tab, b, shards, n_shards, origin, bucket, stream);
    if (!one_pass) {
        st = launch_concat(shards, n_shards, b.S3 * es, bucket, stream);
        if (st != HZP_OK) return st;
        return launch_unpack(plan, b, shards, n_shards, tensors, 0, b.n_tensors, stream);
    }
    // The bucket shard by shard: tensor pieces with the padding behind them, and padding that a shard begins with.
    std::vector<Part> parts;
    auto add = [&](uint32_t j, uint64_t begin, uint64_t end, uint64_t tensor, uint64_t n) {     // [begin, end) of shard j
        const uint64_t src = reinterpret_cast<uint64_t>(shards[j]) + begin * es, dst = out + (j * b.S3 + begin) * es;
        for (uint64_t x = 0; x < end - begin; x += kMostInPart)
            parts.push_back({src + x * es, tensor + x * es, n > x ? std::min(n - x, kMostInPart) : 0, dst + x * es,
                             std::min(end - begin - x, kMostInPart)});
    };
    try {
        parts.reserve(b.pieces.size() + n_shards);
        size_t i = 0;
        for (uint32_t j = 0; j < n_shards; ++j) {
            const uint64_t first = i < b.pieces.size() && b.pieces[i].shard == j ? b.pieces[i].src_off : b.S3;
            if (first > 0) add(j, 0, first, out, 0);
            for (; i < b.pieces.size() && b.pieces[i].shard == j; ++i) {
                const Piece &p = b.pieces[i];
                const bool last = i + 1 == b.pieces.size() || b.pieces[i + 1].shard != j;
                add(j, p.src_off, last ? b.S3 : b.pieces[i + 1].src_off, reinterpret_cast<uint64_t>(tensors[p.tensor]) + p.dst_off * es,
                    p.len);
            }
        }
    } catch (const std::bad_alloc &) {
        return fail(HZP_ERR_NOMEM, "hzp_gather_layer: out of host memory");
    }
    const ListedParts listed{parts.data()};
    return es == 4 ? unpack_parts<4, true>(listed, parts.size(), stream, "hzp_gather_layer")
                   : unpack_parts<2, true>(listed, parts.size(), stream, "hzp_gather_layer");
}

// ---------------------------------------------------------------------------------------
// The same unpack for callers that must not allocate: the bucket's piece table is written, by a
// small kernel that carries it in its arguments, into a fixed array in device memory instead of
// the per-plan tables that device_tables() allocates on first use.
// ---------------------------------------------------------------------------------------
struct StaticTables {
    Piece pieces[HZP_STATIC_MAX_PIECES];
    uint32_t piece_chunk[HZP_STATIC_MAX_PIECES];
};
// One copy per GPU, at an address of its own, held until the process ends.  In host code this
// name is only a handle for hipGetSymbolAddress; kernels get the address that call returns.
static __device__ __align__(256) unsigned char scratch[sizeof(StaticTables)];

constexpr uint32_t kFillWords = 896;    // 3584 bytes of table per launch, in the argument block
struct FillArgs {
    uint32_t word[kFillWords];
    uint32_t *dst;
    uint32_t n;
};
__global__ __launch_bounds__(256) void table_fill_kernel(const FillArgs a)
{
    for (uint32_t i = threadIdx.x; i < a.n; i += 256) a.dst[i] = a.word[i];
}

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up once per device).
static hzp_status_t scratch_address(StaticTables **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(HZP_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(HZP_ERR_UNSUPPORTED, "device %d: more than %d devices", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(HZP_ERR_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        g_scratch_ptr[dev] = ptr;
    }
    *out = static_cast<StaticTables *>(g_scratch_ptr[dev]);
    return HZP_OK;
}

// Enqueue the copy of `bytes` (a multiple of 4) of host data to device memory at `dst`.
static hzp_status_t fill_table(void *dst, const void *src, size_t bytes, hipStream_t stream)
{
    const uint32_t *w = static_cast<const uint32_t *>(src);
    size_t left = bytes / 4;
    uint32_t *d = static_cast<uint32_t *>(dst);
    while (left) {
        FillArgs a;
        a.n = (uint32_t)std::min<size_t>(left, kFillWords);
        std::memcpy(a.word, w, (size_t)a.n * 4);
        a.dst = d;
        const hzp_status_t st = start("hzp_gather_layer_static", table_fill_kernel, dim3(1), dim3(256), 0, stream, a);
        if (st != HZP_OK) return st;
        w += a.n;
        d += a.n;
        left -= a.n;
    }
    return HZP_OK;
}

hzp_status_t launch_unpack_static(const BucketRec &b, const void *const *shards, uint32_t n_shards,
                                  void *const *tensors, hipStream_t stream)
{
    if (b.pieces.size() > HZP_STATIC_MAX_PIECES)        // refused by the entry point; the table below has this many rows
        return fail(HZP_ERR_UNSUPPORTED, "hzp_gather_layer_static: more tensor pieces than the fixed table holds");
    StaticTables *tab = nullptr;
    hzp_status_t st = scratch_address(&tab);
    if (st != HZP_OK) return st;
    uint32_t chunk_begin[HZP_STATIC_MAX_PIECES];
    for (size_t i = 0; i < b.pieces.size(); ++i) chunk_begin[i] = b.pieces[i].chunk_begin;
    static_assert(sizeof(Piece) % 4 == 0, "tables are copied in 32-bit words");
    st = fill_table(tab->pieces, b.pieces.data(), b.pieces.size() * sizeof(Piece), stream);
    if (st == HZP_OK) st = fill_table(tab->piece_chunk, chunk_begin, b.pieces.size() * sizeof(uint32_t), stream);
    if (st != HZP_OK) return st;
    const UnpackCall u{tab->pieces, tab->piece_chunk, b, shards, n_shards, stream};
    return launch_unpack_with(u, tensors, 0, b.n_tensors, "hzp_gather_layer_static");
}

// ---------------------------------------------------------------------------------------
// Per-plan, per-device lookup tables.
// ---------------------------------------------------------------------------------------
hzp_status_t device_tables(const hzp_plan_t *plan, const DeviceTables **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(HZP_ERR_HIP, "hipGetDevice: %s", hipGetErrorString(e));
    std::lock_guard<std::mutex> lock(plan->mu);
    for (const DeviceTables &t : plan->dev)
        if (t.device == dev) {
            *out = &t;
            return HZP_OK;
        }
    DeviceTables t;
    t.device = dev;
    std::vector<Piece> all;
    std::vector<uint32_t> words;        // the pieces' first chunks, and behind them the tensors' spans
    size_t span_at = 0;
    try {
        for (const BucketRec &b : plan->buckets) all.insert(all.end(), b.pieces.begin(), b.pieces.end());
        words.resize(all.size() + all.size() % 2);
        for (size_t i = 0; i < all.size(); ++i) words[i] = all[i].chunk_begin;
        span_at = words.size();
        for (const BucketRec &b : plan->buckets)
            for (uint32_t id : b.tensor_ids) {
                const TensorRec &r = plan->tensors[id];
                words.push_back((uint32_t)r.offset);                // (read only where the bucket is short)
                words.push_back((uint32_t)(r.offset + r.numel));
            }
        // The vector may only grow while no reader holds a pointer into it: reserve once.
        if (plan->dev.capacity() == 0) plan->dev.reserve(64);
    } catch (const std::bad_alloc &) {
        return fail(HZP_ERR_NOMEM, "device tables: out of host memory");
    }
    if (plan->dev.size() == plan->dev.capacity()) return fail(HZP_ERR_UNSUPPORTED, "plan used on more than 64 devices");
    const size_t nr = plan->run_off.size();
    auto upload = [&](void **dptr, const void *src, size_t bytes) -> hipError_t {
        hipError_t err = hipMalloc(dptr, bytes ? bytes : 16);
        if (err != hipSuccess) return err;
        return bytes ? hipMemcpy(*dptr, src, bytes, hipMemcpyHostToDevice) : hipSuccess;
    };
    e = upload((void **)&t.run_off, plan->run_off.data(), nr * sizeof(uint64_t));
    if (e == hipSuccess) e = upload((void **)&t.run_wd, plan->run_wd.data(), nr * sizeof(float));
    if (e == hipSuccess) e = upload((void **)&t.pieces, all.data(), all.size() * sizeof(Piece));
    if (e == hipSuccess) e = upload((void **)&t.piece_chunk, words.data(), words.size() * sizeof(uint32_t));
    t.span = t.piece_chunk + span_at;
    // (a stream created as non-blocking is not ordered behind the null stream's copies, and the call that made the tables may read them)
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) {
        (void)hipFree(t.piece_chunk);
        (void)hipFree(t.run_off);
        (void)hipFree(t.run_wd);
        (void)hipFree(t.pieces);
        return fail(e == hipErrorOutOfMemory ? HZP_ERR_NOMEM : HZP_ERR_HIP, "device tables: %s",
                    hipGetErrorString(e));
    }
    plan->dev.push_back(t);
    *out = &plan->dev.back();
    return HZP_OK;
}

}  // namespace hzp

extern "C" hzp_status_t hzp_plan_prepare(const hzp_plan_t *plan, hipStream_t stream)
{
    if (!plan) return hzp::fail(HZP_ERR_INVALID_ARG, "hzp_plan_prepare: NULL plan");
    const hzp::DeviceTables *tab = nullptr;
    hzp_status_t st = hzp::device_tables(plan, &tab);       // allocates and copies (blocking) on first use
    if (st != HZP_OK) return st;
    // The copies above were blocking host-to-device copies on the null stream; a stream created
    // as non-blocking is not ordered behind them by itself, so wait for them once here.
    hipError_t e = hipStreamSynchronize(stream);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) return hzp::fail(HZP_ERR_HIP, "hzp_plan_prepare: %s", hipGetErrorString(e));
    return HZP_OK;
}

namespace hzp {

void free_device_tables(hzp_plan_t *plan)
{
    for (DeviceTables &t : plan->dev) {
        int cur = -1;
        if (hipGetDevice(&cur) == hipSuccess && cur != t.device) (void)hipSetDevice(t.device);
        (void)hipFree(t.run_off);
        (void)hipFree(t.run_wd);
        (void)hipFree(t.pieces);
        (void)hipFree(t.piece_chunk);
        if (cur >= 0 && cur != t.device) (void)hipSetDevice(cur);
    }
    plan->dev.clear();
}

}  // namespace hzp
