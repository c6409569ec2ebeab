// gfx950 kernels and C-ABI entry points of the bucketed FSDP copy path.
//
// All kernels are HBM-bound streams (no contraction, so no MFMA): one launch
// covers every parameter of a bucket.  The work of a launch is cut into tiles
// that never cross a parameter (and, for the W-way copies, never cross one
// rank's segment of a parameter), so that a tile is a plain contiguous copy,
// cast or reduction with 16-byte vector accesses.  The per-parameter table
// travels in the kernel arguments.  The pack and the reduce number their tiles
// parameter by parameter, the W-way copies chunk by chunk.  The pack holds the
// table in lanes (lane p holds parameter p's entries; a ballot over the first
// tiles finds a tile's parameter); the others look a tile up with scalar
// instructions only (TilePlace).  Tile counts fit in 31 bits (checked on the
// host); grid-stride loops count in 64 bits, or in unsigned 32 (a tile number
// plus a grid size is below 2^32), so the last step cannot overflow.
//
// A bucket buffer of W chunks is addressed either as one allocation (chunk i
// at base + i*stride) or through a table of W chunk pointers, so the same
// kernels can pull from or push to chunks that live in separate buffers (for
// an exchange fused with the copy: the chunks of the peers).
//
// Numerics (SimpleFSDP sections 3.2.1 and 4):
//   * fp32 -> bf16 is IEEE round-half-to-even on the 16 dropped bits (the
//     hardware conversion); NaN gives (bits >> 16) | 0x0040;
//   * bf16 -> fp32 is exact (append 16 zero bits); fp32 copies are bit copies;
//   * the average is an fp32 sum over source ranks in order 0..W-1, starting
//     from the rank-0 value, then one IEEE division by W.  The library is
//     built without fast-math or fp contraction and with fp32 subnormals
//     enabled, so every add and the division are correctly rounded.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cstdint>
#include <string>
#include <type_traits>

#include "plan_impl.h"

namespace fsdp {
namespace {

#ifndef FSDP_REDUCE_WAVES
#define FSDP_REDUCE_WAVES 4
#endif
#ifndef FSDP_REDUCE_CAP_WAVES
#define FSDP_REDUCE_CAP_WAVES 26
#endif
#ifndef FSDP_REDUCE_ONE_WAVES
#define FSDP_REDUCE_ONE_WAVES 10
#endif
#ifndef FSDP_REDUCE_TWO_WAVES
#define FSDP_REDUCE_TWO_WAVES 5
#endif
#ifndef FSDP_BLOCKS_PER_CU
#define FSDP_BLOCKS_PER_CU 16384
#endif
#ifndef FSDP_XCD_RUN
#define FSDP_XCD_RUN 256
#endif
#ifndef FSDP_NT_LOAD
#define FSDP_NT_LOAD 1
#endif
#ifndef FSDP_NT_STORE
#define FSDP_NT_STORE 1
#endif

constexpr int PMAX = FSDP_MAX_PARAMS;
constexpr int kMaxChunks = FSDP_MAX_CHUNKS;
// One parameter per lane of a wave64: the pack's ballot lookup and lane-held
// table need every parameter's entry in one wavefront.
static_assert(PMAX <= 64, "the pack's lookup holds one parameter per lane of a 64-wide wavefront");
static_assert(kCopyBlock % 64 == 0 && kWidenBlock % 64 == 0 && kPackBlock % 64 == 0 && kPackBigBlock % 64 == 0 &&
                  kReduceBlock == 64,
              "workgroups are whole wavefronts, the reduction's one wavefront");
constexpr int kReduceWaves = FSDP_REDUCE_WAVES;           // resident waves per SIMD of a large shard's reduction
constexpr int kReduceCapWaves = FSDP_REDUCE_CAP_WAVES;    // waves per CU from which a shard is large
constexpr int kReduceSomeW = 11;                          // ... and W up to which it is large
constexpr int kReduceSomeWaves = 32;                      // ... from here only;
constexpr int kReducePlainWaves = 192;                    // ... tiles on the lines are in plain order from here
constexpr int kReduceFewestW = 3;                         // ... W up to which no shard is capped
constexpr int kReduceFewW = 7;                            // ... and W up to which none whose tiles are in runs is
constexpr int kReduceWideW = 32;                          // ... W from which one wave fewer is resident
constexpr int kReduceWideWaves = 32;                      // ... in a shard of as many waves per CU,
constexpr int kReduceWidePlainWaves = 96;                 // ... which is in plain order from here
constexpr int kReduceOneWaves = FSDP_REDUCE_ONE_WAVES;    // ... from which a wave keeps one source in flight, not two
constexpr int kReduceTwoWaves = FSDP_REDUCE_TWO_WAVES;    // ... two sources, not four
constexpr int kReduceThroughW = 4;                        // W up to which an fp32 wire's averages always write through
constexpr int kBlocksPerCU = FSDP_BLOCKS_PER_CU;  // workgroups per CU in the grid-stride launch
constexpr int kXcds = 8;                          // accelerator dies; workgroup b runs on die b % 8
constexpr int kXcdRun = FSDP_XCD_RUN;             // consecutive copy tiles dealt to one die
static_assert(kXcdRun >= 1, "a die takes at least one tile at a time");

// ------------------------------------------------------------------ device helpers

// fp32 -> bf16 with gfx950's packed conversion (v_cvt_pk_bf16_f32): IEEE
// round-half-to-even on the 16 dropped bits under the default rounding mode,
// subnormals kept, overflow to infinity; a NaN keeps its sign and top payload
// bits and gets the quiet bit, (bits >> 16) | 0x0040.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t bf16x2_bits(float lo, float hi) {
    const f32x2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

__device__ __forceinline__ uint32_t bf16_bits(float f) { return bf16x2_bits(f, 0.f) & 0xffffu; }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// IEEE binary16: the conversion instruction rounds to nearest even under the
// default mode, keeps subnormals and overflows to infinity; the way back is
// exact.
__device__ __forceinline__ uint32_t f16_bits(float f) {
    return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f));
}
__device__ __forceinline__ float f16_lo(uint32_t w) {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w & 0xffffu)));
}
__device__ __forceinline__ float f16_hi(uint32_t w) {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(w >> 16)));
}

// Element formats a kernel reads or writes on a bucket wire.
constexpr int kF32 = 0;    // fp32, copied bit for bit
constexpr int kBF16 = 1;   // bf16
constexpr int kF16 = 2;    // IEEE binary16

// The exact fp32 value of the low / high 16-bit element of a word.
template <int kFrom>
__device__ __forceinline__ float widen_lo(uint32_t w) { return kFrom == kF16 ? f16_lo(w) : bf16_lo(w); }
template <int kFrom>
__device__ __forceinline__ float widen_hi(uint32_t w) { return kFrom == kF16 ? f16_hi(w) : bf16_hi(w); }

// Parameter owning tile t: the last p with tile_start[p] <= t.  Every lane of
// the wave holds tile_start[lane] (INT_MAX past the last parameter).
__device__ __forceinline__ int param_of_tile(int my_start, int t) {
    const uint64_t m = __ballot(my_start <= t);
    return __builtin_amdgcn_readfirstlane(__popcll(m) - 1);
}

// A pointer into device memory whose origin the compiler cannot see: the round
// trip through the global address space keeps its accesses global.  (As flat
// ones they would count as LDS accesses too, and every wait near them becomes
// a wait for everything.)
template <typename T>
__device__ __forceinline__ T* as_global(T* p) {
    typedef T __attribute__((address_space(1))) Global;
    return (T*)(Global*)(reinterpret_cast<uintptr_t>(p));
}

__host__ __device__ __forceinline__ bool on_line(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 127) == 0; }
__device__ __forceinline__ bool is_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// The same 16 bytes at an address that is only 2- or 4-byte aligned (the
// target's global loads and stores take any alignment).
typedef u32x4 __attribute__((aligned(2))) u32x4_any2;
typedef u32x4 __attribute__((aligned(4))) u32x4_any4;
typedef f32x4 __attribute__((aligned(4))) f32x4_any4;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 __attribute__((aligned(2))) u32x2_any2;

// The pack's accesses; streamed data bypasses cache retention (non-temporal).
// Stores are non-temporal unless kNt is false: a chunk that other workgroups
// read back at once (the first half of a wide push) is stored through the cache.
template <bool kNt = bool(FSDP_NT_STORE)>
__device__ __forceinline__ void st16(void* p, uint4 v) {
    u32x4* q = reinterpret_cast<u32x4*>(p);
    const u32x4 w = {v.x, v.y, v.z, v.w};
    if constexpr (kNt) __builtin_nontemporal_store(w, q);
    else *q = w;
}

template <bool kNt = bool(FSDP_NT_STORE)>
__device__ __forceinline__ void st8(void* p, uint2 v) {
    u32x2* q = reinterpret_cast<u32x2*>(p);
    const u32x2 w = {v.x, v.y};
    if constexpr (kNt) __builtin_nontemporal_store(w, q);
    else *q = w;
}
__device__ __forceinline__ float4 ld16f(const float* p) {
    const f32x4* q = reinterpret_cast<const f32x4*>(p);
#if FSDP_NT_LOAD
    const f32x4 v = __builtin_nontemporal_load(q);
#else
    const f32x4 v = *q;
#endif
    return make_float4(v.x, v.y, v.z, v.w);
}
template <bool kNt = bool(FSDP_NT_STORE)>
__device__ __forceinline__ void st16f(float* p, float4 v) {
    f32x4* q = reinterpret_cast<f32x4*>(p);
    const f32x4 w = {v.x, v.y, v.z, v.w};
    if constexpr (kNt) __builtin_nontemporal_store(w, q);
    else *q = w;
}

// ------------------------------------------------------------------ windows

// A window of `bytes` bytes from a wave-uniform address on, as a raw buffer
// resource (32-bit data format, no stride): an access takes a 32-bit byte
// offset per lane, and one at or past `bytes` reads zero or is dropped.
// Loads are non-temporal.  Stores are non-temporal and write through (sc1:
// system scope), so a streamed line leaves the L2 as it is written instead of
// waiting there to be evicted among the reads: a plain copy of 1.7 GB takes
// 520 us this way, 526 us with the non-temporal bit alone, 546 us with neither.
typedef __amdgpu_buffer_rsrc_t Window;
constexpr int kRawBuffer = 0x00020000;
constexpr int kPolicyNt = 2, kPolicySc1 = 16;
#ifndef FSDP_LOAD_POLICY
#define FSDP_LOAD_POLICY kPolicyNt
#endif
#ifndef FSDP_STORE_POLICY
#define FSDP_STORE_POLICY (kPolicySc1 | kPolicyNt)
#endif
__device__ __forceinline__ Window window(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, int(bytes), kRawBuffer);
}
__device__ __forceinline__ u32x4 ld16(Window w, uint32_t byte) {
    return __builtin_amdgcn_raw_buffer_load_b128(w, int(byte), 0, FSDP_LOAD_POLICY);
}
__device__ __forceinline__ u32x2 ld8(Window w, uint32_t byte) {
    return __builtin_amdgcn_raw_buffer_load_b64(w, int(byte), 0, FSDP_LOAD_POLICY);
}
template <int kPolicy = FSDP_STORE_POLICY>
__device__ __forceinline__ void st16(Window w, uint32_t byte, u32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, w, int(byte), 0, kPolicy);
}
__device__ __forceinline__ void st16(Window w, uint32_t byte, f32x4 v) { st16(w, byte, __builtin_bit_cast(u32x4, v)); }

// ------------------------------------------------------------------ bucket chunk addressing

// One allocation holding W chunks, chunk i at base + i*stride bytes.
struct ContigChunks {
    char* base;
    int64_t stride;
    __device__ __forceinline__ char* at(int i) const { return as_global(base + int64_t(i) * stride); }
    // at(i) for an i that may be W or more: an address that is not accessed then.
    __device__ __forceinline__ char* ahead(int i, int) const { return at(i); }
    __device__ __forceinline__ bool aligned() const { return ((uintptr_t(base) | uintptr_t(stride)) & 15) == 0; }
};

// W chunks anywhere (up to kMaxChunks), chunk i at ptr[i]; the host checks
// that every chunk is 16-byte aligned.
struct TableChunks {
    char* ptr[kMaxChunks];
    __device__ __forceinline__ char* at(int i) const { return as_global(ptr[i]); }
    __device__ __forceinline__ char* ahead(int i, int world) const { return at(min(i, world - 1)); }
    __device__ __forceinline__ bool aligned() const { return true; }
};

// ------------------------------------------------------------------ tile look-up

// The first tile of every parameter, in tile order (a parameter without tiles
// shares its start with the next one).  It is read with scalar loads: one
// round for the pivots, a second for four entries above kPivots parameters.
constexpr int kPivots = 16;
constexpr int kPerPivot = 4;
static_assert(kPivots * kPerPivot >= PMAX, "the pivots cover every parameter");
struct TileTable {
    uint32_t pivot[kPivots];       // first tile of parameter k, or of 4k if `deep`; UINT_MAX past the last
    uint32_t deep;                 // more than kPivots parameters
    uint32_t start[PMAX];          // first tile of every parameter; UINT_MAX past the last
};

// The parameter of tile r, the last one that starts at or before it, and the
// tile's number within it.
struct TilePlace {
    int param;
    uint32_t tile;
    __device__ __forceinline__ TilePlace(const TileTable& c, uint32_t r) {
        int k = 0;
        uint32_t first = 0;
#pragma unroll
        for (int e = 0; e < kPivots; ++e) {
            const bool in = c.pivot[e] <= r;
            k = in ? e : k;
            first = in ? c.pivot[e] : first;
        }
        if (c.deep) {
            const int base = k * kPerPivot;
            k = base;
#pragma unroll
            for (int e = 0; e < kPerPivot; ++e) {
                const uint32_t f = c.start[base + e];
                const bool in = f <= r;
                k = in ? base + e : k;
                first = in ? f : first;
            }
        }
        param = k;
        tile = r - first;
    }
};

// ------------------------------------------------------------------ segment copy

__device__ __forceinline__ int clamp_to(int64_t x, int hi) { return int(min(max(x, int64_t(0)), int64_t(hi))); }

// d[k] = k < v ? s[k] : 0 for the elements k of unit [g, g + kN) that lie below
// `end`, one by one.
template <int kN, typename D, typename S, class Cast>
__device__ __forceinline__ void copy_elements(const S* s, D* d, int64_t g, int64_t v, int64_t end, Cast cast) {
    for (int64_t k = g; k < min(g + kN, end); ++k) d[k] = k < v ? cast(s[k]) : D(0);
}

// d[k] = k < v ? s[k] : 0 for k in [lo, hi), s and d 16-byte aligned at 0: one
// tile of kSteps steps of kCopyBlock threads x 8 elements, in 2-byte units
// (bf16, or the halves of fp32 words for a plain copy).  The source window ends
// with the last whole valid unit and the destination's with the last whole
// unit, so a full and a short tile are the same loads and stores: units past
// the valid ones read zero, units past the tile are dropped.  Only the lanes
// of the units that are cut go element by element.
template <int kSteps>
__device__ __forceinline__ void seg_copy_aligned(const uint16_t* __restrict__ s, uint16_t* __restrict__ d, int64_t lo,
                                                 int64_t hi, int64_t v) {
    const int n = int(hi - lo), nv = clamp_to(v - lo, n);
    const Window in = window(s + lo, uint32_t(nv / kVec) * 16);
    const Window out = window(d + lo, uint32_t(n / kVec) * 16);
    const bool cut = ((nv | n) & (kVec - 1)) != 0;
    u32x4 x[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) x[u] = ld16(in, (u * kCopyBlock + threadIdx.x) * 16);
    if (!cut) {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) st16(out, (u * kCopyBlock + threadIdx.x) * 16, x[u]);
        return;
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int i = u * kCopyBlock + threadIdx.x;
        const bool mine = (i == nv / kVec && (nv & (kVec - 1))) || (i == n / kVec && (n & (kVec - 1)));
        st16(out, mine ? ~0u : uint32_t(i) * 16, x[u]);          // past the window: dropped
        if (mine) copy_elements<kVec>(s, d, lo + i * kVec, v, hi, [](uint16_t x) { return x; });
    }
}

// The same from and to any address (a dense bucket, A < 8, a view of flat
// storage, or a destination off the 128-byte lines).  The stores follow d's
// lines, so that no line is written in parts by two waves (which write-through
// stores would send to memory in parts), and each 16-byte store is fed with
// one load from any 2-byte address: such a load costs little more than an
// aligned one (a plain copy of 1.7 GB: 517 us against 511; stores off the grid
// as well: 555).  A tile stores the lines that start in [lo, hi); its last one
// may run past hi into the next tile's elements (up to the segment's end e),
// and the next tile starts with the line after it.  The segment's first
// elements before its first line (in its first tile) and units cut by v or e
// are written element by element.
template <int kSteps>
__device__ __forceinline__ void seg_copy_any(const uint16_t* __restrict__ s, uint16_t* __restrict__ d, int64_t lo,
                                             int64_t hi, int64_t v, int64_t e) {
    constexpr int kUnits = kSteps * kCopyBlock;
    constexpr int kLine = 64;                          // elements
    const int h = (kLine - (int(reinterpret_cast<uintptr_t>(d + lo) >> 1) & (kLine - 1))) & (kLine - 1);
    const int64_t a = lo + h;                          // the first line at or after lo
    const int t = threadIdx.x;
    const auto same = [](uint16_t x) { return x; };
    if (lo == 0 && t < h) copy_elements<1>(s, d, t, v, min(a, hi), same);
    // units from a on: the tile's, those read whole, and the whole ones of zeros
    const int nu = clamp_to((hi - a + kLine - 1) / kLine * (kLine / kVec), kUnits);
    const int whole = clamp_to((min(v, e) - a) >> 3, nu);
    const int zero_from = clamp_to((v - a + kVec - 1) >> 3, nu), zero_to = clamp_to((e - a) >> 3, nu);
    const Window out = window(d + a, uint32_t(nu) * 16);
    const char* const from = as_global(reinterpret_cast<const char*>(s + a));
    u32x4 x[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int i = u * kCopyBlock + t;
        x[u] = u32x4{0, 0, 0, 0};
        if (i < whole) x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any2*>(from + uint32_t(i) * 16));
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int i = u * kCopyBlock + t;
        const bool unit = i < whole || (i >= zero_from && i < zero_to);
        st16(out, unit ? uint32_t(i) * 16 : ~0u, x[u]);          // past the window: dropped
        if (!unit && i < nu) copy_elements<kVec>(s, d, a + int64_t(i) * kVec, v, e, same);
    }
}

// kAny: the launch has segments that start off the 16-byte grid, or in a large
// bucket are written off the 128-byte lines; those take seg_copy_any (the host
// picks kAny only then, so that the aligned kernels keep their own code).
// (vs, e): the segment's valid elements and its end, for seg_copy_any, whose
// lines may run past hi.
template <int kSteps, bool kAny>
__device__ __forceinline__ void seg_copy(const uint16_t* __restrict__ s, uint16_t* __restrict__ d, int64_t lo,
                                         int64_t hi, int64_t v, int64_t vs, int64_t e) {
    if constexpr (kAny) {
        if (!is_aligned16(s) || !on_line(d)) {
            seg_copy_any<kSteps>(s, d, lo, hi, vs, e);
            return;
        }
    }
    seg_copy_aligned<kSteps>(s, d, lo, hi, v);
}

// As seg_copy, but 16-bit elements (bf16 or fp16, kFrom) in and their exact
// fp32 values out, from and to any element-aligned address: with s and d on
// the 16-byte grid through windows, otherwise from where they are.  Each
// thread handles 4 elements per sub-step (8 bytes in, 16 bytes out), so that
// every load and store instruction of a wave covers one contiguous run.
// kAny: a tile off the 128-byte lines is not written through, which would send
// its first and last line to memory in parts (the host picks it where those
// count: kWidenLineTilesPerCU).
template <int kSteps, int kFrom, bool kAny>
__device__ __forceinline__ void seg_widen(const uint16_t* __restrict__ s, float* __restrict__ d, int64_t lo,
                                          int64_t hi, int64_t v) {
    const int n = int(hi - lo), nv = clamp_to(v - lo, n);
    const bool direct = is_aligned16(s) && is_aligned16(d);
    const bool through = !kAny || on_line(d);          // a tile is a whole number of lines
    const char* const from = as_global(reinterpret_cast<const char*>(s + lo));
    char* const to = as_global(reinterpret_cast<char*>(d + lo));
    const auto cast = [](uint16_t x) { return widen_lo<kFrom>(x); };
    u32x2 x[kSteps];
    if (direct) {
        const Window in = window(s + lo, uint32_t(nv / 4) * 8);
#pragma unroll
        for (int u = 0; u < kSteps; ++u) x[u] = ld8(in, (u * kWidenBlock + threadIdx.x) * 8);
    } else {
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
            const int i = u * kWidenBlock + threadIdx.x;
            x[u] = u32x2{0, 0};
            if (i < nv / 4) x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x2_any2*>(from + uint32_t(i) * 8));
        }
    }
    const Window out = window(d + lo, uint32_t(n / 4) * 16);
    const bool cut = ((nv | n) & 3) != 0;
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
        const int i = u * kWidenBlock + threadIdx.x;
        const f32x4 y = {widen_lo<kFrom>(x[u].x), widen_hi<kFrom>(x[u].x), widen_lo<kFrom>(x[u].y), widen_hi<kFrom>(x[u].y)};
        const bool mine = cut && ((i == nv / 4 && (nv & 3)) || (i == n / 4 && (n & 3)));
        if (direct) {
            const uint32_t byte = mine ? ~0u : uint32_t(i) * 16;
            if (through) st16(out, byte, y);
            else st16<kPolicyNt>(out, byte, __builtin_bit_cast(u32x4, y));
        } else if (!mine && i < n / 4) {
            __builtin_nontemporal_store(y, reinterpret_cast<f32x4_any4*>(to + uint32_t(i) * 16));
        }
        if (mine) copy_elements<4>(s, d, lo + i * 4, v, hi, cast);
    }
}

// ------------------------------------------------------------------ ag_pack

// One destination chunk (the rank's send chunk).
struct OneChunk {
    char* ptr;
    __device__ __forceinline__ char* at(int) const { return ptr; }
};

// Dst is OneChunk, or TableChunks when the packed chunk is pushed to W
// destinations (the peers' gathered buffers), each receiving the same bytes.
template <class Dst>
struct PackArgs {
    const float* src[PMAX];
    int64_t off[PMAX + 1];       // off[P] = S
    int64_t valid[PMAX];         // n_{p,rank} * inner_p
    int32_t tile_start[PMAX];    // first tile of parameter p; INT_MAX past the last parameter
    Dst dst;                     // bf16 or fp32 chunks of S elements
    int32_t ndst;                // destinations (1 for OneChunk)
    int32_t nparams;
    int32_t ntiles;
};

// One fp32 value -> its 16-bit pattern in format kOut (bf16 or fp16); four
// values -> four patterns packed in 8 bytes.
template <int kOut>
__device__ __forceinline__ uint32_t cast1(float f) { return kOut == kF16 ? f16_bits(f) : bf16_bits(f); }
template <int kOut>
__device__ __forceinline__ uint2 cast4(float4 a) {
    if constexpr (kOut == kBF16) return make_uint2(bf16x2_bits(a.x, a.y), bf16x2_bits(a.z, a.w));
    return make_uint2(cast1<kOut>(a.x) | (cast1<kOut>(a.y) << 16), cast1<kOut>(a.z) | (cast1<kOut>(a.w) << 16));
}

// The fields of the parameter a pack tile belongs to.
struct PackParam {
    const float* src;
    int64_t off;       // off_p
    int64_t region;    // off_{p+1} - off_p
    int64_t valid;     // n_{p,rank} * inner_p
};

// Lane-held argument tables.  Lane l of a wave loads entry l of each
// per-parameter table of the kernel arguments, every lane and table in one
// round of independent loads; from_lane then hands entry p to the whole wave.
// A kernel that takes its parameter's fields this way waits on one round trip
// to the argument table before its data loads, not on a chain of them (the
// tile table, then the entries of the parameter it names).  from_lane is only
// called where every lane of the wave is active, on values every lane wrote:
// a lane that is inactive when a value is computed keeps its old register,
// and readlane would return that.  The pack uses them: its look-up runs at the
// start of the launch, where no streams are in the way of a vector load, and
// one round of those is shorter than TilePlace's two or three scalar rounds
// (a 10 MB pack 5.1 us this way, 5.9 with TilePlace; the copies and the
// reduction, whose workgroups keep starting among running streams, are the
// other way round).
__device__ __forceinline__ int lane_index() { return int(threadIdx.x & 63); }
// The table entry a lane loads: its own, or the last one for the lanes past
// PMAX (none while PMAX is the wavefront width; their tile start is INT_MAX,
// so the lookup never selects them).
__device__ __forceinline__ int table_lane() { return min(lane_index(), PMAX - 1); }
__device__ __forceinline__ int32_t from_lane(int32_t v, int p) { return __builtin_amdgcn_readlane(v, p); }
__device__ __forceinline__ int64_t from_lane(int64_t v, int p) {
    const uint64_t u = uint64_t(v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u)), p));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u >> 32)), p));
    return int64_t((uint64_t(hi) << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T* from_lane(T* v, int p) {
    return as_global(reinterpret_cast<T*>(from_lane(reinterpret_cast<int64_t>(v), p)));
}

// The pack's lane-held table: lane l holds parameter l's entries.
struct PackLane {
    int start;          // tile_start[lane]
    const float* src;
    int64_t off, end, valid;

    template <class Dst>
    __device__ __forceinline__ explicit PackLane(const PackArgs<Dst>& a) {
        const int l = table_lane();
        start = lane_index() < PMAX ? a.tile_start[l] : INT_MAX;
        src = a.src[l];
        off = a.off[l];
        end = a.off[l + 1];
        valid = a.valid[l];
    }
    __device__ __forceinline__ PackParam param(int p) const {
        const int64_t o = from_lane(off, p);
        return PackParam{from_lane(src, p), o, from_lane(end, p) - o, from_lane(valid, p)};
    }
};

// A tile whose shard or whose place in the chunk is off the 16-byte grid (a
// dense bucket, A < 8, or a shard that is a view of flat storage): units of 4
// elements, loaded from any fp32 address and stored along the destination's
// 128-byte lines (several destinations share only the 16-byte grid), as in
// seg_copy_any.  The elements before the first line and units cut by the
// shard's or the region's end go one by one.  Two steps at a time: more keep
// no more in flight than HBM takes, and cost registers.
template <int kOut, class Dst, bool kNt, int kB, int kS>
__device__ __forceinline__ void pack_tile_any(const PackArgs<Dst>& a, const PackParam& pp, int64_t lo, int64_t hi) {
    constexpr bool kOne = std::is_same<Dst, OneChunk>::value;
    typedef typename std::conditional<kOut != kF32, uint16_t, uint32_t>::type Out;
    constexpr int kU = 4, kUnits = kB * kVec * kS / kU;
    constexpr int kLine = (kOne ? 128 : 16) / int(sizeof(Out));   // elements
    constexpr int kBytes = kU * int(sizeof(Out));
    constexpr int kPolicy = kNt ? kPolicyNt : 0;
    const int64_t v = pp.valid, region = pp.region;
    const int ndst = kOne ? 1 : a.ndst;
    const int t = threadIdx.x;
    const Out* const d0 = reinterpret_cast<const Out*>(a.dst.at(0)) + pp.off;
    const int h = (kLine - (int(reinterpret_cast<uintptr_t>(d0 + lo) / sizeof(Out)) & (kLine - 1))) & (kLine - 1);
    const int64_t at = lo + h;                                    // the first line at or after lo
    const auto cast = [](float f) { return Out(kOut != kF32 ? cast1<kOut>(f) : __float_as_uint(f)); };
    if (lo == 0 && t < h)
        for (int j = 0; j < ndst; ++j)
            copy_elements<1>(pp.src, reinterpret_cast<Out*>(a.dst.at(j)) + pp.off, t, v, min(at, hi), cast);
    const int nu = clamp_to((hi - at + kLine - 1) / kLine * kLine / kU, kUnits);
    const int whole = clamp_to((min(v, region) - at) >> 2, nu);
    const int zero_from = clamp_to((v - at + kU - 1) >> 2, nu), zero_to = clamp_to((region - at) >> 2, nu);
    const char* const from = as_global(reinterpret_cast<const char*>(pp.src + at));
#pragma unroll 1
    for (int u0 = 0; u0 < nu; u0 += 2 * kB) {
        u32x4 x[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = u0 + u * kB + t;
            x[u] = u32x4{0, 0, 0, 0};
            if (i < whole)
                x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any4*>(from + uint32_t(i) * (kU * 4)));
        }
        for (int j = 0; j < ndst; ++j) {
            Out* const d = reinterpret_cast<Out*>(a.dst.at(j)) + pp.off;
            const Window out = window(d + at, uint32_t(nu) * kBytes);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int i = u0 + u * kB + t;
                const bool unit = i < whole || (i >= zero_from && i < zero_to);
                const uint32_t byte = unit ? uint32_t(i) * kBytes : ~0u;    // past the window: dropped
                if constexpr (kOut == kF32) {
                    __builtin_amdgcn_raw_buffer_store_b128(x[u], out, int(byte), 0, kPolicy);
                } else {
                    const float4 f = {__uint_as_float(x[u].x), __uint_as_float(x[u].y), __uint_as_float(x[u].z),
                                      __uint_as_float(x[u].w)};
                    const uint2 c = cast4<kOut>(f);
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{c.x, c.y}, out, int(byte), 0, kPolicy);
                }
                if (!unit && i < nu) copy_elements<kU>(pp.src, d, at + int64_t(i) * kU, v, region, cast);
            }
        }
    }
}

// Tile lt of parameter pp: its part of [off_p, off_{p+1}) of the chunk, the
// shard's values cast to bf16 or fp16 or copied as fp32 (kOut), zeros past the shard,
// written to every destination.  Each thread handles 4 elements per sub-step
// (16 bytes of fp32 in), so every load and store instruction of a wave covers
// one contiguous run; the full tiles of a 16-bit push take 8 per thread.
// kAny: some parameter is off the 16-byte grid (the host picks it only then).
template <int kOut, class Dst, bool kAny, bool kNt = true, int kB = kPackBlock, int kS = kPackSteps>
__device__ __forceinline__ void pack_tile(const PackArgs<Dst>& a, const PackParam& pp, int lt) {
    constexpr int64_t kTile = int64_t(kB) * kVec * kS;
    constexpr bool kCast = kOut != kF32;
    typedef typename std::conditional<kCast, uint16_t, uint32_t>::type Out;
    constexpr int kSub = 2 * kS;
    constexpr bool kOne = std::is_same<Dst, OneChunk>::value;
    const int ndst = kOne ? 1 : a.ndst;
    const int64_t off = pp.off;
    const int64_t region = pp.region;
    const int64_t valid = pp.valid;
    const float* __restrict__ src = pp.src;
    const int64_t lo = int64_t(lt) * kTile;
    const int64_t hi = min(lo + kTile, region);
    if (lo >= hi) return;
    // every destination chunk is 16-byte aligned, so one test covers them all
    const bool vec = is_aligned16(src) && is_aligned16(reinterpret_cast<Out*>(a.dst.at(0)) + off);
    if constexpr (kAny) {
        if (!vec) {
            pack_tile_any<kOut, Dst, kNt, kB, kS>(a, pp, lo, hi);
            return;
        }
    }
    if constexpr (!kOne && kCast) {
        // Pushed to W destinations, the stores outnumber the loads W to 1:
        // each thread casts 8 consecutive elements and writes them with one
        // 16-byte store per destination.
        if (vec && hi - lo == kTile && lo + kTile <= valid) {
            uint4 y[kS];
#pragma unroll
            for (int u = 0; u < kS; ++u) {
                const float* s8 = src + lo + (int64_t(u) * kB + threadIdx.x) * 8;
                const uint2 c0 = cast4<kOut>(ld16f(s8));
                const uint2 c1 = cast4<kOut>(ld16f(s8 + 4));
                y[u] = make_uint4(c0.x, c0.y, c1.x, c1.y);
            }
            for (int j = 0; j < ndst; ++j) {
                Out* __restrict__ dst = reinterpret_cast<Out*>(a.dst.at(j)) + off;
#pragma unroll
                for (int u = 0; u < kS; ++u) st16<kNt>(dst + lo + (int64_t(u) * kB + threadIdx.x) * 8, y[u]);
            }
            return;
        }
    }
    if (vec && hi - lo == kTile && lo + kTile <= valid) {
        float4 x[kSub];
#pragma unroll
        for (int u = 0; u < kSub; ++u) x[u] = ld16f(src + lo + (int64_t(u) * kB + threadIdx.x) * 4);
        for (int j = 0; j < ndst; ++j) {
            Out* __restrict__ dst = reinterpret_cast<Out*>(a.dst.at(j)) + off;
#pragma unroll
            for (int u = 0; u < kSub; ++u) {
                const int64_t g = lo + (int64_t(u) * kB + threadIdx.x) * 4;
                if (kCast) st8<kNt>(dst + g, cast4<kOut>(x[u]));
                else st16f<kNt>(reinterpret_cast<float*>(dst + g), x[u]);
            }
        }
        return;
    }
    for (int u = 0; u < kSub; ++u) {
        const int64_t g = lo + (int64_t(u) * kB + threadIdx.x) * 4;
        if (g >= hi) break;
        if (vec && g + 4 <= hi && (g + 4 <= valid || g >= valid)) {
            const float4 x = g < valid ? ld16f(src + g) : make_float4(0.f, 0.f, 0.f, 0.f);
            for (int j = 0; j < ndst; ++j) {
                Out* __restrict__ dst = reinterpret_cast<Out*>(a.dst.at(j)) + off;
                if (kCast) st8<kNt>(dst + g, g < valid ? cast4<kOut>(x) : make_uint2(0, 0));
                else st16<kNt>(dst + g, g < valid ? make_uint4(__float_as_uint(x.x), __float_as_uint(x.y),
                                                          __float_as_uint(x.z), __float_as_uint(x.w))
                                             : make_uint4(0, 0, 0, 0));
            }
            continue;
        }
        for (int e = 0; e < 4; ++e) {
            const int64_t k = g + e;
            if (k >= hi) break;
            const Out v = k < valid ? Out(kCast ? cast1<kOut>(src[k]) : __float_as_uint(src[k])) : Out(0);
            for (int j = 0; j < ndst; ++j) (reinterpret_cast<Out*>(a.dst.at(j)) + off)[k] = v;
        }
    }
}

// Tiles numbered across the bucket; the parameter of a tile comes from the
// wave-ballot lookup.  The pack moves few bytes per launch, so its start-up
// chain is kept short: tile_start holds INT_MAX past the last parameter (no
// wait for the parameter count before the table load), the grid never exceeds
// the tile count (the first tile needs no bound check), and every field of
// the tile's parameter comes from the looked-up lane (PackLane), so the only
// wait before the data loads is the one round of table loads.  The big tile's
// registers are held to 64 so that 8 waves fit on each SIMD (the extra lane
// fields had cost one wave).  A tile is kB threads x kS steps of 8 elements.
template <int kOut, class Dst, int kB, int kS, bool kAny>
__global__ void __launch_bounds__(kB) __attribute__((amdgpu_waves_per_eu(8))) ag_pack_kernel(const PackArgs<Dst> a) {
    const PackLane lane(a);
    int64_t step = blockIdx.x;
    do {
        const int t = int(step);
        const int p = param_of_tile(lane.start, t);
        pack_tile<kOut, Dst, kAny, true, kB, kS>(a, lane.param(p), t - __builtin_amdgcn_readlane(lane.start, p));
        step += gridDim.x;
    } while (step < a.ntiles);
}

// The first half of a wide push: the rank's own chunk, stored through the
// cache so that the copies to the other destinations read it back from L2 and
// the MALL.  (Read back at once by many workgroups, a chunk just written with
// non-temporal stores streamed at little more than half the rate.)
template <int kOut, bool kAny>
__global__ void __launch_bounds__(kPackBlock) push_pack_kernel(const PackArgs<OneChunk> a) {
    const PackLane lane(a);
    int64_t step = blockIdx.x;
    do {
        const int t = int(step);
        const int p = param_of_tile(lane.start, t);
        pack_tile<kOut, OneChunk, kAny, false>(a, lane.param(p), t - __builtin_amdgcn_readlane(lane.start, p));
        step += gridDim.x;
    } while (step < a.ntiles);
}

// The second half of a wide push: chunk `from` copied to the other W - 1
// chunks of a table.  One work item is one tile of 16-byte units of one
// destination.  Workgroups are dealt to the 8 XCDs round-robin (workgroup b
// runs on XCD b mod 8; a grid-stride step is a multiple of 8), so the items are
// numbered to put all destinations of a tile on one XCD: the tile is read into
// that XCD's L2 once (cached loads) and written to each destination
// (non-temporal stores), each workgroup writing one contiguous run.
//
// From kRepGroup destinations up, they are copied in groups of kRepGroup,
// one group per grid row (blockIdx.y).  Workgroups are dispatched row by row,
// so the workgroups in flight write long runs into few destinations instead
// of short runs into all W - 1; the chunk is read once per group.
#ifndef FSDP_PUSH_REPLICATE_MIN_W
#define FSDP_PUSH_REPLICATE_MIN_W 8
#endif
constexpr int64_t kRepTile = kCopyBlock;          // 16-byte units per tile (2 KB)
constexpr int kReplicateMinW = FSDP_PUSH_REPLICATE_MIN_W;
constexpr int kRepGroupLog2 = 4;
constexpr int kRepGroup = 1 << kRepGroupLog2;     // destinations per grid row

struct ReplicateArgs {
    TableChunks dst;
    int64_t units;        // whole 16-byte units of a chunk
    int32_t tail;         // 2-byte elements after them
    int32_t from;         // the source chunk
    int32_t ndst;         // W - 1 destinations
    int32_t ntiles;
    int32_t nitems;
};

// Tile t of the source to destination index j (0 .. ndst-1, skipping `from`).
__device__ __forceinline__ void replicate_tile(const ReplicateArgs& a, const u32x4* __restrict__ src, int t, int j) {
    j += j >= a.from;                                // every chunk but the source
    u32x4* __restrict__ d = reinterpret_cast<u32x4*>(a.dst.ptr[j]);
    const int64_t g = int64_t(t) * kRepTile + threadIdx.x;
    if (g < a.units) {
        __builtin_nontemporal_store(src[g], d + g);
    } else if (g == a.units && a.tail > 0) {         // one thread copies the partial unit
        const uint16_t* s2 = reinterpret_cast<const uint16_t*>(src + a.units);
        uint16_t* d2 = reinterpret_cast<uint16_t*>(d + a.units);
        for (int e = 0; e < a.tail; ++e) d2[e] = s2[e];
    }
}

// Fewer than kRepGroup destinations: item i is tile round (i / 8) / ndst,
// destination (i / 8) mod ndst.
__global__ void __launch_bounds__(kCopyBlock) replicate_kernel(const ReplicateArgs a) {
    const u32x4* __restrict__ src = reinterpret_cast<const u32x4*>(a.dst.ptr[a.from]);
    for (int64_t step = blockIdx.x; step < a.nitems; step += gridDim.x) {
        const int i = int(step);
        const int k = i / kXcds;
        const int t = (k / a.ndst) * kXcds + i % kXcds;
        if (t >= a.ntiles) continue;
        replicate_tile(a, src, t, k % a.ndst);
    }
}

// kRepGroup destinations or more: row blockIdx.y holds destinations
// y*kRepGroup .. y*kRepGroup + kRepGroup - 1 (the last row may be short);
// item i of a row is tile round (i / 8) / kRepGroup.  `nitems` counts one row.
__global__ void __launch_bounds__(kCopyBlock) replicate_grouped_kernel(const ReplicateArgs a) {
    const u32x4* __restrict__ src = reinterpret_cast<const u32x4*>(a.dst.ptr[a.from]);
    for (int64_t step = blockIdx.x; step < a.nitems; step += gridDim.x) {
        const int i = int(step);
        const int k = i >> 3;
        const int t = ((k >> kRepGroupLog2) << 3) + (i & 7);
        const int j = int(blockIdx.y) * kRepGroup + (k & (kRepGroup - 1));
        if (t >= a.ntiles || j >= a.ndst) continue;
        replicate_tile(a, src, t, j);
    }
}

// ------------------------------------------------------------------ copy tile order

// The copy tile of workgroup-order index b.  Workgroups are dealt to the 8
// dies (XCDs) round-robin, so in tile order b each die would take every 8th
// 4 KB tile.  Instead, within each group of 8 * kXcdRun tiles, the workgroups
// of one die (b, b + 8, b + 16, ...) take kXcdRun consecutive tiles, a 1 MB
// run per die.  Against it, on the 8B, 70B and 405B blocks and the uneven
// bucket: plain order 1-3 % slower, runs of 16 tiles 8 %, of 128, 512 and 1024
// 0-3 %.  (The reduce takes it for some shards: see there.)  The tiles past the
// last whole group keep order b.  A bijection on [0, n), so a grid-stride loop over
// b still covers every tile once.
__device__ __forceinline__ uint32_t copy_tile(uint32_t b, uint32_t n) {
    constexpr uint32_t kGroup = uint32_t(kXcds) * kXcdRun;
    if (b >= n / kGroup * kGroup) return b;
    const uint32_t r = b % kGroup;
    return b - r + (r % kXcds) * kXcdRun + r / kXcds;
}

// n / d for 0 <= n < 2^31 by a multiplication: with 2^(l-1) < d <= 2^l and
// mul = ceil(2^(31+l) / d) < 2^32, n * mul / 2^(31+l) exceeds n / d by less
// than 1 / d, so its floor is the quotient.
struct Divider {
    uint32_t mul, shift;
    __device__ __forceinline__ uint32_t quotient(uint32_t n) const { return uint32_t((uint64_t(n) * mul) >> shift); }
};
Divider divider(uint32_t d) {
    int l = 0;
    while ((uint64_t(1) << l) < d) ++l;
    const uint64_t one = uint64_t(1) << (31 + l);
    return {uint32_t((one + d - 1) / d), uint32_t(31 + l)};
}

// The tiles of a W-way copy: chunk by chunk and, within a chunk, parameter by
// parameter, so a launch walks the bucket buffer front to front.
//
// What bounds the copies is HBM, and within that two things that are settled
// before a wave's first data load:
//   * the look-up.  A table read by vector loads waits in the same queues as
//     the streams of the waves around it (about one full loaded latency), so
//     everything here comes through the scalar cache: these fields in one
//     round, four entries of the full table above kPivots parameters, then the
//     parameter's record in one 32-byte load; the chunk by a multiplication.
//   * the bytes in flight.  A copy streams fastest with about 40 KB of loads
//     in flight per CU (20 waves of 2 KB, kCopyWaves per SIMD; a plain copy
//     loop peaks at 24-32 KB).  With all 32 waves the reads and writes of too
//     many places meet in the memory controllers, and the copy is slower.
// Both copies of the 70B block (3.42 GB): 530 -> 506 us unpack, 537 -> 512 us
// pack (the look-up without the cap: 548 and 537; the cap without the look-up:
// 531 and 532).  3 waves are 5 % slower, 8 waves 4-7 %; 4 / 5 / 6, contiguous
// buckets: 405B block's unpack 1887 / 1911 / 1920, its pack 1883 / 1885 / 1905;
// 70B 507 / 511 / 517 and 501 / 502 / 509; 8B at W = 8 131.4 / 130.0 / 131.4 and
// 129.7 / 129.0 / 130.5; 70B TP-8 shards 66.0 / 65.0 / 66.3 and 64.7 / 63.7 / 65.0:
// 4 for the largest unpacks, 5 elsewhere.
#ifndef FSDP_COPY_WAVES
#define FSDP_COPY_WAVES 5
#endif
constexpr int kCopyWaves = FSDP_COPY_WAVES;       // resident waves per SIMD
#ifndef FSDP_COPY_ANY_WAVES
#define FSDP_COPY_ANY_WAVES 6
#endif
// ... where some tiles take seg_copy_any, whose addresses take longer: 4 / 5 / 6 /
// 8 waves, uneven bucket, A = 1: unpack 880 / 792 / 771 / 781 us, pack 920 / 810 / 769
// / 771; 30 MB, W = 8, A = 1: unpack 14.9 / 13.6 / 13.1 / 13.3.
constexpr int kCopyAnyWaves = FSDP_COPY_ANY_WAVES;
// The widening pack has half the bytes in flight per wave: no cap.
template <int kWiden, bool kAny> constexpr int kPackMinWaves = kWiden != kF32 ? 4 : kAny ? kCopyAnyWaves : kCopyWaves;
template <int kWiden, bool kAny> constexpr int kPackMaxWaves = kWiden != kF32 ? 8 : kAny ? kCopyAnyWaves : kCopyWaves;

struct CopyTiles {
    uint32_t ntiles;               // W * per_chunk
    uint32_t per_chunk;            // tiles of one chunk
    Divider by_chunk;              // n / per_chunk
    TileTable table;               // of one chunk's tiles
};

// One parameter of a W-way copy, in 2-byte units (or 16-bit elements where
// they are widened to fp32): one 32-byte scalar load.
struct alignas(32) CopyParam {
    uint16_t* data;      // the full parameter or gradient
    int64_t off;         // off_p
    int64_t seg;         // L_p
    int64_t elems;       // N_p * inner_p
    // Elements of chunk i's segment (the last chunks' may be short or empty).
    __device__ __forceinline__ int64_t valid(int i) const {
        const int64_t rest = elems - int64_t(i) * seg;
        return rest < seg ? (rest > 0 ? rest : 0) : seg;
    }
};

// Entry p of the records, all of it loaded here (the fields that are needed
// late would otherwise be loaded late, in a round of their own).
__device__ __forceinline__ CopyParam load_param(const CopyParam* params, int p) {
    CopyParam q = params[p];
    asm volatile("" : "+s"(q.data), "+s"(q.off), "+s"(q.seg), "+s"(q.elems));
    q.data = as_global(q.data);
    return q;
}

// Where the tile of workgroup-order index `step` lies.
struct CopyPlace {
    int chunk, param;
    uint32_t tile;        // within the parameter's segment of that chunk
    __device__ __forceinline__ CopyPlace(const CopyTiles& c, uint32_t step) {
        const uint32_t t = copy_tile(step, c.ntiles);
        const uint32_t i = c.by_chunk.quotient(t);
        const TilePlace at(c.table, t - i * c.per_chunk);
        chunk = int(i);
        param = at.param;
        tile = at.tile;
    }
};

// ------------------------------------------------------------------ ag_unpack

// Sizes in 2-byte units (an fp32 element is two units).
template <class Chunks>
struct UnpackArgs {
    CopyTiles tiles;
    Chunks src;                  // gathered chunks, one per source rank
    CopyParam param[PMAX];
};

template <class Chunks, bool kAny>
__global__ void __launch_bounds__(kCopyBlock)
__attribute__((amdgpu_waves_per_eu(kAny ? kCopyAnyWaves : kCopyWaves, kAny ? kCopyAnyWaves : kCopyWaves)))
ag_unpack_kernel(const UnpackArgs<Chunks> a) {
    uint32_t step = blockIdx.x;
    do {
        const CopyPlace at(a.tiles, step);
        const int i = at.chunk;                          // source rank
        const CopyParam q = load_param(a.param, at.param);
        const int64_t v = q.valid(i);
        const int64_t lo = int64_t(at.tile) * kCopyTile;
        const int64_t hi = min(lo + kCopyTile, v);
        step += gridDim.x;
        if (lo >= hi) continue;
        const uint16_t* s = reinterpret_cast<const uint16_t*>(a.src.at(i)) + q.off;
        uint16_t* d = q.data + int64_t(i) * q.seg;
        seg_copy<kCopySteps, kAny>(s, d, lo, hi, hi, v, v);
    } while (step < a.tiles.ntiles);
}

// ------------------------------------------------------------------ rs_pack

// Sizes in units of the source gradient: 2-byte units for a plain copy, 16-bit
// elements when kWiden (kBF16 or kF16; kF32 = no widening) casts them to an
// fp32 wire.
template <class Chunks>
struct RsPackArgs {
    CopyTiles tiles;
    Chunks dst;                  // send chunks, one per destination rank
    CopyParam param[PMAX + 1];   // param[P].off = S
};

template <class Chunks, int kWiden, bool kAny>
__global__ void __launch_bounds__(kWiden != kF32 ? kWidenBlock : kCopyBlock)
__attribute__((amdgpu_waves_per_eu(kPackMinWaves<kWiden, kAny>, kPackMaxWaves<kWiden, kAny>)))
rs_pack_kernel(const RsPackArgs<Chunks> a) {
    uint32_t step = blockIdx.x;
    do {
        const CopyPlace at(a.tiles, step);
        const int j = at.chunk;                          // destination rank
        const CopyParam q = load_param(a.param, at.param);
        const int64_t region = a.param[at.param + 1].off - q.off;
        const int64_t v = q.valid(j);
        constexpr int64_t kTile = kWiden != kF32 ? kWidenTile : kCopyTile;
        const int64_t lo = int64_t(at.tile) * kTile;
        const int64_t hi = min(lo + kTile, region);
        step += gridDim.x;
        const uint16_t* s = q.data + int64_t(j) * q.seg;
        if constexpr (kWiden != kF32) {
            float* d = reinterpret_cast<float*>(a.dst.at(j)) + q.off;
            seg_widen<kWidenSteps, kWiden, kAny>(s, d, lo, hi, v);
        } else {
            uint16_t* d = reinterpret_cast<uint16_t*>(a.dst.at(j)) + q.off;
            seg_copy<kCopySteps, kAny>(s, d, lo, hi, v, v, region);
        }
    } while (step < a.tiles.ntiles);
}

// ------------------------------------------------------------------ rs_reduce

// One parameter of a reduction: one 32-byte scalar load.
struct alignas(32) ReduceParam {
    float* dst;
    int64_t off;                 // off_p
    int64_t valid;               // n_{p,rank} * inner_p
};

template <class Chunks>
struct ReduceArgs {
    uint32_t ntiles;
    int32_t world;
    TileTable table;
    Chunks src;                  // received chunks, one per source rank
    ReduceParam param[PMAX];
};

// The 16 bytes a lane loads from one source: kPer elements, added to as many
// fp32 sums.
template <typename T> struct Unit;
template <> struct Unit<uint16_t> {
    static constexpr int kPer = 8;
    __device__ __forceinline__ static void add(float (&acc)[8], const u32x4& x) {
        acc[0] += bf16_lo(x.x); acc[1] += bf16_hi(x.x);
        acc[2] += bf16_lo(x.y); acc[3] += bf16_hi(x.y);
        acc[4] += bf16_lo(x.z); acc[5] += bf16_hi(x.z);
        acc[6] += bf16_lo(x.w); acc[7] += bf16_hi(x.w);
    }
    __device__ __forceinline__ static float widen(uint16_t x) { return bf16_lo(x); }
};
template <> struct Unit<_Float16> {
    static constexpr int kPer = 8;
    __device__ __forceinline__ static void add(float (&acc)[8], const u32x4& x) {
        acc[0] += f16_lo(x.x); acc[1] += f16_hi(x.x);
        acc[2] += f16_lo(x.y); acc[3] += f16_hi(x.y);
        acc[4] += f16_lo(x.z); acc[5] += f16_hi(x.z);
        acc[6] += f16_lo(x.w); acc[7] += f16_hi(x.w);
    }
    __device__ __forceinline__ static float widen(_Float16 x) { return static_cast<float>(x); }
};
template <> struct Unit<float> {
    static constexpr int kPer = 4;
    __device__ __forceinline__ static void add(float (&acc)[4], const u32x4& x) {
        acc[0] += __uint_as_float(x.x); acc[1] += __uint_as_float(x.y);
        acc[2] += __uint_as_float(x.z); acc[3] += __uint_as_float(x.w);
    }
    __device__ __forceinline__ static float widen(float x) { return x; }
};

// A lane's 16-byte unit of one source: through a window of the tile's whole
// units (a lane past them reads zero), or (not kDirect) from any
// element-aligned address, `in` saying whether the lane has a unit.
template <bool kDirect, typename T>
__device__ __forceinline__ u32x4 load_unit(const char* tile, uint32_t unit_bytes, uint32_t lane_byte, bool in) {
    if constexpr (kDirect) return ld16(window(tile, unit_bytes), lane_byte);
    typedef typename std::conditional<sizeof(T) == 2, u32x4_any2, u32x4_any4>::type Any;
    return in ? __builtin_nontemporal_load(reinterpret_cast<const Any*>(as_global(tile) + lane_byte)) : u32x4{0, 0, 0, 0};
}

// The sums of a tile's whole units: row r of lane t holds outputs [kPer u,
// kPer u + kPer) with u = r * kB + t.  The W sources of every output are added
// in rank order; the loads of kNB sources are issued before the first of them
// is added.  A sum starts from -0, which leaves the first value as it is (its
// sign of zero too).
template <typename T, int kB, int kRows, int kNB, bool kDirect, class Chunks>
__device__ __forceinline__ void sum_units(float (&acc)[kRows][Unit<T>::kPer], const Chunks& src, int W, int64_t byte,
                                          uint32_t units) {
    const uint32_t t = threadIdx.x;
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int e = 0; e < Unit<T>::kPer; ++e) acc[r][e] = -0.f;
    const char* at[kNB];
#pragma unroll
    for (int b = 0; b < kNB; ++b) at[b] = src.ahead(b, W) + byte;
    u32x4 x[kNB][kRows];
    int i = 0;
    for (; i + kNB <= W; i += kNB) {
#pragma unroll
        for (int b = 0; b < kNB; ++b)
#pragma unroll
            for (int r = 0; r < kRows; ++r)
                x[b][r] = load_unit<kDirect, T>(at[b], units * 16, (r * kB + t) * 16, r * kB + t < units);
        // the next batch's addresses (from the chunk table) while these loads run
#pragma unroll
        for (int b = 0; b < kNB; ++b) at[b] = src.ahead(i + kNB + b, W) + byte;
#pragma unroll
        for (int b = 0; b < kNB; ++b)
#pragma unroll
            for (int r = 0; r < kRows; ++r) Unit<T>::add(acc[r], x[b][r]);
    }
#pragma unroll
    for (int b = 0; b < kNB - 1; ++b)
        if (i + b < W) {
#pragma unroll
            for (int r = 0; r < kRows; ++r)
                x[b][r] = load_unit<kDirect, T>(at[b], units * 16, (r * kB + t) * 16, r * kB + t < units);
        }
#pragma unroll
    for (int b = 0; b < kNB - 1; ++b)
        if (i + b < W) {
#pragma unroll
            for (int r = 0; r < kRows; ++r) Unit<T>::add(acc[r], x[b][r]);
        }
}

// One output, at element `at` of every chunk (the elements past a tile's
// whole units).
template <typename T, int kNB, class Chunks>
__device__ __forceinline__ float sum_one(const Chunks& src, int W, int64_t at) {
    float acc = -0.f;
    for (int i = 0; i < W; i += kNB) {
        T x[kNB];
#pragma unroll
        for (int b = 0; b < kNB; ++b) x[b] = reinterpret_cast<const T*>(src.at(min(i + b, W - 1)))[at];
#pragma unroll
        for (int b = 0; b < kNB; ++b) {
            const float sum = acc + Unit<T>::widen(x[b]);
            acc = i + b < W ? sum : acc;
        }
    }
    return acc;
}

// The averages of a tile's whole units.  A lane holds 8 outputs of a 16-bit
// wire: they pass through the wave's own part of LDS, so that every store
// instruction writes one contiguous run (stored as two halves per lane, every
// 128-byte line is written in two parts: 330 us instead of 285 on the 70B
// block's shape).  No other wave reads it, so no barrier is needed: a wave's
// LDS accesses stay in order, and the fences keep the compiler's order of them
// (release for the lanes' writes, acquire for the reads of other lanes').
//
// through: the stores write through.
template <int kB, int kRows, bool kDirect, int kPer>
__device__ __forceinline__ void store_units(float* tile, uint32_t units, const float (&acc)[kRows][kPer], float wf,
                                            bool through) {
    __shared__ f32x4 stage[kPer == 8 ? kB * 2 : 1];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x & ~63u;
    const uint32_t quads = units * (kPer / 4);       // 16-byte outputs of the tile
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        f32x4 out[kPer / 4];
        if constexpr (kPer == 4) {
            out[0] = f32x4{acc[r][0] / wf, acc[r][1] / wf, acc[r][2] / wf, acc[r][3] / wf};
        } else {
            f32x4* const mine = stage + wave * 2;
            mine[lane * 2] = f32x4{acc[r][0] / wf, acc[r][1] / wf, acc[r][2] / wf, acc[r][3] / wf};
            mine[lane * 2 + 1] = f32x4{acc[r][4] / wf, acc[r][5] / wf, acc[r][6] / wf, acc[r][7] / wf};
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            out[0] = mine[lane];
            out[1] = mine[64 + lane];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int h = 0; h < kPer / 4; ++h) {
            const uint32_t q = (r * kB + wave) * (kPer / 4) + h * 64 + lane;
            if constexpr (kDirect) {
                const Window to = window(tile, quads * 16);
                const u32x4 y = __builtin_bit_cast(u32x4, out[h]);
                if (through) st16(to, q * 16, y);
                else st16<kPolicyNt>(to, q * 16, y);
            } else {
                if (q < quads) __builtin_nontemporal_store(out[h], reinterpret_cast<f32x4_any4*>(tile + q * 4));
            }
        }
    }
}

// Whether a tile's averages are written through.  A tile that starts off the
// lines shares its first and last line with its neighbours, and written through
// such a line goes to memory in parts: 46.2 us so, 44.4 through the cache (bf16
// wire, W = 8, 100 waves per CU, shards 16 bytes off the lines; on them the
// check costs nothing that shows, but 0.1 us in the smallest shards' form,
// which is without it).  With an fp32
// wire of few sources the outputs are a large part of the traffic, and it is
// better for them not to wait in the L2: W = 2, 17.1 us against 18.5.
template <typename T>
__device__ __forceinline__ bool store_through(const float* out, int W) {
    return on_line(out) || (Unit<T>::kPer == 4 && W <= kReduceThroughW);
}

// A tile of a reduction: elements [first, first + n) of every chunk, n <= kElems.
// kRuns: the tiles are dealt to the dies in runs (copy_tile).
template <int kElems, bool kRuns>
struct ReduceSpot {
    int64_t first;
    uint32_t n;
    float* out;
    template <class Args>
    __device__ __forceinline__ ReduceSpot(const Args& a, uint32_t step) {
        const TilePlace at(a.table, kRuns ? copy_tile(step, a.ntiles) : step);
        ReduceParam q = a.param[at.param];
        asm volatile("" : "+s"(q.dst), "+s"(q.off), "+s"(q.valid));   // one load, here
        const int64_t lo = int64_t(at.tile) * kElems;
        const int64_t rest = q.valid - lo;
        n = rest < kElems ? uint32_t(rest) : uint32_t(kElems);        // at least 1
        first = q.off + lo;
        out = as_global(q.dst) + lo;
    }
};

// What bounds the reduction is HBM: W reads for one fp32 write.  As in the
// copies, the bytes in flight decide the rate: 24-32 KB of loads per CU stream
// best, and more make it slower again, because the reads of many places (and
// the few writes among them) then meet in the memory controllers.  So a
// workgroup is one wave with one unit per lane, kNB sources are in flight
// while the kNB before them are added, and the host picks kNB and the resident
// waves per SIMD by the waves that the whole shard makes (ReduceForm).
//
// Every batch issues the same number of loads (a source past W, or a tile past
// the last, has an empty window), so the wait for a batch never waits for the
// next one; the loads of a workgroup's next tile are issued before the current
// one is finished.
//
// kAny: some parameter's sources or outputs are off the 16-byte grid (the
// host picks it only then).  Such tiles load and store at any element, and a
// batch is added before the next one is loaded.  kRuns: see the host's choice
// of it.
template <class Chunks, typename T, int kNB, int kMaxWaves, bool kAny, bool kRuns>
__global__ void __launch_bounds__(kReduceBlock)
__attribute__((amdgpu_waves_per_eu(kMaxWaves < 8 ? kMaxWaves : kNB > 2 ? 4 : 8, kMaxWaves)))
rs_reduce_kernel(const ReduceArgs<Chunks> a) {
    constexpr int kPer = Unit<T>::kPer;
    typedef ReduceSpot<kReduceBlock * kPer, kRuns> Spot;
    const uint32_t t = threadIdx.x;
    const int W = a.world;
    const float wf = float(W);
    uint32_t step = blockIdx.x;
    if constexpr (kAny) {
        do {
            const Spot s(a, step);
            step += gridDim.x;
            const uint32_t units = s.n / kPer;
            const int64_t byte = s.first * int64_t(sizeof(T));
            float acc[1][kPer];
            if (a.src.aligned() && (byte & 15) == 0 && is_aligned16(s.out)) {
                sum_units<T, kReduceBlock, 1, kNB, true>(acc, a.src, W, byte, units);
                store_units<kReduceBlock, 1, true>(s.out, units, acc, wf, kNB > 2 || store_through<T>(s.out, W));
            } else {
                sum_units<T, kReduceBlock, 1, kNB, false>(acc, a.src, W, byte, units);
                store_units<kReduceBlock, 1, false>(s.out, units, acc, wf, false);
            }
            const uint32_t k = units * kPer + t;                  // fewer than kPer elements are left
            if (k < s.n) s.out[k] = sum_one<T, 4>(a.src, W, s.first + k) / wf;
        } while (step < a.ntiles);
        return;
    }
    Spot next(a, step);                         // the tile whose loads are issued
    int i = 0;                                  // its next source
    u32x4 x[2][kNB];
    const auto load = [&](u32x4 (&y)[kNB]) {
        const uint32_t bytes = step < a.ntiles ? next.n / kPer * 16 : 0;
#pragma unroll
        for (int b = 0; b < kNB; ++b)
            y[b] = ld16(window(a.src.ahead(i + b, W) + next.first * int64_t(sizeof(T)), i + b < W ? bytes : 0), t * 16);
        i += kNB;
    };
    load(x[0]);
    do {
        const Spot s = next;
        float acc[1][kPer];
#pragma unroll
        for (int e = 0; e < kPer; ++e) acc[0][e] = -0.f;
        const auto add = [&](const u32x4 (&y)[kNB], int sources) {
#pragma unroll
            for (int b = 0; b < kNB; ++b)
                if (b < sources) Unit<T>::add(acc[0], y[b]);
        };
        int j = 0;
        for (; j + 2 * kNB < W; j += 2 * kNB) {
            load(x[1]);
            __builtin_amdgcn_sched_barrier(0);  // the next batch's loads stay before this one's adds
            add(x[0], kNB);
            load(x[0]);
            __builtin_amdgcn_sched_barrier(0);
            add(x[1], kNB);
        }
        load(x[1]);
        step += gridDim.x;
        if (step < a.ntiles) next = Spot(a, step);
        i = 0;
        __builtin_amdgcn_sched_barrier(0);
        add(x[0], W - j);
        load(x[0]);
        __builtin_amdgcn_sched_barrier(0);
        add(x[1], W - j - kNB);
        const uint32_t units = s.n / kPer;
        store_units<kReduceBlock, 1, true>(s.out, units, acc, wf, kNB > 2 || store_through<T>(s.out, W));
        const uint32_t k = units * kPer + t;                      // fewer than kPer elements are left
        if (k < s.n) s.out[k] = sum_one<T, 4>(a.src, W, s.first + k) / wf;
    } while (step < a.ntiles);
}

// ------------------------------------------------------------------ host side

// From this many big pack tiles per CU up, a single-chunk pack uses them.
constexpr int kPackBigTilesPerCU = 4;

int cu_count(fsdp_status* st) {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        *st = fail(FSDP_ERR_HIP, "hipGetDevice failed");
        return 0;
    }
    if (dev >= 0 && dev < 64) {
        const int c = cache[dev].load(std::memory_order_relaxed);
        if (c > 0) return c;
    }
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
        *st = fail(FSDP_ERR_HIP, "hipDeviceGetAttribute(multiProcessorCount) failed");
        return 0;
    }
    if (dev >= 0 && dev < 64) cache[dev].store(n, std::memory_order_relaxed);
    return n;
}

struct Span {
    uintptr_t lo, hi;   // [lo, hi) bytes
};

// The byte spans of one call's inputs or outputs, on the stack: at most one
// per parameter or one per chunk of a table, so the hot calls allocate
// nothing on the host either.
constexpr int kMaxSpans = (PMAX > kMaxChunks ? PMAX : kMaxChunks) + 1;
struct Spans {
    Span s[kMaxSpans];
    int n = 0;
    bool full = false;   // more spans than kMaxSpans were added (the call is refused)
    void add(const void* p, int64_t bytes) {
        if (n < kMaxSpans) s[n++] = {uintptr_t(p), uintptr_t(p) + uintptr_t(bytes)};
        else full = true;
    }
};

// Outputs must be pairwise disjoint and disjoint from every input.
fsdp_status check_overlap(const Spans& out_spans, const Spans& ins) {
    if (out_spans.full || ins.full) return fail(FSDP_ERR_TOO_MANY, "too many buffers to check for overlap");
    Spans outs = out_spans;
    Span* const b = outs.s;
    Span* const e = outs.s + outs.n;
    std::sort(b, e, [](const Span& x, const Span& y) { return x.lo < y.lo; });
    for (int k = 1; k < outs.n; ++k)
        if (b[k].lo < b[k - 1].hi) return fail(FSDP_ERR_OVERLAP, "two outputs overlap");
    for (int k = 0; k < ins.n; ++k) {
        const Span& in = ins.s[k];
        // first output ending after in.lo
        const Span* it = std::upper_bound(b, e, in.lo, [](uintptr_t v, const Span& x) { return v < x.hi; });
        if (it != e && it->lo < in.hi) return fail(FSDP_ERR_OVERLAP, "an output overlaps an input");
    }
    return FSDP_OK;
}

// `index` >= 0 names element `index` of the array `name`.
fsdp_status check_bucket_ptr(const void* ptr, int64_t elems, const char* name, int index = -1) {
    const bool null = elems > 0 && ptr == nullptr;
    if (!null && (reinterpret_cast<uintptr_t>(ptr) & 15) == 0) return FSDP_OK;
    const std::string what = index < 0 ? std::string(name) : std::string(name) + "[" + std::to_string(index) + "]";
    if (null) return fail(FSDP_ERR_INVALID, what + " is NULL");
    return fail(FSDP_ERR_ALIGN, what + " is not 16-byte aligned");
}

fsdp_status check_param_ptr(const void* ptr, int64_t elems, int elem_bytes, int p, const char* what) {
    if (elems > 0 && ptr == nullptr)
        return fail(FSDP_ERR_INVALID, std::string(what) + "[" + std::to_string(p) + "] is NULL");
    if ((reinterpret_cast<uintptr_t>(ptr) & uintptr_t(elem_bytes - 1)) != 0)
        return fail(FSDP_ERR_ALIGN, std::string(what) + "[" + std::to_string(p) + "] is not element-aligned");
    return FSDP_OK;
}

const Plan* get_plan(const fsdp_plan* h, fsdp_status* st) {
    const Plan* pl = plan_of(h);
    if (!pl) *st = fail(FSDP_ERR_INVALID, "unknown plan handle");
    return pl;
}

bool known_dtype(fsdp_dtype t) { return t == FSDP_DTYPE_BF16 || t == FSDP_DTYPE_F32 || t == FSDP_DTYPE_F16; }
int elem_bytes(fsdp_dtype t) { return t == FSDP_DTYPE_F32 ? 4 : 2; }

// A host array of W chunk pointers, each 16-byte aligned and non-NULL when
// chunks have elements.
fsdp_status load_chunk_table(const Plan& pl, const void* const* chunks, int esize, TableChunks* out,
                             Spans* spans) {
    if (chunks == nullptr) return fail(FSDP_ERR_INVALID, "chunks is NULL");
    if (pl.world > kMaxChunks) return fail(FSDP_ERR_TOO_MANY, "world size exceeds FSDP_MAX_CHUNKS");
    fsdp_status st;
    for (int i = 0; i < pl.world; ++i) {
        if ((st = check_bucket_ptr(chunks[i], pl.chunk, "chunks", i)) != FSDP_OK) return st;
        out->ptr[i] = static_cast<char*>(const_cast<void*>(chunks[i]));
        if (pl.chunk > 0) spans->add(chunks[i], pl.chunk * esize);
    }
    return FSDP_OK;
}

// One launch of `kernel` over `ntiles` work tiles, one tile per workgroup up
// to kBlocksPerCU workgroups per CU (grid-stride beyond that).  The grid also
// keeps its work-item count below 2^31, and below the plan's max_workgroups
// when that is positive.
template <typename Args>
fsdp_status launch(const Plan& pl, void (*kernel)(const Args), const Args& args, int ntiles, int block,
                   hipStream_t stream, int rows = 1) {
    if (ntiles <= 0 || rows <= 0) return FSDP_OK;
    fsdp_status st = FSDP_OK;
    const int cus = cu_count(&st);
    if (st != FSDP_OK) return st;
    int64_t cap = std::min<int64_t>(int64_t(cus) * kBlocksPerCU, (int64_t(1) << 31) / block);
    if (pl.max_workgroups > 0) cap = std::min<int64_t>(cap, pl.max_workgroups);
    const dim3 grid(unsigned(std::min<int64_t>(ntiles, cap)), unsigned(rows));
    void* kargs[] = {const_cast<Args*>(&args)};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3(block), kargs, 0, stream);
    if (e != hipSuccess) return fail(FSDP_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
    return FSDP_OK;
}

int64_t tiles(int64_t n, int64_t tile) { return (n + tile - 1) / tile; }

// Whether every chunk of a bucket buffer starts on the 16-byte grid (the host
// has checked the base and every table entry; a contiguous buffer's stride
// may still be off the grid in a dense bucket).
bool chunks_aligned(const ContigChunks& c) { return ((uintptr_t(c.base) | uintptr_t(c.stride)) & 15) == 0; }
bool chunks_aligned(const TableChunks&) { return true; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// ---- ag_pack

template <int kOut, class Dst>
fsdp_status launch_pack(const Plan& pl, const PackArgs<Dst>& a, bool big, bool cached, bool any, hipStream_t stream) {
    if constexpr (std::is_same<Dst, OneChunk>::value) {
        if (cached && any) return launch(pl, push_pack_kernel<kOut, true>, a, a.ntiles, kPackBlock, stream);
        if (cached) return launch(pl, push_pack_kernel<kOut, false>, a, a.ntiles, kPackBlock, stream);
        if (big && any)
            return launch(pl, ag_pack_kernel<kOut, Dst, kPackBigBlock, kPackBigSteps, true>, a, a.ntiles, kPackBigBlock, stream);
        if (big)
            return launch(pl, ag_pack_kernel<kOut, Dst, kPackBigBlock, kPackBigSteps, false>, a, a.ntiles, kPackBigBlock, stream);
    }
    if (any) return launch(pl, ag_pack_kernel<kOut, Dst, kPackBlock, kPackSteps, true>, a, a.ntiles, kPackBlock, stream);
    return launch(pl, ag_pack_kernel<kOut, Dst, kPackBlock, kPackSteps, false>, a, a.ntiles, kPackBlock, stream);
}

// `dst` is the send chunk (OneChunk) or the W destination chunks
// (TableChunks); `outs` holds their byte spans for the overlap check.
template <class Dst>
fsdp_status do_ag_pack(const Plan& pl, int32_t rank, const float* const* shards, fsdp_dtype wire, const Dst& dst,
                       int ndst, const Spans& outs, hipStream_t stream, bool cached = false) {
    fsdp_status st;
    if (rank < 0 || rank >= pl.world) return fail(FSDP_ERR_INVALID, "rank out of range");
    if (shards == nullptr) return fail(FSDP_ERR_INVALID, "shards is NULL");
    PackArgs<Dst> a{};
    Spans ins;
    int64_t nt = 0, nt_big = 0;   // at most the planner's checked pack tile count
    bool any = false;
    for (int p = 0; p < pl.nparams; ++p) {
        const int64_t v = pl.local_elems(p, rank);
        if ((st = check_param_ptr(shards[p], v, 4, p, "shards")) != FSDP_OK) return st;
        a.src[p] = shards[p];
        a.off[p] = pl.off[p];
        a.valid[p] = v;
        nt += tiles(pl.off[p + 1] - pl.off[p], kPackTile);
        nt_big += tiles(pl.off[p + 1] - pl.off[p], kPackBigTile);
        // Every destination chunk is 16-byte aligned (the host has checked).
        if (!aligned16(shards[p]) || ((pl.off[p] * elem_bytes(wire)) & 15)) any = true;
        if (v > 0) ins.add(shards[p], v * 4);
    }
    a.off[pl.nparams] = pl.chunk;
    a.dst = dst;
    a.ndst = ndst;
    a.nparams = pl.nparams;
    if (nt > INT32_MAX) return fail(FSDP_ERR_OVERFLOW, "too many work tiles");
    if ((st = check_overlap(outs, ins)) != FSDP_OK) return st;
    // A single-chunk pack of at least kPackBigTilesPerCU big tiles per CU
    // takes the big tiles (more bytes in flight per wave); smaller buckets keep
    // the small ones, which spread evenly over the CUs.  (The first HIP call:
    // every argument is checked.)
    bool big = false;
    if constexpr (std::is_same<Dst, OneChunk>::value) {
        if (!cached) {
            const int cus = cu_count(&st);
            if (st != FSDP_OK) return st;
            big = nt_big >= int64_t(kPackBigTilesPerCU) * cus;
        }
    }
    const int64_t tile = big ? kPackBigTile : kPackTile;
    int64_t t0 = 0;
    for (int p = 0; p < pl.nparams; ++p) {
        a.tile_start[p] = int32_t(t0);
        t0 += tiles(pl.off[p + 1] - pl.off[p], tile);
    }
    for (int p = pl.nparams; p < PMAX; ++p) a.tile_start[p] = INT32_MAX;   // never a tile's parameter
    a.ntiles = int32_t(t0);
    if (wire == FSDP_DTYPE_BF16) return launch_pack<kBF16>(pl, a, big, cached, any, stream);
    if (wire == FSDP_DTYPE_F16) return launch_pack<kF16>(pl, a, big, cached, any, stream);
    return launch_pack<kF32>(pl, a, big, cached, any, stream);
}

fsdp_status do_ag_pack_one(const fsdp_plan* h, int32_t rank, const float* const* shards, fsdp_dtype wire,
                           void* send_chunk, hipStream_t stream) {
    clear_error();
    fsdp_status st = FSDP_OK;
    const Plan* pl = get_plan(h, &st);
    if (!pl) return st;
    if (!known_dtype(wire)) return fail(FSDP_ERR_INVALID, "unknown dtype");
    if ((st = check_bucket_ptr(send_chunk, pl->chunk, "send_chunk")) != FSDP_OK) return st;
    Spans outs;
    if (pl->chunk > 0) outs.add(send_chunk, pl->chunk * elem_bytes(wire));
    return do_ag_pack(*pl, rank, shards, wire, OneChunk{static_cast<char*>(send_chunk)}, 1, outs, stream);
}

// The rest of a tile table, once every parameter has its start.
void finish_table(const Plan& pl, TileTable* c) {
    for (int p = pl.nparams; p < PMAX; ++p) c->start[p] = UINT32_MAX;   // never a tile's parameter
    c->deep = pl.nparams > kPivots;
    for (int k = 0; k < kPivots; ++k) c->pivot[k] = c->start[c->deep ? k * kPerPivot : k];
}

// ---- the W-way copies: u = 2-byte units per element

// Parameter p has n tiles per chunk, its first being *nt.
fsdp_status add_copy_tiles(const Plan& pl, int p, int64_t n, CopyTiles* c, int64_t* nt) {
    if (n * pl.world > INT32_MAX || (*nt + n) * pl.world > INT32_MAX)
        return fail(FSDP_ERR_OVERFLOW, "too many work tiles");
    c->table.start[p] = uint32_t(*nt);
    *nt += n;
    return FSDP_OK;
}

// The rest of the table, once every parameter has its tiles (nt in a chunk).
void finish_copy_tiles(const Plan& pl, int64_t nt, CopyTiles* c) {
    finish_table(pl, &c->table);
    c->ntiles = uint32_t(nt * pl.world);
    c->per_chunk = uint32_t(nt);
    c->by_chunk = divider(uint32_t(std::max<int64_t>(nt, 1)));
}

// Whether every chunk of a bucket buffer starts on a 128-byte line.
bool chunks_on_lines(const ContigChunks& c, int) { return ((uintptr_t(c.base) | uintptr_t(c.stride)) & 127) == 0; }
bool chunks_on_lines(const TableChunks& c, int world) {
    uintptr_t all = 0;
    for (int i = 0; i < world; ++i) all |= uintptr_t(c.ptr[i]);
    return (all & 127) == 0;
}
// What a copy's segments are off: the 16-byte grid (read or written), or the
// 128-byte lines (written).
struct Off {
    bool grid, lines;
    // (read, written): the alignments in bytes of a segment's start and length.
    void add(int64_t read, int64_t written) {
        if (((read | written) & 15) != 0) grid = true;
        if ((written & 127) != 0) lines = true;
    }
};

// Whether a launch of `ntiles` copy tiles takes the any-address kernel: if some
// segment is off the grid, and, if one is written off the lines, from
// kCopyLineTilesPerCU tiles per CU on.  A large bucket pays for the lines that two
// tiles share; a small one for the longer way to a tile's first store.
// Line-following / aligned kernel, W = 32, all segments 16 bytes off the lines,
// MB over all ranks: rs_pack of 2 MB 4.8 / 3.6 us, 12 MB 7.7 / 7.1, 40 MB (38 tiles
// per CU) 16.6 / 16.0, 60 MB 21.8 / 22.4, 600 MB 182 / 202; ag_unpack of 2 MB 4.6 /
// 3.6, 12 MB 7.5 / 7.1, 40 MB 16.3 / 16.1, 60 MB 21.9 / 22.7, 600 MB 183 / 200.
constexpr int kCopyLineTilesPerCU = 44;
// From here on the widening pack's tiles off the lines are not written through.
// bf16 on an fp32 wire, segments 32 bytes off the lines, MB of fp32 over all
// ranks, written through / not: W = 1 30 MB 10.6 / 10.5 us, 100 MB (95 tiles per
// CU) 27.1 / 26.3, 400 MB 101 / 95; W = 8 30 MB 10.5 / 10.8, 60 MB 18.3 / 18.1, 100
// MB 28.6 / 27.8, 400 MB 103 / 98; W = 32 20 MB 8.2 / 8.6, 100 MB 27.8 / 27.7, 400 MB
// 105 / 98.
constexpr int kWidenLineTilesPerCU = 96;

fsdp_status copy_takes_any(const Off& off, int64_t ntiles, int line_tiles_per_cu, bool* any) {
    *any = off.grid;
    if (off.grid || !off.lines || ntiles == 0) return FSDP_OK;
    fsdp_status st = FSDP_OK;
    const int cus = cu_count(&st);
    *any = ntiles >= int64_t(line_tiles_per_cu) * cus;
    return st;
}

// ---- ag_unpack

template <class Chunks>
fsdp_status do_ag_unpack(const Plan& pl, const Chunks& src, const Spans& ins, int u,
                         void* const* params, hipStream_t stream) {
    fsdp_status st;
    if (params == nullptr) return fail(FSDP_ERR_INVALID, "params is NULL");
    UnpackArgs<Chunks> a{};
    Spans outs;
    int64_t nt = 0;               // tiles of one chunk
    Off off{!chunks_aligned(src), false};
    for (int p = 0; p < pl.nparams; ++p) {
        const int64_t e = pl.elems[p];
        if ((st = check_param_ptr(params[p], e, 2 * u, p, "params")) != FSDP_OK) return st;
        a.param[p] = {static_cast<uint16_t*>(params[p]), pl.off[p] * u, pl.seg[p] * u, e * u};
        if ((st = add_copy_tiles(pl, p, tiles(pl.seg[p] * u, kCopyTile), &a.tiles, &nt)) != FSDP_OK) return st;
        // Segment i of parameter p is read from chunk i at off_p and written
        // to params[p] at i * L_p.
        off.add(a.param[p].off * 2, (a.param[p].seg * 2) | int64_t(uintptr_t(params[p])));
        if (e > 0) outs.add(params[p], e * 2 * u);
    }
    a.src = src;
    finish_copy_tiles(pl, nt, &a.tiles);
    if ((st = check_overlap(outs, ins)) != FSDP_OK) return st;
    bool any;
    if ((st = copy_takes_any(off, a.tiles.ntiles, kCopyLineTilesPerCU, &any)) != FSDP_OK) return st;
    if (any) return launch(pl, ag_unpack_kernel<Chunks, true>, a, int(a.tiles.ntiles), kCopyBlock, stream);
    return launch(pl, ag_unpack_kernel<Chunks, false>, a, int(a.tiles.ntiles), kCopyBlock, stream);
}

// ---- rs_pack: gradient elements of `gsize` bytes; kWiden (kBF16 / kF16) casts
// 16-bit gradients to fp32, kF32 copies

template <class Chunks, int kWiden>
fsdp_status do_rs_pack(const Plan& pl, const void* const* grads, int gsize, const Chunks& dst,
                       const Spans& outs, hipStream_t stream) {
    fsdp_status st;
    if (grads == nullptr) return fail(FSDP_ERR_INVALID, "grads is NULL");
    const int u = kWiden != kF32 ? 1 : gsize / 2;     // kernel units per element
    constexpr int64_t kTile = kWiden != kF32 ? kWidenTile : kCopyTile;
    constexpr int kBlock = kWiden != kF32 ? kWidenBlock : kCopyBlock;
    RsPackArgs<Chunks> a{};
    Spans ins;
    int64_t nt = 0;               // tiles of one chunk
    Off off{!chunks_aligned(dst), !chunks_on_lines(dst, pl.world)};
    for (int p = 0; p < pl.nparams; ++p) {
        const int64_t e = pl.elems[p];
        if ((st = check_param_ptr(grads[p], e, gsize, p, "grads")) != FSDP_OK) return st;
        a.param[p] = {static_cast<uint16_t*>(const_cast<void*>(grads[p])), pl.off[p] * u, pl.seg[p] * u, e * u};
        const int64_t n = tiles((pl.off[p + 1] - pl.off[p]) * u, kTile);
        if ((st = add_copy_tiles(pl, p, n, &a.tiles, &nt)) != FSDP_OK) return st;
        // Segment j of parameter p is read from grads[p] at j * L_p and written
        // to chunk j at off_p.
        if (kWiden == kF32) off.add((a.param[p].seg * 2) | int64_t(uintptr_t(grads[p])), a.param[p].off * 2);
        else off.add(0, pl.off[p] * 4);
        if (e > 0) ins.add(grads[p], e * gsize);
    }
    a.param[pl.nparams].off = pl.chunk * u;
    a.dst = dst;
    finish_copy_tiles(pl, nt, &a.tiles);
    if ((st = check_overlap(outs, ins)) != FSDP_OK) return st;
    if (kWiden != kF32) off.grid = false;              // the widening pack's one form takes any address
    bool any;
    if ((st = copy_takes_any(off, a.tiles.ntiles, kWiden == kF32 ? kCopyLineTilesPerCU : kWidenLineTilesPerCU, &any)) != FSDP_OK)
        return st;
    if (any) return launch(pl, rs_pack_kernel<Chunks, kWiden, true>, a, int(a.tiles.ntiles), kBlock, stream);
    return launch(pl, rs_pack_kernel<Chunks, kWiden, false>, a, int(a.tiles.ntiles), kBlock, stream);
}

// ---- rs_reduce: received elements of type T

template <class Chunks, typename T, int kNB, int kMaxWaves, bool kAny, bool kRuns>
fsdp_status launch_reduce(const Plan& pl, const ReduceArgs<Chunks>& a, hipStream_t stream) {
    return launch(pl, rs_reduce_kernel<Chunks, T, kNB, kMaxWaves, kAny, kRuns>, a, int(a.ntiles), kReduceBlock, stream);
}

template <class Chunks, typename T, int kNB, int kMaxWaves>
fsdp_status launch_reduce(const Plan& pl, const ReduceArgs<Chunks>& a, bool runs, hipStream_t stream) {
    if (runs) return launch_reduce<Chunks, T, kNB, kMaxWaves, false, true>(pl, a, stream);
    return launch_reduce<Chunks, T, kNB, kMaxWaves, false, false>(pl, a, stream);
}

template <class Chunks, typename T>
fsdp_status do_rs_reduce(const Plan& pl, int32_t rank, const Chunks& src, const Spans& ins,
                         float* const* grad_shards, hipStream_t stream) {
    fsdp_status st = FSDP_OK;
    if (grad_shards == nullptr) return fail(FSDP_ERR_INVALID, "grad_shards is NULL");
    constexpr int64_t kWave = int64_t(kReduceBlock) * Unit<T>::kPer;   // outputs of one wave
    Spans outs;
    int64_t waves = 0, waves_off = 0;   // all waves, those whose sources are off the 128-byte lines
    bool any = !chunks_aligned(src);
    const bool lines = chunks_on_lines(src, pl.world);
    for (int p = 0; p < pl.nparams; ++p) {
        const int64_t v = pl.local_elems(p, rank);
        if ((st = check_param_ptr(grad_shards[p], v, 4, p, "grad_shards")) != FSDP_OK) return st;
        if (v > 0) outs.add(grad_shards[p], v * 4);
        // Sources of parameter p start at off_p in every chunk.
        const int64_t byte = pl.off[p] * int64_t(sizeof(T));
        if ((byte & 15) || !aligned16(grad_shards[p])) any = true;
        waves += tiles(v, kWave);
        if (!lines || (byte & 127)) waves_off += tiles(v, kWave);
    }
    if ((st = check_overlap(outs, ins)) != FSDP_OK) return st;
    if (waves == 0) return FSDP_OK;                      // nothing to write: no launch
    if (waves > INT32_MAX) return fail(FSDP_ERR_OVERFLOW, "too many work tiles");
    // (The first HIP call: every argument is checked.)
    const int cus = cu_count(&st);
    if (st != FSDP_OK) return st;
    // The shard's waves per CU decide how many sources a wave keeps in flight
    // (24-32 KB per CU, as far as the shard goes).  Measured, kNB = 1 / 2 / 4:
    // 8B block at W = 128 (13 waves per CU) 66.8 / 68.0 / 71.3 us; 0.95 M outputs
    // at W = 64 (7 waves) 24.7 / 21.6 / 22.7; 64 norm shards at W = 32 (1 wave on
    // every fourth CU) 7.9 / 5.8 / 4.8.  Off the grid, where a batch is added before
    // the next is loaded, never one source.  There, kNB = 2 with the cap / 4, bf16,
    // W = 24: 3 waves per CU 11.5 / 9.4 us, 8 waves 14.3 / 15.0, 12 waves 16.1 / 17.1, 20
    // waves 27.6 / 25.8, 64 waves 75 / 87; at 5 to 7 waves these bounds, which are
    // the other form's, are not the best ones (6 waves 13.4 / 11.4).  Dense uneven
    // bucket: two sources 437 us, 488 without the cap.
    //
    // Where the waves are more than stream well together, how many are resident
    // per SIMD.  3 / 4 / 8: 70B block, W = 64: 262 / 274 / 283; uneven bucket,
    // W = 48: 404 / 416 / 436; 8B block, W = 8: 88 / 87 / 89; five segments on
    // the lines, W = 16, 31 waves per CU: 26.5 / 24.8 / 26.8, 64 waves: 49.5 / 46.3
    // / 49.5.  A wave of few sources is not long in its stream, and needs the
    // others beside it, with more sources unless the shard takes many rounds: W = 3,
    // 64 waves per CU 19.8 / 18.1 / 16.8; 4 / 8: W = 1, 200 waves 31.0 / 27.3, W = 4, fp32,
    // 600 waves 119 / 125, W = 8, fp16, 28 waves 15.1 / 14.4, W = 64, fp32, 28 waves 68.9 /
    // 73.8.
    const auto from = [&](int per_cu) { return waves >= int64_t(per_cu) * cus; };
    bool large = from(pl.world <= kReduceSomeW ? kReduceSomeWaves : kReduceCapWaves);
    bool wide = pl.world >= kReduceWideW && from(kReduceWideWaves);
    int batch = from(kReduceOneWaves) ? 1 : from(kReduceTwoWaves) ? 2 : 4;
    if (pl.reduce_tiles == FSDP_REDUCE_TILES_FULL) large = true, wide = pl.world >= kReduceWideW, batch = 1;
    if (pl.reduce_tiles == FSDP_REDUCE_TILES_HALF) large = wide = false, batch = 4;
    // Off the 128-byte lines two neighbouring tiles share a line of every source.
    // In plain order they run on different dies, and each die's L2 fetches the
    // line; so the tiles are dealt in runs, as the copies' are, where the sources
    // of most of them are off the lines.  Five segments 16 bytes off the lines,
    // 64 waves per CU, plain / runs: W = 8 31.8 / 29.2 us, W = 32 101 / 90 us;
    // 16 waves per CU, W = 32: 30.0 / 24.6.  (The form for the smallest shards
    // has no such order: 8 runs are 8 waves per CU.)
    //
    // On the lines runs are better where a shard takes a few rounds of resident
    // waves, plain / runs: W = 64, 32 waves per CU 87.9 / 83.5 us, 40 waves 117 / 107; W
    // = 16, 96 waves 73.7 / 71.3, 128 waves 97.4 / 94.4; 70B block's TP-8 shards, W = 8:
    // 45.6 / 44.4.  They are no better where most of it is resident (W = 128, fp32,
    // 30 waves: 146 / 153; 8B block, fp32: 129 / 131) or where it takes many rounds
    // (W = 16, 300 waves: 220 / 226, 600 waves: 437 / 460; 8B block, W = 8, fp32: 150 /
    // 153; 70B block, W = 64: 262 / 264).
    const bool off = 2 * waves_off > waves;
    const bool rounds = pl.world >= kReduceWideW ? wide && !from(kReduceWidePlainWaves) : large && !from(kReducePlainWaves);
    const bool runs = off || rounds;
    // Tiles of the parameters with the fewest tiles are numbered (and so
    // dispatched) first: a ragged last tile sums its W sources in a longer
    // dependent chain, which then overlaps the bulk instead of trailing it.
    // (A stable insertion sort of at most FSDP_MAX_PARAMS entries: equal
    // counts keep the bucket order, and nothing is allocated.)
    int order[PMAX];
    int64_t nts[PMAX];
    for (int p = 0; p < pl.nparams; ++p) {
        nts[p] = tiles(pl.local_elems(p, rank), kWave);
        int q = p;
        for (; q > 0 && nts[order[q - 1]] > nts[p]; --q) order[q] = order[q - 1];
        order[q] = p;
    }
    ReduceArgs<Chunks> a{};
    int64_t t0 = 0;
    for (int q = 0; q < pl.nparams; ++q) {
        const int p = order[q];
        a.param[q] = {grad_shards[p], pl.off[p], pl.local_elems(p, rank)};
        a.table.start[q] = uint32_t(t0);
        t0 += nts[p];
    }
    finish_table(pl, &a.table);
    a.src = src;
    a.world = pl.world;
    a.ntiles = uint32_t(t0);
    if (any) {
        if (batch == 4) return launch_reduce<Chunks, T, 4, 8, true, false>(pl, a, stream);
        if (off) return launch_reduce<Chunks, T, 2, kReduceWaves, true, true>(pl, a, stream);
        return launch_reduce<Chunks, T, 2, kReduceWaves, true, false>(pl, a, stream);
    }
    if (wide) return launch_reduce<Chunks, T, 1, kReduceWaves - 1>(pl, a, runs, stream);
    if (large && pl.world > (rounds ? kReduceFewW : kReduceFewestW))
        return launch_reduce<Chunks, T, 1, kReduceWaves>(pl, a, runs, stream);
    if (batch == 1) return launch_reduce<Chunks, T, 1, 8>(pl, a, runs, stream);
    if (batch == 2) return launch_reduce<Chunks, T, 2, 8>(pl, a, runs, stream);
    return launch_reduce<Chunks, T, 4, 8, false, false>(pl, a, stream);
}

}  // namespace
}  // namespace fsdp

using namespace fsdp;

extern "C" fsdp_status fsdp_ag_pack(const fsdp_plan* h, int32_t rank, const float* const* shards,
                                    uint16_t* send_chunk, hipStream_t stream) {
    return do_ag_pack_one(h, rank, shards, FSDP_DTYPE_BF16, send_chunk, stream);
}

extern "C" fsdp_status fsdp_ag_pack_ex(const fsdp_plan* h, int32_t rank, const float* const* shards,
                                       fsdp_dtype param_dtype, void* send_chunk, hipStream_t stream) {
    return do_ag_pack_one(h, rank, shards, param_dtype, send_chunk, stream);
}

extern "C" fsdp_status fsdp_ag_pack_push(const fsdp_plan* h, int32_t rank, const float* const* shards,
                                         fsdp_dtype param_dtype, void* const* chunks, hipStream_t stream) {
    clear_error();
    fsdp_status st = FSDP_OK;
    const Plan* pl = get_plan(h, &st);
    if (!pl) return st;
    if (!known_dtype(param_dtype)) return fail(FSDP_ERR_INVALID, "unknown dtype");
    if (rank < 0 || rank >= pl->world) return fail(FSDP_ERR_INVALID, "rank out of range");
    const int esize = elem_bytes(param_dtype);
    TableChunks dst{};
    Spans outs;
    if ((st = load_chunk_table(*pl, const_cast<const void* const*>(chunks), esize, &dst, &outs)) != FSDP_OK)
        return st;
    if (pl->world < kReplicateMinW || pl->chunk == 0)
        return do_ag_pack(*pl, rank, shards, param_dtype, dst, pl->world, outs, stream);
    // Many destinations: pack once into the rank's own chunk (through the
    // cache), then copy that chunk to the other W - 1.  Every chunk's span is
    // in the overlap check of the pack.
    ReplicateArgs r{};
    r.dst = dst;
    const int64_t bytes = pl->chunk * esize;
    r.units = bytes / 16;
    r.tail = int32_t(bytes % 16 / 2);
    r.from = rank;
    r.ndst = pl->world - 1;
    const int64_t nt = tiles(r.units + (r.tail > 0), kRepTile);
    const bool grouped = r.ndst >= kRepGroup;
    const int64_t items = tiles(nt, kXcds) * kXcds * (grouped ? kRepGroup : r.ndst);
    if (items > INT32_MAX) return fail(FSDP_ERR_OVERFLOW, "too many work tiles");
    r.ntiles = int32_t(nt);
    r.nitems = int32_t(items);
    if ((st = do_ag_pack(*pl, rank, shards, param_dtype, OneChunk{dst.ptr[rank]}, 1, outs, stream, true)) != FSDP_OK)
        return st;
    if (grouped)
        return launch(*pl, replicate_grouped_kernel, r, r.nitems, kCopyBlock, stream, int(tiles(r.ndst, kRepGroup)));
    return launch(*pl, replicate_kernel, r, r.nitems, kCopyBlock, stream);
}

extern "C" fsdp_status fsdp_ag_unpack(const fsdp_plan* h, const uint16_t* gathered, uint16_t* const* params,
                                      hipStream_t stream) {
    clear_error();
    fsdp_status st = FSDP_OK;
    const Plan* pl = get_plan(h, &st);
    if (!pl) return st;
    const int64_t total = int64_t(pl->world) * pl->chunk;
    if ((st = check_bucket_ptr(gathered, total, "gathered")) != FSDP_OK) return st;
    Spans ins;
    if (total > 0) ins.add(gathered, total * 2);
    const ContigChunks src{reinterpret_cast<char*>(const_cast<uint16_t*>(gathered)), pl->chunk * 2};
    return do_ag_unpack(*pl, src, ins, 1, reinterpret_cast<void* const*>(params), stream);
}

extern "C" fsdp_status fsdp_ag_unpack_ex(const fsdp_plan* h, fsdp_dtype param_dtype, const void* const* chunks,
                                         void* const* params, hipStream_t stream) {
    clear_error();
    fsdp_status st = FSDP_OK;
    const Plan* pl = get_plan(h, &st);
    if (!pl) return st;
    if (!known_dtype(param_dtype)) return fail(FSDP_ERR_INVALID, "unknown dtype");
    const int esize = elem_bytes(param_dtype);
    TableChunks src{};
    Spans ins;
    if ((st = load_chunk_table(*pl, chunks, esize, &src, &ins)) != FSDP_OK) return st;
    return do_ag_unpack(*pl, src, ins, esize / 2, params, stream);
}

extern "C" fsdp_status fsdp_rs_pack(const fsdp_plan* h, const uint16_t* const* grads, uint16_t* send_buf,
                                    hipStream_t stream) {
    clear_error();
    fsdp_status st = FSDP_OK;
    const Plan* pl = get_plan(h, &st);
    if (!pl) return st;
    const int64_t total = int64_t(pl->world) * pl->chunk;
    if ((st = check_bucket_ptr(send_buf, total, "send_buf")) != FSDP_OK) return st;
    Spans outs;
    if (total > 0) outs.add(send_buf, total * 2);
    const ContigChunks dst{reinterpret_cast<char*>(send_buf), pl->chunk * 2};
    return do_rs_pack<ContigChunks, kF32>(*pl, reinterpret_cast<const void* const*>(grads), 2, dst, outs, stream);
}

extern "C" fsdp_status fsdp_rs_pack_ex(const fsdp_plan* h, fsdp_dtype grad_dtype, const void* const* grads,
                                       fsdp_dtype reduce_dtype, void* const* chunks, hipStream_t stream) {
    clear_error();
    fsdp_status st = FSDP_OK;
    const Plan* pl = get_plan(h, &st);
    if (!pl) return st;
    if (!known_dtype(grad_dtype) || !known_dtype(reduce_dtype)) return fail(FSDP_ERR_INVALID, "unknown dtype");
    // the wire keeps the gradients' type or widens 16-bit gradients to fp32;
    // any other pair would be a rounding step the method does not describe
    if (reduce_dtype != grad_dtype && reduce_dtype != FSDP_DTYPE_F32)
        return fail(FSDP_ERR_INVALID, "the wire must have the gradients' type or be fp32");
    TableChunks dst{};
    Spans outs;
    if ((st = load_chunk_table(*pl, chunks, elem_bytes(reduce_dtype), &dst, &outs)) != FSDP_OK) return st;
    if (grad_dtype == FSDP_DTYPE_BF16 && reduce_dtype == FSDP_DTYPE_F32)
        return do_rs_pack<TableChunks, kBF16>(*pl, grads, 2, dst, outs, stream);
    if (grad_dtype == FSDP_DTYPE_F16 && reduce_dtype == FSDP_DTYPE_F32)
        return do_rs_pack<TableChunks, kF16>(*pl, grads, 2, dst, outs, stream);
    return do_rs_pack<TableChunks, kF32>(*pl, grads, elem_bytes(grad_dtype), dst, outs, stream);
}

extern "C" fsdp_status fsdp_rs_reduce(const fsdp_plan* h, int32_t rank, const uint16_t* recv,
                                      float* const* grad_shards, hipStream_t stream) {
    clear_error();
    fsdp_status st = FSDP_OK;
    const Plan* pl = get_plan(h, &st);
    if (!pl) return st;
    if (rank < 0 || rank >= pl->world) return fail(FSDP_ERR_INVALID, "rank out of range");
    const int64_t total = int64_t(pl->world) * pl->chunk;
    if ((st = check_bucket_ptr(recv, total, "recv")) != FSDP_OK) return st;
    Spans ins;
    if (total > 0) ins.add(recv, total * 2);
    const ContigChunks src{reinterpret_cast<char*>(const_cast<uint16_t*>(recv)), pl->chunk * 2};
    return do_rs_reduce<ContigChunks, uint16_t>(*pl, rank, src, ins, grad_shards, stream);
}

extern "C" fsdp_status fsdp_rs_reduce_ex(const fsdp_plan* h, int32_t rank, fsdp_dtype reduce_dtype,
                                         const void* const* chunks, float* const* grad_shards, hipStream_t stream) {
    clear_error();
    fsdp_status st = FSDP_OK;
    const Plan* pl = get_plan(h, &st);
    if (!pl) return st;
    if (!known_dtype(reduce_dtype)) return fail(FSDP_ERR_INVALID, "unknown dtype");
    if (rank < 0 || rank >= pl->world) return fail(FSDP_ERR_INVALID, "rank out of range");
    TableChunks src{};
    Spans ins;
    if ((st = load_chunk_table(*pl, chunks, elem_bytes(reduce_dtype), &src, &ins)) != FSDP_OK) return st;
    if (reduce_dtype == FSDP_DTYPE_F32) return do_rs_reduce<TableChunks, float>(*pl, rank, src, ins, grad_shards, stream);
    if (reduce_dtype == FSDP_DTYPE_F16)
        return do_rs_reduce<TableChunks, _Float16>(*pl, rank, src, ins, grad_shards, stream);
    return do_rs_reduce<TableChunks, uint16_t>(*pl, rank, src, ins, grad_shards, stream);
}
