// gfx950 kernels of libmics and their launchers.
//
// All four steps stream every byte once and do at most a few operations per
// element, so they are bound by HBM bandwidth, not by the matrix or vector
// units.  The kernels therefore aim at: 128-bit global loads and stores that
// cover contiguous memory per wavefront instruction, all of a lane's loads in
// flight before the first use, no re-reads, and grids with one pass per lane:
// workgroups are dispatched in index order, so the lanes in flight cover a
// compact window of every buffer that advances through memory (measured on
// MI355X: a lane that owns several vectors a grid stride apart, or a small
// persistent grid, loses 5-30 % of the bandwidth, stores most of all).
//
// Alignment.  gfx950 executes a 128-bit global access at any address, at full speed from 4 bytes on (2-byte
// aligned ones lose about 20 % of a p = 16 reduction).  What costs is the 128-byte lines that two wavefronts share:
// a 1 KiB access off the lines touches nine instead of eight (Adam, everything 4 bytes off, 20 M elements 92 us ->
// 122).  So the element-wise kernels use 128-bit accesses on under-aligned vector types everywhere, a lane
// that would cross the end of a buffer works element by element inside the same kernel (no tail launches), and
// the gradient pointers, most of a reduction's bytes, are rounded down to the lines (align_gradient_pointers).
//
// Arithmetic rules (they make the results reproducible bit for bit):
//   - no fused multiply-add (-ffp-contract=off and the pragma below),
//   - sums in the order the header states,
//   - correctly rounded fp32 division and square root,
//   - fp32 denormals are kept.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "internal.h"
#include "launch_rules.h"

#pragma clang fp contract(off)

namespace mics {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// The same vectors at the alignment of their elements (see "Alignment" above).
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
typedef u32x2 u32x2_a2 __attribute__((aligned(2)));
typedef uint32_t u32_a2 __attribute__((aligned(2)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
typedef f32x2 f32x2_a4 __attribute__((aligned(4)));

// Launch shape and cache hints per kernel family; the defaults are the measured best on
// MI355X for the h = 8192, p = 16 shard shapes.  *_BLOCK = workgroup size, *_BPC = cap on
// workgroups per compute unit (the grid covers the data with one pass per lane unless the
// cap is reached; lanes stride over the rest), *_NTL = non-temporal loads.
#ifndef MICS_REORDER_BLOCK
#define MICS_REORDER_BLOCK 64
#endif
#ifndef MICS_REORDER_BPC
#define MICS_REORDER_BPC 4096
#endif
#ifndef MICS_REORDER_NTL
#define MICS_REORDER_NTL 1
#endif
#ifndef MICS_RSA_BPC
#define MICS_RSA_BPC 4096
#endif
#ifndef MICS_RSA_NTL
#define MICS_RSA_NTL 1
#endif
#ifndef MICS_RSA_BATCH
#define MICS_RSA_BATCH 16
#endif
#ifndef MICS_AVG_BPC
#define MICS_AVG_BPC 4096
#endif
#ifndef MICS_AVG_NTL
#define MICS_AVG_NTL 1
#endif
#ifndef MICS_ADAM_BPC
#define MICS_ADAM_BPC 4096
#endif
#ifndef MICS_ADAM_NTL
#define MICS_ADAM_NTL 1
#endif
constexpr bool kReorderNtl = MICS_REORDER_NTL;
constexpr bool kRsaNtl = MICS_RSA_NTL;   // gradient loads; the accumulator's hint is chosen per launch
constexpr bool kAvgNtl = MICS_AVG_NTL;   // input loads; the output's hint is chosen per launch
constexpr bool kAdamNtl = MICS_ADAM_NTL;

// Compile-time sized pointer table for the unrolled kernels (keeps the
// kernel-argument segment small); the launcher copies out of PtrTable.
template <int N>
struct SmallTable {
    const void* ptr[N];
};

// What a reduction indexes: a SmallTable itself (constant indices), or a table through the
// kernel-argument segment, so that run-time indices stay scalar loads, of several pointers at once
// where they are consecutive.  (Indexing the by-value parameter at run time makes one dependent
// 8-byte load of every pointer, 64 of them 5 us; the averages' and updates' kernels for any number of copies still do, which
// spaces their loads: in the middle of the range they are faster than unrolled ones, see unrolled_average.)  Its kernels
// have their table as the first parameter: offset 0 of the segment.  The entries of a PtrTable behind its last pointer
// repeat it (pad_table).
struct KernargTable {
    const void* const __attribute__((address_space(4)))* ptr;
};
template <int N>
__device__ __forceinline__ const SmallTable<N>& table_view(const SmallTable<N>& t) { return t; }
__device__ __forceinline__ KernargTable kernarg_table()
{
    return {(const void* const __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr()};
}
__device__ __forceinline__ KernargTable table_view(const PtrTable&) { return kernarg_table(); }

// Load / store through a pointer whose pointee type carries the alignment (macros, not function
// templates: a template parameter would drop the typedef's alignment and promise 16 bytes).
// NT selects the non-temporal form; it is a compile-time constant wherever these are used.
#define MICS_LD(NT, ptr) ((NT) ? __builtin_nontemporal_load(ptr) : *(ptr))
#define MICS_ST(NT, ptr, val) \
    do { if (NT) __builtin_nontemporal_store((val), (ptr)); else *(ptr) = (val); } while (0)

// N consecutive floats at a 4-byte aligned address, as one access.
template <int N, bool NT>
__device__ __forceinline__ void ld_f32(float (&a)[N], const float* p)
{
    static_assert(N == 1 || N == 2 || N == 4 || N == 8, "");
    if constexpr (N == 1) {
        a[0] = MICS_LD(NT, p);
    } else if constexpr (N == 2) {
        const f32x2 t = MICS_LD(NT, (const f32x2_a4*)p);
        a[0] = t.x; a[1] = t.y;
    } else {
        #pragma unroll
        for (int h = 0; h < N / 4; ++h) {
            const f32x4 t = MICS_LD(NT, (const f32x4_a4*)p + h);
            a[4 * h] = t.x; a[4 * h + 1] = t.y; a[4 * h + 2] = t.z; a[4 * h + 3] = t.w;
        }
    }
}

template <int N, bool NT>
__device__ __forceinline__ void st_f32(float* p, const float (&a)[N])
{
    if constexpr (N == 1) {
        MICS_ST(NT, p, a[0]);
    } else if constexpr (N == 2) {
        const f32x2 t = {a[0], a[1]};
        MICS_ST(NT, (f32x2_a4*)p, t);
    } else {
        #pragma unroll
        for (int h = 0; h < N / 4; ++h) {
            const f32x4 t = {a[4 * h], a[4 * h + 1], a[4 * h + 2], a[4 * h + 3]};
            MICS_ST(NT, (f32x4_a4*)p + h, t);
        }
    }
}

// Cache policy bits of a gfx950 buffer store: sc0 + sc1 = system scope, the store is written through
// the L2 at once instead of being left there for a later write-back.
constexpr int kWriteThrough = 17, kNonTemporal = 2;

// A buffer descriptor over `bytes` bytes from a wavefront-uniform address.  Stores outside are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wave_buffer(void* base, int bytes)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)base);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uintptr_t)base >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)((uintptr_t)hi << 32 | lo), 0, bytes, 0x00027000);
}

template <int POLICY>
__device__ __forceinline__ f32x4 load_vec(__amdgpu_buffer_rsrc_t from, unsigned byte)
{
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(from, (int)byte, 0, POLICY));
}

template <int POLICY>
__device__ __forceinline__ void store_vec(__amdgpu_buffer_rsrc_t to, unsigned byte, f32x4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), to, (int)byte, 0, POLICY);
}

// fp32 -> bf16, round to nearest even, two at a time (gfx950 converts a pair
// in one instruction).  Low half = a, high half = b.
__device__ __forceinline__ uint32_t bf16_pack(float a, float b)
{
    f32x2 f = {a, b};
    bf16x2 h = __builtin_convertvector(f, bf16x2);
    return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ uint16_t bf16_single(float a)
{
    __bf16 h = (__bf16)a;
    return __builtin_bit_cast(uint16_t, h);
}

// fp32 -> IEEE binary16, round to nearest even, subnormals kept, overflow to Inf.
__device__ __forceinline__ uint16_t f16_single(float a)
{
    _Float16 h = (_Float16)a;
    return __builtin_bit_cast(uint16_t, h);
}

// Low-precision copy of the parameters that the Adam kernels write next to the fp32 master.
enum { kParamNone = 0, kParamBf16 = 1, kParamF16 = 2 };

template <int OUT>
__device__ __forceinline__ uint32_t param_pack(float a, float b)
{
    if constexpr (OUT == kParamBf16) return bf16_pack(a, b);
    else return (uint32_t)f16_single(a) | ((uint32_t)f16_single(b) << 16);
}
template <int OUT>
__device__ __forceinline__ uint16_t param_single(float a)
{
    if constexpr (OUT == kParamBf16) return bf16_single(a);
    else return f16_single(a);
}

// ---------------------------------------------------------------------------
// Step 1: chunk rearrangement of the hierarchical all-gather (Section 3.3).
// Chunk g of the result comes from slot g div k of the stage-1 buffer of local
// rank g mod k.  blockIdx.y = g mod k, blockIdx.z = g div k (dividing g in
// every wavefront cost 1 % of a coalesced call), blockIdx.x strides over the chunk.
// ---------------------------------------------------------------------------

// Vector i of a wavefront's 64 consecutive ones from d: non-temporal, and through the L2 (nt / nt sc0 sc1:
// p = 16, 268 MB 43.0 / 41.2 us, 3.2 GB 481 / 480).  It needs whole 128-byte lines: with chunks that begin
// in the middle of one, p = 48, 537 MB takes 91.0 (nt: 89.5), with wavefronts moved to the lines 84.0.
// At every size: from 3 to 30 MB calls whose buffers no cache holds would be 1 to 4 % faster without, those whose
// buffers are still in one 2 to 8 % slower (p = 8, 7 MB 2.7, nt 3.0).
__device__ __forceinline__ void put_line(u32x4* d, size_t i, u32x4 v)
{
    const unsigned lane = threadIdx.x & 63u;
    store_vec<kNonTemporal | kWriteThrough>(wave_buffer(d + (i - lane), 1024), 16 * lane, __builtin_bit_cast(f32x4, v));
}

// All addresses and the shard size are multiples of 16 bytes: a remapped copy.
__global__ __launch_bounds__(kMaxBlock) void reorder_vec_kernel(
    u32x4* __restrict__ dst, PtrTable src, size_t shard_vecs, size_t n_valid_bytes, int k)
{
    const size_t l = blockIdx.y, j = blockIdx.z, g = j * (size_t)k + l;
    const size_t chunk_begin = g * shard_vecs * 16;
    if (chunk_begin >= n_valid_bytes) return;
    size_t valid = n_valid_bytes - chunk_begin;
    if (valid > shard_vecs * 16) valid = shard_vecs * 16;
    const size_t nfull = valid / 16;
    const u32x4* __restrict__ s = (const u32x4*)src.ptr[l] + j * shard_vecs;
    u32x4* const d = dst + g * shard_vecs;
    // wavefronts begin on 128-byte lines of the destination
    const unsigned lead = (unsigned)((uintptr_t)d / 16 & 7);

    // One vector per lane and pass.  Workgroups are dispatched in blockIdx order, so the lanes
    // in flight cover one compact, advancing window of the source and of the destination; a
    // lane that strides far ahead (several loads a grid stride apart) measurably lowers the
    // achieved bandwidth, for loads and even more for stores.
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nfull + lead; i += stride)
        if (i >= lead) put_line(d - lead, i, MICS_LD(kReorderNtl, s + (i - lead)));

    // ragged end of the logical buffer: fewer than 16 valid bytes remain
    const size_t tail_halves = (valid - nfull * 16) / 2;
    if (blockIdx.x == 0 && threadIdx.x < tail_halves) {
        const uint16_t* sh = (const uint16_t*)(s + nfull);
        uint16_t* dh = (uint16_t*)(d + nfull);
        dh[threadIdx.x] = sh[threadIdx.x];
    }
}

// Coalesced form (many separately sharded tensors in one launch): blockIdx.y and .z = chunk, blockIdx.x = tile
// x - tile_begin[t] of tensor t's chunk.  reorder_seg_kernel is for calls whose tensors are all 16-byte aligned,
// reorder_shift_kernel for all others, which moves the aligned ones among them the same way (move_tile): one launch, us,
// split by kind / so: 16 tensors with odd shards p = 16, 60 MB 16.1 / 12.8, 200 MB 38.1 / 35.5, 800 MB 131 / 129.  A tile is
// MICS_SEG_U runs of blockDim.x vectors: the table look-up in every wavefront's prologue has to
// be paid for by two vectors per lane (one: -15 %), more spreads the window (four: -3 %).
// Measured on the h = 8192 layer with two vectors per lane (GB/s): 64 lanes 6470, 128: 6540,
// 256: 6180.  A small chunk (a bias of h/p elements) costs one workgroup.
#ifndef MICS_SEG_BLOCK
#define MICS_SEG_BLOCK 128
#endif
constexpr int kSegLanes = MICS_SEG_BLOCK;
#ifndef MICS_SEG_U
#define MICS_SEG_U 2
#endif

// Where the tiles of up to SEGS tensors begin, and the index of the tensor whose tiles hold workgroup x (x < 2^31 - 1):
// begin is ascending, unused entries hold kNoTile.  Counting instead of walking keeps the table reads
// independent of one another (a few wide scalar loads), which matters for workgroups that move
// only a few KiB.  The count is written as integer arithmetic on the sign bit so that it stays
// on the scalar unit: as a sum of comparisons it was compiled into some 300 vector
// instructions per wavefront (-18 % on a layer of 16 unaligned tensors).  Counting only the
// entries in use would need the entry count first, and that dependent load costs more than
// the additions it saves (h = 8192 layer: 6.25 against 6.45 TB/s).  Up to 48 tensors all entries are counted; above, every
// eighth and then the eight from there: with 16 tensors at 400 MB that round costs 1.3 us, with more than 48 a second launch
// costs more (us, 48 / 96 per launch: 95 tensors, p = 2 80 MB 20.8 / 17.2, 400 MB 69.2 / 66.0, p = 96 80 MB 34.5 / 19.7, 1 GB
// equal; all 96 entries counted: 62 tensors 200 MB 28.2 / 26.5).
constexpr unsigned kNoTile = 0x7FFFFFFFu;
template <int SEGS>
struct TileBegin {
    static constexpr int kStep = SEGS <= kMaxSegPerLaunch ? SEGS : 8;
    unsigned coarse[SEGS / kStep];                 // every kStep-th entry
    unsigned begin[SEGS];
    __device__ __forceinline__ unsigned find(unsigned x) const
    {
        unsigned t = 0;
        #pragma unroll
        for (int i = 1; i < SEGS / kStep; ++i) t += (coarse[i] - 1u - x) >> 31;       // 1 iff coarse[i] <= x
        t *= kStep;
        unsigned u = 0;
        #pragma unroll
        for (int i = 1; i < kStep; ++i) u += (begin[t + i] - 1u - x) >> 31;
        return t + u;
    }
    void close(int n)                              // behind the n entries in use
    {
        for (int t = n; t < SEGS; ++t) begin[t] = kNoTile;
        for (int t = 0; t < SEGS; t += kStep) coarse[t / kStep] = begin[t];
    }
};
struct ReorderSeg {
    unsigned long long shard_vecs, valid_bytes, src_vec, dst_vec;
};
template <int SEGS>
struct ReorderSegTable {
    TileBegin<SEGS> tiles;
    ReorderSeg seg[SEGS];
};

// Tile `tile` of an aligned chunk of `valid` bytes.
__device__ __forceinline__ void move_tile(size_t tile, const u32x4* __restrict__ s, u32x4* __restrict__ d, size_t valid)
{
    const size_t nfull = valid / 16;
    const size_t tile_vecs = (size_t)blockDim.x * MICS_SEG_U;
    const size_t tile0 = tile * tile_vecs;
    const unsigned lead = (unsigned)((uintptr_t)d / 16 & 7);          // as in reorder_vec_kernel
    u32x4 v[MICS_SEG_U];
    #pragma unroll
    for (int u = 0; u < MICS_SEG_U; ++u) {
        const size_t i = tile0 + (size_t)u * blockDim.x + threadIdx.x;
        if (i >= lead && i < nfull + lead) v[u] = MICS_LD(kReorderNtl, s + (i - lead));
    }
    #pragma unroll
    for (int u = 0; u < MICS_SEG_U; ++u) {
        const size_t i = tile0 + (size_t)u * blockDim.x + threadIdx.x;
        if (i >= lead && i < nfull + lead) put_line(d - lead, i, v[u]);
    }
    // ragged end of the tensor: the tile that holds vector index nfull moves the last bytes
    const size_t tail_halves = (valid - nfull * 16) / 2;
    if (tail_halves && (nfull + lead) / tile_vecs == tile && threadIdx.x < tail_halves) {
        const uint16_t* sh = (const uint16_t*)(s + nfull);
        uint16_t* dh = (uint16_t*)(d + nfull);
        dh[threadIdx.x] = sh[threadIdx.x];
    }
}

template <int SEGS>
__global__ __launch_bounds__(kMaxBlock) void reorder_seg_kernel(
    u32x4* __restrict__ dst, PtrTable src, ReorderSegTable<SEGS> tab, int k)
{
    const unsigned x = blockIdx.x;
    const unsigned t = tab.tiles.find(x);
    const size_t shard_vecs = tab.seg[t].shard_vecs, valid_bytes = tab.seg[t].valid_bytes;
    const size_t l = blockIdx.y, j = blockIdx.z, g = j * (size_t)k + l;
    const size_t chunk_begin = g * shard_vecs * 16;
    if (chunk_begin >= valid_bytes) return;
    size_t valid = valid_bytes - chunk_begin;
    if (valid > shard_vecs * 16) valid = shard_vecs * 16;
    move_tile(x - tab.tiles.begin[t], (const u32x4*)src.ptr[l] + tab.seg[t].src_vec + j * shard_vecs,
              dst + tab.seg[t].dst_vec + g * shard_vecs, valid);
}

// General case: source and destination of a chunk sit at different offsets
// within their 16-byte lines (odd shard sizes, sub-buffers that start anywhere
// on an element boundary).  Like reorder_seg_kernel the kernel serves many
// tensors per launch: workgroup x moves tile x - tile_begin[t] of chunk
// blockIdx.y of tensor t.
struct ByteSeg {
    unsigned long long shard_bytes, valid_bytes, src_byte, dst_byte;
};
// Where workgroup x works: many tensors (table in the kernel arguments) ...
template <int SEGS>
struct ByteSegTable {
    static constexpr bool kAligned = true;         // aligned tensors may be among them
    TileBegin<SEGS> tiles;
    ByteSeg seg[SEGS];
    __device__ __forceinline__ const ByteSeg& locate(unsigned x, size_t* tile) const
    {
        const unsigned t = tiles.find(x);
        *tile = x - tiles.begin[t];
        return seg[t];
    }
};
// ... or a single tensor: no table, no look-up (4 % faster than a table of one entry).
struct OneTensor {
    static constexpr bool kAligned = false;
    ByteSeg seg;
    __device__ __forceinline__ const ByteSeg& locate(unsigned x, size_t* tile) const
    {
        *tile = x;
        return seg;
    }
};

// The 16 bytes that start 4 * W + sub bytes into `lo`, the rest from the first W + 1 dwords of `next`.
template <int W>
__device__ __forceinline__ u32x4 bytes_from(u32x4 lo, u32x4 next, unsigned sub)
{
    u32x4 out;
    #pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t below = W + d < 4 ? lo[(W + d) & 3] : next[(W + d) & 3];
        const uint32_t above = W + d + 1 < 4 ? lo[(W + d + 1) & 3] : next[(W + d + 1) & 3];
        out[d] = __builtin_amdgcn_alignbyte(above, below, sub);
    }
    return out;
}

// Lane n's `mine` of lane n + 1; lane 63 gets its own `last`.
__device__ __forceinline__ uint32_t from_next_lane(uint32_t mine, uint32_t last)
{
    constexpr int kWaveShiftLeft1 = 0x130;
    return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)mine, kWaveShiftLeft1, 0xf, 0xf, false);
}

// Both sides move whole aligned lines.  A wavefront writes U * 1 KiB of the destination, on 128-byte
// boundaries, from the aligned 16-byte source vectors that cover them; a vector of the destination
// is the end of one of those and the beginning of the next, which is the next lane's (lane 63: lane
// 0's of the next KiB, and behind the last KiB one vector more that it loads itself).  Loads that are
// off 16 bytes by themselves run at full speed on gfx950, but 1 KiB of them touches nine lines
// instead of eight, and so does a store off the lines.  The shift is the same for every vector of a
// chunk.  Partial vectors at the two ends of a chunk go in 2-byte units on lanes 0 .. 15 of the
// chunk's first workgroup; the first and the last whole vector, whose source lines reach beyond the
// chunk, are loaded from where they start: memory is touched only inside the chunk.
// GB/s of a layer with odd shards (2 x 629 MB, p = 32), loads off 16 bytes / so: 5880 / 6300; tensor by
// tensor with 16 per launch (3.2 GB) 5640 / 6340; 40 MB in one call 3700 / 4200.
template <typename Where, int U>
__global__ __launch_bounds__(kMaxBlock) void reorder_shift_kernel(
    unsigned char* __restrict__ dst, PtrTable src, Where where, int k)
{
    size_t tile;
    const ByteSeg& sg = where.locate(blockIdx.x, &tile);
    const size_t shard_bytes = sg.shard_bytes, n_valid_bytes = sg.valid_bytes;
    const size_t l = blockIdx.y, j = blockIdx.z, g = j * (size_t)k + l;
    const size_t chunk_begin = g * shard_bytes;
    if (chunk_begin >= n_valid_bytes) return;
    size_t valid = n_valid_bytes - chunk_begin;
    if (valid > shard_bytes) valid = shard_bytes;

    if constexpr (Where::kAligned) {
        static_assert(U == MICS_SEG_U, "move_tile's tiles");
        const uintptr_t s0 = (uintptr_t)src.ptr[l] + sg.src_byte, d0 = (uintptr_t)dst + sg.dst_byte;
        if (((s0 | d0 | shard_bytes) & 15) == 0) {
            move_tile(tile, (const u32x4*)(s0 + j * shard_bytes), (u32x4*)(d0 + chunk_begin), valid);
            return;
        }
    }
    const uintptr_t d_lo = (uintptr_t)dst + sg.dst_byte + chunk_begin;      // chunk in dst
    const uintptr_t d_hi = d_lo + valid;
    const uintptr_t s_chunk = (uintptr_t)src.ptr[l] + sg.src_byte + j * shard_bytes;
    const uintptr_t a_lo = (d_lo + 15) & ~(uintptr_t)15;                    // first full dst vector
    const size_t nfull = a_lo + 16 <= d_hi ? ((d_hi & ~(uintptr_t)15) - a_lo) / 16 : 0;

    if (tile == 0 && threadIdx.x < 16) {
        const uintptr_t head_end = a_lo < d_hi ? a_lo : d_hi;
        const uintptr_t b = threadIdx.x < 8 ? d_lo + 2 * threadIdx.x
                                            : a_lo + nfull * 16 + 2 * (threadIdx.x - 8);
        const bool on = threadIdx.x < 8 ? b < head_end : (b >= head_end && b < d_hi);
        if (on) *(uint16_t*)b = *(const uint16_t*)(s_chunk + (b - d_lo));
    }

    // vector i is the destination's at d_line + 16 i; the chunk's are [first, last)
    const uintptr_t d_line = d_lo & ~(uintptr_t)127;
    const size_t first = (a_lo - d_line) / 16, last = first + nfull;
    const unsigned lane = threadIdx.x & 63u;
    const size_t w0 = (tile * blockDim.x + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u)) * U;   // of the wavefront
    if (w0 >= last) return;
    const uintptr_t s_line = s_chunk + (d_line - d_lo);                     // source of vector 0
    const unsigned phase = (unsigned)(s_line & 15), sub = phase & 3;        // chunk-uniform
    const uintptr_t s_vec = s_line - phase;                                 // its aligned source line

    auto move = [&](auto ALL) {                    // ALL: every vector, and the one behind, is inside the chunk
        u32x4 v[U + 1];
        #pragma unroll
        for (int u = 0; u <= U; ++u) {
            const size_t i = w0 + 64 * u + (u < U ? lane : 0);
            v[u] = u32x4{0, 0, 0, 0};
            const bool inside = i >= first && i < last && s_vec + 16 * i >= s_chunk;
            if (u < U ? ALL.value || inside : phase != 0 && lane == 63 && (ALL.value || inside))
                v[u] = MICS_LD(true, (const u32x4*)(s_vec + 16 * i));
        }
        auto put = [&](auto W) {
            #pragma unroll
            for (int u = 0; u < U; ++u) {
                u32x4 out = v[u];
                if constexpr (W.value >= 0) {
                    u32x4 next = {0, 0, 0, 0};
                    #pragma unroll
                    for (int d = 0; d <= W.value; ++d)
                        next[d] = from_next_lane(v[u][d], u + 1 < U ? __builtin_amdgcn_readfirstlane(v[u + 1][d]) : v[U][d]);
                    out = bytes_from<W.value>(v[u], next, sub);
                }
                const size_t i = w0 + 64 * u + lane;
                if constexpr (!ALL.value) {
                    if (i < first || i >= last) continue;
                    if (phase != 0 && (s_vec + 16 * i < s_chunk || i + 1 == last))
                        out = MICS_LD(true, (const u32x4_a2*)(s_line + 16 * i));
                }
                MICS_ST(true, (u32x4*)(d_line + 16 * i), out);
            }
        };
        if (phase == 0) put(std::integral_constant<int, -1>{});
        else if (phase < 4) put(std::integral_constant<int, 0>{});
        else if (phase < 8) put(std::integral_constant<int, 1>{});
        else if (phase < 12) put(std::integral_constant<int, 2>{});
        else put(std::integral_constant<int, 3>{});
    };
    if (w0 >= first && w0 + 64 * U < last && s_vec + 16 * w0 >= s_chunk) move(std::true_type{});
    else move(std::false_type{});
}

// Table of up to SEGS (1, or 64 to 128) tensors in the kernel arguments, and the look-up of the tensor whose tiles
// hold workgroup x: lane i takes entry i, the tensor's index is the number of entries at or below x.  Small calls
// (ONE_ROUND, 64 entries) have every lane take entry i's record too, so that nothing waits for the index, and so do
// the large reductions but those of up to 8 two-byte buffers, whose wavefronts move too little for 2 KiB of table (16
// tensors, bf16, p = 4, 79 M elements: 194 us, without 190; p = 6, 335 MB 52.3, 50.7).  Looked up with scalar instructions,
// as the large gathers do, in three dependent rounds, reductions take 1 to 4 % longer (p = 32, 16 tensors, 3.8 M elements 7
// %).
template <typename Seg, int SEGS>
struct TileTable {
    unsigned tile_begin[SEGS];                     // ascending; kNoTile behind the last
    Seg seg[SEGS];
};
__device__ __forceinline__ uint32_t uniform_lane(uint32_t v, unsigned from)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)from);
}
template <bool ONE_ROUND, typename Seg, int SEGS>
__device__ __forceinline__ Seg segment_at(const TileTable<Seg, SEGS>& tab, unsigned x, unsigned* tile)
{
    const unsigned lane = threadIdx.x & 63u;
    const unsigned begin = tab.tile_begin[lane];
    unsigned t;
    if constexpr (SEGS == 64) {
        constexpr int W = sizeof(Seg) / 4;
        struct Words { uint32_t w[W]; } sg;
        if constexpr (ONE_ROUND) sg = __builtin_bit_cast(Words, tab.seg[lane]);
        t = (unsigned)__builtin_popcountll(__builtin_amdgcn_ballot_w64(begin <= x)) - 1;
        *tile = x - uniform_lane(begin, t);
        if constexpr (ONE_ROUND) {
            #pragma unroll
            for (int i = 0; i < W; ++i) sg.w[i] = uniform_lane(sg.w[i], t);
            return __builtin_bit_cast(Seg, sg);
        }
    } else {
        // the second read overlaps the first: its last SEGS - 64 entries count
        const unsigned later = tab.tile_begin[SEGS - 64 + lane];
        t = (unsigned)__builtin_popcountll(__builtin_amdgcn_ballot_w64(begin <= x)) - 1 +
            (unsigned)__builtin_popcountll(__builtin_amdgcn_ballot_w64(lane >= 128 - SEGS && later <= x));
        *tile = x - (t < 64 ? uniform_lane(begin, t) : uniform_lane(later, t - (SEGS - 64)));
    }
    return tab.seg[t];
}

// Small calls.  What bounds them is latency: of dependent reads of the kernel arguments (0.15 to 0.25 us each; the
// kernels above make three or four before their first load), and, with many tensors, of workgroups that have
// nothing to do (one workgroup per chunk is p of them for every bias).  Here a tensor's destination is cut into
// tiles whatever its chunks are, and every lane finds the chunk of its own 16 bytes: a multiplication by a host-made
// reciprocal for the chunk, another for its node, and the stage-1 buffer's address from the lane that holds it.  Up to
// 64 tensors all of the arguments come in one round of loads.  Any alignment: 16 bytes that cross the border of a chunk or an
// end of the tensor go in 2-byte units.  us, one workgroup per chunk / so: 1 MB in one tensor, p = 16 2.45 / 2.06;
// p = 16, 40 tensors, 1 MB 7.3 / 3.2; p = 128, 90 tensors, 5 MB 42.6 / 8.6, 40 tensors, 1 MB 20.9 / 3.4.
struct FlatSeg {
    unsigned long long src_byte, dst_byte;
    unsigned shard_bytes, valid_bytes;             // below 2^31
    unsigned recip, shift;                         // b / shard_bytes = mulhi(b, recip) >> shift for even b below 2^32
};
template <int SEGS> using FlatTable = TileTable<FlatSeg, SEGS>;

// Lane `from`'s value, for a lane index that may differ from lane to lane.
__device__ __forceinline__ uint32_t lane_value(uint32_t v, unsigned from)
{
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4 * from), (int)v);
}

template <int U, int SEGS, bool MANY>
__global__ __launch_bounds__(kMaxBlock) void reorder_flat_kernel(
    unsigned char* __restrict__ dst, PtrTable src, FlatTable<SEGS> tab, unsigned k, unsigned k_recip)
{
    const unsigned lane = threadIdx.x & 63u, x = blockIdx.x;
    const uint64_t p0 = (uint64_t)src.ptr[MANY ? lane : lane & 15], p1 = (uint64_t)src.ptr[MANY ? 64 + lane : 0];
    unsigned tile = x;                                         // of the tensor
    FlatSeg sg;
    if constexpr (SEGS == 1) sg = tab.seg[0];
    else sg = segment_at<true>(tab, x, &tile);
    const unsigned shard = sg.shard_bytes, valid = sg.valid_bytes;
    const uintptr_t d_lo = (uintptr_t)dst + sg.dst_byte;
    const uintptr_t d_line = d_lo & ~(uintptr_t)127;           // tiles begin on the destination's lines

    // every lane takes part in the exchange, whatever it moves
    auto buffer = [&](unsigned l) {
        const uint64_t a = (uint64_t)lane_value((uint32_t)(p0 >> 32), l & 63u) << 32 | lane_value((uint32_t)p0, l & 63u);
        if (!MANY) return a;
        const uint64_t b = (uint64_t)lane_value((uint32_t)(p1 >> 32), l & 63u) << 32 | lane_value((uint32_t)p1, l & 63u);
        return l < 64 ? a : b;
    };
    int off[U];                                                // the lane's first byte, in the tensor
    unsigned j[U], l[U], rest[U];                              // where it is (byte 0 if that lies in front of the tensor)
    uintptr_t s[U];
    u32x4 v[U];
    bool whole[U];
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        off[u] = (int)((tile * U + u) * blockDim.x * 16 + threadIdx.x * 16) - (int)(d_lo - d_line);
        const unsigned b = off[u] < 0 ? 0 : (unsigned)off[u], g = __umulhi(b, sg.recip) >> sg.shift;
        rest[u] = b - g * shard;
        j[u] = g * k_recip >> 16;
        l[u] = g - j[u] * k;
        s[u] = buffer(l[u]) + sg.src_byte + j[u] * shard + rest[u];
        whole[u] = off[u] >= 0 && b + 16 <= valid && rest[u] + 16 <= shard;
        if (whole[u]) v[u] = MICS_LD(true, (const u32x4_a2*)s[u]);
    }
    #pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool parts = !whole[u] && off[u] + 16 > 0 && off[u] < (int)valid;
        if (__builtin_amdgcn_ballot_w64(parts)) {
            const unsigned from = off[u] < 0 ? 0 : (unsigned)off[u];
            const unsigned n = !parts ? 0 : ((unsigned)(off[u] + 16) < valid ? (unsigned)(off[u] + 16) : valid) - from;
            uint16_t h[8];
            if (shard >= 16) {                                 // one border at most
                const unsigned here = shard - rest[u];
                const unsigned l1 = l[u] + 1 == k ? 0 : l[u] + 1, j1 = l[u] + 1 == k ? j[u] + 1 : j[u];
                const uintptr_t s1 = buffer(l1) + sg.src_byte + j1 * shard - here;
                #pragma unroll
                for (unsigned i = 0; i < 8; ++i)
                    if (2 * i < n) h[i] = *(const uint16_t*)((2 * i < here ? s[u] : s1) + 2 * i);
            } else {
                #pragma unroll
                for (unsigned i = 0; i < 8; ++i) {
                    const uintptr_t a = buffer(l[u]) + sg.src_byte + j[u] * shard + rest[u];
                    if (2 * i < n) h[i] = *(const uint16_t*)a;
                    rest[u] += 2;
                    if (rest[u] == shard) {
                        rest[u] = 0;
                        if (++l[u] == k) l[u] = 0, ++j[u];
                    }
                }
            }
            #pragma unroll
            for (unsigned i = 0; i < 8; ++i)
                if (2 * i < n) *(uint16_t*)(d_lo + from + 2 * i) = h[i];
        }
        if (whole[u]) *(u32x4*)(d_lo + off[u]) = v[u];
    }
}

// ---------------------------------------------------------------------------
// Step 2a: reduction of the partition-group reduce-scatter, accumulated over
// micro-steps (Section 3.4).
//
// Gradient formats (KIND): 0 = bf16, 1 = IEEE binary16 (what mixed precision means on GPUs
// without bf16), 2 = binary32 (plain float32 training).  Widening to binary32 is exact.
//
// One kernel for every alignment.  The kernel works in a "virtual" element index space in
// which element 0 of every (rounded-down) gradient pointer sits at a 16-byte aligned address (at
// least a 4-byte aligned one, where the pointers differ); the call's elements are the virtual
// range [lead, lead + count), lead = the elements that the pointers were rounded down by.
// A lane owns the virtual elements [EPL*i, EPL*i + EPL): one load per
// rank buffer, one load and one store of the accumulator (which is then 4-byte aligned at
// worst).  A lane whose elements are not all inside the range -- at most the first and the
// last one -- leaves them to rsa_edges.
//
// VEC = dwords per load: 4 for bandwidth (8 bf16/fp16 or 4 fp32 elements per lane); 1 for
// small messages on large groups, where the time is the launch plus the serial chain of
// load round trips of one lane: one dword per buffer and lane spreads a 1 MB message over
// 32 compute units instead of 1 and lets a lane keep 64 loads in flight, so p = 128 needs
// two round trips.  (Splitting the buffers of p > 64 over two wavefronts, one round trip, takes
// longer than the second one since the pointers arrive in wide loads: 5.3 against 4.5 us for 33 k
// elements at p = 128; 7.9 while each pointer was a load of its own.)
// ---------------------------------------------------------------------------

template <int KIND> struct GradFormat {
    static constexpr int kElemBytes = KIND == 2 ? 4 : 2;
    static constexpr int kPerDword = KIND == 2 ? 1 : 2;
};

template <int KIND>
__device__ __forceinline__ void widen_dword(float* out, uint32_t w)
{
    if constexpr (KIND == 0) {          // the bf16 bits are the upper half of the fp32 bits
        out[0] = __uint_as_float(w << 16);
        out[1] = __uint_as_float(w & 0xFFFF0000u);
    } else if constexpr (KIND == 1) {
        out[0] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xFFFFu));
        out[1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
    } else {
        out[0] = __uint_as_float(w);
    }
}

template <int KIND>
__device__ __forceinline__ float widen_one(const void* buf, size_t x)
{
    if constexpr (KIND == 0) return __uint_as_float((uint32_t)((const uint16_t*)buf)[x] << 16);
    else if constexpr (KIND == 1) return (float)((const _Float16*)buf)[x];
    else return ((const float*)buf)[x];
}

template <int KIND, int VEC> struct GradVec;      // the registers of one load
template <int KIND> struct GradVec<KIND, 4> {
    u32x4 v;
    __device__ __forceinline__ void load(const void* base, size_t elem)
    {
        const char* a = (const char*)base + elem * GradFormat<KIND>::kElemBytes;
        if constexpr (KIND == 2) v = MICS_LD(kRsaNtl, (const u32x4_a4*)a);
        else v = MICS_LD(kRsaNtl, (const u32x4_a2*)a);
    }
    __device__ __forceinline__ uint32_t dword(int d) const { return v[d]; }
};
template <int KIND> struct GradVec<KIND, 1> {
    uint32_t v;
    __device__ __forceinline__ void load(const void* base, size_t elem)
    {
        const char* a = (const char*)base + elem * GradFormat<KIND>::kElemBytes;
        if constexpr (KIND == 2) v = MICS_LD(kRsaNtl, (const uint32_t*)a);
        else v = MICS_LD(kRsaNtl, (const u32_a2*)a);
    }
    __device__ __forceinline__ uint32_t dword(int) const { return v; }
};

template <int KIND, int VEC, bool FIRST>
__device__ __forceinline__ void rsa_add(float* s, const GradVec<KIND, VEC>& v)
{
    constexpr int PD = GradFormat<KIND>::kPerDword;
    #pragma unroll
    for (int d = 0; d < VEC; ++d) {
        float w[PD];
        widen_dword<KIND>(w, v.dword(d));
        #pragma unroll
        for (int e = 0; e < PD; ++e) {
            if constexpr (FIRST) s[PD * d + e] = w[e];
            else s[PD * d + e] = s[PD * d + e] + w[e];
        }
    }
}

// s = (((s + g_q0) + g_{q0+1}) + ...) + g_{q0+n-1} for the lane's elements starting at virtual
// element `elem`, at most N buffers: N loads in flight, unconditional.  n > N - PAD; what is loaded
// beyond n is the last buffer again (see KernargTable) and not added.
template <int KIND, int VEC, int N, int PAD, typename Tab>
__device__ __forceinline__ void rsa_batch(float* s, const Tab& g, int q0, int n, size_t elem)
{
    GradVec<KIND, VEC> v[N];
    #pragma unroll
    for (int b = 0; b < N; ++b) v[b].load(g.ptr[q0 + b], elem);
    // as in rsa_partial; the 64 single dwords of a full batch are better left to the compiler (p = 64,
    // 74 k elements: 4.0 against 4.6 us)
    if constexpr (N < 64) __builtin_amdgcn_sched_barrier(0);
    #pragma unroll
    for (int b = 0; b < N; ++b)
        if (b <= N - PAD || b < n) rsa_add<KIND, VEC, false>(s, v[b]);
}

// The last `n` < N buffers: the smallest batch of a multiple of PAD loads that holds them.  (Found by halving,
// f32, p = 3, 50 k elements took 2.9 us instead of 2.6: the jumps cost more than the comparisons.)
template <int KIND, int VEC, int N, int PAD, typename Tab>
__device__ __forceinline__ void rsa_rest(float* s, const Tab& g, int q0, int n, size_t elem)
{
    if constexpr (N > PAD) {
        if (n > N - 2 * PAD) rsa_batch<KIND, VEC, N - PAD, PAD>(s, g, q0, n, elem);
        else rsa_rest<KIND, VEC, N - PAD, PAD>(s, g, q0, n, elem);
    }
}

// As rsa_batch for any p, in batches of kShallow (large calls of 16 and more buffers, `shallow_call`).  What counts there is
// what all wavefronts of a compute unit have in flight together, 8 x 2 to 4 KiB: deeper batches in fewer wavefronts end at the same rate,
// but a wavefront then lives longer, and with it the end of the call, where units run dry.  The next pointers come while
// these loads are out.  us, bf16, the best cap for each of 3 / 4 / 6 / 8 / 16 loads: p = 24 350 MB 53.3 / 52.7 / 53.3 / 54.0 / 55.6, 730 MB
// 109.3 / 107.4 / 109.6 / 111.3 / 115.9; p = 32 159 MB 24.8 / 24.9 / 25.3 / 26.0 / 25.8; p = 64 301 MB 44.6 / 45.5 / 46.0 /
// 47.8 / 50.1; p = 128 482 MB 73.1 / 71.1 / 76.3 / 76.9 / 80.2; f32, p = 24 325 MB 49.1 / 49.4 / 49.6 / 50.2 / 51.4, p = 64
// 430 MB 63.0 / 65.1 / 65.8 / 66.7 / 68.6.  A ring of 6 or 8 loads that moves on by two is 1 % slower.  The accumulator's
// loads go out with the last batch, of 4 to 7: where it took what 4 left over, one load was alone in flight (speed of this
// against that, means of 40 to 70 calls: p = 17 1.014, 18 1.008, 21 1.011, 25 1.010; f32, 16 tensors, p = 17 318 MB 53.2 /
// 51.5, 1.1 GB 173.4 / 166.9).
constexpr int kShallow = 4;
// The last kShallow to 2 kShallow - 1 of the n buffers from q0; the pointers of the first kShallow are there.
template <int KIND, int N, typename Tab, typename Issue>
__device__ __forceinline__ void rsa_last_batch(float* s, const void* const (&first)[kShallow], const Tab& g, int q0, int n, size_t elem, Issue&& accumulator)
{
    if constexpr (N > kShallow)
        if (n < N) return rsa_last_batch<KIND, N - 1>(s, first, g, q0, n, elem, accumulator);
    GradVec<KIND, 4> v[N];
    #pragma unroll
    for (int b = 0; b < N; ++b) v[b].load(b < kShallow ? first[b] : g.ptr[q0 + b], elem);
    accumulator();
    __builtin_amdgcn_sched_barrier(0);
    #pragma unroll
    for (int b = 0; b < N; ++b) rsa_add<KIND, 4, false>(s, v[b]);
}
template <int KIND, typename Tab, typename Issue>
__device__ __forceinline__ void rsa_shallow(float* s, const Tab& g, int p, size_t elem, Issue&& accumulator)
{
    const void* next[kShallow];
    #pragma unroll
    for (int b = 0; b < kShallow; ++b) next[b] = g.ptr[b];
    int q0 = 0;
    #pragma unroll 1
    for (; q0 + 2 * kShallow <= p; q0 += kShallow) {
        GradVec<KIND, 4> v[kShallow];
        #pragma unroll
        for (int b = 0; b < kShallow; ++b) v[b].load(next[b], elem);
        #pragma unroll
        for (int b = 0; b < kShallow; ++b) next[b] = g.ptr[q0 + kShallow + b];
        __builtin_amdgcn_sched_barrier(0);
        #pragma unroll
        for (int b = 0; b < kShallow; ++b) rsa_add<KIND, 4, false>(s, v[b]);
    }
    rsa_last_batch<KIND, 2 * kShallow - 1>(s, next, g, q0, p - q0, elem, accumulator);
}

// s = ((g_0 + g_1) + ...) + g_{p-1} for the lane's elements starting at virtual element `elem`.
// `accumulator` issues the accumulator's loads, behind those of the first buffers: it needs more instructions,
// and a small call is over in a few times the latency of what stands in front of its loads (in front: 16 tensors, p = 16,
// 50 M elements 309 / 303 us; bf16, p = 32, 0.3 to 1 M as fast).  Windows of loads have it behind the last buffers.
// P > 0: p = P at compile time; P == 0: any p.  The loads go out in batches of BATCH, every
// batch entirely in flight before its first addition (P <= BATCH: all of them at once; a
// batch of 32 128-bit loads would leave room for 3 wavefronts per SIMD only).  -0 is the identity of
// binary32 addition (-0 + x is x, also for x = -0 and x = +0).
template <int KIND, int VEC, int P, int BATCH, bool SHALLOW, bool HOLD, typename Tab, typename Issue>
__device__ __forceinline__ void rsa_partial(float* s, const Tab& g, int p, size_t elem, Issue&& accumulator)
{
    if constexpr (VEC == 4 && ((P == 32 && (KIND != 0 || HOLD)) || (P == 16 && KIND == 1 && !HOLD))) {
        // A window of W loads that moves on by STEP buffers, held in this order.  Left to itself the compiler put as few as
        // one load in flight here and more than enough there, from one change of the source to the next: us, f16, 16
        // tensors, p = 16 900 MB 239 / so 139, 2 GB 524 / 324, p = 32 45 MB 20.5 / 10.6, 2 GB 752 / 313; f32, p = 32, 12 MB in two batches
        // 3.95 / 3.69.  The bf16 kernels are better in the compiler's order (p = 32 300 MB 49.1, held 51).  (Of the calls
        // past the L2, one tensor of 32 gets here below 8 wavefronts per unit and segments of 32 below 12, of two-byte
        // elements also from 40 on; long_call_in_step any.)
        // The accumulator's loads go out behind the last gradients: in front, or behind the first window, they are one of
        // the few in flight while nothing needs them (us, p = 32, 45 MB, in front / behind the first / behind the last: f32
        // 9.0 / 9.2 / 8.6; f16 9.9 / 9.9 / 9.2).
        constexpr int W = HOLD ? 16 : P == 16 ? 4 : 6, STEP = HOLD ? 4 : 2;
        static_assert((P - W) % STEP == 0, "");
        GradVec<KIND, VEC> v[W];
        #pragma unroll
        for (int b = 0; b < W; ++b) v[b].load(g.ptr[b], elem);
        if (HOLD) accumulator();
        __builtin_amdgcn_sched_barrier(0);
        #pragma unroll
        for (int q0 = 0; q0 < P; q0 += STEP) {
            #pragma unroll
            for (int b = q0; b < q0 + STEP; ++b) {
                if (b == 0) rsa_add<KIND, VEC, true>(s, v[0]);
                else rsa_add<KIND, VEC, false>(s, v[b % W]);
            }
            #pragma unroll
            for (int b = q0; b < q0 + STEP; ++b)
                if (b + W < P) v[b % W].load(g.ptr[b + W], elem);
            if (!HOLD && q0 + STEP + W == P) accumulator();
            if (q0 + W < P) __builtin_amdgcn_sched_barrier(0);
        }
    } else if constexpr (P > 0) {
        #pragma unroll
        for (int q0 = 0; q0 < P; q0 += BATCH) {
            GradVec<KIND, VEC> v[BATCH];
            #pragma unroll
            for (int b = 0; b < BATCH; ++b)
                if (q0 + b < P) v[b].load(g.ptr[q0 + b], elem);
            if (q0 == 0) accumulator();
            // Up to 8 buffers: keep the compiler from trading the loads in flight for registers (left to
            // itself it ran f16, p = 8 one load at a time: 172 against 128 us at 33 M elements).  With 16
            // loads it keeps about 10 in flight by itself (f32: 4), and more cost occupancy (one tensor, p = 16, 7.5 M, which
            // is read in shallow batches now: 52.4 against 50.7 us), except in the small calls that HOLD stands for, where
            // latency counts (f32, p = 16, 42 k elements: 2.4 us, not held 4.0; p = 32, 59 k: 3.7, 5.4; bf16, p = 16, 75 k:
            // 2.7, 3.1).
            if constexpr (P <= 8 || HOLD) __builtin_amdgcn_sched_barrier(0);
            #pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                if (q0 + b < P) {
                    if (q0 + b == 0) rsa_add<KIND, VEC, true>(s, v[b]);
                    else rsa_add<KIND, VEC, false>(s, v[b]);
                }
            }
        }
    } else {
        // 128-bit loads: exactly the buffers that are left; single dwords, whose time is latency: whole
        // groups of 8
        constexpr int PAD = VEC == 1 ? 8 : 1;
        #pragma unroll
        for (int e = 0; e < VEC * GradFormat<KIND>::kPerDword; ++e) s[e] = -0.0f;
        if constexpr (SHALLOW) return rsa_shallow<KIND>(s, g, p, elem, accumulator);
        accumulator();
        int q0 = 0;
        for (; q0 + BATCH <= p; q0 += BATCH) rsa_batch<KIND, VEC, BATCH, 1>(s, g, q0, BATCH, elem);
        if (q0 < p) rsa_rest<KIND, VEC, BATCH + (PAD > 1 ? PAD : 0), PAD>(s, g, q0, p - q0, elem);
    }
}

// a[0 .. EPL) = a[0 .. EPL) + partial sum at virtual element `elem`.
template <int KIND, int VEC, int P, int BATCH, bool SHALLOW, bool HOLD, typename Tab, typename Issue>
__device__ __forceinline__ void rsa_sum(float (&a)[VEC * GradFormat<KIND>::kPerDword], const Tab& g, int p, size_t elem,
                                        Issue&& accumulator)
{
    constexpr int EPL = VEC * GradFormat<KIND>::kPerDword;
    float s[EPL];
    rsa_partial<KIND, VEC, P, BATCH, SHALLOW, HOLD>(s, g, p, elem, accumulator);
    #pragma unroll
    for (int e = 0; e < EPL; ++e) a[e] = a[e] + s[e];
}

// One element, the loads in flight 16 at a time (a lane that waited for each of 128 loads in
// turn would hold up a small call for tens of microseconds); any p: the last ones in a whole group
// of 8 (see KernargTable).
template <int KIND, int N, typename Tab>
__device__ __forceinline__ void rsa_element_batch(float& s, const Tab& g, int q0, int n, size_t elem)
{
    float w[N];
    #pragma unroll
    for (int b = 0; b < N; ++b) w[b] = widen_one<KIND>(g.ptr[q0 + b], elem);
    #pragma unroll
    for (int b = 0; b < N; ++b)
        if (b < n) s = s + w[b];
}
template <int KIND, int P, bool ACCUM, typename Tab>
__device__ __forceinline__ void rsa_element(float* acc_e, const Tab& g, int p, size_t elem)
{
    float partial = -0.0f;                          // the identity, see rsa_partial
    if constexpr (P > 0 && P <= 16) {
        rsa_element_batch<KIND, P>(partial, g, 0, P, elem);
    } else {
        int q0 = 0;
        // not unrolled: the 64 scalar registers of 32 pointers leave none to spare
        #pragma unroll 1
        for (; q0 + 16 <= p; q0 += 16) rsa_element_batch<KIND, 16>(partial, g, q0, 16, elem);
        if constexpr (P == 0) {
            if (p - q0 > 8) rsa_element_batch<KIND, 16>(partial, g, q0, p - q0, elem);
            else if (p > q0) rsa_element_batch<KIND, 8>(partial, g, q0, p - q0, elem);
        }
    }
    *acc_e = (ACCUM ? *acc_e : 0.0f) + partial;
}

// Orders LDS accesses of one wavefront's lanes before and after it.  They complete in program order, so this
// is no instruction: it tells the compiler, to whom the lanes' addresses do not alias, to keep that order.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// The lane's virtual elements [v0, v0 + EPL) of a call (or segment) whose elements are the
// virtual range [lead, end): `acc` is the accumulator address of virtual element `lead`, and
// virtual element e sits at element src0 + e of every rank buffer.  Consecutive lanes of a
// wavefront hold consecutive v0, and every lane of the wavefront gets here (lanes past `end`
// find nothing to do).  A lane whose elements are not all inside the range does nothing:
// those elements -- fewer than EPL at either end -- are rsa_edges' work.
//
// PARTS (small segments, of at least EPL elements): such a lane sums the first or the last EPL elements of the
// range instead and keeps those that are its own.  A workgroup that has a segment's ends would otherwise wait for
// a second chain of loads, 16 at a time.  (In the flat kernels, where a workgroup of its own does that, the
// additional instructions cost more: p = 4, 0.1 M elements 2.2 / 2.4 us.)
//
// CACHED (kAccCached): plain accesses, straight from the lane.  A kernel of its own, because in small calls
// every instruction in front of the loads and between sum and store counts (bf16, p = 8, 125 k elements: 2.4
// us; with the choice made at run time, or through LDS, 2.7).
//
// Otherwise accumulators of 8-element lanes are stored through LDS: a lane's two 128-bit stores are 32
// bytes apart, so each store instruction of the wavefront would fill every other 16 bytes of its
// cache lines, which leave the L2 between the two halves.  Passing the results through 2 KiB of LDS
// per wavefront lets every store instruction cover one contiguous KiB.  Vector j of the wavefront's
// 128 holds half of the elements of lane j / 2.
template <int KIND, int VEC, int P, int BATCH, bool SHALLOW, bool ACCUM, bool CACHED, bool PARTS, typename Tab>
__device__ __forceinline__ void rsa_lane(float* acc, const Tab& g, int p, size_t src0, size_t v0,
                                         size_t lead, size_t end, int how)
{
    constexpr int EPL = VEC * GradFormat<KIND>::kPerDword;
    const bool full = v0 >= lead && v0 + EPL <= end;
    float a[EPL];
    #pragma unroll
    for (int e = 0; e < EPL; ++e) a[e] = 0.0f;
    if constexpr (PARTS) {
        static_assert(CACHED, "");
        if (v0 >= end || v0 + EPL <= lead) return;
        const size_t w0 = full ? v0 : v0 < lead ? lead : end - EPL;
        float* const at = acc + (w0 - lead);
        auto own = [&](int e) { return w0 + e >= v0 && w0 + e < v0 + EPL; };
        rsa_sum<KIND, VEC, P, BATCH, false, VEC == 4>(a, g, p, src0 + w0, [&] {
            if constexpr (ACCUM) {
                if (full) {
                    ld_f32<EPL, false>(a, at);
                } else {
                    #pragma unroll
                    for (int e = 0; e < EPL; ++e)
                        if (own(e)) a[e] = at[e];
                }
            }
        });
        if (full) {
            st_f32<EPL, false>(at, a);
        } else {
            #pragma unroll
            for (int e = 0; e < EPL; ++e)
                if (own(e)) at[e] = a[e];
        }
    } else if constexpr (CACHED) {
        if (full) {
            rsa_sum<KIND, VEC, P, BATCH, false, VEC == 4>(a, g, p, src0 + v0, [&] {
                if (ACCUM) ld_f32<EPL, false>(a, acc + (v0 - lead));
            });
            st_f32<EPL, false>(acc + (v0 - lead), a);
        }
    } else {
        const unsigned lane = threadIdx.x & 63u;
        const size_t wave_v0 = v0 - EPL * lane;
        float* const wave_acc = acc + (wave_v0 - lead);
        const __amdgpu_buffer_rsrc_t out = wave_buffer(wave_acc, 64 * EPL * 4);
        const bool whole = (__builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)wave_acc) & 127) == 0;
        const bool wt = how == kAccThrough || (whole && how == kAccThroughLines);
        auto store = [&](unsigned i, f32x4 v) {
            if (wt) store_vec<kWriteThrough>(out, 16 * i, v);
            else MICS_ST(true, (f32x4_a4*)wave_acc + i, v);
        };
        if (full) {
            rsa_sum<KIND, VEC, P, BATCH, SHALLOW, false>(a, g, p, src0 + v0, [&] {
                // with more than 8 buffers the choice between two kinds of loads costs more registers than it
                // gives (p = 32: 158 instead of 99)
                if constexpr (ACCUM && P > 0 && P <= 8) {
                    f32x4 t[EPL / 4];
                    #pragma unroll
                    for (int h = 0; h < EPL / 4; ++h)
                        if (whole) t[h] = load_vec<kNonTemporal>(out, 4 * EPL * lane + 16 * h);
                        else t[h] = load_vec<0>(out, 4 * EPL * lane + 16 * h);
                    #pragma unroll
                    for (int e = 0; e < EPL; ++e) a[e] = t[e / 4][e % 4];
                } else if constexpr (ACCUM) {
                    ld_f32<EPL, true>(a, acc + (v0 - lead));
                }
            });
        }
        if constexpr (EPL == 4) {
            if (full) store(lane, f32x4{a[0], a[1], a[2], a[3]});
        } else {
            extern __shared__ f32x4 stage[];                     // blockDim.x * 2 vectors (launcher)
            f32x4* mine = stage + (threadIdx.x - lane) * 2;      // this wavefront's 128 vectors
            if (full) {
                mine[2 * lane] = f32x4{a[0], a[1], a[2], a[3]};
                mine[2 * lane + 1] = f32x4{a[4], a[5], a[6], a[7]};
            }
            wave_lds_order();
            // a workgroup's last wavefront may be a partial one (even_call), in the kernels that such calls reach
            unsigned half = 64;
            if constexpr (partial_waves(P, SHALLOW)) {
                const unsigned left = blockDim.x - __builtin_amdgcn_readfirstlane(threadIdx.x);
                if (left < 64) half = left;
            }
            #pragma unroll
            for (unsigned h = 0; h < 2; ++h) {
                const unsigned i = half * h + lane;
                const size_t owner = wave_v0 + 8 * (i / 2);
                if (owner >= lead && owner + 8 <= end) store(i, mine[i]);
            }
            wave_lds_order();                                    // the next pass writes there again
        }
    }
}

// A segment of fewer than EPL elements: one per lane of the calling workgroup.
template <int KIND, int P, bool ACCUM, typename Tab>
__device__ __forceinline__ void rsa_short(float* acc, const Tab& g, int p, size_t src0, size_t lead, size_t end)
{
    if (threadIdx.x >= end - lead) return;
    if constexpr (P <= 16) rsa_element<KIND, P, ACCUM>(acc + threadIdx.x, g, p, src0 + lead + threadIdx.x);
    else rsa_element<KIND, P, ACCUM>(acc + threadIdx.x, kernarg_table(), P, src0 + lead + threadIdx.x);
}

// The elements that no lane holds as a full vector: virtual [lead, head) with head = lead
// rounded up to EPL (or `end`), and [tail, end) with tail = `end` rounded down to EPL (or
// head).  One element per lane, lanes 0 .. 2*EPL-1 of the calling workgroup.
template <int KIND, int EPL, int P, bool ACCUM, typename Tab>
__device__ __forceinline__ void rsa_edges(float* acc, const Tab& g, int p, size_t src0, size_t lead, size_t end)
{
    if (threadIdx.x >= 2 * EPL) return;
    size_t head = (lead + EPL - 1) / EPL * EPL;
    if (head > end) head = end;
    size_t tail = end / EPL * EPL;
    if (tail < head) tail = head;
    const size_t e = threadIdx.x < EPL ? lead + threadIdx.x : tail + (threadIdx.x - EPL);
    const size_t stop = threadIdx.x < EPL ? head : end;
    if (e >= stop) return;
    if constexpr (P <= 16) rsa_element<KIND, P, ACCUM>(acc + (e - lead), g, p, src0 + e);
    else rsa_element<KIND, P, ACCUM>(acc + (e - lead), kernarg_table(), P, src0 + e);
}

// The tile of workgroup x of n.  Workgroups go to the 8 XCDs in turn, so neighbouring tiles meet in no L2, and a line
// that two of them share is fetched, or written in parts, twice.  IN_RUNS (reduce_order): rounds of 128 workgroups in which every XCD
// has a run of 16 neighbouring tiles.
constexpr int kInRuns = 4;                         // in a kernel's `how`, beside the accumulator's policy
__device__ __forceinline__ unsigned tile_of(unsigned x, unsigned n, bool in_runs)
{
    constexpr unsigned kXcds = 8, kRun = 16, kRound = kXcds * kRun;
    const unsigned at = x % kRound, base = x - at;
    return in_runs && base + kRound <= n ? base + at % kXcds * kRun + at / kXcds : x;
}

// Workgroups of blockDim.x lanes (64 .. 512 for VEC = 4, a multiple of 8: the launcher takes small ones for
// calls that would otherwise occupy a fraction of the compute units), plus one more workgroup
// for the edge elements, so that their load chains run beside the vector work.
// OTHER: a kernel's other form, with CACHED tiles in runs (of the others `how` says whether: tile_of's few instructions are
// 1 % of a small call), else shallow batches (shallow_call).
template <int KIND, int VEC, int P, bool ACCUM, bool CACHED, bool OTHER, typename Tab>
__global__ __launch_bounds__(VEC == 4 ? kMaxBlock : kNarrowBlock) void rsa_kernel(
    Tab tab, float* __restrict__ acc, int p, unsigned lead, size_t count, int how)
{
    const auto& g = table_view(tab);
    constexpr int BATCH = VEC == 1 ? 64 : MICS_RSA_BATCH;
    constexpr int EPL = VEC * GradFormat<KIND>::kPerDword;
    const size_t end = (size_t)lead + count;
    const size_t nlanes = (end + EPL - 1) / EPL;
    const size_t block = blockDim.x;
    // the last workgroup of the grid does nothing but the edge elements
    if (blockIdx.x == gridDim.x - 1) {
        rsa_edges<KIND, EPL, P, ACCUM>(acc, g, p, 0, lead, end);
        return;
    }
    const size_t stride = (size_t)(gridDim.x - 1) * block;
    const unsigned tile = CACHED && !OTHER ? blockIdx.x : tile_of(blockIdx.x, gridDim.x - 1, CACHED || (how & kInRuns));
    for (size_t base = (size_t)tile * block; base < nlanes; base += stride)   // workgroup-uniform
        rsa_lane<KIND, VEC, P, BATCH, OTHER && !CACHED, ACCUM, CACHED, false>(acc, g, p, 0, (base + threadIdx.x) * EPL, lead, end, how & ~kInRuns);
}

// Coalesced form (many separately sharded tensors in one launch): workgroup x works on
// tile x - tile_begin[t] of segment t.  Every segment has its own virtual index space as in
// rsa_kernel: src0 = position of its virtual element 0 in the rounded-down rank buffers, a
// multiple of a line (align_gradient_pointers) of them, [lead, end) = its elements,
// dst = accumulator index of virtual element `lead`.
struct ReduceSeg {
    unsigned long long end, src0, dst;
    unsigned lead, pad;
};
template <int SEGS> using ReduceTable = TileTable<ReduceSeg, SEGS>;

// Whether a segment's ends get a workgroup of their own in front of the tiles, because a tile would wait for too many of its loads one
// after another: 16 tensors, p = 96, 64 MB 18.5 / 15.9 us, f32 68 tensors 194 MB 45.2 / 40.9.  Not with up to 8 buffers,
// where the additional branch costs more (p = 2, 75 MB 13.9 / 14.4; f32, p = 4, 75 MB 2.5 %), nor with 32 (28 MB 3 %).
template <int P, bool CACHED> constexpr bool kEdgeGroups = !CACHED && P == 0;
template <int KIND, int VEC, int P, bool ACCUM, bool CACHED, bool SHALLOW, int SEGS, typename Tab>
__global__ __launch_bounds__(VEC == 4 ? kMaxBlock : kNarrowBlock) void rsa_seg_kernel(
    Tab gtab, float* __restrict__ acc, int p, ReduceTable<SEGS> tab, int how, unsigned edges)
{
    const auto& g = table_view(gtab);
    constexpr int BATCH = VEC == 1 ? 64 : MICS_RSA_BATCH;
    constexpr int EPL = VEC * GradFormat<KIND>::kPerDword;
    unsigned tile, x = blockIdx.x;
    if constexpr (kEdgeGroups<P, CACHED>) {
        if (x < edges) {                               // workgroup x does nothing but the ends of segment x
            const ReduceSeg& sg = tab.seg[x];
            rsa_edges<KIND, EPL, P, ACCUM>(acc + sg.dst, g, p, sg.src0, sg.lead, sg.end);
            return;
        }
        x -= edges;
    }
    const ReduceSeg sg = segment_at<(CACHED || KIND == 2 || P == 0 || P > 8)>(
        tab, VEC == 1 ? x : tile_of(x, kEdgeGroups<P, CACHED> ? gridDim.x - edges : gridDim.x, how & kInRuns), &tile);
    const size_t end = sg.end, lead = sg.lead;
    float* const dst = acc + sg.dst;
    if constexpr (CACHED) {
        if (end - lead < EPL) {
            rsa_short<KIND, P, ACCUM>(dst, g, p, sg.src0, lead, end);
            return;
        }
    } else if constexpr (!kEdgeGroups<P, CACHED>) {
        if (tile == 0) rsa_edges<KIND, EPL, P, ACCUM>(dst, g, p, sg.src0, lead, end);
    }
    const size_t v0 = ((size_t)tile * blockDim.x + threadIdx.x) * EPL;
    rsa_lane<KIND, VEC, P, BATCH, SHALLOW, ACCUM, CACHED, CACHED>(dst, g, p, sg.src0, v0, lead, end, how & ~kInRuns);
}

// ---------------------------------------------------------------------------
// Step 2b: reduction of the replication-group all-reduce at the accumulation
// boundary and the scaling to a mean (Section 3.4).  One lane owns 4 elements
// per copy and pass (the last count mod 4 elements go one per lane).  `out` may be copies[0]: a lane
// reads its elements of every copy before it writes them, and no other lane touches them.
// ---------------------------------------------------------------------------

// s = ((a_0 + a_1) + ...) + a_{r-1} for the 4 elements from x.  R > 0: r = R at compile time,
// all loads in flight at once; R == 0: any r in batches of 16 loads.
template <int R, bool NT, typename Tab>
__device__ __forceinline__ f32x4 avg_sum4(const Tab& a, int r, size_t x)
{
    if constexpr (R > 0) {
        f32x4 v[R];
        #pragma unroll
        for (int c = 0; c < R; ++c) v[c] = MICS_LD(NT, (const f32x4_a4*)((const float*)a.ptr[c] + x));
        f32x4 sum = v[0];
        #pragma unroll
        for (int c = 1; c < R; ++c) sum = sum + v[c];
        return sum;
    } else {
        constexpr int B = 16;
        f32x4 sum = MICS_LD(NT, (const f32x4_a4*)((const float*)a.ptr[0] + x));
        for (int c0 = 1; c0 < r; c0 += B) {
            f32x4 v[B];
            #pragma unroll
            for (int b = 0; b < B; ++b)
                if (c0 + b < r) v[b] = MICS_LD(NT, (const f32x4_a4*)((const float*)a.ptr[c0 + b] + x));
            #pragma unroll
            for (int b = 0; b < B; ++b)
                if (c0 + b < r) sum = sum + v[b];
        }
        return sum;
    }
}

// One element, the r loads in flight 16 at a time.
template <typename Tab>
__device__ __forceinline__ float avg_sum1(const Tab& a, int r, size_t x)
{
    constexpr int B = 16;
    float sum = ((const float*)a.ptr[0])[x];
    for (int c0 = 1; c0 < r; c0 += B) {
        float w[B];
        #pragma unroll
        for (int b = 0; b < B; ++b)
            if (c0 + b < r) w[b] = ((const float*)a.ptr[c0 + b])[x];
        #pragma unroll
        for (int b = 0; b < B; ++b)
            if (c0 + b < r) sum = sum + w[b];
    }
    return sum;
}

// STORE: average_store.
template <int R, int STORE, typename Tab>
__global__ __launch_bounds__(kMaxBlock) void avg_kernel(
    float* out, Tab a, int r, float scale, size_t count)
{
    const size_t nlanes = (count + 3) / 4;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nlanes; i += stride) {
        const size_t x = 4 * i;
        if (x + 4 <= count) {
            const f32x4 sum = avg_sum4<R, kAvgNtl>(a, r, x);
            [[maybe_unused]] const unsigned lane = threadIdx.x & 63u;
            if constexpr (STORE == kOutThrough)
                store_vec<kWriteThrough>(wave_buffer(out + (x - 4 * lane), 1024), 16 * lane, sum * scale);
            else
                MICS_ST(STORE == kOutStreamed, (f32x4_a4*)(out + x), sum * scale);
        }
    }
    // the last count mod 4 elements: one per lane
    const size_t e = count / 4 * 4 + threadIdx.x;
    if (blockIdx.x == 0 && e < count) out[e] = avg_sum1(a, r, e) * scale;
}

// ---------------------------------------------------------------------------
// Step 3: mixed-precision Adam on the shard (Sections 2.1, 3.2).  One fp32
// operation per line; the order is part of the contract.
// ---------------------------------------------------------------------------

__device__ __forceinline__ void adam_element(float& w, float& m, float& v, float g,
                                             const AdamScalars& hp)
{
    const float t1 = hp.beta1 * m;
    const float t2 = hp.one_minus_beta1 * g;
    const float m_new = t1 + t2;
    const float gg = g * g;
    const float t3 = hp.beta2 * v;
    const float t4 = hp.one_minus_beta2 * gg;
    const float v_new = t3 + t4;
    const float m_hat = m_new / hp.bias_corr1;        // correctly rounded (build flag)
    const float v_hat = v_new / hp.bias_corr2;
    const float root = __builtin_sqrtf(v_hat);       // correctly rounded (build flag)
    const float denom = root + hp.eps;
    const float ratio = m_hat / denom;
    const float decay = hp.weight_decay * w;
    const float update = ratio + decay;
    const float delta = hp.lr * update;
    w = w - delta;
    m = m_new;
    v = v_new;
}

// The update of 4 consecutive elements from x given their gradient, states in place.
template <int OUT>
__device__ __forceinline__ void adam_update4(float* master, float* exp_avg, float* exp_avg_sq,
                                             uint16_t* param_bf16, size_t x, f32x4 g, f32x4 w, f32x4 m,
                                             f32x4 v, const AdamScalars& hp, bool through)
{
    #pragma unroll
    for (int e = 0; e < 4; ++e) {
        float we = w[e], me = m[e], ve = v[e];
        adam_element(we, me, ve, g[e], hp);
        w[e] = we; m[e] = me; v[e] = ve;
    }
    if (through) {                                             // wavefront-uniform
        const unsigned lane = threadIdx.x & 63u;
        const size_t x0 = x - 4 * lane;
        store_vec<kWriteThrough | kNonTemporal>(wave_buffer(master + x0, 1024), 16 * lane, w);
        store_vec<kWriteThrough | kNonTemporal>(wave_buffer(exp_avg + x0, 1024), 16 * lane, m);
        store_vec<kWriteThrough | kNonTemporal>(wave_buffer(exp_avg_sq + x0, 1024), 16 * lane, v);
    } else {
        MICS_ST(true, (f32x4_a4*)(master + x), w);
        MICS_ST(true, (f32x4_a4*)(exp_avg + x), m);
        MICS_ST(true, (f32x4_a4*)(exp_avg_sq + x), v);
    }
    if constexpr (OUT != kParamNone) {
        u32x2 b = {param_pack<OUT>(w.x, w.y), param_pack<OUT>(w.z, w.w)};
        MICS_ST(true, (u32x2_a2*)(param_bf16 + x), b);
    }
}

template <int OUT>
__device__ __forceinline__ void adam_update1(float* master, float* exp_avg, float* exp_avg_sq,
                                             uint16_t* param_bf16, size_t x, float g, const AdamScalars& hp)
{
    float w = master[x], m = exp_avg[x], v = exp_avg_sq[x];
    adam_element(w, m, v, g, hp);
    master[x] = w; exp_avg[x] = m; exp_avg_sq[x] = v;
    if constexpr (OUT != kParamNone) param_bf16[x] = param_single<OUT>(w);
}

// One lane owns 4 consecutive elements per pass, so that every load and store instruction of
// a wavefront covers one contiguous kilobyte (stores that leave gaps between lanes reach
// memory as partial lines and cost extra traffic).  Four 128-bit loads are in flight before
// the first use; the 16-bit parameters (bf16 or binary16, OUT) leave as one 64-bit store.  That
// output may sit anywhere on an element boundary -- for instance inside the stage-1 buffer of
// the next parameter gather, at T_l + j*S.
template <int OUT>
__global__ __launch_bounds__(kMaxBlock) void adam_kernel(
    float* __restrict__ master, float* __restrict__ exp_avg, float* __restrict__ exp_avg_sq,
    uint16_t* __restrict__ param_bf16, const float* __restrict__ grad, size_t count, AdamScalars hp, bool through)
{
    const size_t nlanes = (count + 3) / 4;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nlanes; i += stride) {
        const size_t x = 4 * i;
        if (x + 4 <= count) {
            const f32x4 g = MICS_LD(kAdamNtl, (const f32x4_a4*)(grad + x));
            const f32x4 w = MICS_LD(kAdamNtl, (const f32x4_a4*)(master + x));
            const f32x4 m = MICS_LD(kAdamNtl, (const f32x4_a4*)(exp_avg + x));
            const f32x4 v = MICS_LD(kAdamNtl, (const f32x4_a4*)(exp_avg_sq + x));
            adam_update4<OUT>(master, exp_avg, exp_avg_sq, param_bf16, x, g, w, m, v, hp, through);
        } else {
            for (size_t e = x; e < count; ++e)
                adam_update1<OUT>(master, exp_avg, exp_avg_sq, param_bf16, e, grad[e], hp);
        }
    }
}

// Replica average fused into the Adam step: the averaged gradient of a lane's 4 elements is
// formed in registers from the r accumulator copies (same additions, same order, same multiply
// as avg_kernel) and goes straight into adam_element, so it is neither written nor re-read:
// 4r + 12 bytes read and 14 written per element instead of (4r + 4) + 30.  R > 0: r = R at
// compile time; R == 0: any r in batches of 16 loads.
template <int R, int OUT, typename Tab>
__global__ __launch_bounds__(kMaxBlock) void avg_adam_kernel(
    float* __restrict__ master, float* __restrict__ exp_avg, float* __restrict__ exp_avg_sq,
    uint16_t* __restrict__ param_bf16, Tab a, int r, float scale, size_t count, AdamScalars hp, bool through)
{
    const size_t nlanes = (count + 3) / 4;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nlanes; i += stride) {
        const size_t x = 4 * i;
        if (x + 4 <= count) {
            f32x4 sum, w, m, v;
            auto states = [&] {
                w = MICS_LD(kAdamNtl, (const f32x4_a4*)(master + x));
                m = MICS_LD(kAdamNtl, (const f32x4_a4*)(exp_avg + x));
                v = MICS_LD(kAdamNtl, (const f32x4_a4*)(exp_avg_sq + x));
            };
            if constexpr (R > 0) {
                // every load in flight before the first use: left to itself the compiler may trade the
                // loads for registers (r = 8, 50 M elements: 514 against 440 us)
                f32x4 c[R];
                #pragma unroll
                for (int i = 0; i < R; ++i) c[i] = MICS_LD(kAdamNtl, (const f32x4_a4*)((const float*)a.ptr[i] + x));
                states();
                __builtin_amdgcn_sched_barrier(0);
                sum = c[0];
                #pragma unroll
                for (int i = 1; i < R; ++i) sum = sum + c[i];
            } else {
                sum = avg_sum4<0, kAdamNtl>(a, r, x);
                states();
            }
            adam_update4<OUT>(master, exp_avg, exp_avg_sq, param_bf16, x, sum * scale, w, m, v, hp, through);
        }
    }
    // the last count mod 4 elements: one per lane
    const size_t e = count / 4 * 4 + threadIdx.x;
    if (blockIdx.x == 0 && e < count)
        adam_update1<OUT>(master, exp_avg, exp_avg_sq, param_bf16, e, avg_sum1(a, r, e) * scale, hp);
}

// ---------------------------------------------------------------------------
// Launch helpers
// ---------------------------------------------------------------------------

int compute_units(int* out)
{
    static std::atomic<int> cached[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev >= 0 && dev < 64 && cached[dev].load() > 0) { *out = cached[dev].load(); return 0; }
    int n = 0;
    e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return (int)e;
    if (n < 1) n = 1;
    if (dev >= 0 && dev < 64) cached[dev].store(n);
    *out = n;
    return 0;
}

int compute_units(size_t* out)
{
    int n = 0;
    const int e = compute_units(&n);
    *out = (size_t)n;
    return e;
}

// Workgroups of `block` lanes for `items` lane-sized work items: enough to cover them, at
// most `bpc` per compute unit (the kernels stride over the rest).
int grid_for(size_t items, int block, int bpc, unsigned* blocks)
{
    int cus = 0;
    if (int e = compute_units(&cus)) return e;
    const int forced = g_blocks_per_cu.load();
    if (forced > 0) bpc = forced;
    size_t want = (items + (size_t)block - 1) / (size_t)block;
    const size_t cap = (size_t)cus * (size_t)bpc;
    if (want > cap) want = cap;
    if (want < 1) want = 1;
    *blocks = (unsigned)want;
    return 0;
}

template <typename T> struct same_type { typedef T type; };

// Launches `kernel` with `lds` bytes of dynamic LDS and returns the launch call's own status:
// the caller's HIP error state (an earlier, unrelated error of the thread) is neither reported
// nor cleared here.
template <typename... KArgs>
int launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t st,
           typename same_type<KArgs>::type... args)
{
    void* ptrs[] = {(void*)&args...};
    return (int)hipLaunchKernel((const void*)kernel, grid, block, ptrs, lds, st);
}

// Calls f(std::bool_constant<a>) for a runtime flag.
template <typename F>
int dispatch_bool(bool a, F&& f)
{
    return a ? f(std::true_type{}) : f(std::false_type{});
}

template <int N>
SmallTable<N> small(const PtrTable& t)
{
    SmallTable<N> s;
    for (int i = 0; i < N; ++i) s.ptr[i] = t.ptr[i];
    return s;
}

// Calls f(std::integral_constant<int, P>) with P = p if p has an unrolled kernel, else P = 0.
template <typename F>
int dispatch_group(int p, F&& f)
{
    switch (unrolled_group(p)) {
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        case 8: return f(std::integral_constant<int, 8>{});
        case 16: return f(std::integral_constant<int, 16>{});
        case 32: return f(std::integral_constant<int, 32>{});
        default: return f(std::integral_constant<int, 0>{});
    }
}

// Calls f(std::integral_constant<int, R>, table) for an average of r copies: R = r where there is an unrolled kernel, those
// of 3, 5, 6, 7 and 9 to 16 only if `all`, else R = 0 and the whole table.
template <typename F>
int dispatch_copies(const PtrTable& t, int r, bool all, F&& f)
{
    auto unrolled = [&](auto R) { return f(R, small<R.value>(t)); };
    switch (r) {
        case 1: return unrolled(std::integral_constant<int, 1>{});
        case 2: return unrolled(std::integral_constant<int, 2>{});
        case 4: return unrolled(std::integral_constant<int, 4>{});
        case 8: return unrolled(std::integral_constant<int, 8>{});
        default: break;
    }
    switch (all ? r : 0) {
        case 3: return unrolled(std::integral_constant<int, 3>{});
        case 5: return unrolled(std::integral_constant<int, 5>{});
        case 6: return unrolled(std::integral_constant<int, 6>{});
        case 7: return unrolled(std::integral_constant<int, 7>{});
        case 9: return unrolled(std::integral_constant<int, 9>{});
        case 10: return unrolled(std::integral_constant<int, 10>{});
        case 11: return unrolled(std::integral_constant<int, 11>{});
        case 12: return unrolled(std::integral_constant<int, 12>{});
        case 13: return unrolled(std::integral_constant<int, 13>{});
        case 14: return unrolled(std::integral_constant<int, 14>{});
        case 15: return unrolled(std::integral_constant<int, 15>{});
        case 16: return unrolled(std::integral_constant<int, 16>{});
        default: break;
    }
    return f(std::integral_constant<int, 0>{}, t);
}

}  // namespace

void set_blocks_per_cu(int n) { g_blocks_per_cu.store(n); }

void set_stream_threshold_bytes(size_t n) { g_stream_bytes.store(n); }

void set_launch_shape(int family, int lanes, int waves_per_cu)
{
    g_lanes[family].store(lanes);
    g_waves[family].store(waves_per_cu);
}

const char* hip_error_text(int err) { return hipGetErrorString((hipError_t)err); }

// Most vectors that a chunk's tiles have in front of it, since they begin on 128-byte lines.
static size_t off_line(const void* dst, size_t dst_byte, size_t shard_bytes)
{
    return (((uintptr_t)dst + dst_byte) | shard_bytes) % 128 ? 7 : 0;
}

namespace {

// Vectors per lane (1 or 2) of a call that moves `moved` bytes through reorder_flat_kernel, 0: not its work.  us, flat /
// the kernels with a workgroup per chunk:
//   one tensor, 16-byte aligned, p = 16: 0.3 MB 1.82 / 2.22, 8 MB 3.04 / 3.47, 20 MB (two vectors) 5.08 / 5.97, 28 MB 6.6 /
//   6.9, 36 MB 8.9 / 8.2 (buffers in the L2: 10 MB 3.0 / 2.75); not aligned, whose wavefronts at the borders of chunks make a second
//   round trip, never: 0.6 MB 2.35 / 2.05, 4 MB 3.75 / 3.3, 8 MB 4.3 / 4.0
//   several tensors, all aligned: 16 of a layer, p = 4 33 MB 7.5 / 8.1, 40 MB 9.5 / 9.1, p = 128 33 MB 7.4 / 8.5, 40 MB 9.5 / 9.8
//   not all aligned: 4 of them p = 4 23 MB 6.4 / 6.7, p = 16 22 MB 7.5 / 6.5, p = 64 19 MB 6.9 / 6.2; 16, 40, 60 and 93 of
//   them p = 16 15 MB 5.5 / 6.1, 5.5 / 6.2, 5.7 / 6.0, 5.5 / 6.2, 23 MB 7.5 / 7.3, 8.8 / 7.7, 8.4 / 7.3, 8.6 / 7.5; p = 32
//   19 MB 7.0 / 7.0, 7.3 / 7.6, 7.4 / 7.2, 7.9 / 7.7; p = 64 19 MB 7.2 / 7.4, 7.6 / 8.5, 7.9 / 8.1, 8.4 / 9.4, 27 MB 8.9 /
//   8.5, 9.5 / 9.7, 10.9 / 9.5, 11.4 / 10.7; p = 128 27 MB 9.1 / 9.2, 9.9 / 12.0, 11.7 / 11.6, 12.3 / 13.6, 33 MB 13.1 /
//   10.3, 11.9 / 12.3, 12.2 / 12.5, 12.9 / 14.8.  (Tensors of similar size would rather stay up to 24 MB, p = 16 40 tensors
//   19 MB 6.9 / 7.5, 24 MB 7.9 / 8.2, p = 8 60 tensors 24 MB 7.6 / 8.1; lists that spread over three decades would rather
//   go, 15 to 24 MB 15 % faster by chunks.)
int flat_vectors(int n, size_t moved, int p, bool vec16)
{
    const size_t mb = moved >> 20;
    if (g_blocks_per_cu.load() > 0) return 0;                  // its grid has no cap
    if (n == 1) return !vec16 || mb >= 27 ? 0 : mb < 16 ? 1 : 2;
    const size_t most = vec16 ? (n <= kMaxSegPerLaunch ? 36 : p >= 48 ? 52 : 24)
                        : n < 16 ? 18 : p < 24 ? 17 : p < 48 ? 18 : p < 96 ? 20 : n <= 24 ? 27 : 34;
    return mb >= most ? 0 : mb < 18 ? 1 : 2;
}

template <int U, int SEGS>
int launch_reorder_flat(void* dst, const PtrTable& src, const Segment* segs, int n, size_t moved, int k, size_t eb, hipStream_t st)
{
    // us, one tensor, 64 / 128 / 512 lanes: 1 MB 2.08 / 2.06 / 2.14, 8 MB 3.58 / 3.40 / 3.04; two vectors: 256.  Many, speed against
    // 64 lanes of 256: 0.3 MB 0.93, 2 MB 1.00, 8 MB 1.11
    const int lanes = U == 2 ? 256 : n == 1 ? (moved < (3u << 20) ? 128 : kMaxBlock) : moved < (3u << 19) ? 64 : 256;
    const Shape sh = with_knobs(kFamReorder, Shape{lanes, 0});
    const size_t tile_bytes = (size_t)sh.lanes * U * 16;
    FlatTable<SEGS> tab;
    size_t tiles = 0;
    for (int t = 0; t < n; ++t) {
        const size_t valid = segs[t].numel * eb, shard = segs[t].shard_elems * eb;
        FlatSeg& f = tab.seg[t];
        tab.tile_begin[t] = (unsigned)tiles;
        f.src_byte = segs[t].src_offset * eb;
        f.dst_byte = segs[t].dst_offset * eb;
        f.valid_bytes = (unsigned)valid;
        f.shard_bytes = (unsigned)(shard < valid ? shard : valid);
        // n / d for n < 2^31: with 2^shift >= d the rounded-up 2^(31 + shift) / d is too large by less than 2^shift / d
        const unsigned d = f.shard_bytes / 2;
        f.shift = 0;
        while ((1ull << f.shift) < d) ++f.shift;
        f.recip = (unsigned)(((1ull << (31 + f.shift)) + d - 1) / d);
        tiles += (valid + (((uintptr_t)dst + f.dst_byte) & 127) + tile_bytes - 1) / tile_bytes;
    }
    for (int t = n; t < SEGS; ++t) tab.tile_begin[t] = kNoTile;
    return launch(k <= 16 ? reorder_flat_kernel<U, SEGS, false> : reorder_flat_kernel<U, SEGS, true>, dim3((unsigned)tiles), dim3(sh.lanes),
                  lds_for(sh), st, (unsigned char*)dst, src, tab, (unsigned)k, 65536u / (unsigned)k + 1);
}

// Tensors of at least one byte.
int launch_reorder_small(void* dst, const PtrTable& src, const Segment* segs, int n, int vectors, size_t moved, int k, size_t eb,
                         hipStream_t st)
{
    return dispatch_bool(vectors == 2, [&](auto TWO) {
        constexpr int U = TWO.value ? 2 : 1;
        if (n == 1) return launch_reorder_flat<U, 1>(dst, src, segs, n, moved, k, eb, st);
        if (n <= 64) return launch_reorder_flat<U, 64>(dst, src, segs, n, moved, k, eb, st);
        return launch_reorder_flat<U, kMaxSegMany>(dst, src, segs, n, moved, k, eb, st);
    });
}

}  // namespace

int launch_reorder(void* dst, const PtrTable& src, size_t n_valid_bytes, size_t shard_bytes, int p,
                   int k, bool vec16, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    const Segment one = {n_valid_bytes, shard_bytes, 0, 0};
    if (const int vectors = flat_vectors(1, 2 * n_valid_bytes, p, vec16))
        return launch_reorder_small(dst, src, &one, 1, vectors, 2 * n_valid_bytes, k, 1, st);
    if (vec16) {
        // spread the block budget over the p chunks
        unsigned total = 0;
        const Shape sh = reorder_shape(2 * n_valid_bytes, MICS_REORDER_BLOCK);
        if (int e = grid_for((shard_bytes / 16 + off_line(dst, 0, shard_bytes)) * (size_t)p, sh.lanes, MICS_REORDER_BPC, &total)) return e;
        unsigned bx = (total + (unsigned)p - 1) / (unsigned)p;
        return launch(reorder_vec_kernel, dim3(bx, (unsigned)k, (unsigned)(p / k)), dim3(sh.lanes), lds_for(sh), st, (u32x4*)dst, src,
                      shard_bytes / 16, n_valid_bytes, k);
    }
    return launch_reorder_coalesced(dst, src, &one, 1, p, k, 1, false, stream);
}

namespace {

// Repeats the last of n pointers up to a multiple of 8: kernels may load through those entries.
void pad_table(PtrTable& t, int n)
{
    for (int i = n; i < (n + 7) / 8 * 8; ++i) t.ptr[i] = t.ptr[n - 1];
}

// Rounds gradient pointers down to a 128-byte line when all of them sit at the same position inside
// theirs (rank g's slices of separately allocated buffers do: they all start g*S elements in);
// returns how many elements they moved back (the kernels' `lead`, 0 .. 63).  The p gradient loads of a
// wavefront then cover whole lines and only its accumulator accesses do not, 8 of 2p+8 bytes.  A 1 KiB
// load that is off the lines touches nine of them instead of eight, and with non-temporal loads the
// shared ones are fetched twice.  us with pointers rounded down to 16 / to 128 bytes, all 64 bytes off:
// p = 8, 27 M elements 92 / 84; p = 16, 12.5 M 90 / 82; p = 32, 7 M 90 / 81; 1.7 M 23.9 / 21.8; p = 64, 0.2 M
// 11.0 / 8.8.  Up to 3 buffers the accumulator is most of the traffic: p = 2, 30 MB 6.7 / 6.9, so they go
// down to 16 bytes only, which keeps its vectors of 16 bytes together (down to 4 / to 16 bytes, all 2 or 10
// bytes off: p = 32, 9.8 M 124 / 117; p = 16, 50 M 343 / 322).
// With mixed positions 2-byte elements are still brought to 4 bytes if their parity agrees; else
// the pointers stay and the odd ones are read with 2-byte aligned 128-bit loads.
// *line = the alignment they have afterwards: 128, 16, 4 or 1 bytes (1: that of their elements).
unsigned align_gradient_pointers(PtrTable& g, int p, int elem_bytes, unsigned* line_out)
{
    uintptr_t differ = 0;                                  // address bits in which the pointers differ
    for (int q = 1; q < p; ++q) differ |= (uintptr_t)g.ptr[q] ^ (uintptr_t)g.ptr[0];
    const uintptr_t line = p >= 4 && (differ & 127) == 0 ? 128 : (differ & 15) == 0 ? 16 : (differ & 3) == 0 ? 4 : 1;
    const uintptr_t back = (uintptr_t)g.ptr[0] & (line - 1);
    *line_out = (unsigned)line;
    for (int q = 0; q < p; ++q) g.ptr[q] = (const char*)g.ptr[q] - back;
    pad_table(g, p);
    return (unsigned)(back / (uintptr_t)elem_bytes);
}

// Where the gradients are at one position inside their lines and the accumulator is at another, the lanes' vectors can be laid
// on the lines of either.  The `lead` that lays them on the accumulator's, if the gradients' (`first` = address of the first
// element) are then on 16 bytes, else -1.
int lead_on_accumulator_lines(const float* acc, uintptr_t first, size_t elem_bytes)
{
    const uintptr_t lead = (uintptr_t)acc / 4 % 32;
    return (first - lead * elem_bytes) % 16 ? -1 : (int)lead;
}

// Whether neighbouring tiles meet in one XCD (tile_of), and on whose lines the vectors lie.  From 640 calls and 400 of segments drawn
// over p = 1 .. 96, 12 MB .. 2.2 GB, the formats, positions and both kinds of micro-step; speed against the plain order on the
// gradients' lines:
//   - Gradients off their lines, each buffer at another position: in runs (bf16, p = 8 64 MB 1.06, 411 MB 1.15; p = 12..16 25..60 MB 1.07;
//     p = 32 60..120 MB 1.09; p = 96 1.04; f32, p = 8 54 MB 1.23, 436 MB 1.09); below 12 MB the few instructions cost 1 to
//     2 %.  Not with few buffers, where the accumulator is most of the traffic: one (bf16, 24 MB .77; f32, 160 MB .81), two
//     and three of f32 off 16 bytes (p = 3 666 MB .88; on 16 bytes p = 2, 3 1.01 to 1.09).
//   - Gradients on lines, accumulator not: on the accumulator's lines and in runs, so that the gradients' shared lines are found in the
//     L2 and no accumulator's line is written in parts (bf16, p = 5 321 MB 1.09, runs alone 1.04, 1.2 GB 1.07, .97; p = 8
//     416 MB 1.10, 1.04; p = 12..16 300..700 MB 1.06, 1.03, above 700 MB .97, 1.00; f32, p = 8 250 MB 1.03, .92, 1.8 GB
//     .98, .94; p = 24 and more up to 5 % slower).  Not in runs this loses 1 to 10 %.  If the gradients are then off 16
//     bytes: p = 12 to 16 runs alone (bf16 120..700 MB 1.01 to 1.03, f32 p = 12 200..450 MB 1.05 to 1.08, p = 16 1.04;
//     above 700 MB 1.00, first micro-steps .96), fewer buffers neither (bf16, p = 8 120 MB and more .97 to 1.00).
//   - Everything on lines, or many buffers: in runs in the middle of the range (bf16, p = 4 209 MB 1.06, p = 8 231 MB 1.05,
//     p = 12..16 120..300 MB 1.05, 300..700 MB 1.03, above .98; below 60 MB .99 to 1.00; f32, p = 8 124 MB 1.06, p = 12..16
//     60..120 MB .96, 120..300 MB 1.03, above 700 MB .97; first micro-steps 120..700 MB 1.01 to 1.03, above .95 to .96).
//   - Segments, whose ends lie anywhere: in runs, up to 3 buffers below 60 MB only (bf16, p = 2 45 MB 1.07, 150 MB .97, 600
//     MB .94; f32, p = 3 300..700 MB .84), from 32 on above 24 MB (f32, p = 32 14 MB .83), f32 below 1 GB (p = 16 2 GB
//     .93), up to 8 buffers of f32 not from 300 to 700 MB unless all can be on the accumulator's lines (p = 8 335 MB .93,
//     447 MB .88, 760 MB 1.09; if they can 335 MB 1.04). Accumulating, on the accumulator's lines where that can be (lines
//     / runs alone: bf16, p = 4 300..700 MB 1.06 / 1.01, p = 8 120..300 MB 1.02 / 1.00; f32, p = 8 120..300 MB 1.04 / .93),
//     with 12 to 19 buffers from 60 to 700 MB (p = 16 25 MB 1.01 / 1.02, 400 MB 1.08 / 1.05, above 700 MB .98 / 1.03), with
//     more never (p = 24 25..120 MB .99 / 1.01).  First micro-steps in runs alone (lines / so: p = 8 1.00 / 1.03, p =
//     12..16 .99 / 1.01, p = 24 .97 / 1.00).
struct ReduceOrder {
    bool in_runs, acc_lines;
};
// lane_acc: the accumulator at the lanes' virtual element 0; alignable: the vectors can be laid on its lines.
ReduceOrder reduce_order(int p, int elem_bytes, size_t count, bool accumulate, bool grads_on_lines, bool grads16, const float* lane_acc,
                         bool alignable)
{
    const size_t mb = count * ((size_t)p * elem_bytes + (accumulate ? 8 : 4)) >> 20;
    const bool two = elem_bytes == 2, acc_on_lines = (uintptr_t)lane_acc % 128 == 0;
    if (!grads_on_lines || (p < 4 && !acc_on_lines))
        return {mb >= 12 && (p >= 4 || (p > 1 && (two || (grads16 && (uintptr_t)lane_acc % 16 == 0)))), false};
    const bool below = mb < (two && accumulate ? 700 : 500);
    if (!acc_on_lines && p <= 16) {
        if (alignable && (two && p <= 8 ? mb >= 60 : mb >= 20 && mb < (accumulate ? 700 : 600))) return {true, true};
        if (p < 12) return {false, false};
    }
    const bool few = accumulate ? !two && p < 8 : p < 12;
    return {!few && mb >= (two ? 80 : 120) && below, false};
}
// alignable: all segments can be laid on the accumulator's lines.
ReduceOrder reduce_order_segments(int p, int elem_bytes, size_t mb, bool accumulate, bool alignable)
{
    if (p < 4) return {p > 1 && mb < 60, false};
    if (elem_bytes == 4 && (mb >= 1000 || (accumulate && !alignable && p <= 8 && mb >= 300 && mb < 700))) return {false, false};
    return {p < 32 || (p < 48 && mb >= 24), accumulate && (p < 12 || (p < 20 && mb >= 60 && mb < 700))};
}

// Small messages on large groups take the one-dword-per-lane kernels (VEC = 1; of a coalesced call up to kMaxSegMany
// segments together), MB of gradients up to which they win.  us per call, one dword / 128 bits per lane:
//   bf16, p = 20 5 MB 3.4 / 3.9, 19 MB 6.0 / 6.0, 32 MB 8.9 / 8.2      p = 32 13 MB 4.3 / 4.7, 24 MB 6.4 / 6.3
//         p = 48 13 MB 4.5 / 5.8, 49 MB 10.7 / 12.2, 63 MB 13.7 / 12.9  p = 40 49 MB 10.9 / 11.6, 62 MB 13.6 / 12.9
//         p = 64 1 MB 3.0 / 6.4, 50 MB 10.7 / 11.6, 65 MB 13.5 / 14.6   p = 128 3 MB 4.3 / 11.2, 67 MB 12.7 / 15.9
//   f32 alike: p = 48 59 MB 11.5 / 12.0, 66 MB 13.1 / 12.7; p = 64 67 MB 12.8 / 14.3; p = 96 79 MB 15.0 / 15.2
// and about half of that where the buffers sit at different positions inside their lines, which costs every dword
// load (bf16, p = 24 12 MB 5.4 / 5.5, 23 MB 8.3 / 7.2; p = 48 21 MB 7.1 / 7.1, 35 MB 10.6 / 9.3; p = 64 31 MB 9.2 / 8.9;
// p = 128 52 MB 14.5 / 15.2, 67 MB 18.4 / 17.7; f16, p = 128 59 MB 15.6 / 16.6).
// Few segments change sooner, many as one tensor does (from 32 buffers on): speed against 128 bits a lane, 16 tensors of a
// layer / 60 of 1 k elements and more: bf16, p = 20 10 MB 1.07 / 1.08, 18 MB .97 / .92, 23 MB .91 / .88; p = 32 10 MB 1.06
// / 1.15, 18 MB .88 / 1.13; p = 40 23 MB 1.02 / 1.09, 30 MB .72 / 1.13; p = 48 30 MB 1.18 / 1.22, 50 MB .94 / .95; p = 64
// 30 MB 1.09 / 1.34, 40 MB .86 / 1.22; p = 128 50 MB 1.01 / 1.34, 60 MB .89 / 1.17; f32, p = 40 18 MB 1.13 / 1.20, 30 MB
// .92 / 1.00; p = 48 50 MB .87 / 1.04; p = 96 50 MB .96 / 1.19.  22 tensors go with the 60 (p = 32 20 MB 1.25).
// segments: their number, 0 for one tensor.
inline bool narrow_call(int p, size_t elem_bytes, size_t count, bool same_line, int segments)
{
    int most = p >= 56 ? (same_line ? (p >= 96 ? 72 : 68) : p / 2) : p >= 48 ? (same_line ? 60 : 25)
               : p >= 40 ? (same_line ? 54 : 22) : p >= 20 && elem_bytes == 2 ? (same_line ? 24 : 12) : 0;
    if (segments && (p < 32 || segments <= 20)) {
        const int line = p >= 96 ? 50 : p >= 48 ? 31 : p >= 40 ? 24 : p >= 32 ? 12 : 14;
        most = std::min(most, same_line ? line : line / 2);
    }
    return count <= ((size_t)most << 20) / ((size_t)p * elem_bytes);
}

template <int KIND, int VEC, int P, bool ACCUM, bool CACHED, bool OTHER = false>
int rsa_launch(float* acc, const PtrTable& g, int p, unsigned lead, size_t count, unsigned blocks,
               const Shape& sh, int how, hipStream_t st)
{
    // lanes of 8 elements pass their results through 32 bytes of LDS (rsa_lane)
    const size_t lds = lds_for(sh, !CACHED && KIND != 2 ? (size_t)sh.lanes * 32 : 0);
    if constexpr (P > 0)
        return launch(rsa_kernel<KIND, VEC, P, ACCUM, CACHED, OTHER, SmallTable<P>>, dim3(blocks + 1), dim3(sh.lanes), lds, st,
                      small<P>(g), acc, p, lead, count, how);
    else
        return launch(rsa_kernel<KIND, VEC, 0, ACCUM, CACHED, OTHER, PtrTable>, dim3(blocks + 1), dim3(sh.lanes), lds, st, g,
                      acc, p, lead, count, how);
}

template <int KIND>
int rsa_launch_kind(float* acc, PtrTable g, int p, size_t count, bool accumulate, hipStream_t st)
{
    unsigned line = 0;
    unsigned lead = align_gradient_pointers(g, p, GradFormat<KIND>::kElemBytes, &line);
    constexpr size_t PD = GradFormat<KIND>::kPerDword;
    unsigned blocks = 0;
    // small message on a large group: one dword per lane and buffer
    constexpr int GB = GradFormat<KIND>::kElemBytes;
    if (narrow_call(p, GB, count, line >= 16, 0)) {
        const Shape narrow = {kNarrowBlock, 0};
        const size_t nlanes = (lead + count + PD - 1) / PD;
        if (int e = grid_for(nlanes, kNarrowBlock, MICS_RSA_BPC, &blocks)) return e;
        return accumulate ? rsa_launch<KIND, 1, 0, true, true>(acc, g, p, lead, count, blocks, narrow, kAccCached, st)
                          : rsa_launch<KIND, 1, 0, false, true>(acc, g, p, lead, count, blocks, narrow, kAccCached, st);
    }
    size_t units = 0;
    if (int e = compute_units(&units)) return e;
    const uintptr_t first = (uintptr_t)g.ptr[0] + lead * GB;
    const int other = lead_on_accumulator_lines(acc, first, GB);
    const bool lines = line == 128 || on_lines(g, p);
    const ReduceOrder order = reduce_order(p, GB, count, accumulate, lines, lines || line >= 16, acc - lead, other >= 0);
    if (order.acc_lines) {
        for (int q = 0; q < p; ++q) g.ptr[q] = (const char*)g.ptr[q] + ((ptrdiff_t)lead - other) * GB;
        pad_table(g, p);
        lead = (unsigned)other;
        line = 16;
    }
    const size_t nlanes = (lead + count + 4 * PD - 1) / (4 * PD);
    const bool acc16 = ((uintptr_t)acc - 4 * (uintptr_t)lead) % 16 == 0;
    const int policy = accum_policy(count, p, GB), how = policy | (order.in_runs ? kInRuns : 0);
    const bool shallow = policy != kAccCached && shallow_call(p, nlanes, units) && !long_call_in_step(g, p, nlanes, units);
    const Shape sh = shallow ? shallow_shape(p, nlanes, units)
                             : reduce_shape(p, GB, nlanes, line >= 16, acc16, accumulate, policy == kAccCached, units);
    if (int e = grid_for(nlanes, sh.lanes, MICS_RSA_BPC, &blocks)) return e;
    return dispatch_bool(accumulate, [&](auto A) {
        if (policy == kAccCached)
            return dispatch_bool(order.in_runs, [&](auto R) {
                return dispatch_group(p, [&](auto P) {                 // one buffer is never in runs there
                    return rsa_launch<KIND, 4, P.value, A.value, true, (R.value && P.value != 1)>(acc, g, p, lead, count, blocks, sh, how, st);
                });
            });
        if (shallow) return rsa_launch<KIND, 4, 0, A.value, false, true>(acc, g, p, lead, count, blocks, sh, how, st);
        return dispatch_group(p, [&](auto P) {
            constexpr int N = P.value == 16 ? 0 : P.value;             // 16 are always read in shallow batches
            return rsa_launch<KIND, 4, N, A.value, false>(acc, g, p, lead, count, blocks, sh, how, st);
        });
    });
}

}  // namespace

int launch_reduce_scatter_accum(float* acc, const PtrTable& grads, size_t count, int p, bool accumulate,
                                int kind, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    switch (kind) {
        case 0: return rsa_launch_kind<0>(acc, grads, p, count, accumulate, st);
        case 1: return rsa_launch_kind<1>(acc, grads, p, count, accumulate, st);
        default: return rsa_launch_kind<2>(acc, grads, p, count, accumulate, st);
    }
}

int launch_replica_average(float* out, const PtrTable& a, size_t count, int r, float scale, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    unsigned blocks = 0;
    const bool streamed = stream_acc(count);
    size_t units = 0;
    if (int e = compute_units(&units)) return e;
    const Shape sh = average_shape(r, count, streamed, on_lines(a, r), units);
    const size_t lds = lds_for(sh);
    if (int e = grid_for((count + 3) / 4, sh.lanes, MICS_AVG_BPC, &blocks)) return e;
    const dim3 gr(blocks), bl(sh.lanes);
    auto run = [&](auto SO) {
        return dispatch_copies(a, r, unrolled_average(r, count, streamed, units), [&](auto R, const auto& tab) {
            return launch(avg_kernel<R.value, SO.value, std::decay_t<decltype(tab)>>, gr, bl, lds, st, out, tab, r, scale, count);
        });
    };
    switch (average_store(r, count, streamed)) {
        case kOutPlain: return run(std::integral_constant<int, kOutPlain>{});
        case kOutThrough: return run(std::integral_constant<int, kOutThrough>{});
        default: return run(std::integral_constant<int, kOutStreamed>{});
    }
}

namespace {
// Calls f(std::integral_constant<int, OUT>) for the parameter output of a call.
template <typename F>
int dispatch_param(const void* param_out, bool f16, F&& f)
{
    if (!param_out) return f(std::integral_constant<int, kParamNone>{});
    if (f16) return f(std::integral_constant<int, kParamF16>{});
    return f(std::integral_constant<int, kParamBf16>{});
}
}  // namespace

int launch_adam(float* master, float* exp_avg, float* exp_avg_sq, uint16_t* param_bf16, bool param_f16,
                const float* grad, size_t count, const AdamScalars& hp, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    unsigned blocks = 0;
    const Shape sh = adam_shape(count);
    if (int e = grid_for((count + 3) / 4, sh.lanes, MICS_ADAM_BPC, &blocks)) return e;
    return dispatch_param(param_bf16, param_f16, [&](auto OUT) {
        return launch(adam_kernel<OUT.value>, dim3(blocks), dim3(sh.lanes), lds_for(sh), st, master, exp_avg,
                      exp_avg_sq, param_bf16, grad, count, hp, states_through(count * 30));
    });
}

namespace {

// A launch of SEGS tensors at most, none of them empty.
// Full-size workgroups take tiles of 16 KiB, which small chunks do not fill: below 48 MB they are for calls whose chunks do
// (us, full-size / 128 lanes: 41 MB, 40 tensors, p = 128 (chunks of 4 KB) 22.9 / 13.6, p = 64 (8 KB) 15.9 / 11.7, p = 16
// (32 KB) 11.3 / 10.5; 16 tensors, p = 32 (40 KB) 11.0 / 10.4; 93 tensors, p = 8 (27 KB) 10.6 / 10.7; 60 tensors, p = 4, 28
// MB (58 KB) 7.7 / 7.9).
Shape reorder_tensors_shape(size_t moved, int n, int p)
{
    const size_t chunk = moved / 2 / ((size_t)n * (size_t)p);
    return chunk < (size_t{48} << 10) ? with_knobs(kFamReorder, Shape{kSegLanes, 0}) : reorder_shape(moved, kSegLanes);
}

template <int SEGS>
int launch_reorder_seg(void* dst, const PtrTable& src, const Segment* segs, int n, size_t moved, int p, int k, size_t eb, hipStream_t st)
{
    const Shape sh = reorder_tensors_shape(moved, n, p);
    const size_t tile_vecs = (size_t)sh.lanes * MICS_SEG_U;
    size_t tiles = 0;
    ReorderSegTable<SEGS> tab;
    for (int t = 0; t < n; ++t) {
        const Segment& sg = segs[t];
        tab.tiles.begin[t] = (unsigned)tiles;
        tab.seg[t].shard_vecs = sg.shard_elems * eb / 16;
        tab.seg[t].valid_bytes = sg.numel * eb;
        tab.seg[t].src_vec = sg.src_offset * eb / 16;
        tab.seg[t].dst_vec = sg.dst_offset * eb / 16;
        tiles += (tab.seg[t].shard_vecs + off_line(dst, sg.dst_offset * eb, sg.shard_elems * eb) + tile_vecs - 1) / tile_vecs;
        if (tiles > 0x7FFFFFFFull) return (int)hipErrorInvalidValue;
    }
    tab.tiles.close(n);
    return launch(reorder_seg_kernel<SEGS>, dim3((unsigned)tiles, (unsigned)k, (unsigned)(p / k)), dim3(sh.lanes), lds_for(sh), st,
                  (u32x4*)dst, src, tab, k);
}

ByteSeg byte_seg(const Segment& sg, size_t eb)
{
    return ByteSeg{sg.shard_elems * eb, sg.numel * eb, sg.src_offset * eb, sg.dst_offset * eb};
}

// Tiles start on a 128-byte line of the destination; at least one per tensor, for the chunk ends.
size_t shift_tiles(const ByteSeg& sg, size_t tile_bytes) { return (sg.shard_bytes + 127 + tile_bytes - 1) / tile_bytes; }

// Vectors per lane of reorder_shift_kernel: more of them, fewer wavefronts that share a source line at their ends;
// fewer, a call that is spread further.  Speed against loads off 16 bytes, one tensor, 512
// lanes x 1 / 64 x 4: 39 MB 1.15 / 1.11, 134 MB 1.11 / 1.12 and (p = 48) 1.08 / 1.05, 268 MB 1.04 / 1.10,
// 1.26 GB 1.05 / 1.07; many tensors per launch, whose tile has to be found first, 128 x 2 / 64 x 4 /
// 512 x 1: 315 MB 1.12 / 1.08 / 0.83, 3.2 GB 1.13 / 1.07 / 0.81.
template <int SEGS>
int launch_reorder_shift(void* dst, const PtrTable& src, const Segment* segs, int n, size_t moved, int p, int k, size_t eb, hipStream_t st)
{
    const Shape sh = reorder_tensors_shape(moved, n, p);
    const size_t tile_bytes = (size_t)sh.lanes * MICS_SEG_U * 16;
    size_t tiles = 0;
    ByteSegTable<SEGS> tab;
    for (int t = 0; t < n; ++t) {
        tab.tiles.begin[t] = (unsigned)tiles;
        tab.seg[t] = byte_seg(segs[t], eb);
        tiles += shift_tiles(tab.seg[t], tile_bytes);
        if (tiles > 0x7FFFFFFFull) return (int)hipErrorInvalidValue;
    }
    tab.tiles.close(n);
    return launch(reorder_shift_kernel<ByteSegTable<SEGS>, MICS_SEG_U>, dim3((unsigned)tiles, (unsigned)k, (unsigned)(p / k)),
                  dim3(sh.lanes), lds_for(sh), st, (unsigned char*)dst, src, tab, k);
}

int launch_reorder_shift_one(void* dst, const PtrTable& src, const Segment& one, size_t moved, int p, int k, size_t eb, hipStream_t st)
{
    const bool spread = moved < (160u << 20);
    const Shape sh = reorder_shape(moved, spread ? kMaxBlock : 64);
    const OneTensor where{byte_seg(one, eb)};
    const size_t tiles = shift_tiles(where.seg, (size_t)sh.lanes * (spread ? 1 : 4) * 16);
    if (tiles > 0x7FFFFFFFull) return (int)hipErrorInvalidValue;
    return launch(spread ? reorder_shift_kernel<OneTensor, 1> : reorder_shift_kernel<OneTensor, 4>,
                  dim3((unsigned)tiles, (unsigned)k, (unsigned)(p / k)), dim3(sh.lanes), lds_for(sh), st,
                  (unsigned char*)dst, src, where, k);
}

}  // namespace

int launch_reorder_coalesced(void* dst, const PtrTable& src, const Segment* segs, int n, int p, int k,
                             int elem_bytes, bool vec16, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    const size_t eb = (size_t)elem_bytes;
    size_t moved = 0;
    for (int t = 0; t < n; ++t) moved += 2 * segs[t].numel * eb;
    if (const int vectors = flat_vectors(n, moved, p, vec16)) return launch_reorder_small(dst, src, segs, n, vectors, moved, k, eb, st);
    if (vec16)
        return n <= kMaxSegPerLaunch ? launch_reorder_seg<kMaxSegPerLaunch>(dst, src, segs, n, moved, p, k, eb, st)
                                     : launch_reorder_seg<kMaxSegMany>(dst, src, segs, n, moved, p, k, eb, st);
    if (n == 1) return launch_reorder_shift_one(dst, src, segs[0], moved, p, k, eb, st);
    return n <= kMaxSegPerLaunch ? launch_reorder_shift<kMaxSegPerLaunch>(dst, src, segs, n, moved, p, k, eb, st)
                                 : launch_reorder_shift<kMaxSegMany>(dst, src, segs, n, moved, p, k, eb, st);
}

namespace {

// Virtual index of the first element of a segment that is element `src` of the rounded-down buffers.
template <int KIND>
unsigned segment_lead(const float* acc, const PtrTable& g, size_t src, size_t dst, size_t unit, ReduceOrder order)
{
    constexpr size_t GB = GradFormat<KIND>::kElemBytes;
    if (order.acc_lines && unit * GB == 128) {
        const int lead = lead_on_accumulator_lines(acc + dst, (uintptr_t)g.ptr[0] + src * GB, GB);
        if (lead >= 0) return (unsigned)lead;
    }
    return (unsigned)(src % unit);
}

// `n` segments in one launch, with lanes of VEC dwords.
template <int KIND, int VEC, int SEGS>
int reduce_segments(float* acc, const PtrTable& g, size_t base_lead, size_t unit, const Segment* segs, int n, int p,
                    bool accumulate, const Shape& sh, int policy, ReduceOrder order, bool shallow, hipStream_t st)
{
    const int how = policy | (order.in_runs ? kInRuns : 0);
    constexpr size_t EPL = VEC * GradFormat<KIND>::kPerDword;
    ReduceTable<SEGS> tab;
    const size_t tile_elems = (size_t)sh.lanes * EPL;
    size_t tiles = 0;
    bool ends = false;                             // elements that no lane holds as a full vector
    for (int t = 0; t < n; ++t) {
        const Segment& sg = segs[t];
        // position of the segment's first element in the rounded-down buffers; its virtual
        // element 0 is the one on a line (of 128, 16 or 4 bytes: see align_gradient_pointers) at or below it
        const size_t src = sg.src_offset + base_lead;
        const unsigned lead = segment_lead<KIND>(acc, g, src, sg.dst_offset, unit, order);
        tab.tile_begin[t] = (unsigned)tiles;
        tab.seg[t].lead = lead;
        tab.seg[t].pad = 0;
        tab.seg[t].end = lead + sg.numel;
        ends = ends || lead % EPL || tab.seg[t].end % EPL;
        tab.seg[t].src0 = src - lead;
        tab.seg[t].dst = sg.dst_offset;
        tiles += (lead + sg.numel + tile_elems - 1) / tile_elems;
        if (tiles > 0x7FFFFFFFull) return (int)hipErrorInvalidValue;
    }
    for (int t = n; t < SEGS; ++t) tab.tile_begin[t] = kNoTile;
    auto run = [&](auto P, auto A, auto C, auto S) {
        // lanes of 8 elements pass their results through 32 bytes of LDS
        const size_t lds = lds_for(sh, !C.value && EPL == 8 ? (size_t)sh.lanes * 32 : 0);
        const unsigned edges = kEdgeGroups<P.value, C.value> && ends ? (unsigned)n : 0;
        const dim3 gr((unsigned)tiles + edges), bl(sh.lanes);
        if constexpr (P.value > 0)
            return launch(rsa_seg_kernel<KIND, VEC, P.value, A.value, C.value, S.value, SEGS, SmallTable<P.value>>, gr, bl, lds, st,
                          small<P.value>(g), acc, p, tab, how, edges);
        else
            return launch(rsa_seg_kernel<KIND, VEC, 0, A.value, C.value, S.value, SEGS, PtrTable>, gr, bl, lds, st, g, acc, p, tab, how, edges);
    };
    return dispatch_bool(accumulate, [&](auto A) {
        if constexpr (VEC == 1) {
            return run(std::integral_constant<int, 0>{}, A, std::true_type{}, std::false_type{});
        } else if constexpr (SEGS > 64) {
            return dispatch_group(p, [&](auto P) { return run(P, A, std::true_type{}, std::false_type{}); });
        } else {
            if (shallow) return run(std::integral_constant<int, 0>{}, A, std::false_type{}, std::true_type{});
            return dispatch_bool(policy == kAccCached, [&](auto C) {
                return dispatch_group(p, [&](auto P) { return run(P, A, C, std::false_type{}); });
            });
        }
    });
}

template <int KIND>
int reduce_coalesced_kind(float* acc, PtrTable g, const Segment* segs, int n, int p, bool accumulate, int* taken,
                          hipStream_t st)
{
    constexpr size_t GB = GradFormat<KIND>::kElemBytes, EPL = 4 * GradFormat<KIND>::kPerDword;
    unsigned line = 0;
    const size_t base_lead = align_gradient_pointers(g, p, (int)GB, &line);
    size_t units = 0;
    if (int e = compute_units(&units)) return e;
    const size_t unit = line >= 16 ? line / GB : 4 / GB;             // elements that a segment's lead is counted in
    auto elements_of = [&](int m) {
        size_t sum = 0;
        for (int t = 0; t < m; ++t) sum += segs[t].numel;
        return sum;
    };
    size_t elements = elements_of(n);
    *taken = n;
    if (narrow_call(p, GB, elements, line >= 16, n)) {
        const Shape sh = {kNarrowBlock, 0};
        return n <= 64 ? reduce_segments<KIND, 1, 64>(acc, g, base_lead, unit, segs, n, p, accumulate, sh, kAccCached, {false, false}, false, st)
                       : reduce_segments<KIND, 1, kMaxSegMany>(acc, g, base_lead, unit, segs, n, p, accumulate, sh, kAccCached, {false, false}, false, st);
    }
    // Small calls carry more than 64 segments, whose records then come in a second round: us, 64 / 96 per launch, f16, p = 12,
    // 79 segments 7.3 / 4.0; larger ones keep to 64 and to half as many kernels.
    if (n > 64 && accum_policy(elements, p, (int)GB) != kAccCached) {
        *taken = n = 64;
        elements = elements_of(n);
    }
    bool alignable = unit * GB == 128;
    for (int t = 0; t < n; ++t)
        alignable = alignable && lead_on_accumulator_lines(acc + segs[t].dst_offset, (uintptr_t)g.ptr[0] + (segs[t].src_offset + base_lead) * GB, GB) >= 0;
    const ReduceOrder order = reduce_order_segments(p, (int)GB, elements * (p * GB + (accumulate ? 8 : 4)) >> 20, accumulate, alignable);
    bool acc16 = true;
    size_t waves = 0, full = 0, half = 0;                            // workgroups of 64 lanes, of kMaxBlock and of half as many
    for (int t = 0; t < n; ++t) {
        const size_t lead = segment_lead<KIND>(acc, g, segs[t].src_offset + base_lead, segs[t].dst_offset, unit, order);
        waves += (lead + segs[t].numel + 64 * EPL - 1) / (64 * EPL);
        full += (lead + segs[t].numel + kMaxBlock * EPL - 1) / (kMaxBlock * EPL);
        half += (lead + segs[t].numel + kMaxBlock / 2 * EPL - 1) / (kMaxBlock / 2 * EPL);
        acc16 = acc16 && ((uintptr_t)(acc + segs[t].dst_offset) - 4 * lead) % 16 == 0;
    }
    const int policy = accum_policy(elements, p, (int)GB);
    const size_t nlanes = (elements + EPL - 1) / EPL;
    const bool shallow = policy != kAccCached && shallow_segments(p, (int)GB, nlanes, units) && !long_call_in_step(g, p, nlanes, units);
    const Shape sh = shallow ? shallow_shape_segments(p, waves, full, half, n, units)
                             : reduce_shape_segments(p, (int)GB, nlanes, n, line >= 16, acc16, accumulate, policy == kAccCached, units);
    return n <= 64 ? reduce_segments<KIND, 4, 64>(acc, g, base_lead, unit, segs, n, p, accumulate, sh, policy, order, shallow, st)
                   : reduce_segments<KIND, 4, kMaxSegMany>(acc, g, base_lead, unit, segs, n, p, accumulate, sh, policy, order, shallow, st);
}

}  // namespace

int launch_reduce_coalesced(float* acc, const PtrTable& grads, const Segment* segs, int n, int p,
                            bool accumulate, int kind, int* taken, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    switch (kind) {
        case 0: return reduce_coalesced_kind<0>(acc, grads, segs, n, p, accumulate, taken, st);
        case 1: return reduce_coalesced_kind<1>(acc, grads, segs, n, p, accumulate, taken, st);
        default: return reduce_coalesced_kind<2>(acc, grads, segs, n, p, accumulate, taken, st);
    }
}

int launch_avg_adam(float* master, float* exp_avg, float* exp_avg_sq, uint16_t* param_bf16, bool param_f16,
                    const PtrTable& copies, int r, float scale, size_t count, const AdamScalars& hp,
                    void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    unsigned blocks = 0;
    size_t units = 0;
    if (int e = compute_units(&units)) return e;
    const bool lines = on_lines(copies, r) && on_lines({master, exp_avg, exp_avg_sq});
    const Shape sh = fused_shape(r, count, lines, units);
    // off the lines: 17.6 M elements, r = 2, 110 us, through the L2 124
    const size_t traffic = count * (4 * (size_t)r + 26);
    const bool through = lines && states_through(traffic);
    const size_t lds = lds_for(sh);
    if (int e = grid_for((count + 3) / 4, sh.lanes, MICS_ADAM_BPC, &blocks)) return e;
    return dispatch_param(param_bf16, param_f16, [&](auto BF) {
        const dim3 gr(blocks), bl(sh.lanes);
        return dispatch_copies(copies, r, unrolled_update(r, count, units), [&](auto R, const auto& tab) {
            return launch(avg_adam_kernel<R.value, BF.value, std::decay_t<decltype(tab)>>, gr, bl, lds, st, master, exp_avg, exp_avg_sq, param_bf16,
                          tab, r, scale, count, hp, through);
        });
    });
}

}  // namespace mics
