// How the kernels are launched: workgroup sizes, caps on wavefronts, kernels for ranges of sizes, paths through the
// caches.  Host code without HIP, so that its arithmetic is tested where there is no GPU.  Every rule has both sides measured beside it.
#pragma once

#include <algorithm>
#include <atomic>
#include <cmath>
#include <initializer_list>

#include "internal.h"

namespace mics {
namespace {                                // its includer's own: the knobs are one library's, not a process's

constexpr int kMaxBlock = 512;           // most lanes per workgroup of the element-wise kernels
constexpr int kNarrowBlock = 64;         // ... of the one-dword-per-lane reduction

std::atomic<int> g_blocks_per_cu{0};

// How a reduction passes its accumulator through the caches (accum_policy): plain loads and stores
// (kernels of their own); otherwise write-through stores from the wavefronts whose lines are whole and
// non-temporal or write-through ones from the others; non-temporal stores from all.  Wavefronts whose lines
// are whole load it non-temporally, the others plainly up to 8 buffers and non-temporally above.
enum { kAccCached = 0, kAccThroughLines = 1, kAccThrough = 2, kAccStreamed = 3 };

// Accumulators and averages of up to 224 MiB -- what the 256 MB Infinity Cache absorbs -- are written so
// that the next call can find them there, larger ones are streamed.  An explicit threshold (0 = none)
// replaces this line.
constexpr size_t kDefaultStreamBytes = 224u << 20;
std::atomic<size_t> g_stream_bytes{0};

inline bool stream_acc(size_t elements)
{
    const size_t t = g_stream_bytes.load();
    return elements * 4 > (t ? t : kDefaultStreamBytes);
}

// The optimizer states are written non-temporally, and through the L2 as well (nt sc0 sc1) in calls
// that no cache could hold: Adam, 50 M elements 227.4 -> 226.3 us, 101 M 456 -> 453; average + Adam,
// 50 M, r = 2 257.3 -> 253.4, r = 4 322 -> 317, r = 8 442 -> 433.  A call at 150 to 250 MB loses 2 to 3 %.
inline bool states_through(size_t traffic) { return traffic >= (300u << 20); }

// A large accumulator is read with non-temporal loads and written through the L2 (sc0 sc1): the next
// micro-step finds it in the Infinity Cache if nothing has displaced it, and if something has, the
// writes have reached memory in the order of the stream.  us per call, accumulator resident on
// consecutive calls / not:
//                                 plain          NT loads,       NT loads, write-
//                                                NT stores       through stores
//   p = 16, 50 M elements (201 MB)  304 / 335    311 / 311       291 / 315
//   p = 8,  25 M (101 MB)           89  / 103    97  / 97        88  / 96
//   p = 8,  9.8 M (39 MB)           40.2 / 40.0  40.0 / 38.9     36.5 / 37.0
// Non-temporal stores win where the accumulator is beyond the 224 MiB that the cache absorbs (p = 8,
// 101 M elements: 364 against 375), for 32 and more buffers beyond 64 MiB (p = 32, 25 M: 289, 302),
// and where the lines at the two ends of a wavefront's piece are not whole (accumulator off 128
// bytes: p = 16, 50 M: 324, 374; p = 32, 9.8 M: 123, 129) unless few buffers are read (p = 2, 42 M: 85.5, 79.8;
// f32, p = 3, 40 M: 137, 132) or the accumulator is small (p = 8, 9.8 M: 40.6, 37.9).  Those wavefronts load it
// plainly up to 8 buffers, so that the second one to need a line finds it in the L2 (all with non-temporal
// loads / so: f32, p = 1, 16.7 M 38.8 / 33.5, p = 2, 50 M 142 / 134).
// A small accumulator is left in the L2 (8 x 4 MB).  Speed of that against write-through, over resident and not, first
// micro-step and accumulating, geometric means with buffers rotating through 1 GB / through three sets:
//   p = 4..11         10 MiB 1.04 / 1.00   12 MiB 1.01 / 0.98   16..20 MiB 0.95..0.99 in both   28 MiB 0.98 / 0.98
//   f32, p = 1..3     8 MiB  1.06 / 0.98   12 MiB 1.02 / 0.96   20 MiB 0.98 / 0.97              28 MiB 0.96 / 0.96
//   bf16, p = 1..3    4 MiB  1.03 / 0.95   7 MiB  1.04 / 0.96   8 MiB  0.97 / 0.86              16 MiB 0.95 / 0.84
// Calls that accumulate in a resident buffer still gain from it beyond the lines (p = 4..11, 16..24 MiB 1.03..1.07;
// bf16, p = 4, 28 MiB 17.7 / 19.8 us); first micro-steps lose more (16 MiB 0.91..0.93).  With many gradients it would be
// gone before its turn (p = 16, 3 M, 12 MB 18.9 / 21.2, 19.9 / 20.2; 7.5 M, 30 MB 51.9 / 52.2, 48.6 / 49.3; p = 32, 0.6 M,
// 2.5 MB 9.4 / 10.5, 10.0 / 9.9; of 32 and more buffers only the calls that are all latency). 16 to 31 buffers of f32 up to
// 4 MiB, since what passes the L2 is read in shallow batches; us, left there / past it, accumulating and first micro-step:
// p = 16 4.2 MiB 15.5 / 14.4, 14.8 / 13.8, 6 MiB 20.6 / 19.9, 19.8 / 19.1, 7.9 MiB 25.0 / 24.1, 23.5 / 23.1; p = 24 4.2 MiB
// 21.6 / 19.4, 20.9 / 18.9, 7.9 MiB 35.7 / 33.6, 34.1 / 32.8; p = 31 6 MiB 34.6 / 33.4, 33.6 / 32.7.  (Below, 3.2 MiB, 3 to
// 8 % too with buffers in no cache; resident ones were not compared there.)
inline int accum_policy(size_t count, int p, int elem_bytes)
{
    constexpr size_t kSmall = 64u << 20;
    const size_t cached = p < 4 && elem_bytes == 2 ? 7u << 20 : p < 12 ? 12u << 20 : p < 16 ? 8u << 20 : p < 32 ? (elem_bytes == 2 ? 8u : 4u) << 20 : 1u << 20;
    if (stream_acc(count)) return kAccStreamed;
    if (count * 4 <= cached) return kAccCached;
    if (g_stream_bytes.load() == 0 && p >= 32 && count * 4 > kSmall) return kAccStreamed;
    return p < 4 || (p < 16 && count * 4 <= kSmall) ? kAccThrough : kAccThroughLines;
}

enum { kOutPlain = 0, kOutThrough = 1, kOutStreamed = 2 };         // how an average passes them (average_store)

// Launch shape: lanes per workgroup and the most wavefronts a compute unit may hold at a time (0 =
// whatever fits).
//
// These streaming kernels run fastest in single-wavefront workgroups -- a finished wavefront's slot
// is refilled at once instead of when the last of a workgroup's 8 wavefronts has finished -- and,
// the reorder aside, with fewer wavefronts per compute unit than fit, i.e. with fewer but longer
// request streams at the memory controllers.  Measured on MI355X (GB/s of algorithmic bytes; lanes
// x wavefronts per compute unit, 32 = no cap; 50 M elements):
//   reorder (3.2 GB)  256x32 6335  64x32 6580  64x16 5990  64x8  3860
//   average r = 2                  64x32 6540  64x16 6470  64x11 6200
//   average r = 8     512x32 5935  64x32 6325  64x9 6580  64x8  6650
//   Adam              128x32 6040  64x32 5965  64x11 6670  64x9 6630
//   average + Adam, r = 8          64x11 6290  64x8  6530  64x5  6740
// The cap is enforced with otherwise unused dynamic LDS: a workgroup that asks for 1/n of a
// compute unit's LDS shares the unit with at most n - 1 others.
struct Shape {
    int lanes, waves_per_cu;
};
std::atomic<int> g_lanes[kFamilies], g_waves[kFamilies];       // 0 = built-in choice

inline Shape with_knobs(int family, Shape sh)
{
    if (const int l = g_lanes[family].load()) sh.lanes = l;
    if (const int w = g_waves[family].load()) sh.waves_per_cu = w;
    if (sh.waves_per_cu >= 32) sh.waves_per_cu = 0;
    return sh;
}

// A call that is over before a capped pipeline has filled: uncapped, in full-size workgroups.  Where a
// compute unit gets fewer than four of them, all run at once and the slowest unit decides: the
// largest workgroups whose rounded-up number per unit wastes at most 12 % (reduce, p = 64, 1.1 M
// elements, 269 workgroups of 512 lanes on 256 units: 34.6 us, of 64 lanes 27.6; p = 16, 2.5 M: 512
// lanes 19.7, 256 lanes 18.8; p = 8, 4.2 M, where 512 fits: 17.2, 64 lanes 18.4; average + Adam,
// r = 2, 0.74 M: 512 lanes 9.9, 64 lanes 8.7).  Up to one full-size workgroup per unit the launch of many
// small ones takes longer than idle units cost (reduce, p = 8, 0.88 M: 5.0 us, 64 lanes 5.6), but a call
// that gives a unit less than half of one runs in single wavefronts: a unit moves about 100 GB/s on
// its own (reduce, 0.5 M elements at p = 16: 5.3 us instead of 6.2).
inline Shape small_call(size_t nlanes, size_t units)
{
    auto waste = [&](size_t lanes) {                           // of the fullest unit against an even share
        const size_t wgs = (nlanes + lanes - 1) / lanes;
        return (double)((wgs + units - 1) / units * units * lanes) / (double)nlanes;
    };
    if (nlanes >= units * (4 * kMaxBlock)) return Shape{kMaxBlock, 0};
    if (nlanes * 2 <= (size_t)kMaxBlock * units) return Shape{64, 0};
    if (nlanes <= (size_t)kMaxBlock * units) return Shape{kMaxBlock, 0};
    return Shape{waste(512) <= 1.12 ? 512 : waste(256) <= 1.12 ? 256 : 64, 0};
}

// A reduction with more than half of and less than seven eighths of a full-size workgroup for every compute unit (from 16
// buffers on, more than a quarter, f32 up to 31 a third): one workgroup per unit, of as many lanes as that takes, so that
// no unit idles and none has more than another.  Tiles begin on the gradients' lines (8 lanes).  us, full-size workgroups
// or single wavefronts / so, wavefronts per unit in front: bf16, p = 4 4.3 8 % faster, p = 8 10, p = 12 11, 5.5 5 to 7; p =
// 16 2.3 3.9 / 3.4, 4.2 5.45 / 4.77, 6.3 6.15 / 6.1; p = 32 4.2 9.1 / 7.5; p = 64 5.2 16.5 / 15.3; p = 128 2.3 17.8 / 15.0,
// 4.2 27.3 / 23.4; f32, p = 12 4.3 4.3 / 3.8, p = 16 2.4 3.4 / 3.6, p = 32 2.3 16 % faster, 4.2 8.0 / 6.9, p = 128 4.2 26.3
// / 22.3.  With few buffers single wavefronts are 2 to 6 % faster below; two or more such workgroups per unit are faster or
// slower by 5 %, from one size to the next.
// With n segments, so many workgroups less as may have a partial tile; every wavefront, the last and partial one too, needs n lanes to look
// its segment up (segment_at).  us, 512 lanes / so: bf16, 16 tensors, p = 8 4.2 wavefronts per unit 13 % faster, p = 48 4.2
// 54 MB 14.2 / 11.3, p = 64 4.2 72 MB f32 16.5 / 13.6, p = 96 4.2 107 MB f32 24.0 / 19.7.
inline Shape even_call(size_t nlanes, size_t units, size_t least = 256, size_t most = 448, size_t n = 0)
{
    const size_t groups = units - n;
    if (n >= 64 || units <= n || nlanes > groups * most || nlanes <= units * least) return small_call(nlanes, units);
    size_t lanes = ((nlanes + groups - 1) / groups + 7) / 8 * 8;
    if (lanes % 64 && lanes % 64 < n) lanes += (n + 7) / 8 * 8 - lanes % 64;
    return Shape{(int)lanes, 0};
}
// The P of a reduction's kernel: that of p buffers where there is an unrolled one, else 0.
constexpr int unrolled_group(int p) { return p <= 8 || p == 16 || p == 32 ? p : 0; }
// Whether a kernel that passes its stores through LDS (two-byte gradients, accumulator not left in the L2) knows a
// workgroup's partial last wavefront (rsa_lane).
constexpr bool partial_waves(int P, bool shallow) { return (P == 0 || P == 32) && !shallow; }
// The line from which a reduction does so.
inline size_t even_least(int p, int elem_bytes, bool cached)
{
    if (!cached && elem_bytes == 2 && !partial_waves(unrolled_group(p), false)) return (size_t)1 << 40;
    return p < 16 ? 256 : p < 32 && elem_bytes == 4 ? 170 : 128;
}

// True if the buffers begin on 128-byte lines.
inline bool on_lines(std::initializer_list<const void*> buffers)
{
    uintptr_t bits = 0;
    for (const void* b : buffers) bits |= (uintptr_t)b;
    return bits % 128 == 0;
}
inline bool on_lines(const PtrTable& t, int n)
{
    uintptr_t bits = 0;
    for (int i = 0; i < n; ++i) bits |= (uintptr_t)t.ptr[i];
    return bits % 128 == 0;
}

// Where a single buffer spans gigabytes (all the shards of a group in one call), still fewer request
// streams are better, us with the caps above / with those for huge calls: reduce p = 16, 805 M elements
// 5436 / 5278, p = 8, 201 M 742 / 730; Adam, 402 M 1940 / 1900, 805 M 3980 / 3830; average + Adam, r = 4,
// 402 M 2660 / 2590; average r = 2, 402 M 749 / 735.
constexpr size_t kHugeElements = 192u << 20;

// Wavefronts whose copies or states begin off the 128-byte lines share a line at each end with the next one,
// which finds it in the L2 only if both run at about the same time: full-size workgroups, uncapped.  us, everything 4
// bytes off, 64 lanes / 512: average + Adam, r = 8, 1.4 M elements 18.0 / 16.5, r = 6, 4 M 41 / 38; average, r = 4, 10 M
// 34.4 / 32.3.
inline Shape off_lines(size_t nlanes, size_t units)
{
    return nlanes * 2 <= (size_t)kMaxBlock * units ? Shape{64, 0} : Shape{kMaxBlock, 0};
}

// The average's result is left in the L2 by calls of a middle size and written through it by larger ones and by
// the smallest, which end sooner without a write-back behind them, us plain / through: r = 2, 0.12 M elements 1.88 /
// 1.81, 1.2 M 3.7 / 4.0, 3.3 M 7.3 / 7.7, 6.7 M 15.0 / 14.5; r = 4, 0.15 M 2.6 / 2.25, 1 M 4.85 / 5.0, 3 M 11.0 / 10.7, 5.5 M
// 20.8 / 18.4; r = 8, 0.11 M 2.7 / 2.4; r = 16, 0.88 M 10.9 / 11.2, 1.6 M 19.3 / 19.2.  A single copy: 0.25 M 2.0 / 1.8, 1 M 3.0 /
// 3.2, 2.5 M 5.0 / 4.75.  (Copies that no cache holds.  If one still does, writing through wins from about 40 MB on: r = 3,
// 3.4 M 10.6 / 9.9, r = 6, 2 M 10.5 / 9.9.)
inline int average_store(int r, size_t count, bool streamed)
{
    if (streamed) return kOutStreamed;
    const size_t traffic = count * (4 * (size_t)r + 4);
    const bool middle = traffic >= ((r < 4 ? 3u : 12u) << 20) && traffic < ((r < 2 ? 12u : 44u) << 20);
    return middle ? kOutPlain : kOutThrough;
}

// The lines below which a call is small, us (buffers rotating), full-size workgroups / single wavefronts: average, r = 4 at
// 50 MB 8.6 / 8.6, 90 MB 15.7 / 15.0, r = 5 90 MB 16.2 / 15.3, r = 6 90 MB 16.6 / 15.4, 150 MB 25.8 / 24.3, r = 12 50 MB
// 8.8 / 8.8, 90 MB 16.2 / 15.1; average + Adam, r = 1 40 MB 8.5 / 8.5, 80 MB 15.6 / 15.0, 180 MB 31.4 / 30.1, r = 4 40 MB
// 8.4 / 8.7, 80 MB 15.4 / 15.0, 180 MB 32.2 / 30.2, r = 6 120 MB 21.6 / 20.5, r = 8 40 MB 8.3 / 8.3, 120 MB 21.7 / 20.8;
// reorder at 32 MB 7.7, 64x32 8.7, at 64 MB 13.1, 12.0.
constexpr size_t kLargeAverage = 60u << 20;
// Updates of more copies later: us, full-size workgroups, any r / single wavefronts, unrolled: r = 9 160 MB 27.5 / 31.5,
// 240 MB 44.8 / 40.6, r = 11 180 MB 30.6 / 32.5, 200 MB 36.5 / 35.2, r = 12 120 MB 23.1 / 24.6, r = 13 180 MB 31.8 / 32.4,
// 240 MB 44.1 / 41.4, r = 16 140 MB 24.1 / 27.9, 240 MB 48.1 / 41.1; above 16, all of them any r: r = 20 180 MB 36.3 /
// 34.5, r = 24 200 MB 40.8 / 37.8.
inline size_t large_update(int r) { return (r <= 8 ? size_t{76} : r < 12 ? size_t{180} : r <= 16 ? size_t{200} : size_t{160}) << 20; }
// ... and up to 8 copies not below 25 wavefronts a unit, which all run at once as full-size workgroups: us, so / single
// wavefronts, r = 6 80 MB 15.5 / 16.3, r = 7 80 MB 14.8 / 16.1, 84 MB 15.2 / 16.8, 88 MB 17.3 / 17.7, r = 8 88 MB 16.0 /
// 16.9, 92 MB 18.3 / 18.3.
inline bool single_waves_update(int r, size_t count, size_t units)
{
    return count * (4 * (size_t)r + 26) >= large_update(r) && (r > 8 || (count + 3) / 4 >= units * 1600);
}
// Copies in numbers other than 1, 2, 4 and 8 have unrolled kernels up to 16, whose loads need no pointer's load before each
// of them, and the one for any r, which spaces its loads by that.  Averages, us, any r / unrolled: r = 3 3 MB 2.63 / 2.29,
// 90 MB 15.3 / 14.7, r = 6 3 MB 2.7 / 2.3, 11 MB 3.8 / 3.55, 20 MB 5.05 / 5.4, 38 MB 7.8 / 8.3, 90 MB 16.7 / 15.4, 800 MB
// 119.7 / 121.6, r = 7 9 MB 3.5 / 3.1, 24 MB 5.7 / 6.3, 56 MB 11.3 / 12.2, r = 5 800 MB 122.3 / 122.4; r = 9 4 MB 2.9 /
// 2.5, 130 MB 22.9 / 22.2, 300 MB 46.8 / 45.7, r = 12 8 MB 3.4 / 3.1, 19 MB 5.35 / 4.9, 26 MB 5.85 / 5.5, 28 MB 6.5 / 7.2,
// 130 MB 22.8 / 24.2, 300 MB 47.1 / 46.4, r = 13 500 MB 75.2 / 75.9, 1 GB 146.6 / 146.3, r = 16 12 MB 4.1 / 3.8, 40 MB 8.7
// / 9.2, 250 MB 41.3 / 42.7.
// So from 6 copies on: unrolled in calls of up to one full-size workgroup a unit, which are all latency, and in large ones.
inline bool unrolled_average(int r, size_t count, bool streamed, size_t units)
{
    const size_t traffic = count * (4 * (size_t)r + 4);
    if (r > 5 && (count + 3) / 4 <= units * kMaxBlock) return true;
    if (r > 8) return r < 14 && traffic >= (200u << 20);
    return r == 3 ? !streamed : (r < 6 || traffic >= kLargeAverage) && traffic < (500u << 20);
}
// Updates: r = 3 5 MB 3.4 / 2.9, 40 MB 7.2 / 8.6, 180 MB 33.0 / 30.5; r = 5 5 MB 3.6 / 3.0, 40 MB 7.9 / 8.3, 180 MB 32.4 /
// 30.6; r = 9 4 MB 3.5 / 2.9, 20 MB 5.4 / 5.7, 300 MB 49.7 / 48.1, 900 MB 152 / 135; r = 13 20 MB 5.35 / 4.9, 40 MB 8.1 /
// 8.15, 300 MB 53.7 / 50.3; r = 12 33 MB 7.0 / 7.4; r = 16 3 MB 3.6 / 2.8, 28 MB 10 % faster, 80 MB 15.7 / 16.9, 400 MB
// 69.9 / 66.9.
inline bool unrolled_update(int r, size_t count, size_t units)
{
    return single_waves_update(r, count, units) || count * (4 * (size_t)r + 26) < (r < 12 ? 12u << 20 : 30u << 20);
}

inline Shape average_shape(int r, size_t count, bool streamed, bool lines, size_t units)
{
    const size_t traffic = count * (4 * (size_t)r + 4), nlanes = (count + 3) / 4;
    // a single copy below 18 MB: 1 M elements 2.94, 64x32 3.02; 1.7 M 3.8, 4.0
    if (!lines || (r < 2 && traffic < (18u << 20))) return with_knobs(kFamAverage, off_lines(nlanes, units));
    // few copies, few loads in flight per lane: every wavefront that fits (3 copies 300 MB 42.3, a cap of 14 46.1, but 800
    // MB 127.3, 120.6, streamed 2.1 GB 328, 345)
    if (r < 4) return with_knobs(kFamAverage, Shape{64, count >= kHugeElements ? 16 : r == 3 && !streamed && traffic >= (600u << 20) ? 14 : 0});
    if (traffic < kLargeAverage) return with_knobs(kFamAverage, r < 5 ? small_call(nlanes, units) : even_call(nlanes, units, 256, r < 12 ? 384 : 448));
    // more than 8 copies stay with full-size workgroups up to 96 MiB, if all that a unit gets run at once, up to three of
    // them (25 wavefronts), or as many that their number no longer matters: us, full-size workgroups / single wavefronts,
    // per unit in front, r = 11 22 12.5 / 13.5, r = 13 19 12.7 / 13.5, 27 20.1 / 18.3, r = 16 22 17.1 / 18.3, r = 14 25.4
    // 20.6 / 18.4, r = 9 27 14.4 / 13.5, 38 17.1 / 18.0, r = 10 34 17.5 / 18.0, r = 64 6 17.5 / 19.2
    const size_t waves = nlanes / (64 * units);
    if (r > 8 && traffic < (96u << 20) && (waves < 25 || waves >= 32)) return with_knobs(kFamAverage, even_call(nlanes, units, 256, 448));
    // us, caps of 9 / 10 / 11 / 12 / 14 / 16 / 18: 4 copies 90 MB 17.1 / 16.6 / 16.4 / 16.0 / 15.7 / 15.3 / 15.0, 300 MB
    // 48.9 / 47.4 / 46.4 / 45.8 / 45.0 / 44.6 / 44.6, 800 MB 127.6 / 124.5 / 121.3 / 122.4 / 125.2 / 126.7 / 127.7,
    // streamed 1.5 GB a cap of 16 232, 11 254; 5 copies 90 MB 16.8 / 16.2 / 16.4 / 16.1 / 15.4 / 15.3 / 15.3, 300 MB 46.5 /
    // 45.7 / 45.6 / 45.5 / 45.1 / 45.6 / 45.8, 800 MB 123.2 / 122.4 / 123.3 / 125.3; 6 copies 90 MB 16.6 / 16.2 / 16.1 /
    // 15.7 / 15.4, 300 MB 46.8 / 46.2 / 45.9 / 46.0 / 46.4; 8 copies 90 MB 15.7 / 15.4 / 15.3 / 15.4, 300 MB 46.2 / 46.3 /
    // 46.3.  Caps of 7 / 8 / 9 / 10, unrolled: 9 copies 300 MB 46.7 / 45.7 / 45.5 / 45.6, 1 GB 146.0 / 142.9 / 145.0 /
    // 144.9, 11 copies 1 GB 145.1 / 145.6 / 146.0 / 146.8, 13 copies 1 GB 147.0 / 146.3 / 147.3 / 147.7; any r: 9 copies
    // 130 MB 24.1 / 23.5 / 23.0 / 22.9, 12 copies 160 MB 28.0 / 28.1 / 27.3 / 27.4, 16 copies 160 MB 28.2 / 28.7 / 27.9 /
    // 28.1, 300 MB 47.7 / 48.3 / 48.1 / 48.4, 1 GB 147.2 / 148.9 / 150.0 / 151.0, 24 copies 250 MB 44.2 / 45.1 / 42.3 /
    // 42.4, 64 copies 250 MB 47.8 / 49.0 / 47.2 / 45.0, 700 MB 111.1 / 113.1 / 113.0 / 114.3
    const bool wide = traffic < (500u << 20) || (r < 5 && streamed);
    int cap = 0;
    if (r < 5) cap = traffic < (200u << 20) ? 18 : wide ? 16 : 11;
    else if (r < 6) cap = wide ? 14 : 11;
    else if (r < 8) cap = traffic < (120u << 20) ? 14 : wide ? 11 : 9;
    else if (r < 9) cap = traffic < (200u << 20) ? 10 : 9;
    else if (r < 14) cap = traffic >= (200u << 20) ? 8 : r < 12 ? 10 : 9;
    else cap = traffic < (280u << 20) ? 9 : 7;
    return with_knobs(kFamAverage, Shape{64, cap});
}

inline Shape adam_shape(size_t count) { return with_knobs(kFamAdam, Shape{64, count >= kHugeElements ? 8 : 11}); }

inline Shape fused_shape(int r, size_t count, bool lines, size_t units)
{
    const size_t traffic = count * (4 * (size_t)r + 26);
    if (!lines) return with_knobs(kFamFused, off_lines((count + 3) / 4, units));
    if (!single_waves_update(r, count, units)) return with_knobs(kFamFused, r < 12 ? small_call((count + 3) / 4, units) : even_call((count + 3) / 4, units));
    if (count >= kHugeElements) return with_knobs(kFamFused, Shape{64, r < 4 ? 8 : r < 8 ? 6 : 4});
    // us, caps of 4 / 5 / 6 / 7 / 8 / 9 / 10 / 11, at 120 MB: r = 1 .. / 25.4 / 23.9 / 22.7 / 21.7 / 21.1 / 20.9, r = 3
    // 22.8 / 21.9 / 21.3 / 21.1 / 21.1 / 21.2 from 6 on, r = 4 22.0 / 21.2 / 21.0 / 21.0 / 21.1, r = 6 21.2 / 20.8 / 20.8 /
    // 20.7 / 20.5, r = 8 22.9 / 21.4 / 21.0 / 21.1 / 21.2 / 20.8; at 400 MB: r = 1
    // 9 to 11 63.3 / 62.6 / 62.7, r = 2 62.5 at 9, r = 3 62.6 at 8, r = 4 61.6 at 7, r = 5 75.9 / 66.9 / 63.1 / 63.2 /
    // 64.1, r = 6 71.9 / 64.2 / 62.2 / 62.9, r = 8 68.5 / 63.5 / 64.0 / 65.2, r = 9 65.4 / 62.6 / 63.7, r = 11 63.5 / 63.5
    // / 64.2, r = 13 64.4 / 65.2 / 65.7, r = 16 66.9 / 67.6 / 68.1; at 800 MB: r = 5 121.8 / 120.8 / 123.7 at 6 to 8, r = 6
    // 140.9 / 124.8 / 120.3 / 122.6; at 2.2 GB: r = 9 350.8 / 340.1 / 344.2, r = 11 343.3 / 345.0 / 345.5, r = 13 333.3 /
    // 341.6 / 342.9, r = 16 337.7 / 347.4 / 350.9.  Any r, caps of 5 / 8 or 9: r = 20 240 MB 47.0 / 43.0, 300 MB 56.0 /
    // 52.3, r = 32 240 MB 47.5 / 43.9, 900 MB 148.8 / 154.6, r = 64 300 MB 58.0 / 54.6, 2.2 GB 374.5 / 377.6
    constexpr int kCapSmall[9] = {0, 11, 10, 10, 9, 8, 8, 8, 9}, kCap[9] = {0, 10, 9, 8, 7, 7, 6, 6, 5};
    const bool below = traffic < (220u << 20);
    return with_knobs(kFamFused, Shape{64, r <= 8 ? (below ? kCapSmall[r] : kCap[r]) : r <= 16 ? (r < 12 ? 5 : 4) : traffic < (300u << 20) ? 9 : 5});
}

inline Shape reorder_shape(size_t traffic, int lanes)
{
    return with_knobs(kFamReorder, traffic < (48u << 20) ? Shape{kMaxBlock, 0} : Shape{lanes, 0});
}

// Dynamic LDS that keeps the wavefronts of `sh` on a compute unit at or below its cap, at least `needed` bytes (what the
// kernel itself uses).  A workgroup's LDS is handed out in pieces of 1280 bytes (counted on the chip: 16384 bytes a
// workgroup leave room for 9, 14848 for 10), and m pieces leave room for 128 / m workgroups: 12, 14, 16, 18, 21, 25 and
// every number below, not those between.  So a workgroup asks for the fewest pieces that keep one more of them out.  A
// partial last wavefront counts as one.  Without an opt-in a workgroup gets at most 64 KiB, which leaves room for 2.
inline size_t lds_for(const Shape& sh, size_t needed = 0)
{
    constexpr size_t kPiece = 1280, kPieces = (160u << 10) / kPiece, kMost = (64u << 10) / kPiece;
    const int waves_per_wg = (sh.lanes + 63) / 64;
    if (sh.waves_per_cu <= 0 || sh.waves_per_cu / waves_per_wg >= 32) return needed;
    const size_t wgs = std::max(sh.waves_per_cu / waves_per_wg, 1);
    const size_t bytes = std::min(kPieces / (wgs + 1) + 1, kMost) * kPiece;
    return bytes > needed ? bytes : needed;
}

// Launch shape of a reduction over p buffers with `nlanes` lanes of work that is not read in shallow batches.  Measured per call on
// buffers that rotate through 1 GB, p = 1 .. 128, 16 MB .. 2.4 GB of traffic, three formats; the lines
// below lie where the best shape changes, and the shapes next to the chosen one lose 1 to 3 %.
//   - Small calls, see small_call; single-wavefront workgroups are capped at 16 here (p = 24, 2.7 M: 28.2 us,
//     uncapped 28.7).
//   - One tensor, 4 buffers and more: from 25 wavefronts per compute unit on, single-wavefront workgroups with a cap on the
//     wavefronts of a unit that falls with the buffers a lane reads: what counts is the number of request streams.  Wherever the
//     buffers lie: us, 512 lanes uncapped (gradients off 16 bytes: capped at 16) / so: bf16, p = 4, odd rows 59 MB 11.1 /
//     10.8, 179 MB 29.5 / 26.9; p = 5, odd rows 99 MB 17.3 / 16.6; p = 6, odd rows 218 MB 34.3 / 32.1; p = 8, 99 MB 16.9 /
//     16.1, odd rows 218 MB 34.3 / 32.2; p = 12, 149 MB 24.8 / 23.9, accumulator off 348 MB 54.5 / 52.1; f32, p = 5, 54 MB
//     10.0 / 9.1; p = 8, 82 MB 14.7 / 13.6, accumulator off 290 MB 46.5 / 44.8; p = 10, accumulator off 153 MB 27.3 / 25.4.
//     (17 to 25 wavefronts per unit: f32, p = 8, accumulator off 58 MB 9.8 / 10.6.)  Four two-byte buffers on their lines
//     with the accumulator off need more of them, because the partial lines between two wavefronts then meet in one
//     workgroup (bf16, 99 MB 16.8 / 17.4, 497 MB 82.4 / 82.2).  First micro-steps take more wavefronts (bf16, p = 4, 129 MB
//     caps of 14 / 16 17.0 / 16.7; p = 8, 149 MB 10 / 11 21.1 / 20.6), and fewer again from 200 per unit on (p = 8, 995 MB
//     10 / 7 135.5 / 128.2; p = 12, 2.2 GB 9 / 6 299 / 292; f32, p = 12, 1.9 GB 276 / 269.5), as do long calls that
//     accumulate (f32, p = 4, 1.1 GB 14 / 11 176.5 / 171.6; p = 6, 1.2 GB 12 / 10 184.8 / 180.7; p = 8, 1.2 GB 10 / 8 191.4
//     / 187.5).
//   - Up to 3 two-byte buffers with either off 16 bytes: 256 lanes, uncapped (p = 2,
//     67 M: 127, 512 x 16 136; accumulator 4 bytes off, 17 M: 33.3, 64 lanes 34.5).
inline int reduce_cap(int p, bool two, size_t nlanes, bool accumulate, size_t units)
{
    const size_t per_unit = nlanes / (64 * units);
    const bool many = per_unit >= (!accumulate ? 200 : two ? 1500 : 350);
    if (p < 6) return accumulate ? (many ? 11 : two ? 14 : 16) : p > 4 ? 16 : many && !two ? 14 : 0;
    if (p < 8) return accumulate ? (many ? 10 : 12) : many ? 11 : 14;
    if (p < 12) return accumulate ? (many ? 8 : 10) : many ? (two ? 7 : 9) : 11;
    if (p >= 32) return 5;                                 // long_call_in_step
    return accumulate ? (many ? 7 : 8) : many ? (two ? 6 : 7) : 10;
}
inline Shape reduce_shape(int p, int elem_bytes, size_t nlanes, bool grads16, bool acc16, bool accumulate, bool cached, size_t units)
{
    const bool two = elem_bytes == 2;
    size_t many = p < 6 ? 1600 : 1800;
    if (p < 4 || (p == 4 && two && grads16 && !acc16)) many = !acc16 ? 8000 : 3200;
    Shape sh;
    if (nlanes < units * many) {
        sh = even_call(nlanes, units, even_least(p, elem_bytes, cached));
        if (sh.lanes == 64 && p >= 6 && nlanes * 2 > (size_t)kMaxBlock * units) sh.waves_per_cu = 16;
    } else if (p >= 4) {
        sh = !two && !grads16 && p > 4 && p < 8 && nlanes >= units * 9600 ? Shape{kMaxBlock, 16} : Shape{64, reduce_cap(p, two, nlanes, accumulate, units)};
    } else if (grads16) {
        sh = Shape{two && !acc16 ? 256 : 64, 0};
    } else {
        sh = two ? Shape{256, 0} : Shape{kMaxBlock, 16};
    }
    return with_knobs(kFamReduce, sh);
}

// The same for the segments of a coalesced call, whose last tiles are partial ones: workgroups of 512 lanes that would just
// fill the compute units no longer do (16 tensors, bf16, p = 8, 49 MB 11.9 us, of 256 lanes 9.6; p = 4, 99 MB 17.6, 16.7),
// and wherever single wavefronts do not pay yet 256 lanes are faster (p = 6, 99 MB 18.1 / 17.2, f32 18.3 / 17.3).  Single
// wavefronts, us: p = 8, 279 MB caps of 9 / 12 42.7 / 41.4, f32 478 MB 73.8 / 71.1, 899 MB 141 / 135.5; p = 12, 169 MB 512
// lanes 28.8, caps of 8 / 10 / 12 27.6 / 27.6 / 27.5, f32 477 MB 8 / 9 / 10 74.0 / 73.2 / 73.0, 899 MB 137.0 / 136.2 /
// 137.1; p = 16, 169 MB 512 lanes 30.6, caps of 8 / 10 / 12 28.6 / 28.1 / 28.1, f32 478 MB 75.2 / 75.8 / 76.5. Two two-byte
// buffers take 256 lanes, capped at 16 wavefronts but in first micro-steps (318 MB 64 lanes 55.5, 256 53.2, 805 MB 122 /
// 126), up to 3 of f32 below 50 wavefronts per unit (speed of 256 lanes against 64, 200 calls, per unit in front: p = 1 to
// 25 1.10, 37 1.03, 50 .99, 75 .955, 100 .92, 300 .96; p = 2 25 1.03, 50 .98, 75 .96, 100 .96, 300 .98; p = 3 25 1.00, 50
// 1.00, 75 1.00, 100 .99, 300 .985).
inline Shape reduce_shape_segments(int p, int elem_bytes, size_t nlanes, int n, bool grads16, bool acc16, bool accumulate, bool cached, size_t units)
{
    const bool two = elem_bytes == 2;
    const size_t per_unit = nlanes / (64 * units);
    Shape sh;
    if (p >= 32 ? per_unit < 37 : p >= 12 ? per_unit < 30 : per_unit < 16) {
        sh = n > 32 ? small_call(nlanes, units) : even_call(nlanes, units, even_least(p, elem_bytes, cached), 448, (size_t)n);
        if (sh.lanes == 64 && p >= 6 && nlanes * 2 > (size_t)kMaxBlock * units) sh.waves_per_cu = 16;
    } else if (!grads16) {
        sh = p < 4 && two ? Shape{256, 0} : Shape{kMaxBlock, 16};
    } else if (p < 4) {
        const bool small = per_unit < (acc16 ? 50 : 125);
        if (two) sh = !accumulate && p == 2 && per_unit >= 650 ? Shape{64, 0} : Shape{256, !small && p > 1 && (p == 3 || accumulate) ? 16 : 0};
        else sh = Shape{per_unit < 50 ? 256 : 64, 0};
    } else if (p < 12) {
        sh = per_unit < 50 ? Shape{256, 0} : Shape{64, p < 6 ? 16 : p < 8 ? 14 : 12};
    } else {
        sh = Shape{64, p > 32 ? 5 : p == 32 ? 8 : two ? 10 : p < 16 ? 9 : 8};   // 33 and more: long_call_in_step
    }
    return with_knobs(kFamReduce, sh);
}

// Whether a reduction past the L2 reads its buffers in shallow batches (rsa_shallow): from 16 buffers on, if a compute unit gets wavefronts
// enough, as it does wherever the accumulator of up to 31 does not stay in the L2.
// us, batches of 16 / so, wavefronts per unit in front: p = 32 7 11.7 / 12.2, f32 7 11.2 / 11.4, 9 13.1 / 12.9; p = 48 5.2
// 13.2 / 13.3, 6.3 15.2 / 14.1; p = 64 5.2 16.5 / 16.3; p = 128 4.2 27.3 / 27.6, 5.2 29.5 / 29.4, 6.3 34.8 / 32.1.  At 8, one
// full-size workgroup for every unit: p = 32 12.9 / 13.9, f32 12.1 / 13.0, p = 33 14.0 / 14.4, p = 40 15.8 / 15.2; 8 elements
// more: p = 32 16.0 / 14.3.
inline bool shallow_call(int p, size_t nlanes, size_t units)
{
    if (p < 32) return p >= 16;
    return p < 40 ? nlanes > units * kMaxBlock : nlanes >= units * (p < 48 ? 512 : 352);
}

// Whether buffers lie 16 MiB (up to 63 of them also 32) from one to the next.  Four of them at a time meet in few memory
// channels, which long calls feel: us, 58 wavefronts per unit, batches of 16 with 5 wavefronts / of 4, 16 MiB: p = 32 84.2
// / 86.0, p = 48 122.5 / 140.8, f32 115.7 / 131.7, p = 64 162.9 / 167.3, f32 153.0 / 159.5, p = 96 237.1 / 244.0, p = 128
// 311.1 / 313.4; 32 MiB: p = 48 119.6 / 125.3, p = 64 155.8 / 157.3, p = 96 231.5 / 228.9; 20 MiB: p = 64 160.4 / 157.7; 48
// MiB 159.2 / 154.4; 64 MiB 158.5 / 150.9; 16 MiB, 29 per unit: p = 64 82.7 / 79.1.
inline bool in_step(const PtrTable& g, int p)
{
    constexpr ptrdiff_t kStep = 16 << 20;
    const ptrdiff_t step = (intptr_t)g.ptr[1] - (intptr_t)g.ptr[0];
    if (step != kStep && step != -kStep && (p >= 64 || (step != 2 * kStep && step != -2 * kStep))) return false;
    for (int q = 2; q < p; ++q)
        if ((intptr_t)g.ptr[q] - (intptr_t)g.ptr[q - 1] != step) return false;
    return true;
}
inline bool long_call_in_step(const PtrTable& g, int p, size_t nlanes, size_t units) { return p >= 32 && nlanes >= units * (46 * 64) && in_step(g, p); }

// The same for segments.  16 buffers stay with the unrolled kernel (us, the best cap of each, unrolled / shallow: 172 MB
// 28.4 / 29.2, 307 MB 49.4 / 49.6, f32 906 MB 138.5 / 139.0), 32 two-byte ones in long calls (453 MB 71.6 / 72.0, first
// micro-step 69.0 / 69.7; 276 MB 45.8 / 45.6); below 64 buffers it takes 12 wavefronts per unit (p = 48, odd shards 149 MB,
// 11 per unit 27.5 / 28.2; p = 64, 146 MB, 8.4 per unit 26.7 / 25.0).
inline bool shallow_segments(int p, int elem_bytes, size_t nlanes, size_t units)
{
    return p > 16 && nlanes >= units * (p < 64 ? 768 : 352) && !(p == 32 && elem_bytes == 2 && nlanes >= units * 2560);
}

// A call's wavefronts start together and read the same number of bytes, so they end together too: a compute unit goes through
// them in rounds of as many as it holds, and a last round that is half empty costs almost as much as a full one.  So the cap
// is the one that leaves the least of the last round empty, beside what a cap costs in calls of many rounds.  us, bf16, p =
// 128, 17 wavefronts per unit (585 MB), caps of 6 / 7 / 8 / 9 / 10 / 12 / 16: 89.7 / 93.7 / 101.8 / 87.8 / 90.1 / 97.9 /
// 101.9; p = 64, 20 per unit (354 MB) 60.0 / 53.5 / 56.3 / 60.1 / 54.6 / 56.2 / 57.4; p = 24, 70 per unit (511 MB) 82.8 /
// 79.3 / 75.9 / 79.3 / 79.2 / 79.7 / 78.6.  An empty round costs about 0.4 of a full one. All in one round is as good up to
// 12 per unit (p = 64, 11: 30.3, two rounds 31.3; 14: 38.9, two 37.8; odd rows, 13: 39.5, 36.5).  The workgroup for the
// ends does not count: without one, calls of exactly full rounds take as long (p = 4 to 128, 2 to 24 per unit, 130 sizes
// within .5 %).
inline Shape shallow_shape(int p, size_t nlanes, size_t units)
{
    // {waves, cost up to 19 buffers in calls of less than 46 wavefronts per unit, up to 48 otherwise, from 64 on, from 64
    // on in calls of 46 and more} Few buffers take more wavefronts in short calls: caps of 7 / 8 / 9 / 10 / 11 / 12 / 14 /
    // none, speed against 16 in flight, p = 16 to 19, 21 per unit 1.04 / 1.04 / 1.01 / .98 / 1.07 / 1.05 / 1.02 / 1.07, 24
    // .99 / 1.04 / 1.04 / 1.01 / .98 / 1.05 / 1.02 / 1.05, 34 1.04 / 1.01 / 1.05 / 1.03 / 1.02 / 1.07 / 1.03 / 1.03. Long
    // calls of many, us, caps of 6 / 7 / 8: p = 64 1.25 GB, first micro-step, 197.1 / 193.4 / 197.7, 2.1 GB 322.8 / 312.3 /
    // 307.5, 2.5 GB, first, 387.4 / 368.6 / 380.3, p = 96 1.8 GB 274.7 / 267.9 / 271.4, 2.5 GB 372.1 / 377.2 / 377.4, p =
    // 128 2.5 GB 379.1 / 378.5 / 389.7; f32, p = 64 2.5 GB 361.8 / 357.8 / 365.5.
    static constexpr struct { int waves; double cost[4]; } kCaps[] = {
        {6, {.06, .06, .02, .008}}, {7, {.045, .04, 0, 0}}, {8, {.02, 0, 0, .012}}, {9, {.015, .04, .012, .03}}, {10, {.01, .035, .025, .05}},
        {11, {0, .04, .03, .06}}, {12, {.01, .035, .035, .06}}, {14, {.005, .035, .04, .07}}, {16, {.015, .03, .04, .07}}};
    const double per_unit = (double)((nlanes + 63) / 64) / (double)units;
    const int column = p < 64 ? !(p < 20 && per_unit < 46) : per_unit < 46 ? 2 : 3;
    int best = 8;
    double least = 1e9;
    for (const auto& c : kCaps) {
        const double rounds = per_unit / c.waves;
        const double cost = rounds > 1 ? .4 * (std::ceil(rounds) / rounds - 1) + c.cost[column] : per_unit <= 12 ? .03 : .085;
        if (cost < least) least = cost, best = c.waves;
    }
    return with_knobs(kFamReduce, Shape{64, best});
}

// The same for n segments, whose partial tiles add wavefronts to an even number.  From 48 buffers on full-size workgroups
// (`full` of them for the whole call) where a unit gets one at most, and from 8 segments on where they fill two or three a
// unit evenly: speed of single wavefronts / of these against 16 loads in flight, 64 to 128 buffers, wavefronts per unit in
// front, mean and worst: 6 1.10, 1.06 / 1.19, 1.12 (bf16, p = 64, 16 tensors, 105 MB 23.2 / 18.8 us); 7 .96, .86 / 1.12,
// 1.07; 13.5 1.06, 1.02 / 1.10, 1.09; 14.5 1.05, .98 / 1.09, 1.03; 22 1.04, 1.00 / 1.06, 1.03; 23.5 .99, .96 / 1.06, 1.04;
// not filled evenly 12.5 1.05 / 1.07, 17 1.11 / 1.02, 26 1.13 / 1.04, 30 1.10 / 1.05; 2 segments, p = 128 15.4 82.3 / 88.6
// us. From 16 segments on workgroups of 256 lanes, two, three or five of which fill a unit: speed against single
// wavefronts, means of 40 to 60 calls, 9.5 to 12 per unit 1.014, 17.5 to 20 1.024.
inline Shape shallow_shape_segments(int p, size_t waves, size_t full, size_t half, int n, size_t units)
{
    // the wavefronts if all units get as many workgroups as the fullest one, by those that there are
    auto waste = [&](size_t groups, size_t of) { return (double)((groups + units - 1) / units * units * of) / (double)waves; };
    if (p >= 48 && (full <= units || (n >= 8 && full <= 3 * units && waste(full, 8) <= 1.2))) return with_knobs(kFamReduce, Shape{kMaxBlock, 0});
    if (p >= 48 && n >= 16 && half <= 5 * units && waste(half, 4) <= 1.12) return with_knobs(kFamReduce, Shape{kMaxBlock / 2, 0});
    return shallow_shape(p, 64 * waves, units);
}

}  // namespace
}  // namespace mics
