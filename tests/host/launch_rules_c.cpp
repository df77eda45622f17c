// C names for the launch rules (launch_rules.h), for tests/test_launch_rules.py.
#include "launch_rules.h"

using namespace mics;

static long long code(Shape sh) { return sh.lanes * 64 + sh.waves_per_cu; }

extern "C" {
size_t rules_lds(int lanes, int waves_per_cu, size_t needed) { return lds_for(Shape{lanes, waves_per_cu}, needed); }

// Lanes and cap of an average's (fused = 0) or an update's shape as lanes * 64 + cap, buffers on their lines.
long long rules_copies(int fused, int r, size_t count, size_t units)
{
    return code(fused ? fused_shape(r, count, true, units) : average_shape(r, count, stream_acc(count), true, units));
}
int rules_unrolled(int fused, int r, size_t count, size_t units)
{
    return fused ? unrolled_update(r, count, units) : unrolled_average(r, count, stream_acc(count), units);
}

long long rules_shallow(int p, size_t nlanes, size_t units) { return code(shallow_shape(p, nlanes, units)); }
// n equal segments of `lanes` lanes each.
long long rules_shallow_segments(int p, size_t lanes, size_t n, size_t units)
{
    return code(shallow_shape_segments(p, n * ((lanes + 63) / 64), n * ((lanes + 511) / 512), n * ((lanes + 255) / 256), (int)n, units));
}
long long rules_segments(int p, int elem_bytes, size_t nlanes, int n, int accumulate, size_t units)
{
    return code(reduce_shape_segments(p, elem_bytes, nlanes, n, true, true, accumulate, false, units));
}
int rules_in_step(const size_t* addresses, int p, size_t nlanes, size_t units)
{
    PtrTable g = {};
    for (int q = 0; q < p; ++q) g.ptr[q] = (const void*)addresses[q];
    return long_call_in_step(g, p, nlanes, units);
}
long long rules_reduce(int p, int elem_bytes, size_t nlanes, int cached, size_t units)
{
    return code(reduce_shape(p, elem_bytes, nlanes, true, true, true, cached, units));
}
int rules_partial_waves(int p) { return partial_waves(unrolled_group(p), false); }
int rules_shallow_call(int p, size_t nlanes, size_t units) { return shallow_call(p, nlanes, units); }
}
