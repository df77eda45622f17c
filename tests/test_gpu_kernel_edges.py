"""Edges of the kernels' tiles, lines and dispatch rules, against the oracle (bit for bit: the
contract fixes the order and the rounding of every operation)."""
import ctypes
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

mics = pytest.importorskip("paper_2205_00119_amd")
from gpu_util import Guarded  # noqa: E402

FORMATS = {"bf16": (0, np.uint16), "f16": (1, np.uint16), "f32": (2, np.float32)}


def grad_table(gen, name):
    if name == "bf16":
        return gen.normal_table(1e-3, "bf16")
    if name == "f16":
        return gen.normal_table(1e-2, "f32").astype(np.float16).view(np.uint16)
    return gen.normal_table(1e-3, "f32")


def rank_buffers(gen, name, p, n, skews, seed=4100):
    tab = grad_table(gen, name)
    host = [gen.fill_host(gen.stream_key(seed, gen.ROLE_GRAD, 0, 0, q), 0, n, tab) for q in range(p)]
    dev = [Guarded(n, FORMATS[name][1], skew=skews[q % len(skews)], fill=h) for q, h in enumerate(host)]
    return host, dev


def start_acc(gen, n, skew=0):
    ref = gen.fill_host(gen.stream_key(4101, gen.ROLE_ACC), 0, n, gen.normal_table(1e-2, "f32"))
    return ref, Guarded(n, np.float32, skew=skew, fill=ref)


def same_bits(dev, ref):
    return np.array_equal(dev.numpy().view(np.uint32), ref.view(np.uint32)) and dev.guards_intact()


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("p", [3, 16, 48, 72])
def test_reduce_at_every_position_inside_a_line(orc, gen, name, p):
    """Gradient pointers are rounded down to a line (128 bytes from 4 buffers on, else 16): the first 16 bytes'
    positions, at counts around a lane's, a wavefront's and a workgroup's elements, flat and as segments of
    one call."""
    code = FORMATS[name][0]
    for phase in range(8 if name != "f32" else 4):
        for count in (1, 6, 8, 9, 511, 513, 4099):
            host, dev = rank_buffers(gen, name, p, phase + count + 3, [0])
            for accumulate in (False, True):
                ref, acc = start_acc(gen, count, skew=phase % 3)
                mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], phase, count, accumulate, code)
                orc.reduce_scatter_accum_typed(ref, host, phase, accumulate, code)
                torch.cuda.synchronize()
                assert same_bits(acc, ref), (phase, count, accumulate)
    numels, src, dst, segs = (1, 8, 515, 7, 1030), 0, 0, []
    for i, n in enumerate(numels):
        src += i                                            # segments start at changing positions
        segs.append((n, 0, src, dst))
        src, dst = src + n, dst + n
    for skew in (0, 1, 5):
        host, dev = rank_buffers(gen, name, p, src + 2, [skew])
        ref, acc = start_acc(gen, dst, skew=1)
        mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, True, code)
        orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, True, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), skew


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("p", [1, 3, 5, 9, 15, 17, 20, 24, 31, 32, 33, 39, 40, 47, 63, 65, 71, 72, 100, 127, 128])
def test_reduce_with_every_remainder_of_the_load_batches(orc, gen, name, p):
    """Loads go out in batches; what is left of a group takes a batch of its own, padded with repeats of
    the last buffer in the one-dword kernel and in the edge elements.  Flat and as segments, whose
    kernels have 128-bit lanes at every size."""
    code = FORMATS[name][0]
    count = 1027
    host, dev = rank_buffers(gen, name, p, count + 2, [0])
    for accumulate in (False, True):
        ref, acc = start_acc(gen, count)
        mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], 1, count, accumulate, code)
        orc.reduce_scatter_accum_typed(ref, host, 1, accumulate, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), accumulate
        segs = [(515, 0, 0, 0), (512, 0, 517, 515)]
        ref, acc = start_acc(gen, count)
        mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, accumulate, code)
        orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), accumulate


@pytest.mark.parametrize("elem_bytes,p,limit,skews", [(2, 20, 24, [0]), (2, 40, 54, [0]), (4, 40, 54, [0]), (2, 64, 68, [0]),
                                                      (4, 96, 72, [0]), (2, 24, 12, [0, 1]), (4, 48, 25, [0, 1]), (2, 64, 32, [0, 3]),
                                                      (2, 100, 50, [1, 0])])
def test_reduce_on_both_sides_of_the_one_dword_rule(orc, gen, elem_bytes, p, limit, skews):
    limit <<= 20
    for count in (limit // (p * elem_bytes), limit // (p * elem_bytes) + 1):
        name = "bf16" if elem_bytes == 2 else "f32"
        host, dev = rank_buffers(gen, name, p, count, skews)
        ref, acc = start_acc(gen, count)
        mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], 0, count, True, FORMATS[name][0])
        orc.reduce_scatter_accum_typed(ref, host, 0, True, FORMATS[name][0])
        torch.cuda.synchronize()
        assert same_bits(acc, ref), count


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("p", [2, 3, 4, 8, 16, 48])
def test_reduce_at_positions_inside_a_128_byte_line(orc, gen, name, p):
    """Groups of 4 and more round their pointers down to the line: calls that end before, at and behind
    the first whole vector of the first wavefront, flat and as segments."""
    code, per_line = FORMATS[name][0], 64 if name != "f32" else 32
    for phase in (4, 8, per_line // 2, per_line - 9, per_line - 1, per_line + 5):
        for count in (1, 5, 8, 9, 63, 64, 449, 512, 1537):
            host, dev = rank_buffers(gen, name, p, phase + count + 3, [0])
            ref, acc = start_acc(gen, count, skew=phase % 5)
            mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], phase, count, True, code)
            orc.reduce_scatter_accum_typed(ref, host, phase, True, code)
            torch.cuda.synchronize()
            assert same_bits(acc, ref), (phase, count)
    segs, src, dst = [], 3, 0
    for i, n in enumerate((1, 8, 515, 70, 1030, 64, 129)):
        src += (8, 24, 1, 32, 57, 0, 13)[i]
        segs.append((n, 0, src, dst))
        src, dst = src + n, dst + n
    for skews in ([0], [8], [40], [0, 32], [16, 48]):       # the last two: 16-byte lines only
        host, dev = rank_buffers(gen, name, p, src + 2, skews)
        ref, acc = start_acc(gen, dst, skew=1)
        mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, False, code)
        orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, False, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), skews


@pytest.mark.parametrize("p,count", [(2, 530001), (2, 3200001), (8, 4000001), (6, 530001), (6, 1250003), (6, 2500000), (6, 4194311), (6, 6600001), (16, 1250001)])
@pytest.mark.parametrize("threshold", [0, 1, 1 << 40])
def test_reduce_in_every_launch_shape_and_store_kind(orc, gen, p, count, threshold):
    """Sizes on both sides of the launch rule's lines (64, 256 and 512 lanes, capped and not), with the
    accumulator on and off the 128-byte lines that decide how it is stored."""
    host, dev = rank_buffers(gen, "bf16", p, count + 9, [0])
    try:
        mics.mics_set_stream_threshold_bytes(threshold)
        for offset, skew in ((0, 0), (3, 0), (0, 5)):
            ref, acc = start_acc(gen, count, skew=skew)
            mics.mics_reduce_scatter_accum(acc.t, [d.t for d in dev], offset, count, True)
            orc.reduce_scatter_accum(ref, host, offset, True)
            torch.cuda.synchronize()
            assert same_bits(acc, ref), (offset, skew)
    finally:
        mics.mics_set_stream_threshold_bytes(0)


@pytest.mark.parametrize("name,p,count", [("bf16", 2, 17000003), ("bf16", 2, 1835011), ("bf16", 7, 3145731), ("f32", 3, 3145736), ("f16", 11, 3145729),
                                          ("bf16", 16, 2097159), ("f32", 32, 262147), ("bf16", 32, 3300001)])
def test_reduce_at_the_largest_accumulator_that_stays_in_the_l2(orc, gen, name, p, count):
    """Accumulators beyond what the caches are left with take the kernels that store whole lines, by groups; at
    the line and behind it, on and off the 128-byte lines."""
    code = FORMATS[name][0]
    host, dev = rank_buffers(gen, name, p, count + 5, [0])
    for n, offset, skew in ((count - 8, 0, 0), (count, 0, 0), (count, 5, 0), (count, 0, 3)):
        ref, acc = start_acc(gen, n, skew=skew)
        mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], offset, n, True, code)
        orc.reduce_scatter_accum_typed(ref, host, offset, True, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), (n, offset, skew)


@pytest.mark.parametrize("r,count,skew", [(2, 300001, 0), (2, 2100003, 1), (3, 9000001, 0), (1, 11000003, 0),
                                          (1, 900001, 0), (1, 2700001, 1), (8, 5600001, 32), (5, 6000002, 3), (8, 2600001, 0), (8, 3600001, 1), (8, 6000003, 0), (11, 300007, 1)])
def test_average_and_update_in_every_launch_shape_and_store_kind(orc, gen, r, count, skew):
    """Sizes on both sides of the lines of the average's and the update's launch rules and of the
    kinds of store, with a ragged end."""
    hp = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)
    scale = float(np.float32(1.0 / (r * 16)))
    tab = gen.normal_table(1e-2, "f32")
    copies_h = [gen.fill_host(gen.stream_key(4200, gen.ROLE_ACC, c), 0, count, tab) for c in range(r)]
    copies = [Guarded(count, np.float32, skew=skew, fill=h) for h in copies_h]
    grad = orc.replica_average(copies_h, scale)
    avg = Guarded(count, np.float32, skew=skew)
    mics.mics_replica_average(avg.t, [c.t for c in copies], count, scale)
    torch.cuda.synchronize()
    assert same_bits(avg, grad)
    start = [gen.fill_host(gen.stream_key(4201, gen.ROLE_MASTER), 0, count, gen.normal_table(0.02, "f32")),
             gen.fill_host(gen.stream_key(4202, gen.ROLE_MASTER), 0, count, gen.normal_table(1e-3, "f32")),
             np.abs(gen.fill_host(gen.stream_key(4203, gen.ROLE_MASTER), 0, count, gen.normal_table(1e-5, "f32")))]
    ref = [s.copy() for s in start]
    param_ref = orc.adam_shard(*ref, grad, step=3, f32=True, **hp)
    for fused in (False, True):
        dev = [Guarded(count, np.float32, skew=skew, fill=s) for s in start]
        param = Guarded(count, np.uint16, skew=skew)
        state = [d.t for d in dev] + [param.t]
        if fused:
            mics.mics_replica_average_adam_shard(*state, [c.t for c in copies], count, scale, step=3, **hp)
        else:
            mics.mics_adam_shard(*state, avg.t, count, step=3, **hp)
        torch.cuda.synchronize()
        assert all(same_bits(d, x) for d, x in zip(dev, ref)), fused
        assert np.array_equal(param.numpy(), param_ref) and param.guards_intact(), fused


@pytest.mark.parametrize("src_skew", range(8))
@pytest.mark.parametrize("eb,dst_skew", [(2, 0), (2, 3), (2, 7), (4, 0), (4, 1)])
def test_gather_at_every_shift_between_source_and_destination(orc, gen, eb, src_skew, dst_skew):
    """All byte shifts of a chunk, at chunks around a vector's, a 128-byte line's, a wavefront's and a
    tile's bytes, one tensor and several per launch."""
    dtype = np.uint16 if eb == 2 else np.uint32
    tab = gen.normal_table(1.0, "bf16") if eb == 2 else gen.normal_table(1.0, "f32").view(np.uint32)
    p, k = 4, 2
    shards_of = (1, 7, 8, 9, 63, 65, 511, 513, 1025, 2049, 4095, 8193, 16391)
    segs, src, dst_at = [], 0, 0
    for S in shards_of:
        segs.append((p * S - S // 3, S, src, dst_at))
        src, dst_at = src + p // k * S + 1, dst_at + p * S + 2
    T = [gen.fill_host(gen.stream_key(4300 + l, gen.ROLE_PARAM), 0, src, tab) for l in range(k)]
    T_dev = [Guarded(src, dtype, skew=(src_skew + l) % 8, fill=t) for l, t in enumerate(T)]
    dst = Guarded(dst_at, dtype, skew=dst_skew)
    want = dst.numpy().copy()
    mics.mics_hier_gather_reorder_coalesced(dst.t, [t.t for t in T_dev], segs, p, k, eb)
    orc.hier_gather_reorder_coalesced(T, segs, p, want)
    torch.cuda.synchronize()
    assert np.array_equal(dst.numpy(), want) and dst.guards_intact()
    for n, S, at, _ in segs:
        one = Guarded(p * S, dtype, skew=dst_skew)
        before = one.numpy().copy()
        mics.mics_hier_gather_reorder(one.t, [t.t[at:] for t in T_dev], n, S, p, k, eb)
        torch.cuda.synchronize()
        got = one.numpy()
        assert np.array_equal(got[:n], orc.hier_gather_reorder([t[at:at + p // k * S] for t in T], n, S, p)), S
        assert np.array_equal(got[n:], before[n:]) and one.guards_intact(), S


@pytest.mark.parametrize("skews", [(0, 1), (3, 0), (1, 4), (5, 5)])
def test_gather_of_a_large_unaligned_tensor(gen, skews):
    """Beyond 160 MB moved a lane holds four vectors."""
    S = 21_000_003
    bufs = [Guarded(S, np.uint16, skew=(skews[0] + l) % 8, fill=gen.fill_host(
        gen.stream_key(4400 + l, gen.ROLE_PARAM), 0, S, gen.normal_table(1.0, "bf16"))) for l in range(2)]
    dst = Guarded(2 * S, np.uint16, skew=skews[1])
    before = dst.t[2 * S - 5:].clone()
    mics.mics_hier_gather_reorder(dst.t, [b.t for b in bufs], 2 * S - 5, S, 2, 2, 2)
    torch.cuda.synchronize()
    assert torch.equal(dst.t[:S], bufs[0].t) and torch.equal(dst.t[S:2 * S - 5], bufs[1].t[:S - 5])
    assert torch.equal(dst.t[2 * S - 5:], before) and dst.guards_intact()


@pytest.mark.parametrize("dst_vecs", [0, 1, 5, 7])
@pytest.mark.parametrize("unit", [8, 24, 64])
def test_aligned_gather_off_the_128_byte_lines(orc, gen, dst_vecs, unit):
    """16-byte aligned geometry: wavefronts begin on 128-byte lines of the destination, at every
    position of a chunk in its line; with ragged ends around a tile's last vector."""
    p, k = 6, 3
    skew = 8 * dst_vecs
    segs, src, dst_at = [], 0, 0
    for i, vecs in enumerate((1, 2, 31, 64, 127, 128, 129, 255, 256, 257, 1025)):
        S = vecs * unit
        n = p * S - (0, 1, 7, 8, S // 2, 8 * 8 + 3, S + 5)[i % 7]
        segs.append((max(n, 1), S, src, dst_at))
        src, dst_at = src + p // k * S, dst_at + p * S
    T = [gen.fill_host(gen.stream_key(4500 + l, gen.ROLE_PARAM), 0, src, gen.normal_table(1.0, "bf16")) for l in range(k)]
    T_dev = [Guarded(src, np.uint16, skew=8 * l, fill=t) for l, t in enumerate(T)]
    dst = Guarded(dst_at, np.uint16, skew=skew)
    want = dst.numpy().copy()
    mics.mics_hier_gather_reorder_coalesced(dst.t, [t.t for t in T_dev], segs, p, k, 2)
    orc.hier_gather_reorder_coalesced(T, segs, p, want)
    torch.cuda.synchronize()
    assert np.array_equal(dst.numpy(), want) and dst.guards_intact()
    for n, S, at, _ in segs:
        one = Guarded(p * S, np.uint16, skew=skew)
        before = one.numpy().copy()
        mics.mics_hier_gather_reorder(one.t, [t.t[at:] for t in T_dev], n, S, p, k, 2)
        torch.cuda.synchronize()
        got = one.numpy()
        assert np.array_equal(got[:n], orc.hier_gather_reorder([t[at:at + p // k * S] for t in T], n, S, p)), S
        assert np.array_equal(got[n:], before[n:]) and one.guards_intact(), S


@pytest.mark.parametrize("p,k,eb,sizes", [
    (4, 2, 2, [3, 1, 17, 40, 130]), (128, 128, 2, [191, 127, 900, 70000, 33]), (96, 48, 4, [95, 4097, 130000]),
    (6, 3, 2, [5] * 64), (24, 8, 2, list(range(1, 700, 11))), (12, 4, 4, list(range(7, 20000, 199))),
    (48, 8, 2, [3_000_017, 1_500_001, 12_345]), (2, 2, 2, [100_003] * 70), (8, 8, 2, [9_000_000, 2_000_001])])
@pytest.mark.parametrize("align,skew", [(1, 0), (1, 3), (8, 0), (8, 5)])
@pytest.mark.parametrize("cap", [0, 4096])
def test_gather_of_small_tensors(orc, gen, p, k, eb, sizes, align, skew, cap):
    """Small calls find the chunk of every 16 bytes by a reciprocal: chunks from one element to megabytes, more tensors
    than a wavefront has lanes and than a launch carries, more stage-1 buffers than 16 and than 64, one and two
    vectors per lane.  A capped grid takes the kernels of larger calls."""
    dtype = np.uint16 if eb == 2 else np.uint32
    tab = gen.normal_table(1.0, "bf16") if eb == 2 else gen.normal_table(1.0, "f32").view(np.uint32)
    segs, src, dst_at = [], 0, 0
    for n in sizes:
        S = -(-(-(-n // p)) // align) * align
        segs.append((n, S, src, dst_at))
        src, dst_at = src + p // k * S, dst_at + n
    T = [gen.fill_host(gen.stream_key(4600 + l, gen.ROLE_PARAM), 0, src, tab) for l in range(k)]
    T_dev = [Guarded(src, dtype, skew=skew, fill=t) for t in T]
    dst = Guarded(dst_at, dtype, skew=skew)
    want = dst.numpy().copy()
    orc.hier_gather_reorder_coalesced(T, segs, p, want)
    try:
        mics.mics_set_blocks_per_cu(cap)
        mics.mics_hier_gather_reorder_coalesced(dst.t, [t.t for t in T_dev], segs, p, k, eb)
        torch.cuda.synchronize()
        assert np.array_equal(dst.numpy(), want) and dst.guards_intact()
        for n, S, at, _ in (segs[0], segs[-1]):
            one = Guarded(n, dtype, skew=skew)
            mics.mics_hier_gather_reorder(one.t, [t.t[at:] for t in T_dev], n, S, p, k, eb)
            torch.cuda.synchronize()
            assert np.array_equal(one.numpy(), orc.hier_gather_reorder([t[at:at + p // k * S] for t in T], n, S, p)), n
            assert one.guards_intact()
    finally:
        mics.mics_set_blocks_per_cu(0)


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("p", [1, 3, 4, 8, 12, 24, 32, 48, 100])
@pytest.mark.parametrize("n_segs,threshold", [(64, 0), (65, 0), (150, 0), (70, 1)])
def test_reduce_of_many_small_segments(orc, gen, name, p, n_segs, threshold):
    """More segments than a wavefront has lanes and than a launch carries, down to one element, at changing positions
    inside a lane's elements; with a threshold, through the kernels of large accumulators."""
    code = FORMATS[name][0]
    segs, src, dst = [], 1, 0
    for t in range(n_segs):
        n = (1, 2, 7, 8, 9, 63, 130, 600)[t % 8]
        src += t % 5
        segs.append((n, 0, src, dst))
        src, dst = src + n, dst + n
    host, dev = rank_buffers(gen, name, p, src + 3, [0])
    try:
        mics.mics_set_stream_threshold_bytes(threshold)
        for accumulate in (False, True):
            ref, acc = start_acc(gen, dst, skew=1)
            mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, accumulate, code)
            orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
            torch.cuda.synchronize()
            assert same_bits(acc, ref), accumulate
    finally:
        mics.mics_set_stream_threshold_bytes(0)


@pytest.mark.parametrize("p,k,n_tensors", [(2, 2, 2), (4, 4, 47), (16, 8, 48), (8, 8, 49), (6, 3, 96), (16, 8, 97), (64, 8, 96)])
@pytest.mark.parametrize("kinds", ["aligned", "mixed", "odd"])
def test_gather_of_tensors_of_two_kinds(orc, gen, p, k, n_tensors, kinds):
    """Larger coalesced calls: 16-byte aligned tensors and others share a launch; the numbers of tensors around those of
    the two tables.  Every other tensor is small, the first is too large for the kernel of small calls."""
    segs, src, dst_at, align = [], 0, 0, 8 if kinds != "odd" else 1
    for t in range(n_tensors):
        n = 14_200_000 if t == 0 else (130_024 if t % 2 else 24 + 8 * t)
        if kinds == "odd" or (kinds == "mixed" and t % 3 == 2):
            n += 3
        S = -(-(-(-n // p)) // align) * align
        segs.append((n, S, src, dst_at))
        src, dst_at = src + p // k * S, dst_at + (-(-n // 8) * 8 if kinds == "aligned" else n + t % 2)
    tab = gen.normal_table(1.0, "bf16")
    T = [gen.fill_host(gen.stream_key(4700 + l, gen.ROLE_PARAM), 0, src, tab) for l in range(k)]
    T_dev = [Guarded(src, np.uint16, fill=t) for t in T]
    dst = Guarded(dst_at, np.uint16)
    want = dst.numpy().copy()
    orc.hier_gather_reorder_coalesced(T, segs, p, want)
    mics.mics_hier_gather_reorder_coalesced(dst.t, [t.t for t in T_dev], segs, p, k, 2)
    torch.cuda.synchronize()
    assert np.array_equal(dst.numpy(), want) and dst.guards_intact()


@pytest.mark.parametrize("name,p,count", [
    ("bf16", 2, 66_003), ("f32", 3, 40_001), ("f16", 6, 131_077), ("bf16", 8, 2_700_011), ("f16", 16, 560_003), ("f32", 5, 1_000_003),
    ("bf16", 24, 1_600_007), ("f32", 32, 70_001), ("f32", 32, 300_017), ("f16", 32, 300_017)])
@pytest.mark.parametrize("skews", [[0], [0, 8, 16], [3, 0, 5]])
def test_reduce_in_runs_of_tiles(orc, gen, name, p, count, skews):
    """Calls of more than a round of workgroups, whose tiles are dealt to the XCDs in runs: buffers at one position and at
    several inside their lines, vectors on the gradients' lines and on the accumulator's; the last round is partial."""
    code = FORMATS[name][0]
    host, dev = rank_buffers(gen, name, p, count + 40, skews)
    for offset, acc_skew in ((0, 0), (24, 0), (24, 8), (5, 1)):
        for accumulate in (False, True):
            ref, acc = start_acc(gen, count, skew=acc_skew)
            mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], offset, count, accumulate, code)
            orc.reduce_scatter_accum_typed(ref, host, offset, accumulate, code)
            torch.cuda.synchronize()
            assert same_bits(acc, ref), (offset, acc_skew, accumulate)


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("p", [2, 4, 16, 24, 32])
@pytest.mark.parametrize("threshold", [0, 1])
def test_reduce_segments_in_runs_of_tiles(orc, gen, name, p, threshold):
    """Segments whose vectors lie on the accumulator's lines where the gradients then are on 16 bytes, the first of them
    at the very start of the buffers, others where they are not; more than a round of workgroups."""
    code = FORMATS[name][0]
    segs, src, dst = [], 0, 24
    for n, gap in ((60_000, 0), (8, 8), (33_000, 24), (4_097, 1), (50_003, 3), (640, 16)):
        src += gap
        segs.append((n, 0, src, dst))
        src, dst = src + n, dst + n
    host, dev = rank_buffers(gen, name, p, src, [0])
    try:
        mics.mics_set_stream_threshold_bytes(threshold)
        for accumulate in (False, True):
            ref, acc = start_acc(gen, dst)
            mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, accumulate, code)
            orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
            torch.cuda.synchronize()
            assert same_bits(acc, ref), accumulate
    finally:
        mics.mics_set_stream_threshold_bytes(0)


def kernels_of(call):
    """Kernel launches of a call, from its capture (never replayed)."""
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    graph, side = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        call()
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("n_segs", [1, 64, 65, 96, 97, 128, 129, 192, 193])
@pytest.mark.parametrize("numel,per_launch", [(64, 96), (100_000, 64)])
def test_launches_of_coalesced_reductions(n_segs, numel, per_launch):
    """64 tensors in a launch, 96 in small calls (accumulators up to 12 MiB); the last launch takes what is left."""
    segs = [(numel, 0, t * numel, t * numel) for t in range(n_segs)]
    grads = [torch.zeros(n_segs * numel, dtype=torch.int16, device="cuda:0") for _ in range(4)]
    acc = torch.zeros(n_segs * numel, device="cuda:0")
    assert kernels_of(lambda: mics.mics_reduce_scatter_accum_coalesced(acc, grads, segs, True)) == -(-n_segs // per_launch)


@pytest.mark.parametrize("n_tensors,shard,launches", [(16, 64, 1), (96, 64, 1), (97, 64, 2), (60, 500_000, 1), (60, 1_500_000, 2), (2, 64, 1)])
@pytest.mark.parametrize("odd", [0, 1, 2])
def test_launches_of_coalesced_gathers(n_tensors, shard, launches, odd):
    """96 tensors in a launch and 48 from 640 MiB moved on, aligned, not aligned, or both in turn."""
    segs, src, dst_at = [], 0, 0
    for t in range(n_tensors):
        S = shard + (t % 2 if odd == 2 else odd)
        segs.append((2 * S, S, src, dst_at))
        src, dst_at = src + S, dst_at + 2 * S
    T = [torch.zeros(src, dtype=torch.int16, device="cuda:0") for _ in range(2)]
    dst = torch.zeros(dst_at, dtype=torch.int16, device="cuda:0")
    assert kernels_of(lambda: mics.mics_hier_gather_reorder_coalesced(dst, T, segs, 2, 2, 2)) == launches


@pytest.mark.parametrize("name,count", [("f32", 262_147), ("f32", 524_281), ("f32", 524_293), ("f32", 794_377), ("f16", 794_377), ("f16", 1_048_561), ("f16", 1_048_585),
                                        ("bf16", 400_003), ("bf16", 1_048_561), ("bf16", 1_048_585)])
def test_reduce_of_32_buffers_on_both_sides_of_the_shallow_batches(orc, gen, name, count):
    """The window of 6 loads in flight (bf16: two batches of 16) and, from 8 wavefronts per compute unit on, batches of 4; the accumulator on the lanes' lines and off them."""
    code = FORMATS[name][0]
    host, dev = rank_buffers(gen, name, 32, count + 8, [0])
    for offset, skew in ((0, 0), (5, 3)):
        for accumulate in (False, True):
            ref, acc = start_acc(gen, count, skew=skew)
            mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], offset, count, accumulate, code)
            orc.reduce_scatter_accum_typed(ref, host, offset, accumulate, code)
            torch.cuda.synchronize()
            assert same_bits(acc, ref), (offset, skew, accumulate)


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("p", [2, 3, 4, 5, 6, 7, 8, 12, 16, 32])
@pytest.mark.parametrize("skews", [[0, 8, 16], [3, 0, 5]])
def test_small_accumulators_in_runs_of_tiles(orc, gen, name, p, skews):
    """Just above and below the 12 MiB moved from which calls with gradients off their lines are dealt out in runs; the accumulator
    is small enough to stay in the L2 up to 16 buffers.  (32: held loads as well, see the next test.)"""
    code, dtype = FORMATS[name]
    per_element = p * np.dtype(dtype).itemsize + 8
    above = -(-(12 << 20) // per_element) + 5
    host, dev = rank_buffers(gen, name, p, above + 40, skews)
    for count in (above - 5000, above):
        for offset, acc_skew in ((0, 0), (24, 8), (5, 1)):
            for accumulate in (False, True):
                ref, acc = start_acc(gen, count, skew=acc_skew)
                mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], offset, count, accumulate, code)
                orc.reduce_scatter_accum_typed(ref, host, offset, accumulate, code)
                torch.cuda.synchronize()
                assert same_bits(acc, ref), (count, offset, acc_skew, accumulate)


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("count", [150_001, 196_608, 196_609, 230_003, 262_144, 262_145])
@pytest.mark.parametrize("skews", [[0], [0, 8, 16], [3, 0, 5]])
def test_reduce_of_32_buffers_into_a_small_accumulator(orc, gen, name, count, skews):
    """Between the calls that take one dword per lane (two-byte buffers at different positions: up to 196608 elements) and the
    accumulators that do not stay in the L2 (from 262145 on): the loads of a window of 16, held."""
    code = FORMATS[name][0]
    host, dev = rank_buffers(gen, name, 32, count + 24, skews)
    for accumulate in (False, True):
        ref, acc = start_acc(gen, count)
        mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], 8, count, accumulate, code)
        orc.reduce_scatter_accum_typed(ref, host, 8, accumulate, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), accumulate


@pytest.mark.parametrize("name", list(FORMATS))
@pytest.mark.parametrize("p", [2, 5, 6, 7, 16])
@pytest.mark.parametrize("n_segs", [65, 96, 97])
def test_reduce_of_up_to_96_segments_unrolled(orc, gen, name, p, n_segs):
    """The unrolled kernels that the any-p ones and those of 1, 3, 4, 8 and 32 buffers above leave out."""
    code = FORMATS[name][0]
    segs, src, dst = [], 3, 0
    for t in range(n_segs):
        n = (1, 2, 7, 8, 9, 63, 130, 2_000)[(t + 1) % 8]
        src += t % 5
        segs.append((n, 0, src, dst))
        src, dst = src + n, dst + n
    host, dev = rank_buffers(gen, name, p, src + 3, [0])
    for accumulate in (False, True):
        ref, acc = start_acc(gen, dst, skew=1)
        mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, accumulate, code)
        orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), accumulate


@pytest.mark.parametrize("name,p,mb", [("bf16", 20, 14), ("f16", 32, 12), ("f16", 32, 24), ("f32", 40, 24), ("bf16", 48, 31), ("bf16", 40, 54), ("f32", 96, 50)])
@pytest.mark.parametrize("n_segs", [5, 20, 21, 70])
def test_segments_around_the_limit_of_one_dword_per_lane(orc, gen, name, p, mb, n_segs):
    """MiB of gradients up to which a lane takes one dword of each buffer, for few and for many segments: both sides of each limit,
    ends anywhere, the segments of unequal sizes."""
    code, dtype = FORMATS[name]
    limit = (mb << 20) // (p * np.dtype(dtype).itemsize)
    small = [3 + t % 40 for t in range(n_segs - 1)]
    for total in (limit, limit + 1):
        segs, src, dst = [], 0, 0
        for n in (*small, total - sum(small)):
            segs.append((n, 0, src, dst))
            src, dst = src + n + 1, dst + n
        host, dev = rank_buffers(gen, name, p, src, [0])
        for accumulate in (False, True):
            ref, acc = start_acc(gen, dst, skew=1)
            mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, accumulate, code)
            orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
            torch.cuda.synchronize()
            assert same_bits(acc, ref), (total, accumulate)


@pytest.mark.parametrize("p,k", [(4, 4), (64, 8)])
@pytest.mark.parametrize("n_tensors,mb", [(1, 27), (2, 18), (15, 18), (16, 24), (16, 36), (49, 24), (49, 52)])
@pytest.mark.parametrize("odd", [0, 1])
def test_gather_on_both_sides_of_the_small_calls(orc, gen, p, k, n_tensors, mb, odd):
    """MiB moved up to which a gather finds the chunk of every 16 bytes, by the number of tensors, aligned or not: the last ones
    below each limit and the first above it."""
    for total in ((mb << 20) // 4 - 8 * n_tensors, (mb << 20) // 4 + 8 * p * n_tensors):
        each = total // n_tensors // (8 * p) * (8 * p) + odd
        segs, src, dst_at = [], 0, 0
        for n in (*[each] * (n_tensors - 1), total - each * (n_tensors - 1) | odd):
            S = -(-n // p) if odd else -(-n // (8 * p)) * 8
            segs.append((n, S, src, dst_at))
            src, dst_at = src + p // k * S, dst_at + n
        tab = gen.normal_table(1.0, "bf16")
        T = [gen.fill_host(gen.stream_key(4800 + l, gen.ROLE_PARAM), 0, src, tab) for l in range(k)]
        T_dev = [Guarded(src, np.uint16, fill=t) for t in T]
        dst = Guarded(dst_at, np.uint16)
        want = dst.numpy().copy()
        orc.hier_gather_reorder_coalesced(T, segs, p, want)
        mics.mics_hier_gather_reorder_coalesced(dst.t, [t.t for t in T_dev], segs, p, k, 2)
        torch.cuda.synchronize()
        assert np.array_equal(dst.numpy(), want) and dst.guards_intact(), total


@pytest.mark.parametrize("name,p,count", [
    ("bf16", 16, 5_003), ("f16", 16, 2_097_153), ("f32", 17, 3_001), ("bf16", 18, 2_100_011), ("f16", 19, 1_033), ("f32", 24, 70_001), ("bf16", 31, 20_011),
    ("bf16", 32, 1_048_513), ("bf16", 32, 1_048_577), ("f32", 33, 524_289), ("bf16", 47, 1_048_577), ("bf16", 48, 720_961), ("f16", 50, 720_897),
    ("f32", 67, 360_449), ("f16", 127, 720_905), ("bf16", 128, 720_897)])
def test_reduce_in_shallow_batches(orc, gen, name, p, count):
    """Every remainder of the batches of 4, the largest group, and both sides of the number of wavefronts from which they are taken
    (up to 31 buffers: any number, where the accumulator passes the L2); gradients on one line, on several and odd, accumulator off."""
    code = FORMATS[name][0]
    for skews, acc_skew in (([0], 0), ([5], 3), ([0, 8], 1), ([3, 0, 6], 0)):
        host, dev = rank_buffers(gen, name, p, count + 6, skews)
        for threshold, offset, accumulate in ((1, 0, True), (0, 6, False)):
            try:
                mics.mics_set_stream_threshold_bytes(threshold)
                ref, acc = start_acc(gen, count, skew=acc_skew)
                mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], offset, count, accumulate, code)
                orc.reduce_scatter_accum_typed(ref, host, offset, accumulate, code)
                torch.cuda.synchronize()
                assert same_bits(acc, ref), (skews, acc_skew, accumulate)
            finally:
                mics.mics_set_stream_threshold_bytes(0)


@pytest.mark.parametrize("name,p,numel", [
    ("bf16", 17, 1_600_003), ("f32", 24, 800_011), ("f16", 32, 1_600_009), ("bf16", 33, 1_580_001), ("f32", 48, 790_003), ("bf16", 64, 725_005),
    ("f16", 96, 730_001), ("f32", 128, 362_003), ("bf16", 12, 2_100_003), ("f16", 40, 300_007),
    ("bf16", 64, 900_003), ("f32", 48, 983_003), ("f16", 49, 1_990_003), ("f32", 128, 458_003)])
@pytest.mark.parametrize("threshold", [0, 1])
def test_reduce_segments_in_shallow_batches(orc, gen, name, p, numel, threshold):
    """Segments that are read in batches of 4, by single wavefronts, full-size workgroups and those of 256 lanes, and any-p ones that are not: their ends in workgroups of their own, a segment shorter than
    a lane's vector and one without ends among them."""
    code = FORMATS[name][0]
    segs, src, dst = [], 3, 0
    for n in (5, numel - 90_000, 64, 40_001, 50_017, 1):
        segs.append((n, 0, src, dst))
        src, dst = src + n + 2, dst + n
    segs.append((4096, 0, -(-src // 64) * 64, dst))
    src, dst = -(-src // 64) * 64 + 4096, dst + 4096
    host, dev = rank_buffers(gen, name, p, src, [0])
    try:
        mics.mics_set_stream_threshold_bytes(threshold)
        for accumulate in (False, True):
            ref, acc = start_acc(gen, dst, skew=threshold)
            mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, accumulate, code)
            orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
            torch.cuda.synchronize()
            assert same_bits(acc, ref), accumulate
    finally:
        mics.mics_set_stream_threshold_bytes(0)


@pytest.mark.parametrize("name,p,step,ends", [("bf16", 33, 16, 3), ("f32", 32, -16, 1), ("f16", 48, -32, 5), ("bf16", 64, 16, 0)])
@pytest.mark.parametrize("segments", [False, True])
def test_reduce_of_buffers_in_step(orc, gen, name, p, step, ends, segments):
    """Long calls over buffers 16 and 32 MiB from one another, upwards and downwards, which are read in batches of 16."""
    code, dtype = FORMATS[name]
    units = torch.cuda.get_device_properties(0).multi_processor_count
    size = np.dtype(dtype).itemsize
    count, pitch = 46 * 64 * units * 16 // size + 8 * 17 + ends, abs(step) * 2**20 // size
    if count + 64 > pitch:
        pytest.skip("a call of this length does not fit between the buffers")
    whole = torch.empty(p * pitch, dtype=torch.float32 if name == "f32" else torch.int16, device="cuda:0")
    host, tab = [], grad_table(gen, name)
    for q in range(p):
        host.append(gen.fill_host(gen.stream_key(4400, gen.ROLE_GRAD, 0, 0, q), 0, count + 8, tab))
    views = [whole[q * pitch:q * pitch + count + 8] for q in (range(p) if step > 0 else reversed(range(p)))]
    for v, h in zip(views, host):
        v.copy_(torch.from_numpy(h if name == "f32" else h.view(np.int16)))
    segs = [(count // 3 + 1, 0, 2, 0), (count - count // 3 - 1, 0, count // 3 + 5, count // 3 + 1)]
    for accumulate in (True, False):
        ref, acc = start_acc(gen, count)
        if segments:
            mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, views, segs, accumulate, code)
            orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
        else:
            mics.mics_reduce_scatter_accum_typed(acc.t, views, 1, count, accumulate, code)
            orc.reduce_scatter_accum_typed(ref, host, 1, accumulate, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), accumulate


@pytest.mark.parametrize("name,p,per_unit", [("bf16", 64, 5.7), ("f16", 49, 12.6), ("f32", 48, 14.9), ("bf16", 50, 11.5), ("f32", 66, 11.7), ("f16", 48, 19.2)])
def test_reduce_many_segments_in_shallow_batches(orc, gen, name, p, per_unit):
    """17 segments by workgroups of 512 and 256 lanes and by single wavefronts, most of them with a partial last tile."""
    code, dtype = FORMATS[name]
    units = torch.cuda.get_device_properties(0).multi_processor_count
    each = int(per_unit * 64 * units) * (16 // np.dtype(dtype).itemsize) // 17
    segs, src, dst = [], 1, 0
    for t in range(17):
        n = each + (t - 8) * 333
        segs.append((n, 0, src, dst))
        src, dst = src + n + t % 3, dst + n
    host, dev = rank_buffers(gen, name, p, src, [0])
    for accumulate in (True, False):
        ref, acc = start_acc(gen, dst)
        mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, accumulate, code)
        orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
        torch.cuda.synchronize()
        assert same_bits(acc, ref), accumulate


@pytest.mark.parametrize("name,p,per_unit", [
    ("bf16", 4, 4.1), ("f16", 8, 5.2), ("f32", 12, 6.9), ("bf16", 16, 2.1), ("f32", 24, 3.0), ("bf16", 24, 6.3), ("f16", 32, 2.3), ("bf16", 32, 5.4),
    ("f32", 33, 4.7), ("bf16", 48, 5.1), ("f16", 72, 4.4), ("f32", 128, 2.6)])
@pytest.mark.parametrize("tensors", [0, 3, 16, 31, 33])
def test_reduce_in_one_even_workgroup_per_unit(orc, gen, name, p, per_unit, tensors):
    """Workgroups of a multiple of 8 lanes whose last wavefront is a partial one: as one tensor, and as segments, of which that wavefront
    has to find its own; accumulators in the L2 and past it, gradients on and off their lines."""
    code, dtype = FORMATS[name]
    units = torch.cuda.get_device_properties(0).multi_processor_count
    total = int(per_unit * 64 * units) * (16 // np.dtype(dtype).itemsize) + 3
    segs, src, dst = [], 0, 0
    for t in range(tensors):
        n = 17 + 900 * (t % 5) if t else total - sum(17 + 900 * (i % 5) for i in range(1, tensors))
        segs.append((n, 0, src, dst))
        src, dst = src + n + t % 3, dst + n
    for skews, threshold in (([0], 0), ([5], 1), ([3, 0, 8], 1)):
        host, dev = rank_buffers(gen, name, p, (src if tensors else total) + 1, skews)
        try:
            mics.mics_set_stream_threshold_bytes(threshold)
            for accumulate in (True, False):
                ref, acc = start_acc(gen, dst if tensors else total)
                if tensors:
                    mics.mics_reduce_scatter_accum_coalesced_typed(acc.t, [d.t for d in dev], segs, accumulate, code)
                    orc.reduce_scatter_accum_coalesced_typed(ref, host, segs, accumulate, code)
                else:
                    mics.mics_reduce_scatter_accum_typed(acc.t, [d.t for d in dev], 1, total, accumulate, code)
                    orc.reduce_scatter_accum_typed(ref, host, 1, accumulate, code)
                torch.cuda.synchronize()
                assert same_bits(acc, ref), (skews, accumulate)
        finally:
            mics.mics_set_stream_threshold_bytes(0)


@pytest.mark.parametrize("r,count", [
    (3, 5), (3, 331_127), (3, 331_131), (3, 2_097_149), (3, 2_097_155), (5, 1_733_000), (5, 1_733_001), (6, 77_003), (6, 1_600_003), (6, 524_288), (7, 524_289), (12, 524_285), (7, 1_500_001), (7, 260_003), (7, 1_610_003), (8, 1_500_003),
    (5, 262_147), (5, 300_003), (7, 393_216), (7, 393_221), (11, 393_216), (11, 393_221),
    (9, 1_048_579), (9, 140_003), (9, 419_431), (9, 5_242_883), (10, 262_147), (11, 300_003), (13, 349_531), (13, 3_744_923), (14, 280_003), (15, 4_191), (16, 246_727),
    (17, 1_783_003), (24, 700_001), (12, 510_103), (12, 510_104), (12, 1_416_993), (13, 40_001), (16, 420_003), (16, 1_515_002)])
@pytest.mark.parametrize("skew", [0, 1])
def test_average_and_update_of_numbers_of_copies(orc, gen, r, count, skew):
    """Numbers of copies that have kernels of their own, for both ends of the range in updates, and ones that have none: both sides of
    the lines between them and between full-size workgroups, even ones and single wavefronts."""
    test_average_and_update_in_every_launch_shape_and_store_kind(orc, gen, r, count, skew)


@pytest.mark.parametrize("p,k,n_tensors,mb", [(8, 4, 20, 17), (32, 8, 17, 18), (64, 8, 60, 20), (96, 8, 24, 27), (128, 8, 25, 34), (32, 8, 40, 44), (8, 8, 16, 44), (128, 8, 12, 30)])
@pytest.mark.parametrize("odd", [0, 1])
def test_gather_of_small_chunks(orc, gen, p, k, n_tensors, mb, odd):
    """Both sides of the sizes from which several tensors go by chunks, and chunks that fill full-size workgroups' tiles and that do not."""
    test_gather_on_both_sides_of_the_small_calls(orc, gen, p, k, n_tensors, mb, odd)
