"""Workgroups of the direct algorithm for more than eight ranks, where two
units per thread become four times the workgroups (no GPU)."""
from __future__ import annotations

import pytest

import paper_2603_11438_amd as ar


@pytest.mark.parametrize("parts,count,want", [
    (4, 16 * 4 * 1000, 16),        # four times, with units for all of them
    (4, 16 * 4 * 9, 9),            # as far as there is a unit for each
    (32, 16 * 4 * 9, 32),          # the tuner's own number is not lowered
])
def test_parts_beyond_eight_ranks(parts, count, want):
    ar.lib()
    ar.ar_set_tuner(lambda ctx: {"algo": ar.AR_ALGO_DIRECT, "direct_parts": parts, "direct_unroll": 2})
    try:
        info = ar.ar_plan_geometry(ar.make_desc(16, count, "f32"))
    finally:
        ar.ar_set_tuner(None)
    assert info["nchannels"] == want and info["direct_unroll"] == 1


@pytest.mark.parametrize("n,count,waves", [(8, 1001, 16), (8, 1001, 4), (16, 16 * 4 * 1000, 4), (16, 1 << 39, 9),
                                           (2, 1 << 42, 1), (11, 5, 16)])
@pytest.mark.parametrize("parts", [(1 << 28) - 1, 1 << 28, (1 << 28) + 1, 1 << 29, (1 << 31) - 1])
def test_parts_no_launch_can_hold(parts, n, count, waves):
    """A launch holds fewer than 2^32 threads.  A number of workgroups beyond
    that becomes one per unit of the segment, as far as a launch holds those;
    grid 0 is kept for plans that launch nothing."""
    ar.lib()
    ar.ar_set_tuner(lambda ctx: {"algo": ar.AR_ALGO_DIRECT, "direct_parts": parts, "direct_nwaves": waves})
    try:
        info = ar.ar_plan_geometry(ar.make_desc(n, count, "f32"))
    finally:
        ar.ar_set_tuner(None)
    units = -(-(-(-count // n)) // 4)
    split = -(-waves // 8)  # a workgroup of more than eight waves is launched as two
    threads = 64 * -(-waves // split)
    room = (((1 << 32) - 1) // threads - 1) // (split * n)
    assert info["nchannels"] == (parts if parts <= room else min(units, room))
    assert info["grid"] == info["nchannels"] * n > 0
    assert (info["grid"] * split + 1) * threads < 1 << 32
