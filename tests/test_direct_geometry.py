"""Workgroups of the direct algorithm for more than eight ranks, where two
units per thread become four times the workgroups (no GPU)."""
from __future__ import annotations

import pytest

import paper_2603_11438_amd as ar


@pytest.mark.parametrize("parts,count,want", [
    (4, 16 * 4 * 1000, 16),        # four times, with units for all of them
    (4, 16 * 4 * 9, 9),            # as far as there is a unit for each
    (32, 16 * 4 * 9, 32),          # the tuner's own number is never lowered
    (1 << 29, 16 * 4 * 1000, 1 << 29),
])
def test_parts_beyond_eight_ranks(parts, count, want):
    ar.lib()
    ar.ar_set_tuner(lambda ctx: {"algo": ar.AR_ALGO_DIRECT, "direct_parts": parts, "direct_unroll": 2})
    try:
        info = ar.ar_plan_geometry(ar.make_desc(16, count, "f32"))
    finally:
        ar.ar_set_tuner(None)
    assert info["nchannels"] == want and info["direct_unroll"] == 1
