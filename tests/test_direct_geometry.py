"""Workgroups and waves of the direct algorithm: a caller's tuner is taken at
its word, the rows of the built-in table are fitted to the rank count, and no plan
has more workgroups than a launch holds (no GPU)."""
from __future__ import annotations

import pytest

import paper_2603_11438_amd as ar


def _geometry(answer, *desc, **kw):
    ar.lib()
    ar.ar_set_tuner(lambda ctx: {"algo": ar.AR_ALGO_DIRECT, **answer})
    try:
        return ar.ar_plan_geometry(ar.make_desc(*desc, **kw))
    finally:
        ar.ar_set_tuner(None)


@pytest.mark.parametrize("unroll", (0, 1, 2))
@pytest.mark.parametrize("n,coll,count", [(16, "allreduce", 16 * 4 * 1000), (9, "reducescatter", 4096), (2, "allgather", 4096),
                                          (2, "allreduce", 99), (8, "allgather", 1 << 20)])
@pytest.mark.parametrize("parts,waves", [(4, 4), (32, 1), (7, 16)])
def test_a_tuners_answer_is_kept(parts, waves, n, coll, count, unroll):
    info = _geometry({"direct_parts": parts, "direct_nwaves": waves, "direct_unroll": unroll}, n, count, "f32", coll=coll)
    assert (info["nchannels"], info["nwaves"]) == (parts, waves)
    if n > 8:
        assert info["direct_unroll"] == 1


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("coll", ("allreduce", "reducescatter", "allgather"))
@pytest.mark.parametrize("n", range(2, 17))
def test_table_rows_at_other_rank_counts(n, coll, dtype):
    """A row's workgroups keep the grid of eight ranks, beyond 8 MiB never a
    little above a multiple of 256; more than eight ranks take four times as
    many where the row has two units per thread, as far as there is a unit for
    each; a two-rank AllGather takes twice the waves; and sums over more
    than four ranks that are no multiple of four take 1024 workgroups beyond 8
    MiB."""
    ar.lib()
    c = ar.COLLS[coll]
    a = 4 if dtype == "f32" else 8
    odd = coll != "allgather" and n in (5, 6, 7, 9, 10, 11, 13, 14, 15)
    for lg in range(8, 28):
        for size in (1 << lg, (3 << lg) // 2 // (16 * n) * 16 * n):
            row = ar.ar_tuner_raw("table", size, 8, dtype, coll=c)
            got = ar.ar_tune(size, n, dtype, coll=c)
            units = -(-(-(-(size * a // 16) // n)) // a)
            parts, waves, unroll = row["direct_parts"], row["direct_nwaves"], row["direct_unroll"]
            if parts:
                parts = max(1, (parts * 8 + n // 2) // n)
                if size > 8 << 20:
                    parts -= parts > 1 and 0 < parts * n % 256 < n
                    assert not (parts > 1 and 0 < parts * n % 256 < n)
            if odd and size > 8 << 20:
                one = coll == "allreduce" and n < 8 and size > 64 << 20
                parts, waves, unroll = 1024 // n, 1 if one else 4, 2 if one else 1
            elif n > 8 and unroll == 2:
                parts, unroll = max(parts, min(4 * parts, units)), 1
            elif coll == "allgather" and n == 2 and parts < units:
                waves *= 2
            assert (got["direct_parts"], got["direct_nwaves"], got["direct_unroll"]) == (parts, waves, unroll), size


@pytest.mark.parametrize("n,count,waves", [(8, 1001, 16), (8, 1001, 4), (16, 16 * 4 * 1000, 4), (16, 1 << 39, 9),
                                           (2, 1 << 42, 1), (11, 5, 16)])
@pytest.mark.parametrize("parts", [(1 << 28) - 1, 1 << 28, (1 << 28) + 1, 1 << 29, (1 << 31) - 1])
def test_parts_no_launch_can_hold(parts, n, count, waves):
    """A launch holds fewer than 2^32 threads.  A number of workgroups beyond
    that becomes one per unit of the segment, as far as a launch holds those;
    grid 0 is kept for plans that launch nothing."""
    info = _geometry({"direct_parts": parts, "direct_nwaves": waves}, n, count, "f32")
    units = -(-(-(-count // n)) // 4)
    split = -(-waves // 8)  # a workgroup of more than eight waves is launched as two
    threads = 64 * -(-waves // split)
    room = (((1 << 32) - 1) // threads - 1) // (split * n)
    assert info["nchannels"] == (parts if parts <= room else min(units, room))
    assert info["grid"] == info["nchannels"] * n > 0
    assert (info["grid"] * split + 1) * threads < 1 << 32


def test_no_opinion_on_other_collectives():
    """A collective that is not tabulated gets the default, at every rank count."""
    ar.lib()
    for n in (2, 5, 7, 8, 16):
        got = ar.ar_tune(64 << 20, n, "f32", coll=9)
        assert (got["direct_parts"], got["direct_nwaves"], got["direct_unroll"]) == (0, 0, 0)
        assert (got["proto_name"], got["nchannels"]) == ("simple", 16)
