"""The direct algorithm where its geometry can go wrong: every rank count's
own kernel, one and several iterations per thread, workgroups launched as two,
the partial unit's own workgroup; against the oracle, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import ring_oracle as ro
from tests.gpu_helpers import draw, oracle_bits, run_case, say, to_bits, to_device

pytestmark = pytest.mark.gpu

CFGS = [dict(nchannels=1, nwaves=1, direct_unroll=1), dict(nchannels=1, nwaves=1, direct_unroll=2),
        dict(nchannels=2, nwaves=9), dict(nchannels=3, nwaves=2)]


@pytest.fixture(scope="module")
def ar():
    import torch

    import paper_2603_11438_amd as ar

    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    ar.lib()
    ar.ar_set_tuner(None)
    return ar


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("n", range(2, 17))
def test_allreduce(ar, n, dtype):
    """Segments that end in a partial unit, one unit short of, at and one past
    what one wave covers in an iteration (64 lanes, 1 to 8 units), and after
    several iterations; and data smaller than one unit."""
    a = 4 if dtype == "f32" else 8
    counts = [1, a - 1, n * a + 1, n * 64 * a - 1, n * 64 * a + n * a, n * 64 * 8 * a + 3, n * 64 * 19 * a - a - 2]
    for i, count in enumerate(counts):
        x = draw(n, count, dtype, "normal", seed=700 + 13 * n + i)
        for cfg in (CFGS[i % 4], CFGS[(i + 1) % 4]):
            run_case(ar, x, dtype, f"direct-{n}-{dtype}-{count}", algo="direct", **cfg)


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("n", (2, 3, 4, 7, 8, 9, 16))
def test_blocks(ar, n, dtype):
    import torch

    a = 4 if dtype == "f32" else 8
    for i, count in enumerate((a, 64 * a, 65 * a, 64 * 8 * a + a, 64 * 21 * a)):
        cfg = CFGS[i % 4]
        x = draw(n, n * count, dtype, "normal", seed=n + count)
        send = to_device(x, dtype)
        want = ro.reduce_scatter(x, dtype)
        want = want.view(np.uint32) if dtype == "f32" else want
        say(f"direct blocks N={n} count={count} {dtype} {cfg}")
        recv = [torch.full((count,), float("nan"), device="cuda:0").to(send[0].dtype) for _ in range(n)]
        with ar.Plan(n, count, dtype, coll="reducescatter", algo="direct", **cfg) as plan:
            plan.run_oop(send, recv)
            torch.cuda.synchronize()
        for r in range(n):
            assert np.array_equal(to_bits(recv[r], dtype), want[r]), ("reducescatter", n, count, cfg, r)
        blocks = [t[:count].clone() for t in send]
        full = [torch.zeros(n * count, dtype=send[0].dtype, device="cuda:0") for _ in range(n)]
        with ar.Plan(n, count, dtype, coll="allgather", algo="direct", **cfg) as plan:
            plan.run_oop(blocks, full)
            torch.cuda.synchronize()
        whole = np.concatenate([to_bits(b, dtype) for b in blocks])
        for r in range(n):
            assert np.array_equal(to_bits(full[r], dtype), whole), ("allgather", n, count, cfg, r)


@pytest.mark.parametrize("n", (8, 16))
def test_more_workgroups_than_a_launch_holds(ar, n):
    """A tuner's number of workgroups that no launch can hold: the plan is
    bounded by the segment's units and every element is summed."""
    count = 1001
    x = draw(n, count, "f32", "normal", seed=71)
    ar.ar_set_tuner(lambda ctx: {"algo": ar.AR_ALGO_DIRECT, "direct_parts": 1 << 28, "direct_nwaves": 16})
    try:
        info = ar.ar_plan_geometry(ar.make_desc(n, count, "f32"))
        assert 0 < info["nchannels"] <= 32
        run_case(ar, x, "f32", f"direct-{n}-bounded")
    finally:
        ar.ar_set_tuner(None)


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("n", (2, 3, 5, 8, 11))
def test_segments_off_the_lines(ar, n, dtype):
    """Buffers that start at every 16-byte place of a 128-byte line, each rank's
    at another, and segments that are no multiple of a line, with outputs of
    12 MiB in all, from which on iterations start on lines: ends around the
    units of whole iterations, where the shift to the line's start just fits
    or would cost an iteration; in place and out of place."""
    import torch

    a = 4 if dtype == "f32" else 8
    for coll in ("allreduce", "reducescatter", "allgather"):
        u = 4 if coll == "allgather" else 2 if n <= 4 else 1  # units per thread and iteration
        least = -(-(12 << 20) // 16 // (n if coll == "reducescatter" else n * n))  # units of a segment
        parts = min(100, least // (1024 * u) + 1)
        one = parts * 1024 * u  # units of one iteration: workgroups of sixteen waves
        k = -(-(least + 8) // one)
        for i, units in enumerate((k * one - 8, k * one - 7, k * one - 6, k * one, (k + 1) * one - 71)):
            count = units * a * (n if coll == "allreduce" else 1) - (1 if coll == "allreduce" and i % 2 else 0)
            ns, nr = {"allreduce": (count, count), "reducescatter": (n * count, count), "allgather": (count, n * count)}[coll]
            x = draw(n, ns, dtype, "normal", seed=31 * n + i)
            if coll == "allreduce":
                want = np.stack([oracle_bits(x, dtype)] * n)
            else:
                want = ro.reduce_scatter(x, dtype) if coll == "reducescatter" else np.stack([ro.all_gather(x)] * n)
                want = want.view(np.uint32) if dtype == "f32" else want
            host = to_device(x, dtype)

            def placed(length):
                whole = [torch.full((length + 16 * a,), float("nan"), device="cuda:0").to(host[0].dtype) for _ in range(n)]
                at = [(3 * r + i) % 8 * a for r in range(n)]
                return whole, [w[o:o + length] for w, o in zip(whole, at)], at

            _, send, _ = placed(ns)
            for t, h in zip(send, host):
                t.copy_(h)
            whole, recv, at = placed(nr)
            say(f"off the lines {coll} N={n} {dtype} units={units} count={count}")
            with ar.Plan(n, count, dtype, coll=coll, algo="direct", nchannels=parts, nwaves=16, direct_unroll=1) as plan:
                plan.run_oop(send, recv)
                torch.cuda.synchronize()
                for r in range(n):
                    assert np.array_equal(to_bits(recv[r], dtype), want[r]), (coll, units, r)
                    # nothing before or after the output is written
                    assert bool(whole[r][:at[r]].isnan().all()) and bool(whole[r][at[r] + nr:].isnan().all()), (coll, units, r)
                if coll == "allreduce":
                    plan.run(send)
                    torch.cuda.synchronize()
                    for r in range(n):
                        assert np.array_equal(to_bits(send[r], dtype), want[r]), (coll, units, r, "in place")
