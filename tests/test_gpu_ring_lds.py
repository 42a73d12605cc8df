"""The ring with its links in LDS against the oracle and against the same
plan with its links in memory, bit for bit, where its pieces, its prefetch
and its partial unit can go wrong; and the production build of the rings in
memory (FIFO-only plans) with poisoned FIFOs."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import ring_oracle as ro
from tests.gpu_helpers import assert_ranks_equal, draw, oracle_bits, run_case, say, to_bits, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ar():
    import torch

    import paper_2603_11438_amd as ar

    assert torch.cuda.is_available()
    torch.cuda.set_device(0)
    ar.lib()
    ar.ar_set_tuner(None)
    return ar


def _piece_units(n, coll="allreduce"):
    """16-byte units of one piece of a segment."""
    return 64 * (2 if n == 2 else 1) * (2 if coll == "allgather" else 1)


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("n", range(2, 17))
def test_allreduce_edges(ar, n, dtype):
    """Counts whose last segment ends inside, at and just past a piece, a lane
    and a unit; one channel of one wave, so max(n, 4) rings share the pieces: one
    piece or fewer per ring, and two and three with the next one loaded ahead."""
    a = 4 if dtype == "f32" else 8
    p = _piece_units(n) * a  # elements of a piece
    rings = max(n, 4)
    counts = [1, a + 1, n * a, n * p - 1, n * p, n * p + 1, n * p + n * a - a + 1, n * (rings + 1) * p + 3,
              n * (2 * rings + 1) * p - p - 5]
    for i, count in enumerate(counts):
        x = draw(n, count, dtype, "normal", seed=900 + 31 * n + i)
        proto = ("simple", "ll", "ll128")[i % 3]
        run_case(ar, x, dtype, f"lds-{n}-{dtype}-{count}-{proto}", proto=proto, nchannels=1, nwaves=1)


@pytest.mark.parametrize("coll", ("reducescatter", "allgather"))
@pytest.mark.parametrize("n", (2, 3, 4, 8, 13, 16))
def test_blocks_against_links_in_memory(ar, coll, n):
    """Out of place and in place, blocks around a piece and of several pieces
    per ring, against the oracle and the FIFO-only plan."""
    import torch

    for dtype in ("f32", "bf16"):
        a = 4 if dtype == "f32" else 8
        p = _piece_units(n, coll) * a
        for count in (a, p - a, p + a, (2 * max(n, 4) + 1) * p + 3 * a):
            ns, nr = (n * count, count) if coll == "reducescatter" else (count, n * count)
            x = draw(n, ns, dtype, "normal", seed=count + n)
            want = ro.reduce_scatter(x, dtype) if coll == "reducescatter" else np.stack([ro.all_gather(x)] * n)
            want = want.view(np.uint32) if dtype == "f32" else want
            send = to_device(x, dtype)
            for flags in (0, ar.AR_PLAN_FIFO_ONLY):
                say(f"lds {coll} N={n} count={count} {dtype} flags={flags}")
                recv = [torch.full((nr,), float("nan"), device="cuda:0").to(send[0].dtype) for _ in range(n)]
                with ar.Plan(n, count, dtype, coll=coll, proto="simple", nchannels=1, nwaves=1, flags=flags) as plan:
                    plan.run_oop(send, recv)
                    full = [torch.zeros(n * count, dtype=t.dtype, device="cuda:0") for t in send]
                    for r in range(n):
                        if coll == "reducescatter":
                            full[r].copy_(send[r])
                        else:
                            full[r][r * count:(r + 1) * count] = send[r]
                    plan.run(full)
                    torch.cuda.synchronize()
                    assert plan.status() == ar.AR_OK
                for r in range(n):
                    mine = full[r][r * count:(r + 1) * count] if coll == "reducescatter" else full[r]
                    assert np.array_equal(to_bits(recv[r], dtype), want[r]), (coll, n, count, dtype, flags, r)
                    assert np.array_equal(to_bits(mine, dtype), want[r]), (coll, n, count, dtype, flags, r, "in place")


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("n", (2, 3, 5, 8))
def test_rings_of_a_plan(ar, n, dtype):
    """Result bits of plans whose channels and waves give few and many rings,
    with more pieces than rings, the last ones partial."""
    a = 4 if dtype == "f32" else 8
    count = n * (2100 if n == 2 else 1030) * _piece_units(n) * a - 7
    x = draw(n, count, dtype, "normal", seed=40 + n)
    want = oracle_bits(x, dtype)
    for channels, waves in ((1, 2), (7, 3), (16, 4), (min(128, 256 // n), 4)):
        say(f"rings N={n} {dtype} C={channels} W={waves}")
        with ar.Plan(n, count, dtype, proto="simple", nchannels=channels, nwaves=waves) as plan:
            ts = to_device(x, dtype)
            plan.run(ts)
            assert_ranks_equal(ts, want, dtype, f"rings {n} {channels} {waves}")


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
def test_special_values(ar, dtype):
    """Infinities, NaN, signed zeros and the largest values come out of the
    chain as they do from the oracle; an AllGather keeps every bit."""
    import torch

    n, count = 8, 5003
    x = draw(n, count, "f32", "normal", seed=77)
    for i, v in enumerate((np.inf, -np.inf, np.nan, 0.0, -0.0, 3.4028235e38, -3.4028235e38, 1e-45)):
        x[i % n, i::17] = v
    if dtype == "bf16":
        x = (x.view(np.uint32) >> 16).astype(np.uint16)
    send = to_device(x, dtype)
    recv = [torch.zeros_like(t) for t in send]
    with ar.Plan(n, count, dtype, algo="ring", proto="simple", nchannels=3) as plan:
        plan.run_oop(send, recv)
        with ar.Plan(n, count, dtype, algo="direct") as direct:
            other = [torch.zeros_like(t) for t in send]
            direct.run_oop(send, other)
        torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        want = oracle_bits(x, dtype)
    finite = ~np.isnan((want.astype(np.uint32) << 16 if dtype == "bf16" else want).view(np.float32))
    for r in range(n):
        got = to_bits(recv[r], dtype)
        assert np.array_equal(got, to_bits(other[r], dtype))
        assert np.array_equal(got[finite], want[finite])


def test_runs_of_one_plan_on_two_streams_after_each_other(ar):
    """No state between runs: two plans on two streams, many runs each, while
    a FIFO-only ring runs on a third."""
    import torch

    n, count = 8, 40001
    x = draw(n, count, "f32", "uniform", seed=5)
    want = oracle_bits(x, "f32")
    plans, streams = [], [torch.cuda.Stream() for _ in range(3)]
    bufs = []
    for i, flags in enumerate((0, 0, ar.AR_PLAN_FIFO_ONLY)):
        plans.append(ar.Plan(n, count, "f32", proto="simple", nchannels=2 + i, flags=flags))
        bufs.append((to_device(x, "f32"), [torch.full((count,), float("nan"), device="cuda:0") for _ in range(n)]))
    torch.cuda.synchronize()
    for rep in range(8):
        for p, s, (send, recv) in zip(plans, streams, bufs):
            p.run_oop(send, recv, s)
    torch.cuda.synchronize()
    for p, (_, recv) in zip(plans, bufs):
        assert p.status() == ar.AR_OK
        assert_ranks_equal(recv, want, "f32", "streams")
        p.destroy()


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
@pytest.mark.parametrize("proto", ("simple", "ll", "ll128"))
def test_links_in_memory_with_poisoned_fifo(ar, proto, dtype):
    """FIFO-only plans run the production build of the rings in memory: every
    run with its FIFOs poisoned gives the oracle's bits."""
    import torch

    n, count = 5, 20011
    plan = ar.Plan(n, count, dtype, proto=proto, nchannels=3, fifo_depth=2, flags=ar.AR_PLAN_FIFO_ONLY)
    assert plan.workspace_bytes > plan.info["fifo_bytes"] > 0
    for i in range(6):
        x = draw(n, count, dtype, "normal", seed=60 + i)
        ts = to_device(x, dtype)
        plan.poison()
        say(f"poisoned {proto} {dtype} run {i}")
        plan.run(ts)
        torch.cuda.synchronize()
        assert plan.status() == ar.AR_OK
        assert_ranks_equal(ts, oracle_bits(x, dtype), dtype, f"{proto} run {i}")
    plan.destroy()
