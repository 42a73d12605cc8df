"""The direct algorithm where its geometry can go wrong: every rank count's
own kernel, one and several iterations per thread, workgroups launched as two,
the partial unit's own workgroup; against the oracle, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import ring_oracle as ro
from tests.gpu_helpers import draw, run_case, say, to_bits, to_device

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
