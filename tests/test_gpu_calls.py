"""The native call path of the Python binding (csrc/tensor_args.cpp): what it
accepts runs and gives the oracle's bits, what it leaves to the checks in
Python is accepted or refused as those checks always did.  The same without
the native part, where every call takes those checks and ctypes."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_helpers import assert_ranks_equal, draw, oracle_bits, to_device

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


@pytest.fixture(params=("native", "python"))
def path(ar, request, monkeypatch):
    """The binding's call path: native (which has to be there), or without it."""
    if request.param == "native":
        assert ar._native() is not None
    else:
        monkeypatch.setattr(ar, "_native_path", False)
    return request.param


@pytest.mark.parametrize("dtype", ("f32", "bf16"))
def test_accepted_forms(ar, path, dtype):
    """Lists and tuples of tensors, parameters, views with an offset, a
    stacked tensor (iterated), a subclass, and a stream of the caller's."""
    import torch

    n, count = 4, 1016
    x = draw(n, count, dtype, "normal", seed=11)
    want = oracle_bits(x, dtype)

    class Sub(torch.Tensor):
        pass

    def views(ts):
        big = [torch.zeros(count + 64, dtype=t.dtype, device=t.device) for t in ts]
        for b, t in zip(big, ts):
            b[32:32 + count] = t
        return [b[32:32 + count] for b in big]

    forms = {"list": lambda ts: ts, "tuple": tuple, "views": views,
             "parameters": lambda ts: [torch.nn.Parameter(t, requires_grad=False) for t in ts],
             "stacked": lambda ts: torch.stack(ts), "subclass": lambda ts: [t.as_subclass(Sub) for t in ts]}
    with ar.Plan(n, count, dtype) as plan:
        for name, make in forms.items():
            send = make(to_device(x, dtype))
            def nans():
                return make([torch.full((count,), float("nan"), dtype=t.dtype, device="cuda:0") for t in send])
            calls = {"run_oop": lambda r: plan.run_oop(send, r), "bind": lambda r: plan.bind(send, r)(),
                     "run_noalloc": lambda r: ar.run_noalloc(send if name in ("list", "tuple") else list(send),
                                                             list(r), algo="ring")}
            for what, run in calls.items():
                recv = nans()
                run(recv)
                torch.cuda.synchronize()
                assert_ranks_equal(list(recv), want, dtype, f"{name} {what}")
            plan.run(send)
            torch.cuda.synchronize()
            assert_ranks_equal(list(send), want, dtype, name + " in place")
        side = torch.cuda.Stream()
        send = to_device(x, dtype)
        with torch.cuda.stream(side):
            current, given = ([torch.full((count,), float("nan"), dtype=t.dtype, device="cuda:0") for t in send]
                              for _ in range(2))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            plan.run_oop(send, current)       # the current stream
        plan.run_oop(send, given, side)       # a stream that is not the current one
        side.synchronize()
        assert_ranks_equal(current, want, dtype, "current stream")
        assert_ranks_equal(given, want, dtype, "given stream")


def test_refused_forms(ar, path):
    import torch

    n, count = 4, 64
    good = [torch.ones(count, device="cuda:0") for _ in range(n)]
    out = [torch.full((count,), 7.0, device="cuda:0") for _ in range(n)]
    bad = {
        "short list": good[:3], "cpu": good[:3] + [torch.ones(count)], "size": good[:3] + [torch.ones(count + 1, device="cuda:0")],
        "strided": good[:3] + [torch.ones(2 * count, device="cuda:0")[::2]],
        "dtype": good[:3] + [torch.ones(count, device="cuda:0", dtype=torch.bfloat16)],
    }
    with ar.Plan(n, count, "f32") as plan:
        for name, ts in bad.items():
            for args in ((ts, out), (good, ts)):
                with pytest.raises(ValueError):
                    plan.run_oop(*args)
            with pytest.raises(ValueError):
                plan.run(ts)
        with pytest.raises(TypeError):
            plan.run_oop(good[:3] + [torch.ones(count, device="cuda:0", dtype=torch.float16)], out)
        with pytest.raises(TypeError):
            plan.run_oop(good, None)
        with pytest.raises(TypeError):
            plan.run(None)
        with pytest.raises(ar.ARError) as e:     # one rank's output over another's input
            plan.run_oop(good, good[1:] + good[:1])
        assert e.value.code == ar.AR_ERR_ARG
        off = torch.ones(count + 1, device="cuda:0")[1:]
        with pytest.raises(ar.ARError) as e:     # not on 16 bytes
            plan.run_oop(good[:3] + [off], out)
        assert e.value.code == ar.AR_ERR_ARG
        call = plan.bind(good, out)
    with pytest.raises(ar.ARError):              # the plan is gone
        call()
    with pytest.raises(ar.ARError):
        plan.run_oop(good, out)
    torch.cuda.synchronize()
    assert all(bool((t == 7.0).all()) for t in out) and all(bool((t == 1.0).all()) for t in good)
