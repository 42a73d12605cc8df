"""The work this library is measured on: collectives over N rank buffers that
live in one GPU's memory, through the public entry points of the Python
binding, from 4 KiB to 128 MiB per rank.

Result bits depend only on (ranks, count, data type): every algorithm,
protocol and channel count gives the same bits, so every case is compared
exactly.
"""
from __future__ import annotations

import math

import torch

import paper_2603_11438_amd as ar

KiB = 1024
MiB = 1024 * 1024
ELEM = {"f32": 4, "bf16": 2}
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}

# A case:
#   coll    allreduce / reducescatter / allgather
#   n       ranks
#   count   elements: AllReduce, each rank's buffer; the others, one block
#   dtype   f32 / bf16 (fp32 partial sums)
#   dist    values: int8 (integers -8..8), uniform [-1, 1), normal
#   choice  how the call is routed: "tuned" (no wishes: the size -> algorithm
#           table decides), "ring" (the ring; the table picks protocol,
#           channels, chunk and waves), "default" (the fixed default policy:
#           Simple protocol, 16 channels), "ll" / "ll128" (that protocol with
#           `channels` channels)
#   entry   bind (buffers checked once, one C call per run), oop (checked on
#           every call, out of place), inplace (checked on every call, in
#           place), noalloc (no plan, no allocation)


def _case(name, coll, n, count, dtype, dist, choice, entry, channels=0):
    return {"name": name, "coll": coll, "n": n, "count": count, "dtype": dtype, "dist": dist,
            "choice": choice, "entry": entry, "channels": channels}


def listed():
    return [
        # The smallest gradient or statistics AllReduce: a call's latency.
        _case("tuned_4KiB_f32", "allreduce", 8, 1024, "f32", "int8", "tuned", "bind"),
        # A layer's worth of bf16 gradients, odd length, from a program that
        # hands its tensors over afresh on every call.
        _case("tuned_195KiB_bf16_oop", "allreduce", 8, 100003, "bf16", "normal", "tuned", "oop"),
        # A medium bucket, resident in the last-level cache.
        _case("tuned_4MiB_f32", "allreduce", 8, 1 * MiB, "f32", "uniform", "tuned", "bind"),
        # The usual bucket of data-parallel training in bf16.
        _case("tuned_32MiB_bf16", "allreduce", 8, 16 * MiB, "bf16", "normal", "tuned", "bind"),
        # The ring at the smallest size, where its hops are all latency.
        _case("ring_4KiB_f32", "allreduce", 8, 1024, "f32", "int8", "ring", "bind"),
        # The ring at the largest size: the flagship step of bench.py.
        _case("ring_128MiB_f32", "allreduce", 8, 32 * MiB, "f32", "uniform", "ring", "bind"),
        # A program (or a tuner without an opinion) that stays on the fixed
        # default policy, ragged bf16 bucket.
        _case("default_9MiB_bf16", "allreduce", 8, 4718597, "bf16", "normal", "default", "bind"),
        # The size-aware policy of the paper's B300 system: LL128 between 4
        # and 32 MiB.
        _case("ll128_8MiB_f32", "allreduce", 8, 2 * MiB, "f32", "uniform", "ll128", "bind", 32),
        # Sharded training: gradients reduced and scattered, 64 MiB per rank.
        _case("rs_tuned_64MiB_bf16", "reducescatter", 8, 4 * MiB, "bf16", "normal", "tuned", "bind"),
        # Sharded training: parameters gathered in place, ring, 12 MiB.
        _case("ag_ring_12MiB_f32", "allgather", 8, 393216, "f32", "uniform", "ring", "inplace"),
        # A serving loop that may not allocate: four ranks, ring.
        _case("noalloc_ring_66KB_f32", "allreduce", 4, 16411, "f32", "uniform", "ring", "noalloc"),
        # Two ranks, as a pair of tensor-parallel shards, large activations.
        _case("tuned_2ranks_48MiB_bf16", "allreduce", 2, 24 * MiB, "bf16", "normal", "tuned", "bind"),
    ]


def draw(rng):
    """One more case: sizes from 4 KiB to 128 MiB per rank (all ranks together
    at most 1 GiB), 2 to 16 ranks, every collective, type, route and entry."""
    coll = rng.choice(("allreduce", "allreduce", "allreduce", "reducescatter", "allgather"))
    dtype = rng.choice(("f32", "bf16"))
    choice = rng.choice(("tuned", "tuned", "tuned", "ring", "ring", "default", "ll", "ll128"))
    entry = rng.choice(("bind", "bind", "oop", "noalloc", "inplace"))
    n = rng.choice((2, 3, 4, 5, 8, 8, 8, 8, 16))
    # Largest buffer per rank: 1 GiB over all ranks; less where the route
    # moves more bytes, where LL is only used small, and where the ring has
    # to fit the static scratch of the allocation-free entry.
    top = 128 * MiB * min(8, 8 / n)
    if choice != "tuned":
        top = min(top, 32 * MiB * 8 / n if dtype == "bf16" else 64 * MiB * 8 / n)
    if choice in ("default", "ll128"):
        top = min(top, 16 * MiB)
    if choice == "ll" or (entry == "noalloc" and choice != "tuned"):
        top = min(top, 1 * MiB)
    size = math.exp(rng.uniform(math.log(4 * KiB), math.log(min(top, 128 * MiB))))
    e = ELEM[dtype]
    if coll == "allreduce":
        count = max(1, int(size) // e)  # any length, mostly odd against the 16-byte unit
        if entry == "inplace":
            entry = "oop"  # sums in place would grow from pass to pass
    else:
        a = 16 // e
        count = max(a, int(size) // (e * n) // a * a)  # blocks start on 16 bytes
        if coll == "reducescatter" and entry == "inplace":
            entry = "oop"  # likewise
    dist = "normal" if dtype == "bf16" else "uniform"
    return {"coll": coll, "n": n, "count": count, "dtype": dtype, "dist": dist, "choice": choice, "entry": entry,
            "channels": rng.choice((2, 4, 8, 16)) if choice in ("ll", "ll128") else 0}


def _lengths(case):
    """Elements of each rank's send and recv buffer."""
    n, c = case["n"], case["count"]
    return {"allreduce": (c, c), "reducescatter": (n * c, c), "allgather": (c, n * c)}[case["coll"]]


def _inputs(case, seed):
    """One tensor per rank, drawn on the GPU from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(11438 + 7919 * seed)
    length = _lengths(case)[0]
    out = []
    for _ in range(case["n"]):
        if case["dist"] == "int8":
            x = torch.randint(-8, 9, (length,), generator=g, device="cuda").float()
        elif case["dist"] == "uniform":
            x = torch.rand(length, generator=g, device="cuda") * 2.0 - 1.0
        else:
            x = torch.randn(length, generator=g, device="cuda")
        out.append(x.to(TORCH[case["dtype"]]))
    return out


def _wishes(case):
    """The plan settings a case's route stands for."""
    if case["choice"] == "tuned":
        return {}
    if case["choice"] == "ring":
        return {"algo": "ring"}
    if case["choice"] == "default":
        return {"proto": "simple", "nchannels": 16, "chunk_bytes": 256 * KiB, "nwaves": 4}
    return {"proto": case["choice"], "nchannels": case["channels"]}


def prepare(case, seed):
    send = _inputs(case, seed)
    length = _lengths(case)[1]
    state = {"case": case, "wishes": dict(_wishes(case), coll=case["coll"])}
    if case["entry"] == "inplace":
        # AllGather: rank r's block lies at r * count of its full buffer
        full = [torch.zeros(length, dtype=TORCH[case["dtype"]], device="cuda") for _ in send]
        for r, (t, x) in enumerate(zip(full, send)):
            t[r * case["count"]:(r + 1) * case["count"]] = x
        state["full"] = full
    else:
        state["send"] = send
        state["recv"] = [torch.zeros(length, dtype=TORCH[case["dtype"]], device="cuda") for _ in send]
    if case["entry"] != "noalloc":
        state["plan"] = ar.Plan(case["n"], case["count"], case["dtype"], **state["wishes"])
        if case["entry"] == "bind":
            state["call"] = state["plan"].bind(state["send"], state["recv"])
    return state


def run(state):
    entry = state["case"]["entry"]
    if entry == "bind":
        state["call"]()
    elif entry == "oop":
        state["plan"].run_oop(state["send"], state["recv"])
    elif entry == "inplace":
        state["plan"].run(state["full"])
        return state["full"]
    else:
        ar.run_noalloc(state["send"], state["recv"], **state["wishes"])
    return state["recv"]


def work(case):
    n, c, e = case["n"], case["count"], ELEM[case["dtype"]]
    if case["coll"] == "allreduce":
        return {"bytes": 2 * n * c * e, "flops": (n - 1) * c}
    # one side holds n blocks per rank, the other one block per rank
    return {"bytes": (n + 1) * n * c * e, "flops": (n - 1) * n * c if case["coll"] == "reducescatter" else 0}


def tolerance(case):
    # The summation order and its roundings are part of the interface.
    return "exact"


def exact(case, seed):
    xs = _inputs(case, seed)
    n, c = case["n"], case["count"]
    if case["coll"] == "allgather":
        y = torch.cat(xs).double()
        return [y] * n
    total = torch.zeros(xs[0].numel(), dtype=torch.float64, device="cuda")
    for x in xs:
        total += x.double()
    if case["coll"] == "allreduce":
        return [total] * n
    return [total[r * c:(r + 1) * c] for r in range(n)]
