"""The native marshaller against the binding's own checks: every call that it
takes gives the outputs of the general path, and every call that the general
path refuses is refused with the same error."""

from __future__ import annotations

import pytest
import torch

from paper_2411_00284_amd import FsdpError

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

if torch.cuda.is_available():
    from paper_2411_00284_amd import BucketPlan

W, DIMS = 3, [(10, 8), (0, 4), (7, 3), (1, 1)]
DT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def state(wire, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    plan = BucketPlan(W, DIMS, 8)
    S = plan.chunk_elems

    def rand(n, dt):
        return torch.randn(n, device="cuda", generator=g).to(DT[dt])

    full = [n * k for n, k in DIMS]
    return plan, {
        "shards": [rand(plan.local_elems(p, 1), "f32") for p in range(len(DIMS))],
        "send": torch.zeros(S, dtype=DT[wire], device="cuda"),
        "gathered": rand(W * S, wire), "chunks": [rand(S, wire) for _ in range(W)],
        "params": [torch.zeros(n, dtype=DT[wire], device="cuda") for n in full],
        "grads": [rand(n, wire) for n in full],
        "outgoing": torch.zeros(W * S, dtype=DT[wire], device="cuda"),
        "outs": [torch.zeros(S, dtype=DT[wire], device="cuda") for _ in range(W)],
        "averages": [torch.zeros(plan.local_elems(p, 1), device="cuda") for p in range(len(DIMS))],
    }


CALLS = {
    "ag_pack": lambda p, s, w, **k: p.ag_pack(1, s["shards"], s["send"], **k),
    "ag_unpack": lambda p, s, w, **k: p.ag_unpack(s["gathered"], s["params"], **k),
    "rs_pack": lambda p, s, w, **k: p.rs_pack(s["grads"], s["outgoing"], **k),
    "rs_reduce": lambda p, s, w, **k: p.rs_reduce(1, s["gathered"], s["averages"], **k),
    "ag_pack_ex": lambda p, s, w, **k: p.ag_pack_ex(1, s["shards"], s["send"], w, **k),
    "ag_pack_push": lambda p, s, w, **k: p.ag_pack_push(1, s["shards"], s["outs"], w, **k),
    "ag_unpack_ex": lambda p, s, w, **k: p.ag_unpack_ex(s["chunks"], s["params"], w, **k),
    "rs_pack_ex": lambda p, s, w, **k: p.rs_pack_ex(s["grads"], s["outs"], w, **k),
    "rs_reduce_ex": lambda p, s, w, **k: p.rs_reduce_ex(1, s["chunks"], s["averages"], w, **k),
}
OUTPUTS = ("send", "params", "outgoing", "outs", "averages")


def outputs(s):
    return [t.clone() for k in OUTPUTS for t in (s[k] if isinstance(s[k], list) else [s[k]])]


@pytest.mark.parametrize("name", CALLS)
@pytest.mark.parametrize("wire", ["bf16", "f16", "f32"])
def test_same_outputs(name, wire):
    if wire != "bf16" and not name.endswith(("_ex", "_push")):
        pytest.skip("the plain calls take bf16")
    side = torch.cuda.Stream()
    for how in ("plain", "tuples", "none", "stream"):
        got = []
        for native in (True, False):
            plan, s = state(wire)
            torch.cuda.synchronize()
            taken = []
            run = plan._caller.run
            plan._run = (lambda *a: taken.append(run(*a)) or taken[-1]) if native else (lambda *a: None)
            if how == "tuples":
                s.update({k: tuple(v) for k, v in s.items() if isinstance(v, list)})
            if how == "none":                               # an empty parameter as None
                for k in ("shards", "params", "grads", "averages"):
                    s[k][1] = None
            print(f"[gpu] {name} {wire} {how} native={native}", flush=True)
            CALLS[name](plan, s, wire, **({"stream": side} if how == "stream" else {}))
            torch.cuda.synchronize()
            assert not native or taken == [0]               # the native path did it
            s.update({k: [t for t in v if t is not None] for k, v in s.items() if isinstance(v, (list, tuple))})
            got.append(outputs(s))
            plan.close()
        assert all(torch.equal(a, b) for a, b in zip(*got))


BAD = {
    "short list": lambda s: s["shards"].pop(),
    "missing": lambda s: s["shards"].__setitem__(0, None),
    "type": lambda s: s["shards"].__setitem__(0, s["shards"][0].double()),
    "int shards": lambda s: s["shards"].__setitem__(0, s["shards"][0].int()),
    "size": lambda s: s["shards"].__setitem__(0, s["shards"][0][:-1]),
    "strides": lambda s: s["shards"].__setitem__(0, s["shards"][0].repeat(2)[::2]),
    "host": lambda s: s["shards"].__setitem__(0, s["shards"][0].cpu()),
    "no tensor": lambda s: s["shards"].__setitem__(0, [1.0]),
    "bucket size": lambda s: s.__setitem__("send", s["send"][1:]),
    "bucket type": lambda s: s.__setitem__("send", s["send"].float()),
    "bucket alignment": lambda s: s.__setitem__("send", torch.zeros(s["send"].numel() + 1, dtype=torch.bfloat16,
                                                                    device="cuda")[1:]),
    "overlap": lambda s: s.__setitem__("send", s["shards"][0].view(torch.bfloat16)[:0]
                                       if s["send"].numel() > 2 * s["shards"][0].numel()
                                       else s["shards"][0].view(torch.bfloat16)[:s["send"].numel()]),
}


@pytest.mark.parametrize("what", BAD)
@pytest.mark.parametrize("rank", [1, -1, W])
def test_same_refusals(what, rank):
    errors = []
    for native in (True, False):
        plan, s = state("bf16")
        BAD[what](s)
        if not native:
            plan._run = lambda *a: None
        with pytest.raises((TypeError, ValueError, FsdpError)) as e:
            plan.ag_pack(rank, s["shards"], s["send"])
        errors.append((e.type, str(e.value)))
        plan.close()
    assert errors[0] == errors[1]


def test_a_closed_plan_is_refused():
    plan, s = state("bf16")
    plan.close()
    with pytest.raises((FsdpError, ValueError)):
        plan.ag_pack(1, s["shards"], s["send"])


TENSORS = {"ag_pack": "shards", "ag_unpack": "params", "rs_pack": "grads", "rs_reduce": "averages"}
BUFFERS = {"ag_pack": "send", "ag_pack_ex": "send", "ag_pack_push": "outs", "ag_unpack": "gathered",
           "ag_unpack_ex": "chunks", "rs_pack": "outgoing", "rs_pack_ex": "outs", "rs_reduce": "gathered",
           "rs_reduce_ex": "chunks"}


def tensors_of(name):
    return TENSORS[name.removesuffix("_ex").removesuffix("_push")]


def put(group, i, change):
    return lambda s, k: s[k[group]].__setitem__(i, change(s[k[group]][i]))


# what is wrong -> the change of the call's tensors ("t") or bucket buffer ("b")
ANY_CALL = {
    "one tensor fewer": lambda s, k: s[k["t"]].pop(),
    "no list": lambda s, k: s.__setitem__(k["t"], iter(s[k["t"]])),
    "missing tensor": put("t", 0, lambda t: None),
    "short tensor": put("t", 2, lambda t: t[:-1]),
    "long tensor": put("t", 2, lambda t: t.repeat(2)),
    "tensor type": put("t", 0, lambda t: t.double()),
    "every tensor's type": lambda s, k: s.__setitem__(k["t"], [t.double() for t in s[k["t"]]]),
    "host tensor": put("t", 0, lambda t: t.cpu()),
    "strided tensor": put("t", 0, lambda t: t.repeat(2)[::2]),
    "no tensor": put("t", 0, lambda t: [1.0]),
}
ONE_BUFFER = {
    "short buffer": lambda s, k: s.__setitem__(k["b"], s[k["b"]][:-1]),
    "long buffer": lambda s, k: s.__setitem__(k["b"], s[k["b"]].repeat(2)),
    "buffer type": lambda s, k: s.__setitem__(k["b"], s[k["b"]].double()),
    "host buffer": lambda s, k: s.__setitem__(k["b"], s[k["b"]].cpu()),
    "strided buffer": lambda s, k: s.__setitem__(k["b"], s[k["b"]].repeat(2)[::2]),
    "buffer off the grid": lambda s, k: s.__setitem__(k["b"], s[k["b"]].repeat(2)[1:1 + s[k["b"]].numel()]),
    "no buffer": lambda s, k: s.__setitem__(k["b"], None),
}
CHUNK_LIST = {
    "one chunk fewer": lambda s, k: s[k["b"]].pop(),
    "one chunk more": lambda s, k: s[k["b"]].append(s[k["b"]][0].clone()),
    "missing chunk": put("b", W - 1, lambda t: None),
    "short chunk": put("b", W - 1, lambda t: t[:-1]),
    "long chunk": put("b", W - 1, lambda t: t.repeat(2)),
    "chunk type": put("b", 1, lambda t: t.double()),
    "host chunk": put("b", 1, lambda t: t.cpu()),
    "strided chunk": put("b", 1, lambda t: t.repeat(2)[::2]),
    "chunk off the grid": put("b", 1, lambda t: t.repeat(2)[1:1 + t.numel()]),
    "one tensor for the chunks": lambda s, k: s.__setitem__(k["b"], torch.cat(s[k["b"]])),
}
GRADIENTS = {
    "mixed gradients": (put("t", 3, lambda t: t.float() if t.dtype != torch.float32 else t.half()), "bf16"),
    "f16 gradients on a bf16 wire": (lambda s, k: s.__setitem__("grads", [t.half() for t in s["grads"]]), "bf16"),
    "fp32 gradients on a bf16 wire": (lambda s, k: s.__setitem__("grads", [t.float() for t in s["grads"]]), "bf16"),
    "bf16 gradients on an f16 wire": (lambda s, k: s.__setitem__("grads", [t.bfloat16() for t in s["grads"]]), "f16"),
}


def refusal(name, wire, change, native, stated=None):
    """The error of a call whose tensors (of ``wire``) were changed; the call
    is given ``stated`` as the wire's name."""
    plan, s = state(wire)
    if change:
        change(s, {"t": tensors_of(name), "b": BUFFERS[name]})
    if not native:
        plan._run = lambda *a: None
    print(f"[gpu] {name} {wire} {stated} native={native}", flush=True)
    with pytest.raises((TypeError, ValueError, AttributeError, FsdpError)) as e:
        CALLS[name](plan, s, wire if stated is None else stated)
    plan.close()
    return e.type, str(e.value)


def wires_of(name):
    return ["bf16", "f16", "f32"] if name.endswith(("_ex", "_push")) else ["bf16"]


@pytest.mark.parametrize("name", CALLS)
def test_every_call_refuses_the_same(name):
    """Bad tensors, buffers and chunk lists, each with the same error with and
    without the native path."""
    lists = isinstance(state("bf16")[1][BUFFERS[name]], list)
    for what, change in {**ANY_CALL, **(CHUNK_LIST if lists else ONE_BUFFER)}.items():
        for wire in wires_of(name):
            got = [refusal(name, wire, change, native) for native in (True, False)]
            assert got[0] == got[1], (what, wire)


@pytest.mark.parametrize("what", GRADIENTS)
def test_gradient_types_are_refused_the_same(what):
    change, wire = GRADIENTS[what]
    got = [refusal("rs_pack_ex", wire, change, native) for native in (True, False)]
    assert got[0] == got[1]


@pytest.mark.parametrize("name", [n for n in CALLS if n.endswith(("_ex", "_push"))])
@pytest.mark.parametrize("stated", ["f64", "bfloat16", "", "f32"])
def test_wire_names_are_refused_the_same(name, stated):
    """A name that is none, and one that the tensors are not of."""
    got = [refusal(name, "bf16", None, native, stated=stated) for native in (True, False)]
    assert got[0] == got[1]


@pytest.mark.parametrize("name", [n for n in CALLS if n.startswith(("ag_pack", "rs_reduce"))])
def test_ranks_are_refused_the_same(name):
    call = {"ag_pack": lambda p, s, r: p.ag_pack(r, s["shards"], s["send"]),
            "ag_pack_ex": lambda p, s, r: p.ag_pack_ex(r, s["shards"], s["send"], "bf16"),
            "ag_pack_push": lambda p, s, r: p.ag_pack_push(r, s["shards"], s["outs"], "bf16"),
            "rs_reduce": lambda p, s, r: p.rs_reduce(r, s["gathered"], s["averages"]),
            "rs_reduce_ex": lambda p, s, r: p.rs_reduce_ex(r, s["chunks"], s["averages"], "bf16")}[name]
    for rank in (-1, W, 1 << 40, 1.0, "1", None):
        errors = []
        for native in (True, False):
            plan, s = state("bf16")
            if not native:
                plan._run = lambda *a: None
            with pytest.raises(Exception) as e:
                call(plan, s, rank)
            errors.append((e.type, str(e.value)))
            plan.close()
        assert errors[0] == errors[1], rank


@pytest.mark.parametrize("name", CALLS)
def test_raw_stream_handle(name):
    """A stream given as its integer handle: the binding's general path runs it,
    with the outputs of the native one."""
    side = torch.cuda.Stream()
    got = []
    for stream in (side, side.cuda_stream):
        plan, s = state("bf16")
        torch.cuda.synchronize()
        CALLS[name](plan, s, "bf16", stream=stream)
        torch.cuda.synchronize()
        got.append(outputs(s))
        plan.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))
