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
