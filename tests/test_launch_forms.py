"""Which kernel each call launches, on the host: the library is loaded against
a stub of the HIP runtime that records launches by kernel name and runs
nothing (a child process, so that the real runtime is not in the way)."""

from __future__ import annotations

import itertools
import json
import os
import re
import subprocess
import sys

import pytest

import bench
from paper_2411_00284_amd import BucketPlan
from synth import WORKLOADS

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2411_00284_amd", "libfsdp_bucket.so")
CUS = 256


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """calls -> the kernels that each launched; and the names of all kernels
    in the library's device code (whose symbols end in .kd)."""
    stub = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-std=gnu99", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    os.path.join(HERE, "hip_stub.c"), "-o", stub], check=True)

    def demangled(names):
        out = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True, check=True).stdout
        return [n.replace("fsdp::(anonymous namespace)::", "").split("(", 1)[0].removeprefix("void ")
                for n in out.splitlines()]

    def run(calls):
        res = subprocess.run([sys.executable, os.path.join(HERE, "launch_worker.py"), stub, LIB], text=True,
                             input=json.dumps(calls), capture_output=True, timeout=120)
        assert res.returncode == 0, res.stderr
        got = json.loads(res.stdout)
        assert got["cus"] == CUS
        with open(LIB, "rb") as f:
            built = {n.decode() for n in re.findall(rb"(_ZN4fsdp\w+)\.kd", f.read())}
        assert set(got["kernels"]) <= built
        return [demangled(names) for names in got["launched"]], demangled(sorted(built))

    return run


def shard_of(world, tiles, per_tile=512):
    """A bucket whose rank 0 holds `tiles` reduction tiles (one parameter)."""
    return [[world * tiles * per_tile, 1]]


# What puts a reduction off the 16-byte grid: a segment's offset, the chunks'
# stride (one buffer only), an output.
OFF_GRID = {"offset": {"dims": [[9, 1], [64, 64]], "align": 1}, "stride": {"dims": [[28, 1]], "align": 1},
            "output": {"dims": [[64, 64]], "shift": 4}}


@pytest.mark.parametrize("why", OFF_GRID)
@pytest.mark.parametrize("tiles,form", [("full", "2, 4, true"), ("half", "4, 8, true"), ("auto", "4, 8, true")])
def test_forced_reduce_form_off_the_grid(launches, why, tiles, form):
    """A small shard off the grid: reduce_tiles="full" forces the form for
    large shards there too."""
    got, _ = launches([{"call": "rs_reduce", "world": 4, "tiles": tiles, **OFF_GRID[why]}])
    runs = "true" if tiles == "full" and why != "output" else "false"
    assert got == [[f"rs_reduce_kernel<ContigChunks, unsigned short, {form}, {runs}>"]]


@pytest.mark.parametrize("world,form", [(4, "1, 8, false, true"), (8, "1, 4, false, true"), (32, "1, 3, false, true")])
@pytest.mark.parametrize("tiles", ["full", "half", "auto"])
def test_forced_reduce_form(launches, tiles, world, form):
    small = "4, 8, false, false"
    got, _ = launches([{"call": "rs_reduce", "world": world, "tiles": tiles, "dims": [[world * 64, 64]]},
                       {"call": "rs_reduce", "world": world, "tiles": tiles, "dims": shard_of(world, 64 * CUS)}])
    want = {"full": [form, form], "half": [small, small], "auto": [small, form]}[tiles]
    assert got == [[f"rs_reduce_kernel<ContigChunks, unsigned short, {f}>"] for f in want]


@pytest.mark.parametrize("world,forms", [
    (1, {4: "4, 8, false", 5: "2, 8, false", 10: "1, 8, false", 31: "1, 8, false", 32: "1, 8, true",
         191: "1, 8, true", 192: "1, 8, false"}),
    (3, {192: "1, 8, false"}),
    (4, {191: "1, 8, true", 192: "1, 4, false"}),
    (7, {9: "2, 8, false", 10: "1, 8, false", 31: "1, 8, false", 32: "1, 8, true", 191: "1, 8, true",
         192: "1, 4, false"}),
    (8, {9: "2, 8, false", 10: "1, 8, false", 31: "1, 8, false", 32: "1, 4, true", 191: "1, 4, true",
         192: "1, 4, false"}),
    (11, {31: "1, 8, false", 32: "1, 4, true"}),
    (12, {25: "1, 8, false", 26: "1, 4, true", 191: "1, 4, true", 192: "1, 4, false"}),
    (31, {25: "1, 8, false", 26: "1, 4, true", 191: "1, 4, true", 192: "1, 4, false"}),
    (32, {25: "1, 8, false", 26: "1, 4, false", 31: "1, 4, false", 32: "1, 3, true", 95: "1, 3, true", 96: "1, 3, false"}),
    (128, {26: "1, 4, false", 31: "1, 4, false", 32: "1, 3, true", 96: "1, 3, false", 200: "1, 3, false"}),
])
def test_reduce_form_by_size(launches, world, forms):
    """Resident waves and tile order of a shard on the lines, on both sides of
    every bound; "sources in flight, resident waves, in runs"."""
    got, _ = launches([{"call": "rs_reduce", "world": world, "dims": shard_of(world, w * CUS)} for w in forms])
    want = [[n, m, "false", runs] for n, m, runs in (f.split(", ") for f in forms.values())]
    assert [g[0].rstrip(">").rsplit(", ", 4)[1:] for g in got] == want


def reduce_call(world, waves, wire="bf16", off=0, **more):
    """A reduction of `waves` waves per CU of five parameters whose segments
    start `off` elements past a 128-byte line."""
    n = waves * CUS * (256 if wire == "f32" else 512) // 5 // 64 * 64
    return {"call": "rs_reduce_ex" if more else "rs_reduce", "world": world, "wire": wire,
            "dims": [[off * world, 1]] * (off > 0) + [[n * world, 1]] * 5, **more}


OFF_LINES = {"segments": {"off": 8}, "chunks": {"chunk_shift": 16}, "f32 chunks": {"chunk_shift": 64, "wire": "f32"}}


@pytest.mark.parametrize("why", OFF_LINES)
@pytest.mark.parametrize("world,waves,form", [(8, 7, "2, 8"), (8, 20, "1, 8"), (48, 20, "1, 8"), (48, 100, "1, 3")])
def test_reduce_off_the_lines_in_runs(launches, why, world, waves, form):
    """Where the sources of most tiles are off the 128-byte lines, the tiles are
    dealt to the dies in runs; a few such tiles, or outputs there, change nothing."""
    few = reduce_call(world, waves)
    few["dims"] = few["dims"] + [[8 * world, 1], [56 * world, 1]]  # the chunks stay on the lines
    got, _ = launches([reduce_call(world, waves, **OFF_LINES[why]), few, reduce_call(world, waves, shift=64)])
    plain = [*form.split(", "), "false", "false>"]
    assert [n[0].rsplit(", ", 4)[1:] for n in got] == [[*form.split(", "), "false", "true>"], plain, plain]


@pytest.mark.parametrize("call", ["ag_unpack", "ag_unpack_ex", "rs_pack", "rs_pack_ex"])
@pytest.mark.parametrize("first,align,any_from", [(2048, 8, None), (2040, 8, 44), (2047, 1, 0)])
def test_copy_form_by_size(launches, call, first, align, any_from):
    """On the 16-byte grid the form that follows the 128-byte lines is for large
    buckets off the lines (44 tiles of 4 KB per CU); off the grid it is for all.
    Segments of `first` elements, and of whole tiles after it."""
    world, least = 8, (any_from or 0) * CUS // 8
    tiles = [2, 44 * CUS // 8 - 1, 44 * CUS // 8, 200 * CUS // 8]           # of one chunk
    # (the tables' chunks are on the lines whatever their length: only the second segment is off)
    got, _ = launches([{"call": call, "world": world, "dims": [[world * first, 1], [world * (t - 1) * 2048, 1]],
                        "align": align} for t in tiles])
    assert [g[0].endswith("true>") for g in got] == [any_from is not None and t >= least for t in tiles]


@pytest.mark.parametrize("grad", ["bf16", "f16"])
@pytest.mark.parametrize("first,align,shift", [(2048, 8, 0), (2040, 8, 0), (2047, 1, 0), (2048, 8, 64)])
def test_widening_pack_form_by_size(launches, grad, first, align, shift):
    """The widening pack does not write through off the 128-byte lines in buckets
    of 96 tiles of 1024 elements per CU and more; the gradients' place changes nothing."""
    world = 8
    tiles = [4, 96 * CUS // world - 1, 96 * CUS // world, 200 * CUS // world]       # of one chunk
    got, _ = launches([{"call": "rs_pack_ex", "world": world, "wire": "f32", "grad": grad, "align": align, "shift": shift,
                        "dims": [[world * first, 1], [world * (t - 2) * 1024, 1]]} for t in tiles])
    widen = {"bf16": 1, "f16": 2}[grad]
    assert [g[0] for g in got] == [
        f"rs_pack_kernel<TableChunks, {widen}, {'true' if first < 2048 and t >= tiles[2] else 'false'}>" for t in tiles]


def every_form():
    """Calls that between them take every branch of the dispatch."""
    small, large = [[64, 64], [9, 64]], [[64, 64], [40_000_000, 1]]
    odd = {"shift": 4, "align": 1}
    calls = []
    for wire in ("bf16", "f16", "f32"):
        for off in ({}, odd):
            calls += [{"call": "ag_pack_ex", "world": 2, "dims": dims, "wire": wire, **off} for dims in (small, large)]
            calls += [{"call": "ag_pack_push", "world": w, "dims": small, "wire": wire, **off} for w in (4, 8, 20)]
            calls += [{"call": "rs_pack_ex", "world": 4, "dims": small, "wire": wire, **off},
                      {"call": "ag_unpack_ex", "world": 4, "dims": small, "wire": wire, **off}]
            if wire != "f32":
                calls += [{"call": "rs_pack_ex", "world": 4, "dims": dims, "wire": "f32", "grad": wire, **off}
                          for dims in (small, [[9, 1], [40_000_000, 1]])]
    calls += [{"call": c, "world": 4, "dims": small, **off}
              for c in ("ag_pack", "ag_unpack", "rs_pack") for off in ({}, odd)]
    reduces = [("rs_reduce", "bf16"), ("rs_reduce_ex", "bf16"), ("rs_reduce_ex", "f16"), ("rs_reduce_ex", "f32")]
    for world, waves, (call, wire) in itertools.product((2, 8, 40), (1, 7, 20, 28, 40, 70, 100), reduces):
        dims = shard_of(world, waves * CUS, 256 if wire == "f32" else 512)
        calls += [{"call": call, "world": world, "wire": wire, "dims": d, "align": align}
                  for d, align in ((dims, 8), ([[8 * world, 1], *dims], 8), ([[9, 1], *dims], 1))]
        calls.append({"call": call, "world": world, "wire": wire, "dims": dims, "shift": 4})
    return calls


def test_every_kernel_is_reached(launches):
    """No kernel is built that no call launches."""
    launched, kernels = launches(every_form())
    assert all(launched)
    assert sorted(set(kernels) - {k for names in launched for k in names}) == []


@pytest.mark.parametrize("align", [8, 1])
def test_the_benchmark_names_the_kernels(launches, align):
    """The symbols that the benchmark gives for a call without a trace are the
    kernels that the library launches."""
    calls, names = [], []
    for wl in WORKLOADS.values():
        plan = BucketPlan(wl.world_size, wl.dims, align)
        for name, rank in itertools.product(bench.KERNELS, sorted({0, wl.world_size // 2, wl.world_size - 1})):
            if any(plan.local_elems(p, rank) for p in range(plan.num_params)):
                calls.append({"call": name, "world": wl.world_size, "dims": [list(d) for d in wl.dims], "rank": rank,
                              "align": align})
                names.append([bench.kernel_symbol(name, plan, rank, CUS)])
        plan.close()
    assert launches(calls)[0] == names
