"""Child of test_launch_forms.py: calls of the library against tests/hip_stub.c.

``launch_worker.py STUB LIB`` reads a JSON list of calls on stdin and prints
the mangled names of the kernels that each launched, and of all there are.
Every address is made up: nothing is read or written.
"""

import ctypes
import json
import sys

CODE = {"bf16": 0, "f32": 1, "f16": 2}
SIZE = {"bf16": 2, "f32": 4, "f16": 2}
TILES = {"auto": 0, "full": 1, "half": 2}
PLACE = 1 << 40


class Options(ctypes.Structure):
    _fields_ = [("max_workgroups", ctypes.c_int64), ("reduce_tiles", ctypes.c_int32), ("reserved", ctypes.c_int32)]


def main():
    stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    lib = ctypes.CDLL(sys.argv[2])
    stub.stub_kernel.restype = stub.stub_launch.restype = ctypes.c_char_p
    lib.fsdp_plan_chunk_elems.restype = lib.fsdp_plan_local_rows.restype = ctypes.c_int64
    lib.fsdp_last_error.restype = ctypes.c_char_p
    at = [PLACE]

    def place(nbytes, shift=0):
        """An address `shift` bytes past a 512-byte boundary, of its own."""
        p = at[0] + shift
        at[0] = (p + max(nbytes, 1) + 511) // 512 * 512
        return p

    def array(addresses):
        return (ctypes.c_void_p * len(addresses))(*addresses)

    launched = []
    for c in json.load(sys.stdin):
        W, dims, rank, shift = c["world"], c["dims"], c.get("rank", 0), c.get("shift", 0)
        n = len(dims)
        plan, options = ctypes.c_void_p(), Options(0, TILES[c.get("tiles", "auto")], 0)
        rows, inner = (ctypes.c_int64 * n)(*[d[0] for d in dims]), (ctypes.c_int64 * n)(*[d[1] for d in dims])
        status = lib.fsdp_bucket_plan_ex(W, n, rows, inner, c.get("align", 8), ctypes.byref(options),
                                         ctypes.byref(plan))
        assert status == 0, c
        S = lib.fsdp_plan_chunk_elems(plan)
        local = [lib.fsdp_plan_local_rows(plan, p, rank) * dims[p][1] for p in range(n)]
        wire = c.get("wire", "bf16")
        grad = c.get("grad", wire)
        call, e = c["call"], CODE[wire]
        shards = array([place(4 * k, shift) for k in local])
        full = array([place(4 * a * b, shift) for a, b in dims])
        one = ctypes.c_void_p(place(S * SIZE[wire] * (1 if call.startswith("ag_pack") else W)))
        chunks = array([place(S * SIZE[wire], c.get("chunk_shift", 0)) for _ in range(W)])
        stub.stub_reset()
        args = {"ag_pack": (rank, shards, one), "ag_unpack": (one, full), "rs_pack": (full, one),
                "rs_reduce": (rank, one, shards), "ag_pack_ex": (rank, shards, e, one),
                "ag_pack_push": (rank, shards, e, chunks), "ag_unpack_ex": (e, chunks, full),
                "rs_pack_ex": (CODE[grad], full, e, chunks), "rs_reduce_ex": (rank, e, chunks, shards)}[call]
        status = getattr(lib, "fsdp_" + call)(plan, *args, None)
        assert status == 0, (c, status, lib.fsdp_last_error())
        launched.append([stub.stub_launch(k).decode() for k in range(stub.stub_launches())])
        lib.fsdp_plan_free(plan)
    print(json.dumps({"launched": launched, "cus": stub.stub_cus(),
                      "kernels": [stub.stub_kernel(k).decode() for k in range(stub.stub_kernels())]}))


main()
