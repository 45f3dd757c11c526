"""What libmeft asks of the HIP runtime, without a GPU: record([(shape, calls), ...]) makes the calls of the C ABI in a
process where tests/hip_recorder.c stands in for the runtime, and returns the launches, copies, event records and stream
waits of each entry, in order.  The call names "capture" and "no_capture" set what the runtime says of the stream from then on;
"flip N" has another thread call meft_debug_global_loads(1) while the N-th launch from then on is under way.
Addresses are made up; the library does not follow them on the host."""
import ctypes
import json
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2406_04984_amd", "libmeft.so")
STREAM = 0x77


def shape(T, d, n_blocks, block_size, top_e, top_k, dtype, flags=0):
    return [T, d, n_blocks * block_size, n_blocks, block_size, top_e, top_k, {"f32": 0, "bf16": 1}[dtype], 0, flags]


def record(jobs):
    with tempfile.TemporaryDirectory() as tmp:
        rec = os.path.join(tmp, "hip_recorder.so")
        subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-Wextra", "-o", rec,
                               os.path.join(ROOT, "tests", "hip_recorder.c"), "-ldl", "-pthread"])
        p = subprocess.run([sys.executable, os.path.abspath(__file__), rec], input=json.dumps(jobs), text=True,
                           stdout=subprocess.PIPE, stderr=subprocess.PIPE, timeout=300)
    assert p.returncode == 0, p.stderr[-4000:]
    return json.loads(p.stdout)


class _Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("T", "d", "N", "n_blocks", "block_size", "top_e", "top_k", "dtype",
                                              "activation")] + [("flags", ctypes.c_uint32)]


class _Rec(ctypes.Structure):
    _fields_ = [("what", ctypes.c_char * 8), ("name", ctypes.c_char * 256), ("grid", ctypes.c_uint32 * 3),
                ("block", ctypes.c_uint32 * 3), ("lds", ctypes.c_uint64), ("stream", ctypes.c_uint64),
                ("event", ctypes.c_uint64), ("dst", ctypes.c_uint64), ("src", ctypes.c_uint64),
                ("bytes", ctypes.c_uint64)]


def _main(rec_path):
    rec = ctypes.CDLL(rec_path, mode=ctypes.RTLD_GLOBAL)   # before the library: its symbols come first
    lib = ctypes.CDLL(LIB)
    rec.rec_at.restype = ctypes.POINTER(_Rec)
    sz, vp = ctypes.c_size_t, ctypes.c_void_p
    for f in (lib.meft_workspace_bytes, lib.meft_union_workspace_bytes):
        f.restype = sz

    def ptr(name):   # one address per operand, far apart
        names = ("h", "Wg", "K", "V", "block_idx", "block_score", "out", "idx", "act", "dOut", "dh", "dK", "dV",
                 "touched", "n_touched", "ws", "ws2")
        return vp((names.index(name) + 1) << 44)

    def call(s, what):
        p = ctypes.byref(s)
        ws = "ws2" if what.endswith("2") else "ws"
        n = (lib.meft_union_workspace_bytes if what.startswith("union") else lib.meft_workspace_bytes)(p)
        tail = (ptr(ws), sz(n), vp(STREAM))
        what = what.rstrip("2")
        if what == "route":
            return lib.meft_route(p, ptr("h"), ptr("Wg"), None, ptr("block_idx"), ptr("block_score"), *tail)
        if what == "fwd":
            return lib.meft_sparse_fwd(p, ptr("h"), ptr("K"), ptr("V"), ptr("block_idx"), ptr("out"), ptr("idx"),
                                       ptr("act"), *tail)
        if what == "bwd":
            return lib.meft_sparse_bwd(p, ptr("h"), ptr("K"), ptr("V"), ptr("idx"), ptr("act"), ptr("dOut"), ptr("dh"),
                                       ptr("dK"), ptr("dV"), ptr("touched"), ptr("n_touched"), *tail)
        if what == "stage":
            return lib.meft_hostkv_stage(p, ptr("block_idx"), ptr("K"), ptr("V"), *tail)
        if what == "union_fwd":
            return lib.meft_union_fwd(p, ptr("h"), ptr("K"), ptr("V"), ptr("idx"), ptr("out"), ptr("touched"),
                                      ptr("n_touched"), *tail)
        if what == "union_bwd":
            return lib.meft_union_bwd(p, ptr("h"), ptr("K"), ptr("V"), ptr("touched"), ptr("n_touched"), ptr("dOut"),
                                      ptr("dh"), ptr("dK"), ptr("dV"), *tail)
        raise ValueError(what)

    out = []
    for fields, calls in json.load(sys.stdin):
        s = _Shape(*fields)
        rec.rec_clear()
        rec.rec_capture(0)
        for c in calls:
            if c.endswith("capture"):
                rec.rec_capture(int(c == "capture"))
                continue
            if c.startswith("flip "):
                rec.rec_flip(int(c[5:]), lib.meft_debug_global_loads)
                continue
            rc = call(s, c)
            assert rc == 0, (fields, c, rc)
        if any(c.startswith("flip ") for c in calls):
            assert rec.rec_flipped(), calls
            lib.meft_debug_global_loads(0)
        rows = []
        for i in range(rec.rec_count()):
            r = rec.rec_at(i).contents
            rows.append(dict(what=r.what.decode(), name=r.name.decode(), grid=list(r.grid), block=list(r.block), lds=r.lds,
                             stream=r.stream, event=r.event, dst=r.dst, src=r.src, bytes=r.bytes))
        out.append(rows)
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main(sys.argv[1])
