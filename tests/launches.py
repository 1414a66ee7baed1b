"""What the library's entry points launch, found out without a GPU: the launch functions of the HIP runtime are replaced
by tests/launch_recorder.c in a process of its own (pointers are made up and never read)."""
import ctypes as C
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2601_11676_amd", "libhalo.so")


def record(calls):
    """calls: dicts with fn (an entry point without its halo_ prefix), shape (d, n_groups, group_size, rank, dtype 0 | 1), T, K
    and, where it is not the queried one, ws (bytes), and where it is not 0, device (up to 7).  Returns per call (status, workspace bytes, [(kernel, grid x, y, z, threads)])."""
    with tempfile.TemporaryDirectory() as tmp:
        shim = os.path.join(tmp, "recorder.so")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(HERE, "launch_recorder.c")], check=True)
        p = subprocess.run([sys.executable, os.path.abspath(__file__), shim], input=json.dumps(calls), capture_output=True,
                           text=True, timeout=120)
    assert p.returncode == 0, p.stderr
    return [(rc, ws, [tuple(l) for l in launches]) for rc, ws, launches in json.loads(p.stdout)]


def _child(shim):
    recorder = C.CDLL(shim, mode=C.RTLD_GLOBAL)
    recorder.recorder_take.restype = C.c_char_p
    lib = C.CDLL(LIB)
    for f in (lib.halo_workspace_bytes, lib.halo_workspace_bytes_q4):
        f.restype = C.c_size_t
    p = C.c_void_p(1 << 30)
    null, other = C.c_void_p(0), C.c_void_p(1 << 31)
    out = []
    for c in json.load(sys.stdin):
        d, G, gs, rank, dtype = c["shape"]
        shape = C.byref((C.c_int32 * 6)(d, G * gs, gs, G, rank, dtype))
        recorder.recorder_device(c.get("device", 0))
        T, K, fn = C.c_int32(c["T"]), C.c_int32(c.get("K", 0)), c["fn"]
        q4 = fn.endswith("_q4")
        size = lib.halo_workspace_bytes_q4 if q4 else lib.halo_workspace_bytes
        ws = c.get("ws", size(shape, T, K))
        w = [p] * (6 if q4 else 3)
        tail = [p, C.c_size_t(ws), null]
        args = {"predict_scores": [p, T, p, p, p],
                "group_sparse_ffn": [p, T, *w, p, p],
                "ffn_forward": [p, p, T, p, p, *w, K, p, 4, null, p, null, null, null, null, null, null],
                "ffn_forward_ahead": [p, T, *w, p, p, other, p, p, K, p, 4, null, null, null, null, other, null, null],
                }[fn.replace("_q4", "")]
        rc = getattr(lib, "halo_" + fn)(shape, *args, *tail)
        lines = recorder.recorder_take().decode().split("\n")[:-1]
        out.append((rc, ws, [(n, *map(int, rest)) for n, *rest in map(str.split, lines)]))
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _child(sys.argv[1])
