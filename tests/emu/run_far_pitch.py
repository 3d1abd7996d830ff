"""One SpMM of the host-emulated library whose rows lie 2^40 elements apart (the largest pitch the library takes), in
reserved address space of which only the rows themselves are backed by memory.  Called as a subprocess by
tests/test_far_pitches.py; prints one JSON line.
usage: python run_far_pitch.py out_type with_sum"""
import ctypes
import json
import mmap
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path.insert(0, ROOT)
sys.path.insert(0, HERE)
PITCH = 1 << 40
libc = ctypes.CDLL(None, use_errno=True)
libc.mmap.restype = ctypes.c_void_p
libc.mmap.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long]
libc.mprotect.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
NORESERVE = 0x4000


def far_rows(rows, M, dtype):
    """Address of a [rows][PITCH] matrix and its rows as arrays of M elements."""
    item = np.dtype(dtype).itemsize
    base = libc.mmap(None, (rows - 1) * PITCH * item + mmap.PAGESIZE, 0, mmap.MAP_PRIVATE | mmap.MAP_ANONYMOUS | NORESERVE, -1, 0)
    assert base not in (None, ctypes.c_void_p(-1).value), os.strerror(ctypes.get_errno())
    out = []
    for r in range(rows):
        at = base + r * PITCH * item
        assert libc.mprotect(at, mmap.PAGESIZE, mmap.PROT_READ | mmap.PROT_WRITE) == 0
        out.append(np.frombuffer((ctypes.c_char * (M * item)).from_address(at), dtype=dtype))
    return base, out


def main():
    out_type, with_sum = sys.argv[1], sys.argv[2] == "1"
    os.environ["EMU_CUS"] = "4"
    import build_emu
    import paper_2306_16601_amd.binding as b
    b.LIB_PATH = build_emu.LIB
    import paper_2306_16601_amd as sp
    import oracle
    N, K, M = 3, 2, 21
    rng = np.random.default_rng(40)
    W = rng.integers(-127, 128, size=(N, K), dtype=np.int8)
    X = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    scale, bias = rng.uniform(0.5, 1.0, N).astype(np.float32), rng.standard_normal(N).astype(np.float32)
    R = rng.standard_normal((N, M)).astype(np.float32)
    x_at, x_rows = far_rows(K, M, np.uint8)
    o_at, o_rows = far_rows(N, M, {"s8": np.int8, "f32": np.float32}[out_type])
    for k in range(K):
        x_rows[k][:] = X[k]
    s_at, ld_sum = None, 0
    if with_sum:
        s_at, s_rows = far_rows(N, M, np.float32)
        ld_sum = PITCH
        for n in range(N):
            s_rows[n][:] = R[n]
    h = sp.spmm_pack(W)
    ep = sp.make_epilogue(scale.ctypes.data, 0.01, 0, bias.ctypes.data, "none", out_type, 2.0, 3, 1.0, None, s_at, ld_sum)
    sp.spmm_run(h, x_at, M, PITCH, ep, o_at, PITCH, None)
    ref = oracle.spmm(W, X, scale, 0.01, bias, "none", out_type, 2.0, 3, 1.0, 0, **({"sum": R} if with_sum else {}))
    print(json.dumps({"match": bool(np.array_equal(np.stack(o_rows), ref))}))


main()
