"""Packs a weight with the host-emulated library while device memory is short, and runs it.  Called as a subprocess by
tests/test_short_memory.py; prints one JSON line.
usage: python run_short_memory.py N K failing [pending] [copies] (bit i: the i-th device allocation of the pack fails; pending: the
error that some earlier call left for whoever asks next; bit i: the i-th copy finds no memory)"""
import ctypes
import json
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path.insert(0, ROOT)
sys.path.insert(0, HERE)


def main():
    N, K, failing, pending, copies = (int(v) for v in (sys.argv[1:] + ["0", "0"])[:5])
    os.environ["EMU_CUS"] = "4"
    import build_emu
    import paper_2306_16601_amd.binding as b
    b.LIB_PATH = build_emu.LIB
    import paper_2306_16601_amd as sp
    import oracle
    L = b.lib()
    L.emu_alloc.restype = ctypes.c_void_p
    L.emu_alloc.argtypes = [ctypes.c_size_t]
    M = 40
    rng = np.random.default_rng(N + K)
    W = np.where(rng.random((N, K)) < 0.1, rng.integers(-128, 128, (N, K)), 0).astype(np.int8)
    X = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    x, out = L.emu_alloc(X.nbytes), L.emu_alloc(4 * N * M)
    ctypes.memmove(x, X.ctypes.data, X.nbytes)
    whole = sp.spmm_pack(W)
    both = sp.spmm_info(whole)[4]
    sp.spmm_destroy(whole)
    before = L.emu_allocations()
    L.emu_fail_mallocs(failing)
    L.emu_fail_copies(copies)
    L.emu_leave_error(pending)
    try:
        h = sp.spmm_pack(W)
    except Exception as e:
        print(json.dumps({"error": str(e), "left": L.emu_allocations() - before}))
        return
    L.emu_fail_mallocs(0)
    error_left = L.emu_error_left()
    sp.spmm_set_tuning(h, 32, 134)
    kernel = sp.spmm_kernel_variant(h, M, "s32", "none")
    sp.spmm_run(h, x, M, M, sp.make_epilogue(None, 1.0, 0, None, "none", "s32"), out, M, None)
    got = np.empty((N, M), dtype=np.int32)
    ctypes.memmove(got.ctypes.data, out, got.nbytes)
    match = bool(np.array_equal(got, W.astype(np.int64) @ X.astype(np.int64)))
    unpacked = bool(np.array_equal(sp.spmm_unpack(h), W))
    device_bytes = sp.spmm_info(h)[4]
    sp.spmm_destroy(h)
    print(json.dumps({"match": match, "unpacked": unpacked, "kernel": kernel, "device_bytes": device_bytes, "both": both, "error_left": error_left,
                      "left": L.emu_allocations() - before}))


main()
