"""Which kernels a call of the C ABI launches, seen without a GPU.

``record(calls)`` runs the calls in a process of its own whose HIP runtime is
``hip_recorder.cpp``: launches are noted, nothing runs, pointers are never
followed. Only the host side of the library is exercised (its checks and its
choice of kernels and grids).
"""
from __future__ import annotations

import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2607_04164_amd", "libbrownout_moe.so")
PTR = 1 << 20  # 256-byte aligned, never followed


def ffn_part(part, n_seg, rows_cap, d, d_ff, dtype=1, workspace=False, **device):
    """A call of one GEMM of the FFN: ``part`` is "up" or "down"."""
    ws = [["p", PTR if workspace else 0], ["z", (1 << 32) if workspace else 0], ["p", 0]]
    ptrs = {"up": 5, "down": 4}[part]  # offsets, operands and the output
    return {"fn": {"up": "brownout_moe_ffn_gate_up", "down": "brownout_moe_ffn_down"}[part],
            "args": [["i", v] for v in (dtype, n_seg, rows_cap, d, d_ff)] + [["p", PTR]] * ptrs + ws, **device}


def record(calls, tmp_path):
    """For each call (status, [(kernel, grid), ...]); a call may name the
    device's answers: device, device_status, cus, cus_status."""
    so = os.path.join(str(tmp_path), "hip_recorder.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_recorder.cpp")], check=True)
    out = subprocess.run([sys.executable, os.path.abspath(__file__), so, LIB], input=json.dumps(calls), text=True,
                         capture_output=True, timeout=120)
    assert out.returncode == 0, out.stderr
    return [(r["status"], [(n, tuple(g)) for n, g in r["launches"]]) for r in json.loads(out.stdout)]


def _main(recorder, lib):
    import ctypes
    rec = ctypes.CDLL(recorder, mode=ctypes.RTLD_GLOBAL)
    rec.recorder_name.restype = ctypes.c_char_p
    bmoe = ctypes.CDLL(lib)
    kinds = {"i": ctypes.c_int32, "p": ctypes.c_void_p, "z": ctypes.c_size_t}
    res = []
    for c in json.load(sys.stdin):
        rec.recorder_device(c.get("device", 0), c.get("device_status", 0), c.get("cus", 256), c.get("cus_status", 0))
        status = getattr(bmoe, c["fn"])(*[kinds[k](v) for k, v in c["args"]])
        grid = (ctypes.c_uint32 * 3)()
        launches = []
        for i in range(rec.recorder_count()):
            rec.recorder_grid(i, grid)
            launches.append([rec.recorder_name(i).decode(), list(grid)])
        res.append({"status": status, "launches": launches})
    print(json.dumps(res))


if __name__ == "__main__":
    _main(*sys.argv[1:])
