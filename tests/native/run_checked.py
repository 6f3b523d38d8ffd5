"""Runs hadfl_local_steps of the networks read from standard input (JSON) on the stand-in for the HIP runtime
(launch_check.cpp, already built: first argument) and writes a report and the kernels' names for each.  A process of its own:
the stand-in has to be loaded before the library and torch's HIP runtime must not be."""
import ctypes
import json
import sys
import types

import numpy as np

fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.check_report.restype = fake.check_trace.restype = ctypes.c_char_p
sys.modules["torch"] = types.ModuleType("torch")
from paper_2111_08274_amd import hadfl  # noqa: E402


def buffer(n):
    """n zero bytes, 256-byte aligned, untouched pages"""
    a = np.zeros(n + 512, dtype=np.uint8)
    at = -a.ctypes.data % 256
    return a[at:at + n]


def run(case):
    n = len(case["ratio"])
    cfg = hadfl.make_config(n, 1, net="custom", bf16=case["bf16"], batch=case["batch"], n_samples=2 * case["batch"],
                            in_shape=case["shape"], n_classes=case["classes"], lr=0.1, momentum=case.get("momentum", 0.9), custom_ops=case["ops"])
    pb, sb = hadfl.workspace_bytes(cfg)
    bufs = [buffer(v) for v in (pb, sb, 8 * n * case["batch"] * int(np.prod(case["shape"])), 8 * n * case["batch"],
                                4 * hadfl.param_count(cfg)[1])]
    spans = (ctypes.c_ulonglong * 10)(*[v for b in bufs for v in (b.ctypes.data, b.size)])
    fake.check_reset(spans, len(bufs))
    h, ptr = ctypes.c_void_p(), [b.ctypes.data for b in bufs]
    ratio = np.asarray(case["ratio"], dtype=np.int32)
    L = hadfl.lib()
    hadfl._check(L.hadfl_init_replicas(ctypes.byref(cfg), ptr[4], ptr[0], ptr[1], ptr[2], ptr[3], hadfl._np_ptr(ratio), None, ctypes.byref(h)))
    for option, value in case.get("options", []):
        hadfl._check(L.hadfl_set_option(h, option, value), h)
    if "steps" in case:
        hadfl._check(L.hadfl_set_steps(h, hadfl._np_ptr(np.asarray(case["steps"], dtype=np.int32))), h)
    if case.get("profile"):
        hadfl._check(L.hadfl_profile_enable(h, 2))
    status = L.hadfl_local_steps(h)
    out = dict(status=status, report=fake.check_report().decode(), trace=fake.check_trace().decode().split())
    if case.get("profile"):
        rows, count = (hadfl.HadflKernelTime * 256)(), ctypes.c_int32()
        hadfl._check(L.hadfl_profile_read(h, rows, 256, ctypes.byref(count)), h)
        out["profile"] = {r.name.decode(): [r.launches, r.flops, r.bytes] for r in rows[:count.value]}
    L.hadfl_destroy(h)
    return out


json.dump([run(c) for c in json.load(sys.stdin)], sys.stdout)
