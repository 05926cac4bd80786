"""Runs host code of the library against hip_stub.c, a stand-in for the HIP
runtime (no GPU): `run(code, env)` starts a child process in which `stub` and
`pmp` are the two libraries and `log()` is what the runtime was asked to do.
The child must not load torch: its HIP runtime would come first."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_1610_10061_amd", "libpmp.so")

PREAMBLE = """
import ctypes as C, os, sys, threading, time
stub = C.CDLL({stub!r}, mode=C.RTLD_GLOBAL)
pmp = C.CDLL({lib!r})
stub.stub_log.restype = C.c_char_p
stub.stub_fail_malloc.argtypes = [C.c_long]
pmp.pmp_last_error.restype = C.c_char_p
vp, i32, i64 = C.c_void_p, C.c_int32, C.c_int64
for f, a in dict(
        pmp_preprocess=[vp, i64, i32, i32, i32, C.c_uint32, vp, vp],
        pmp_eval_population=[vp, vp, i32, vp, vp, C.c_uint32, vp],
        pmp_eval_population_noalloc=[vp, vp, i32, vp, vp, C.c_uint32, vp],
        pmp_instance_destroy=[vp], pmp_instance_check=[vp, vp], pmp_instance_tables=[vp, vp, vp, vp, C.c_uint32, vp],
        pmp_ga_create=[vp, vp, vp], pmp_ga_step=[vp, i32, vp], pmp_ga_best=[vp, vp, vp, vp, vp], pmp_ga_destroy=[vp],
        pmp_batch_create=[vp, i32, vp], pmp_batch_step=[vp, i32, vp], pmp_batch_check=[vp, vp, vp], pmp_batch_destroy=[vp],
        pmp_batch_autotune=[vp, vp, vp], pmp_apsp=[vp, i64, i32, vp, i64, C.c_uint32, vp],
        pmp_hbp_reduce=[vp, vp, vp], pmp_hbp_destroy=[vp]).items():
    getattr(pmp, f).argtypes = a
ON_DEVICE, ASYNC = 1, 2


def log(*kinds):
    rows = [r.split() for r in stub.stub_log().decode().splitlines()]
    return [r for r in rows if not kinds or r[0] in kinds]


def clear():
    stub.stub_clear()


def new_stream():
    s = vp()
    stub.hipStreamCreateWithFlags(C.byref(s), 1)
    return s


def buf(bytes):
    p = vp()
    assert stub.hipMalloc(C.byref(p), C.c_size_t(bytes)) == 0
    return p


def ok(status):
    assert status == 0, (status, pmp.pmp_last_error())


def instance(n, m, p, flags=ON_DEVICE, stream=None, d=None):
    out = vp()
    ok(pmp.pmp_preprocess(d or buf(4 * n * m), m, n, m, p, flags, stream, C.byref(out)))
    return out


class Params(C.Structure):
    _fields_ = [("seed", C.c_uint64)] + [(k, i32) for k in (
        "population", "group_size", "generations", "saturation", "crossover_iters",
        "mutation_iters", "migration", "init")]


def ga(inst, P, NT=64):
    out = vp()
    ok(pmp.pmp_ga_create(inst, C.byref(Params(1, P, NT, 1000, 0, 0, 0, 0, 0)), C.byref(out)))
    return out


def batch(gas):
    out = vp()
    ok(pmp.pmp_batch_create((vp * len(gas))(*gas), len(gas), C.byref(out)))
    return out
"""


def build(folder):
    out = os.path.join(str(folder), "libhipstub.so")
    if not os.path.exists(out):
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-pthread",
                        os.path.join(HERE, "hip_stub.c"), "-o", out], check=True)
    return out


def run(folder, code, env=None):
    stub = build(folder)
    e = {k: v for k, v in os.environ.items() if not k.startswith("PMP_")}
    r = subprocess.run([sys.executable, "-c", PREAMBLE.format(stub=stub, lib=LIB) + code],
                       capture_output=True, text=True, timeout=100, env={**e, **(env or {})})
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout
