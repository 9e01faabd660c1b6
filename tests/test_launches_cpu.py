"""Which kernels a call enqueues, shown without a GPU: the library runs on the recording HIP runtime of
_hip_recorder.c, in a process of its own."""

import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, sys
sys.path.insert(0, {root!r})
rec = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
rec.rec_name.restype = ctypes.c_char_p
rec.rec_threads.restype = rec.rec_blocks.restype = ctypes.c_long
from paper_2203_01291_amd import _lib
lib = ctypes.CDLL(_lib.LIB_PATH)
for name, (res, args) in _lib.EXPORTS.items():
    getattr(lib, name).restype, getattr(lib, name).argtypes = res, args
P = ctypes.c_void_p(1 << 20)  # a device pointer that nothing reads
def lattice(L, Ltau):
    return _lib.Lattice(L, Ltau, 0.1, 1.0, 0.0, 1.0)
def handle(L, Ltau, n):
    h = ctypes.c_void_p()
    rc = lib.fph_create(ctypes.byref(h), ctypes.byref(lattice(L, Ltau)), n)
    return h if rc == 0 else rc
def opts(prec, precond=1, maxiter=2):
    return ctypes.byref(_lib.PcgOpts(1e-8, maxiter, precond, prec, 1, 0.0, 0, 0, 1, 0, 1.0, 1.0))
def names():
    out = [rec.rec_name(i).decode() for i in range(rec.rec_count())]
    rec.rec_reset()
    return out
out = {{}}
"""


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    from paper_2203_01291_amd import _lib
    gcc = shutil.which("gcc")
    if gcc is None or not os.path.exists(_lib.LIB_PATH):
        pytest.skip("needs gcc and the built library")
    so = str(tmp_path_factory.mktemp("rec") / "rec.so")
    subprocess.run([gcc, "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "_hip_recorder.c")], check=True)

    def run(body):
        code = PRELUDE.format(root=ROOT, so=so) + body + "\nprint(json.dumps(out))"
        r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout.splitlines()[-1])

    return run


# Block matrices are built in the precision a solve reads, once per field, and only where its series
# kernel reads any: not by k_kpm (FP32 L = 32 with many blocks), not for many right-hand sides.
def test_matrices_are_built_where_they_are_read(record):
    out = record("""
def solve(h, prec, n, sync=False):
    names()
    f = lib.pcg_solve_sync if sync else lib.pcg_solve
    assert f(h, n, P, P, opts(prec), P if not sync else None, None) == 0
    return sorted({"d" if "k_pc_denseId" in k else "f" for k in names()
                   if "k_pc_dense" in k and "done" not in k})
F64, F32 = _lib.FPH_F64, _lib.FPH_F32_REFINED
h = handle(32, 400, 10)
lib.fph_set_field(h, P, 1.0, 1.0, None)
out["unread"] = solve(h, F32, 10) + solve(h, F32, 3, True)
out["read"] = solve(h, F32, 2)
h = handle(16, 160, 40)
lib.fph_set_field(h, P, 1.0, 1.0, None)
out["many"] = solve(h, F64, 40) + solve(h, F32, 17)
out["f64"] = solve(h, F64, 4)
out["again"] = solve(h, F64, 4) + solve(h, F64, 7, True)
out["fewer"] = solve(h, F64, 1)
out["f32"] = solve(h, F32, 4, True)
rec.rec_capturing(1)
out["captured"] = solve(h, F64, 4)
rec.rec_capturing(0)
lib.fph_set_fields(h, 2, 2, P, 1.0, 1.0, None)
out["fields"] = solve(h, F64, 4)
""")
    assert out == {"unread": [], "read": ["f"], "many": [], "f64": ["d"], "again": [], "fewer": ["d"],
                   "f32": ["f"], "captured": ["d"], "fields": []}


# A handle needs no room for block matrices: refused, it runs the series.
def test_no_room_for_matrices(record):
    out = record("""
def built(h):
    names()
    lib.fph_set_field(h, P, 1.0, 1.0, None)
    assert lib.pcg_solve(h, 1, P, P, opts(_lib.FPH_F64), P, None) == 0
    return any("k_pc_dense" in k for k in names())
out["room"] = built(handle(16, 16, 1))
rec.rec_limit(ctypes.c_size_t(1 << 20))  # the matrices are 11 MB, all else is smaller
h = handle(16, 16, 1)
out["created"] = isinstance(h, ctypes.c_void_p)
out["built"] = built(h)
out["free"] = lib.fph_destroy(h)
rec.rec_limit(ctypes.c_size_t(1 << 10))
out["refused"] = handle(16, 16, 1)
""")
    assert out == {"room": True, "created": True, "built": False, "free": 0, "refused": -100}


# Threads of an untuned batch: more while a compute unit (256 of them) has one item, fewer once it has
# several, by unknowns and not by items.
def test_batch_shapes(record):
    out = record("""
def threads(*systems):
    arr = (_lib.System * len(systems))(*[_lib.System(lattice(L, Ltau), P, n, P, P) for L, Ltau, n in systems])
    b, got = ctypes.c_void_p(), []
    assert lib.fph_batch_create(ctypes.byref(b), arr, len(systems)) == 0
    for precond in (0, 1):
        rec.rec_reset()
        assert lib.fph_batch_solve(b, opts(_lib.FPH_F32_REFINED, precond), None, None) == 0
        got += [rec.rec_threads(i) for i in range(rec.rec_count()) if b"k_batch_solve" in rec.rec_name(i)]
    lib.fph_batch_destroy(b)
    return got
out["few small"] = threads((4, 40, 256))
out["many small"] = threads((4, 40, 257))
out["largest of the small"] = threads((16, 20, 300))
out["above"] = threads((8, 100, 300))
out["large"] = threads((16, 60, 100))
out["many large"] = threads((16, 60, 300))
out["wide"] = threads((32, 8, 16))
out["many wide"] = threads((32, 8, 1200))
out["uneven"] = threads((4, 40, 700), (16, 40, 20))
""")
    assert out == {"few small": [512, 512], "many small": [256, 256], "largest of the small": [256, 256],
                   "above": [512, 256], "large": [512, 1024], "many large": [512, 256], "wide": [512, 1024],
                   "many wide": [512, 256], "uneven": [512, 1024]}


# The series kernel: real and imaginary parts on separate lanes while the longest block sets the time; at
# 33 to 64 and 129 to 256 plaquettes by the load, at L = 32 in FP32 by the blocks.
def test_series_kernel_by_load(record):
    out = record("""
def kernel(L, Ltau, prec, n, a=(1.0, 1.0)):
    h = handle(L, Ltau, n)
    lib.fph_set_field(h, P, *a, None)
    names()
    assert lib.fph_precond_apply(h, _lib.FPH_PC_FFT, prec, n, P, P, None) == 0
    k = [(rec.rec_name(i).decode(), rec.rec_threads(i)) for i in range(rec.rec_count())]
    k = [("split" if "split" in name else "whole", t) for name, t in k if "k_kpm" in name]
    lib.fph_destroy(h)
    return k[0]
F64, F32 = _lib.FPH_F64, _lib.FPH_F32
S = (0.15, 12.0)  # short series, about as long at every frequency
out["L=10"] = [kernel(10, 32, p, 256, S) for p in (F64, F32)]
out["L=16"] = [kernel(16, 32, F64, 60), kernel(16, 32, F64, 31, S), kernel(16, 32, F64, 32, S)]
out["L=22"] = [kernel(22, 32, p, 64, S) for p in (F64, F32)]
out["L=24"] = [kernel(24, 32, F64, 35), kernel(24, 32, F64, 36), kernel(24, 32, F32, 8, S), kernel(24, 32, F32, 9, S)]
out["L=30"] = [kernel(30, 32, F64, 8, S), kernel(30, 32, F64, 9, S)]
out["L=32"] = [kernel(32, 32, F64, 33), kernel(32, 32, F32, 32), kernel(32, 32, F32, 33)]
out["L=34"] = [kernel(34, 4, F64, 1), kernel(34, 4, F32, 1)]
""")
    s, w = "split", "whole"
    assert out == {"L=10": [[s, 64], [s, 64]], "L=16": [[s, 128], [s, 128], [w, 64]], "L=22": [[s, 256], [s, 256]],
                   "L=24": [[s, 512], [w, 192], [s, 512], [w, 192]], "L=30": [[s, 512], [w, 256]],
                   "L=32": [[s, 512], [s, 512], [w, 256]], "L=34": [[w, 512], [w, 512]]}


# Every right-hand side's state is set before a solve.
def test_every_state_is_initialised(record):
    out = record("""
h = handle(16, 32, 200)
lib.fph_set_field(h, P, 1.0, 1.0, None)
for n in (1, 64, 65, 200):
    rec.rec_reset()
    assert lib.pcg_solve(h, n, P, P, opts(_lib.FPH_F64, 0), P, None) == 0
    k = [i for i in range(rec.rec_count()) if b"k_solve_init" in rec.rec_name(i)]
    out[n] = len(k) == 1 and rec.rec_blocks(k[0]) * rec.rec_threads(k[0]) >= n
""")
    assert out == {"1": True, "64": True, "65": True, "200": True}
