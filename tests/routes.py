"""The layout that the library's host rules pick for a plain call (routes.cpp, compiled
against the built library on first use), so that a test can show that its cases reach the
path it is named for."""
import ctypes as C
import functools
import os
import subprocess
import tempfile
from collections import namedtuple

import numpy as np

from paper_2502_00115_amd import dses, synth

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
# windows: parts of a lane group's windows; parts: of a rotation's slabs
Route = namedtuple("Route", "bits wide nslabs pps sorted gref group windows arrange parts")


@functools.lru_cache(maxsize=None)
def _lib():
    dses.lib()
    out = os.path.join(tempfile.mkdtemp(), "routes.so")
    subprocess.check_call([
        "g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
        f"-I{ROCM}/include", f"-I{HERE}/../include", f"-I{os.path.dirname(dses.LIB_PATH)}/csrc",
        os.path.join(HERE, "routes.cpp"), "-o", out, dses.LIB_PATH, f"-L{ROCM}/lib", "-lamdhip64",
        f"-Wl,-rpath,{os.path.dirname(dses.LIB_PATH)}"])
    return C.CDLL(out)


def route(n, tgt, k, eps, box=1.0, lane_group=0, batched=False):
    tgt = np.ascontiguousarray(tgt, np.float32)
    out = (C.c_int32 * 10)()
    st = _lib().route(C.c_void_p(tgt.ctypes.data), len(tgt), n, k, C.c_float(eps),
                      C.c_float(box), lane_group, int(batched), out)
    assert st == 0, st
    return Route(*out)


def parts_and_sort_us(tgt, slabs, k):
    parts, sort = C.c_double(), C.c_double()
    _lib().parts_and_sort_us(C.c_void_p(tgt.ctypes.data), len(tgt), slabs, k, C.byref(parts),
                             C.byref(sort))
    return parts.value, sort.value


def clouds(n, m, seed, clustered=0):
    """A source cut from an m-point reference, moved and jittered, and five rotations;
    clustered: that many reference points lie within a tenth of a millimetre."""
    rng = np.random.default_rng(seed)
    shape = synth.multi_primitive_shape(rng)
    tgt = synth.sample_surface(rng, shape, m)
    if clustered:
        tgt[:clustered] = tgt[0] + rng.uniform(-5e-5, 5e-5, (clustered, 3))
    R, t = synth.random_transform(rng)
    src = synth.jitter(rng, synth.sample_surface(rng, shape, n), 0.01) @ R.T + t
    rot = synth.random_rotations(rng, 5).reshape(-1, 9)
    return tuple(np.ascontiguousarray(a, np.float32) for a in (src, tgt, rot))
