"""The library's host sources built with g++ against a HIP runtime on host
memory (host_runtime.cpp), behind the ordinary binding: paths that need a
failing allocation or another current device are tested without a GPU."""

import concurrent.futures as cf
import contextlib
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2010_09746_amd import build as B
from paper_2010_09746_amd import qsim as Q

SOURCES = ["api.cpp", "server_api.cpp", "batch_api.cpp", "compiler.cpp"]
HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(maxsize=None)
def _built():
    tmp = tempfile.TemporaryDirectory(prefix="qsim_host_")
    flags = [f if f != "-O2" else "-O1" for f in B.CXX_FLAGS] + [
        "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include", "-Wno-unused", "-pthread"]
    srcs = [os.path.join(B.CSRC, s) for s in SOURCES] + [os.path.join(HERE, "host_runtime.cpp")]
    objs = [os.path.join(tmp.name, os.path.basename(s) + ".o") for s in srcs]
    with cf.ThreadPoolExecutor(len(srcs)) as ex:
        list(ex.map(lambda so: subprocess.run(["g++"] + flags + ["-c", so[0], "-o", so[1]], check=True),
                    zip(srcs, objs)))
    out = os.path.join(tmp.name, "libqsim_host.so")
    # symbols bind inside: torch's HIP runtime may be loaded in this process
    subprocess.run(["g++", "-shared", "-pthread", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", out] + objs, check=True)
    return tmp, out


@contextlib.contextmanager
def host_library():
    """The binding on the host build inside the with-block; gives the test's switches."""
    lib, path = Q._lib, Q.LIB_PATH
    Q._lib, Q.LIB_PATH = None, _built()[1]
    try:
        L = Q.load()
        L.host_set_budget.argtypes = [ctypes.c_size_t]
        L.host_used.restype = ctypes.c_size_t
        L.host_mallocs.restype = ctypes.c_long
        L.host_set_budget(2 ** 64 - 1)
        L.host_set_malloc_error(0)
        L.host_set_device(0)
        yield L
    finally:
        Q._lib, Q.LIB_PATH = lib, path
