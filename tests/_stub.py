"""The library's host code on the stub of the HIP calls (tests/host/hip_stub.cpp), built on first use: a
binding of its own beside the product's, and the stub's counters."""
import ctypes
import importlib.util
import os
import shutil
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
HAVE = shutil.which(HIPCC) is not None and shutil.which("g++") is not None
_loaded = None


def _build(folder):
    csrc, host = os.path.join(ROOT, "paper_2306_04467_amd", "csrc"), os.path.join(ROOT, "tests", "host")
    include = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(HIPCC)))), "include")
    objs = [os.path.join(folder, n) for n in ("api.o", "mesh.o", "stub.o")]
    gxx = ["g++", "-O1", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-isystem", include, "-c"]
    jobs = [[HIPCC, "-O1", "-std=c++17", "-fPIC", "--offload-host-only", "--offload-arch=gfx950", "-fuse-cuid=none", "-c",
             os.path.join(csrc, "gks_api.hip"), "-o", objs[0]],
            gxx + [os.path.join(csrc, "mesh_setup.cpp"), "-o", objs[1]],
            gxx + [os.path.join(host, "hip_stub.cpp"), "-o", objs[2]]]
    for p in [subprocess.Popen(j, stderr=subprocess.DEVNULL) for j in jobs]:
        assert p.wait(timeout=600) == 0
    lib = os.path.join(folder, "libgks_stub.so")
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *objs, "-o", lib, "-pthread"], check=True, timeout=600)
    return lib


def load():
    """(binding, stub): the package's binding on the stubbed library, and the library with its counters."""
    global _loaded
    if _loaded is None:
        with tempfile.TemporaryDirectory() as folder:
            before = os.environ.get("GKS_LIBRARY")
            os.environ["GKS_LIBRARY"] = _build(folder)
            try:
                spec = importlib.util.spec_from_file_location(
                    "gks_on_stub", os.path.join(ROOT, "paper_2306_04467_amd", "gks.py"))
                gks = importlib.util.module_from_spec(spec)
                spec.loader.exec_module(gks)
                stub = gks.load()
            finally:
                if before is None:
                    del os.environ["GKS_LIBRARY"]
                else:
                    os.environ["GKS_LIBRARY"] = before
        stub.stub_stream.restype = ctypes.c_void_p
        stub.stub_stream_free.argtypes = [ctypes.c_void_p]
        stub.stub_capture.argtypes = [ctypes.c_void_p, ctypes.c_int]
        stub.stub_malloc_limit.argtypes = [ctypes.c_size_t]
        stub.stub_count.argtypes, stub.stub_count.restype = [ctypes.c_char_p], ctypes.c_long
        _loaded = gks, stub
    return _loaded


def count(stub, what):
    return stub.stub_count(what.encode())
