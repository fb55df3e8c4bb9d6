"""The library's host code on a machine without a GPU.

Every unit of csrc is compiled for the host only and linked with
tests/host_stub.cpp, which stands in for the HIP runtime, rocBLAS, rocSOLVER
and roctx: device memory is zeroed host memory, copies are memcpy, kernels and
library routines do nothing, and every call is one line of a log.  The result,
tests/_build/libsparchost.so (ignored by git), has the C ABI of the library, so
tests can check on the CPU what the host side allocates, copies, waits for and
launches."""
import ctypes
import glob
import os
import re
import shutil
import subprocess

import numpy as np

from paper_1603_04334_amd import binding, inputs

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1603_04334_amd", "csrc")
BUILD = os.path.join(HERE, "_build", "host")
LIB = os.path.join(HERE, "_build", "libsparchost.so")
STUB = os.path.join(HERE, "host_stub.cpp")
HIPCC = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")

_lib = None


def available():
    return os.path.exists(HIPCC) and shutil.which("nm") is not None


def _build():
    os.makedirs(BUILD, exist_ok=True)
    headers = glob.glob(os.path.join(CSRC, "*.hpp")) + [binding.HEADER]
    newest = max(os.path.getmtime(h) for h in headers)
    cmd = [HIPCC, "-std=c++17", "-O1", "-g", "-fPIC", "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-c"]
    objs, todo = [], []
    for src in sorted(glob.glob(os.path.join(CSRC, "*.hip"))) + [STUB]:
        obj = os.path.join(BUILD, os.path.basename(src) + ".o")
        objs.append(obj)
        if not os.path.exists(obj) or os.path.getmtime(obj) < max(newest, os.path.getmtime(src)):
            todo.append([*cmd, src, "-o", obj])
    if not todo and os.path.exists(LIB) and os.path.getmtime(LIB) >= max(map(os.path.getmtime, objs)):
        return
    while todo:
        part, todo = todo[:8], todo[8:]
        procs = [subprocess.Popen(c, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True) for c in part]
        for p in procs:
            text, _ = p.communicate()
            assert p.returncode == 0, text
    # the units refer to device code that a host-only compilation has none of
    names = subprocess.run(["nm", "--undefined-only", *objs], capture_output=True, text=True, check=True).stdout
    code = os.path.join(BUILD, "fatbin.c")
    with open(code, "w") as f:
        for n in sorted(set(re.findall(r"__hip_fatbin_[0-9a-f]+", names))):
            f.write(f"char {n}[64];\n")
    subprocess.run(["gcc", "-fPIC", "-c", code, "-o", code + ".o"], check=True)
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-o", tmp, *objs, code + ".o", "-lpthread"], check=True)
    os.replace(tmp, LIB)


def load():
    """The host library with the binding's signatures."""
    global _lib
    if _lib is None:
        _build()
        L = ctypes.CDLL(LIB)
        for name, (res, args) in binding._SIGS.items():
            fn = getattr(L, name)
            fn.restype, fn.argtypes = res, args
        L.stub_log.restype = ctypes.c_char_p
        L.stub_throw.argtypes = [ctypes.c_char_p]
        _lib = L
    return _lib


def calls(*names):
    """The logged calls of these names (all: none given), in order: (name, {field: value})."""
    out = []
    for line in load().stub_log().decode().splitlines():
        name, _, rest = line.partition(" ")
        if names and name not in names:
            continue
        fields = dict(re.findall(r"(\w+)=(\S+)", rest.split(" name=")[0]))
        if " name=" in rest:
            fields["name"] = rest.split(" name=")[1]
        out.append((name, {k: _value(k, v) for k, v in fields.items()}))
    return out


def _value(key, v):
    if key == "name":
        return v
    if key in ("grid", "block"):
        return tuple(int(x) for x in v.split(","))
    if v == "(nil)":
        return 0
    return int(v, 16) if v.startswith("0x") else int(v)


def create(cluster):
    """sparc_op_create of an inputs.Cluster: (status, handle)."""
    g, atoms, veff, keep = binding._cluster_arrays(cluster)
    h = ctypes.c_void_p()
    st = load().sparc_op_create(ctypes.byref(g), veff.ctypes.data_as(binding._dp), len(cluster.atoms), atoms,
                                ctypes.byref(h))
    return st, h


def cluster(n, boxes, nproj=2, h=0.5, radius=6, seed=1):
    """A cluster with one atom per (lo, ext) box and random projector values."""
    rng = np.random.default_rng(seed)
    atoms = [inputs.Atom(pos=np.zeros(3), Z=1, sigma=1.0, lo=tuple(lo), ext=tuple(ext),
                         chi=rng.standard_normal((nproj, *ext)), gamma=rng.uniform(0.5, 1.0, nproj))
             for lo, ext in boxes]
    return inputs.Cluster(n=tuple(n), h=h, radius=radius, veff=rng.standard_normal(int(np.prod(n))), atoms=atoms,
                          seed=seed)
