"""The library's host code linked with host_stub.cpp in place of the HIP
runtime, and scripts run on it in a child process."""
import concurrent.futures as cf
import os
import re
import shutil
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0712_0813_amd", "csrc")

PRELUDE = """
import ctypes, sys, threading
sys.path.insert(0, {root!r})
sys.modules["torch"] = None   # the stand-in is the only runtime here
from paper_0712_0813_amd import ce
ce.LIB_PATH = {lib!r}
lib = ce.load_library()
lib.stub_calls.restype = lib.stub_blocks.restype = ctypes.c_long
lib.stub_fail.argtypes = [ctypes.c_char_p, ctypes.c_long]
def calls(name):
    return lib.stub_calls(name.encode())
COOP, KERNEL = "hipLaunchCooperativeKernel", "hipLaunchKernel"
SPEC = ce.make_init_spec(1, [3.0, 3.0, 3.0])
def params(dims, N, nf, **kw):
    return ce.make_params(dims, N, nf, 0.15 * N, 0.01, **kw)
def sim(dims, N, nf, **kw):
    s = ce.Simulation(dims, N, nf, 0.15 * N, 0.01, **kw)
    s.generate(SPEC)
    return s
"""


_built = []   # one library serves every module of a run


def build(folder) -> str:
    if not _built:
        _built.append(_build(folder))
    return _built[0]


def _build(folder) -> str:
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not available")
    from paper_0712_0813_amd import build as libbuild
    base = [hipcc, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-ffp-contract=off",
            "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    jobs, objs = [], []
    for src, extra, name in libbuild.compile_units():
        objs.append(str(folder / name))
        jobs.append(base + extra + ["-c", src, "-o", objs[-1]])
    objs.append(str(folder / "stub.o"))
    jobs.append(["g++", "-O1", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-c",
                 os.path.join(ROOT, "tests", "host_stub.cpp"), "-o", objs[-1]])
    with cf.ThreadPoolExecutor(8) as ex:
        for r in ex.map(lambda c: subprocess.run(c, capture_output=True, text=True, timeout=600), jobs):
            assert r.returncode == 0, r.stderr[-2000:]
    # no device code: the names the objects register are defined empty
    nm = subprocess.run(["nm", "-u"] + objs, capture_output=True, text=True).stdout
    fat = folder / "fat.c"
    fat.write_text("".join(f"char {n}[8];\n" for n in sorted(set(re.findall(r"\b__hip_fatbin_\w+", nm)))))
    lib = str(folder / "libce_stub.so")
    r = subprocess.run(["g++", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", lib, "-x", "c", str(fat), "-x", "none", *objs, "-lpthread"],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    return lib


def run(lib: str, script: str) -> str:
    code = PRELUDE.format(root=ROOT, lib=lib) + textwrap.dedent(script) + "\nprint('script done')\n"
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "script done" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout
