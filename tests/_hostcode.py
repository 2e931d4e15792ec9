"""Runs the library's own host code, and device code that compiles for the host,
without a GPU: what a kernel decides, which launches a call makes and what it asks
of the runtime.

`run` compiles a driver program for the host alone and returns what it prints; a
crash or a non-zero exit fails the test.  With `library`, every source of the
library is linked in, host code only, over the runtime of _fake_hip.h."""
import glob
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1002_3094_amd", "csrc")
FLAGS = ["--offload-arch=gfx950", "--cuda-host-only", "-x", "hip", "-O0", "-std=c++17", "-fPIC", "-w",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", HERE]


def _compile(src, obj):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *FLAGS, "-c", "-o", obj, src], check=True)
    return obj


_library = []   # the library's objects, compiled once per test session


def _library_objects(tmp_path_factory):
    if not _library:
        out = str(tmp_path_factory.mktemp("hostcode"))
        srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip"))) + [os.path.join(HERE, "_fake_hip.cpp")]
        with ThreadPoolExecutor(max_workers=4) as ex:
            objs = list(ex.map(lambda s: _compile(s, os.path.join(out, os.path.basename(s) + ".o")), srcs))
        # the device code that the host objects refer to is not built: empty stand-ins
        und = subprocess.run(["nm", "-u", *objs], capture_output=True, text=True, check=True).stdout
        names = sorted({w for w in und.split() if w.startswith("__hip_fatbin_")})
        stubs = os.path.join(out, "stubs.c")
        with open(stubs, "w") as f:
            f.write("".join(f"char {n}[8];\n" for n in names))
        subprocess.run(["gcc", "-fPIC", "-c", "-o", stubs + ".o", stubs], check=True)
        _library.extend([*objs, stubs + ".o"])
    return _library


def run(tmp_path_factory, driver, library=False):
    out = str(tmp_path_factory.mktemp("driver"))
    src = os.path.join(out, "driver.cpp")
    with open(src, "w") as f:
        f.write(driver)
    objs = [_compile(src, src + ".o")] + (list(_library_objects(tmp_path_factory)) if library else [])
    exe = os.path.join(out, "driver")
    subprocess.run(["g++", "-o", exe, *objs, "-lpthread"], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, (p.returncode, p.stdout[-2000:], p.stderr[-2000:])
    return p.stdout
