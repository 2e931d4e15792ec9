"""Compiles pieces of the library's HIP sources for the host alone and runs them
here: what a kernel decides, or what a launcher asks of the HIP runtime, can be
checked without a GPU.

`run` builds one program out of a driver text and, optionally, sources of the
library; with sources, the HIP runtime is a small fake of the test's own, whose
calls the driver sees (device memory is host memory, launches do nothing)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1002_3094_amd", "csrc")


def run(tmp_path, driver, sources=()):
    """Output of the program; a crash or a non-zero exit fails the test."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    text = os.path.join(str(tmp_path), "driver.hip")
    with open(text, "w") as f:
        f.write(driver)
    objs = []
    for src in [text] + [os.path.join(CSRC, s) for s in sources]:
        obj = os.path.join(str(tmp_path), os.path.basename(src) + ".o")
        subprocess.run([hipcc, "--offload-arch=gfx950", "--cuda-host-only", "-O0", "-std=c++17", "-fPIC", "-w",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", "-o", obj, src], check=True)
        objs.append(obj)
    exe = os.path.join(str(tmp_path), "driver")
    subprocess.run(["g++", "-o", exe, *objs], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, (p.returncode, p.stdout[-2000:], p.stderr[-2000:])
    return p.stdout
