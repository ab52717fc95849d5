"""Small C++ programs that look at the library's host side and shared index code from inside, on the CPU:
compiled with g++ against the library's headers, linked with the built librelax.so, run as a child."""
import os
import shutil
import subprocess

import pytest

import paper_1405_0942_amd as R
from paper_1405_0942_amd import build as B

ROCM = "/opt/rocm"


def run(source, tmp_path, *args):
    """stdout of the program `source` (which exits with 0)."""
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("g++ or the HIP headers are not here")
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(source)
    libdir = os.path.dirname(R.LIB_PATH)
    cmd = ["g++", "-std=c++17", "-O1", "-w", "-rdynamic", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{B.CSRC}",
           f"-I{os.path.join(B.ROOT, 'include')}", str(src), "-o", str(exe), f"-L{libdir}", "-l:librelax.so",
           f"-L{ROCM}/lib", "-lamdhip64", f"-Wl,-rpath,{libdir}:{ROCM}/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"exit {r.returncode}\n{r.stdout}{r.stderr}"[-3000:]
    return r.stdout
