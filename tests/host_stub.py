"""Runs the library's host code over the HIP stand-in (helpers/hip_stub.cpp) in
a process of its own: no GPU is used or needed, and calls can be watched and
made to fail."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, re, sys
S = C.CDLL({so!r}, mode=C.RTLD_GLOBAL)
S.stub_log.restype = C.c_char_p
S.stub_device_block.restype = C.c_void_p
sys.path.insert(0, {root!r})
import numpy as np
import workloads
from paper_2512_02175_amd import binding as B
B._torch_stream = lambda: None
L = B.lib()
def log():
    return S.stub_log().decode().splitlines()
def fail(name, skip=0, count=1 << 30):
    S.stub_fail(name.encode(), skip, count)
def steps(lines):
    # the step launches: (kernel, grid, arguments)
    out = []
    for l in lines:
        m = re.match(r"(?:launch|node) (\\S*(?:k_pool|k_step|k_batch)\\S*) grid=(\\d+).* nsteps=", l)
        if m and "reset" not in m[1]:
            out.append((m[1], int(m[2]), {{k: int(v) for k, v in re.findall(r"(\\w+)=(\\d+)", l)}}))
    return out
"""


def build(tmp):
    so = os.path.join(str(tmp), "hip_stub.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-o", so,
                    os.path.join(HERE, "helpers", "hip_stub.cpp")], check=True)
    return so


def run(so, code, **env):
    """The standard output of the code, run after PRELUDE."""
    e = {k: v for k, v in os.environ.items() if k != "MG_TUNE_CACHE"}
    e.update(env)
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(so=so, root=ROOT) + code], env=e,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
