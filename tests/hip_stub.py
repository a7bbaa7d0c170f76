"""The library bound to a HIP runtime without a device (hip_stub.cpp), for a child process that never loads
torch: ``run(code)`` runs ``code`` there with ``B`` (the binding), ``I`` (the instances), ``stub`` (the
runtime's controls), ``bind(plan)`` (a solver handle in host memory) and ``launches()`` (the kernels since
the last call) in scope."""
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SO = os.path.join(ROOT, "paper_2009_00481_amd", "libbddmp.so")

# each function at the version the library asks for
VERSIONS = """hip_4.2 { global: *; };
hip_4.3 { global: hipGraph*; hipStreamBeginCapture; hipStreamEndCapture; } hip_4.2;
"""

PRELUDE = """
import ctypes as C, sys
sys.path.insert(0, {root!r})
stub = C.CDLL({stub!r}, mode=C.RTLD_GLOBAL)
stub.stub_log.restype = C.c_char_p
import numpy as np
from paper_2009_00481_amd import binding as B, instances as I
L = B.lib()
assert "torch" not in sys.modules
_keep = []

def bind(plan):
    n = int(plan.stats.device_bytes)
    raw = np.zeros(n + 256, np.uint8)
    _keep.append(raw)
    h = C.c_void_p()
    B._check(L.bddmp_solver_bind(plan.h, C.c_void_p((raw.ctypes.data + 255) // 256 * 256), C.c_size_t(n), None, C.byref(h)))
    return h

def launches():
    out = stub.stub_log().decode().split()
    stub.stub_clear()
    return out
"""


def build(tmp) -> str:
    """Compiles the stub runtime into the folder tmp."""
    out = os.path.join(str(tmp), "libamdhip64.so")
    vers = os.path.join(str(tmp), "versions")
    with open(vers, "w") as f:
        f.write(VERSIONS)
    need = subprocess.run(["readelf", "-d", SO], capture_output=True, text=True, check=True).stdout
    soname = re.search(r"\[(libamdhip64\.so[^\]]*)\]", need).group(1)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-Wno-attributes",
                    "-I/opt/rocm/include", os.path.join(HERE, "hip_stub.cpp"), f"-Wl,-soname,{soname}",
                    f"-Wl,--version-script,{vers}", "-o", out], check=True)
    return out


def run(stub: str, code: str) -> str:
    """Standard output of code, run in a child process against the stub runtime."""
    env = dict(os.environ, BDDMP_HOST_ONLY_LIB=SO)
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, stub=stub) + code], cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
