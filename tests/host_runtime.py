"""The library's host code built against the stand-in runtime of fake_hip.cpp
(kernel launchers that it does not define return success)."""
from __future__ import annotations

import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def build(out_dir) -> str:
    out = os.path.join(str(out_dir), "libswe_host.so")
    cxx = ["g++", "-O1", "-g", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w"]
    src = {"api": os.path.join(ROOT, "paper_2311_11348_amd", "csrc", "swe_api.cpp"),
           "fake": os.path.join(HERE, "fake_hip.cpp")}
    obj = {k: os.path.join(str(out_dir), k + ".o") for k in src}
    jobs = [subprocess.Popen([*cxx, "-c", src[k], "-o", obj[k]]) for k in src]
    assert [j.wait() for j in jobs] == [0, 0]

    def names(k, flag):
        r = subprocess.run(["nm", flag, obj[k]], capture_output=True, text=True, check=True)
        return {line.split()[-1] for line in r.stdout.splitlines()}

    missing = sorted(n for n in names("api", "-u") - names("fake", "--defined-only") if n.startswith("_ZN3swe"))
    stubs = os.path.join(str(out_dir), "stubs.c")
    with open(stubs, "w") as f:
        f.writelines(f"int {n}(void) {{ return 0; }}\n" for n in missing)
    subprocess.run(["gcc", "-fPIC", "-c", stubs, "-o", stubs + ".o"], check=True)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", out, obj["api"], obj["fake"], stubs + ".o",
                    "-lpthread"], check=True)
    return out


PRELUDE = """
import ctypes, sys, threading
sys.path.insert(0, {root!r})
import numpy as np
from paper_2311_11348_amd import inputs as I, swe
swe.LIB_PATH = {lib!r}
L = swe.lib()
L.fake_count.restype = ctypes.c_long
count = lambda what: int(L.fake_count(what.encode()))

"""


def run(lib: str, body: str) -> None:
    """The body in a process of its own, which has to end well."""
    text = PRELUDE.format(root=ROOT, lib=lib) + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
