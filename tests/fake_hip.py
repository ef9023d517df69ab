"""The library's host side without a GPU: a child process loads libgplbm.so over
tests/fake_hip.c (a HIP runtime that launches nothing and logs every launch and
copy) and runs a script with these names:

  B        the package's binding module
  wl       the workloads module
  context(p, precision, schedule)   a context on 256-byte aligned "device" memory
  alloc(base, size, kind=2, device=0)   declare memory (2 device, 1 pinned host)
  log()    the launches and copies since the last log(): ("launch", kernel name,
           grid, block, planes of a z-march's chunk) and ("copy", bytes)

`out` is what the script returns (anything JSON can hold)."""
from __future__ import annotations

import ctypes
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "fake_hip.c")


def build(folder) -> str:
    from paper_2111_05960_amd import build as hipbuild
    if not os.path.exists(hipbuild.LIB):
        hipbuild.build()
    lib = os.path.join(str(folder), "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", lib, SOURCE], check=True)
    return lib


def run(lib: str, script: str):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), lib], input=script, text=True,
                       capture_output=True, cwd=ROOT, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


def _main(lib: str):
    sys.path[0] = ROOT
    sys.modules["torch"] = None  # the child's only HIP runtime is the stand-in
    fake = ctypes.CDLL(lib, mode=ctypes.RTLD_GLOBAL)
    fake.fake_log.restype = ctypes.c_char_p
    fake.fake_alloc.argtypes = [ctypes.c_size_t, ctypes.c_size_t, ctypes.c_int, ctypes.c_int]
    from paper_2111_05960_amd import binding as B
    import workloads as wl
    B.load()

    def alloc(base, size, kind=2, device=0):
        fake.fake_alloc(base, size, kind, device)

    def context(p, precision="fp64", schedule="auto"):
        q = B.make_params(p, precision, schedule)
        return B.gplbm_create(q, 1 << 40, B.gplbm_state_bytes(q), 0)

    def log():
        out = []
        for line in fake.fake_log().decode().splitlines():
            w = line.split()
            out.append(["copy", int(w[1])] if w[0] == "copy" else
                       ["launch", w[1], [int(v) for v in w[2:5]], [int(v) for v in w[5:8]], int(w[8])])
        fake.fake_clear()
        return out

    env = dict(B=B, wl=wl, alloc=alloc, context=context, log=log, out=None)
    exec(sys.stdin.read(), env)
    print(json.dumps(env["out"]), flush=True)


if __name__ == "__main__":
    _main(sys.argv[1])
