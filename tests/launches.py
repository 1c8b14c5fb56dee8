"""Which kernels a library call launches, and with which grids, found without a
GPU: the calls run in a process of their own on a HIP runtime that records
launches instead of making them (hip_recorder.c)."""
from __future__ import annotations

import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

# stand for device buffers far apart from each other
IMG, LABELS, OUT, COUNT = 1 << 40, 1 << 44, 1 << 48, 1 << 50


def record(calls, tmp_path):
    """Run `calls`, a list of (function, arguments): integers, None, texts, or
    ("cfg", tile_h, waves).  Returns one (status, launches) per call; a launch
    is (kernel, workgroups in x, in y, threads per workgroup, refused)."""
    lib = os.path.join(str(tmp_path), "libamdhip64_recorder.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "hip_recorder.c")],
                   check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), lib, json.dumps(calls)], cwd=ROOT,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return [(rc, [tuple(x) for x in ls]) for rc, ls in json.loads(r.stdout)]


def _main(lib_path, calls):
    import ctypes
    import re

    sys.path.insert(0, ROOT)
    rec = ctypes.CDLL(lib_path, mode=ctypes.RTLD_GLOBAL)
    rec.rec_name.restype = ctypes.c_char_p
    from paper_1708_08180_amd import binding

    lib = ctypes.CDLL(binding.library_path())
    for name, (res, args) in binding.SIGNATURES.items():
        getattr(lib, name).restype, getattr(lib, name).argtypes = res, args
    out = []
    for fn, args in calls:
        conv = []
        for a in args:
            if isinstance(a, list):
                a = ctypes.byref(binding.Config(*a[1:]))
            conv.append(a.encode() if isinstance(a, str) else a)
        if fn == "ccl_label_2d_timed":
            conv[-1] = (ctypes.c_float * 3)()
        rec.rec_clear()
        rc = getattr(lib, fn)(*conv)
        ls = []
        for i in range(rec.rec_count()):
            v = (ctypes.c_uint32 * 4)()
            rec.rec_get(i, v)
            name = subprocess.run(["c++filt", rec.rec_name(i).decode()], capture_output=True, text=True).stdout
            ls.append([re.sub(r"^void |ccl::|\(anonymous namespace\)::|\(.*$", "", name.strip()), v[0], v[1], v[2], v[3]])
        out.append([rc, ls])
    print(json.dumps(out))


if __name__ == "__main__":
    _main(sys.argv[1], json.loads(sys.argv[2]))
