"""Which kernels a call of the library launches, found out on the CPU: a child
process loads launch_recorder.cpp in place of the HIP runtime, runs a piece of
test code against the C ABI and hands back what the code puts in `result`."""
from __future__ import annotations

import json
import os
import subprocess
import sys
import tempfile
from functools import lru_cache
from pathlib import Path

HERE = Path(__file__).resolve().parent
ROOT = HERE.parent

PREAMBLE = '''
import ctypes, json, re, sys
sys.path.insert(0, {root!r})
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rec.rec_name.restype = ctypes.c_char_p
for f in (rec.rec_in, rec.rec_out, rec.rec_arg_ptr):
    f.restype = ctypes.c_void_p
rec.rec_price.argtypes = [ctypes.c_char_p, ctypes.c_double]
from paper_2603_19789_amd import binding, inputs
from paper_2603_19789_amd.binding import Launch, Params
lib = binding.library()
GIB = 1 << 30
rho, scratch, extra = (ctypes.c_void_p(k << 40) for k in (1, 2, 3))

def params(d_dead=0.0):
    return inputs.from_sigma_mu(0.5, 0.2, 0.1, 0.01, (2e-2, 1e-3, 5e-3, 1e-2, d_dead))

def context(nx, ny, dtype="f32", d_dead=0.0, bc=binding.PERIODIC):
    h = ctypes.c_void_p()
    code = binding.F32 if dtype == "f32" else binding.F64
    assert lib.sslbm_init(ctypes.byref(h), nx, ny, code, bc,
                          ctypes.byref(Params.of(params(d_dead)))) == 0
    return h

def ensemble(sizes, dtype="f32", d_dead=0.0):
    n = len(sizes)
    h, bad = ctypes.c_void_p(), ctypes.c_int()
    code = binding.F32 if dtype == "f32" else binding.F64
    assert lib.sslbm_ensemble_create(
        ctypes.byref(h), n, (ctypes.c_int * n)(*[s[0] for s in sizes]),
        (ctypes.c_int * n)(*[s[1] for s in sizes]), code, binding.PERIODIC,
        (Params * n)(*[Params.of(params(d_dead))] * n), ctypes.byref(bad)) == 0
    return h

def launched():
    """(kernel, template arguments, grid, block, in, out) since the last call."""
    out = []
    for i in range(rec.rec_count()):
        name = rec.rec_name(i).decode()
        m = re.search(r"(\\w+)<([^>]*)>", name)
        kernel, args = (m[1], [a.strip() for a in m[2].split(",")]) if m else (name, [])
        out.append((kernel, args, rec.rec_grid(i), rec.rec_block(i), rec.rec_in(i),
                    rec.rec_out(i)))
    return out

def passes(call):
    """The kernels of a call as (kind, steps or None, rows a lane or columns a lane or None)."""
    rec.rec_clear()
    assert call() == 0
    out = []
    for i, (kernel, args, *_) in enumerate(launched()):
        if kernel == "sslbm_march_kernel":
            out.append(("march", int(args[1]), int(args[3])))
        elif kernel == "sslbm_march_mid_kernel":
            out.append(("mid", int(args[1]), int(args[3])))
        elif kernel == "bgk_march_kernel":
            out.append(("bgk", int(args[1]), None))
        elif kernel == "bgk_step_kernel":
            out.append(("bgk", 1, None))
        elif "tile_kernel" in kernel:
            out.append(("tile", None, int(args[1])))
        else:
            out.append((kernel, None, None))
    return out
'''


@lru_cache(maxsize=1)
def recorder() -> str:
    out = Path(tempfile.mkdtemp(prefix="launch_recorder_")) / "librecorder.so"
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    f"-I{rocm}/include", "-o", str(out), str(HERE / "launch_recorder.cpp"),
                    "-ldl"], check=True)
    return str(out)


def record(code: str):
    """Run `code` after the preamble in a child process; its `result`."""
    src = PREAMBLE.replace("{root!r}", repr(str(ROOT))) + code + "\nprint(json.dumps(result))\n"
    res = subprocess.run([sys.executable, "-c", src, recorder()], capture_output=True, text=True,
                         cwd=ROOT, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    return json.loads(res.stdout.splitlines()[-1])
