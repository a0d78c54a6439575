"""What libuniql launches for a list of calls, without a GPU: a child process loads launch_recorder.cpp in place of the HIP runtime.

A call is a dict: "specs", a list of (rows, stored columns, keep rule as a dict) -- one for uniql_w4_linear, several for
uniql_w4_linear_multi, two with "glu" for uniql_w4_gate_up_silu_batch --, "M", and "bits", "bf16" where they are not 4 and fp16.  The answer
for each is (status, [Launch]); `kernel` is the name with its template arguments."""
import ctypes as C
import json
import os
import re
import subprocess
import sys
from collections import namedtuple

HERE = os.path.dirname(os.path.abspath(__file__))
Launch = namedtuple("Launch", "kernel blocks threads lds limit")


def record(calls, directory, compute_units=256):
    so = os.path.join(str(directory), "librecorder.so")
    if not os.path.exists(so):
        rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
        subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"), os.path.join(HERE, "launch_recorder.cpp"), "-o", so], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), so], input=json.dumps(calls), capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, RECORDER_COMPUTE_UNITS=str(compute_units)))
    assert r.returncode == 0, r.stderr
    out = json.loads(r.stdout)
    mangled = sorted({k for _, ls in out for k, *_ in ls})
    plain = dict(zip(mangled, subprocess.run(["c++filt"], input="\n".join(mangled), capture_output=True, text=True, check=True).stdout.split("\n")))
    short = {k: re.sub(r"void |uniql::|__device_stub__|\(.*| ", "", v) for k, v in plain.items()}
    return [(rc, [Launch(short[k], *sizes) for k, *sizes in ls]) for rc, ls in out]


def _child(so):
    recorder = C.CDLL(so, mode=C.RTLD_GLOBAL)
    recorder.recorded_kernel.restype = C.c_char_p
    sys.path.insert(0, os.path.dirname(HERE))
    import paper_2512_03383_amd as uq
    L, at, out = uq.lib(), 4096, []   # at: an address that is never read
    for c in json.load(sys.stdin):
        n, M, bits, dtype = len(c["specs"]), c["M"], c.get("bits", 4), uq.UNIQL_BF16 if c.get("bf16") else uq.UNIQL_F16
        W = (uq.W4 * n)(*[uq.W4(at, at, at, N, K, 128, dtype, 0, bits) for N, K, _ in c["specs"]])
        keep = (uq.KeepDesc * n)(*[uq.KeepDesc(**k) for _, _, k in c["specs"]])
        ldx, ldy = (C.c_int64 * n)(*[K for _, K, _ in c["specs"]]), (C.c_int64 * n)(*[N for N, _, _ in c["specs"]])
        if c.get("glu"):
            rc = L.uniql_w4_gate_up_silu_batch(W, keep, at, ldx[0], at, ldy[0], M, None)
        elif n == 1:
            rc = L.uniql_w4_linear(W, keep, at, ldx[0], at, ldy[0], M, None)
        else:
            p = (C.c_void_p * n)(*[at] * n)
            rc = L.uniql_w4_linear_multi(n, W, keep, p, ldx, p, ldy, M, None)
        s, ls = (C.c_long * 4)(), []
        for i in range(recorder.recorded()):
            recorder.recorded_sizes(i, s)
            ls.append([recorder.recorded_kernel(i).decode(), *s])
        recorder.recorded_clear()
        out.append((rc, ls))
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _child(sys.argv[1])
