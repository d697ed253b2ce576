"""Which kernels a call launches, found on the host: a child process binds the library's runtime calls to stand-ins
that note the launches and refuse what HIP refuses; the tensors are addresses that nothing reads."""
import json
import os
import subprocess
import sys

from paper_2603_13420_amd import binding as pk

STAND_INS = r"""
#include <cstddef>
#include <cstring>
struct dim3 { unsigned x, y, z; };
static const void *kernel[256];
static char name[256][256];
static unsigned long long noted[16][2];
static int which[16], kernels, n;
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *dev, unsigned, void *, void *, void *, void *, int *)
{
    if (kernels < 256) { kernel[kernels] = host; std::strncpy(name[kernels++], dev, 255); }
}
int hipLaunchKernel(const void *k, dim3 g, dim3 b, void **, size_t, void *)
{
    if (n < 16) {
        noted[n][0] = g.x; noted[n][1] = b.x;
        for (which[n] = kernels - 1; which[n] >= 0 && kernel[which[n]] != k; --which[n]) {}
        ++n;
    }
    return (unsigned long long)g.x * b.x > 0xffffffffull ? 9 : 0; /* hipErrorInvalidConfiguration */
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int take_launches(unsigned long long *out) { int k = n; std::memcpy(out, noted, sizeof noted); n = 0; return k; }
const char *launched(int i) { return which[i] >= 0 ? name[which[i]] : ""; }
}
"""

CHILD = """
import ctypes, json, sys
sys.path.insert(0, sys.argv[2])
stand_ins = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stand_ins.launched.restype = ctypes.c_char_p
from paper_2603_13420_amd import binding as pk
lib = pk.load()
vp = ctypes.c_void_p
t = [vp((1 + i) << 42) for i in range(14)]          # addresses 4 TB apart
for c in json.load(sys.stdin):
    p = pk.make_multi_params(pk.make_params(c["B"], c["S"], c["P"], c["Hq"], c["Hkv"], c["D"], c["dtype"]), c["Np"])
    lens = (t[13] if c["Np"] > 1 else None, t[12] if c["lens"] else None)
    if c["call"] == "fwd":
        rc = lib.pskv_attn_fwd_multi(ctypes.byref(p), *t[:5], *lens, t[5], None, None, 0, None)
    else:
        rc = lib.pskv_attn_bwd_multi(ctypes.byref(p), *t[:5], *lens, *t[5:11], None, 0, None)
    got = (ctypes.c_ulonglong * 32)()
    k = stand_ins.take_launches(got)
    print(json.dumps([rc, [[got[2 * i], got[2 * i + 1], stand_ins.launched(i).decode()] for i in range(k)]]), flush=True)
"""


def named(mangled, kernel):
    """Whether a mangled name is that of `kernel`_kernel, with its first template arguments if "<true,false>", "<2,1>" or the like is behind it."""
    name, _, args = kernel.partition("<")
    name += "_kernel"
    args = "I" + "".join({"true": "Lb1E", "false": "Lb0E"}.get(x, f"Li{x}E") for x in args.rstrip(">").split(",")) if args else ""
    return f"{len(name)}{name}{args}" in mangled


def case(call, dtype, D, B, P, S, Hq, Hkv, Np=1, lens=False):
    """lens: the call brings suffix lengths."""
    return dict(call=call, dtype=dtype, D=D, B=B, P=P, S=S, Hq=Hq, Hkv=Hkv, Np=Np, lens=lens)


def launches(tmp_path, cases):
    """[status, [[workgroups, threads of one, the kernel's mangled name], ...]] of every case, on 256 compute units."""
    src, lib = str(tmp_path / "s.cpp"), str(tmp_path / "s.so")
    with open(src, "w") as f:
        f.write(STAND_INS)
    subprocess.run(["g++", "-shared", "-fPIC", "-o", lib, src], check=True)
    res = subprocess.run([sys.executable, "-c", CHILD, lib, os.path.dirname(os.path.dirname(os.path.abspath(pk.__file__)))],
                         input=json.dumps(cases), stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    lines = [json.loads(x) for x in res.stdout.splitlines()]
    assert len(lines) == len(cases)
    return lines
