"""A HIP launch holds fewer than 2^32 work-items per dimension.  What the vector kernels can be launched for
is served: where a matrix-core kernel's grid, of larger workgroups, would not fit, they take the problem.
Checked on the host: a child process binds the library's runtime calls to stand-ins that note the
launches and refuse what HIP refuses; the tensors are addresses that nothing reads."""
import json
import os
import subprocess
import sys

from paper_2603_13420_amd import binding as pk

STAND_INS = r"""
#include <cstddef>
#include <cstring>
struct dim3 { unsigned x, y, z; };
static unsigned long long noted[16][2];
static int n;
extern "C" {
int hipLaunchKernel(const void *, dim3 g, dim3 b, void **, size_t, void *)
{
    if (n < 16) { noted[n][0] = g.x; noted[n][1] = b.x; ++n; }
    return (unsigned long long)g.x * b.x > 0xffffffffull ? 9 : 0; /* hipErrorInvalidConfiguration */
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int take_launches(unsigned long long *out) { int k = n; std::memcpy(out, noted, sizeof noted); n = 0; return k; }
}
"""

CHILD = """
import ctypes, json, sys
sys.path.insert(0, sys.argv[2])
stand_ins = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from paper_2603_13420_amd import binding as pk
lib = pk.load()
vp = ctypes.c_void_p
t = [vp((1 + i) << 42) for i in range(14)]          # addresses 4 TB apart
for c in json.load(sys.stdin):
    p = pk.make_multi_params(pk.make_params(c["B"], c["S"], c["P"], c["Hq"], c["Hkv"], c["D"], c["dtype"]), c["Np"])
    if c["call"] == "fwd":
        rc = lib.pskv_attn_fwd_multi(ctypes.byref(p), *t[:5], None, None, t[5], None, None, 0, None)
    else:
        rc = lib.pskv_attn_bwd_multi(ctypes.byref(p), *t[:5], None, None, *t[5:11], None, 0, None)
    got = (ctypes.c_ulonglong * 32)()
    k = stand_ins.take_launches(got)
    print(json.dumps([rc, [[got[2 * i], got[2 * i + 1]] for i in range(k)]]), flush=True)
"""

MOST = 1 << 24                    # workgroups of 256 from which on a launch does not fit


def case(call, dtype, D, groups, Np=1, S=1, P=8):
    """groups (candidate, KV head) pairs of one position each."""
    return dict(call=call, dtype=dtype, D=D, B=groups // 16, Hq=16, Hkv=16, Np=Np or groups // 16, S=S, P=P)


def test_large_grids_go_to_kernels_that_can_be_launched(tmp_path):
    src, lib = str(tmp_path / "s.cpp"), str(tmp_path / "s.so")
    with open(src, "w") as f:
        f.write(STAND_INS)
    subprocess.run(["g++", "-shared", "-fPIC", "-o", lib, src], check=True)
    # bwd: one unit of 256 threads per pair, for fp32 together with the dq blocks of 16 rows each
    # fwd, Np instructions of one candidate each: one 16-row block per pair
    cases = [(case("bwd", "bf16", 64, MOST - 16), 256), (case("bwd", "bf16", 64, MOST), 64),
             (case("bwd", "f32", 64, MOST - MOST // 16), 256), (case("bwd", "f32", 64, MOST), 64), (case("bwd", "f32", 128, MOST), 64),
             (case("fwd", "f32", 64, MOST - 16, Np=0), 256), (case("fwd", "f32", 128, MOST, Np=0), 64),
             (case("fwd", "bf16", 64, MOST, Np=0), 512)]
    res = subprocess.run([sys.executable, "-c", CHILD, lib, os.path.dirname(os.path.dirname(os.path.abspath(pk.__file__)))],
                         input=json.dumps([c for c, _ in cases]), stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    lines = [json.loads(x) for x in res.stdout.splitlines()]
    assert len(lines) == len(cases)
    for (c, threads), (rc, launches) in zip(cases, lines):
        assert rc == pk.PSKV_OK and launches, (c, rc, launches)
        assert all(g * b < 1 << 32 for g, b in launches), (c, launches)
        assert launches[-1][1] == threads, (c, launches)
