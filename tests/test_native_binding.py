"""The native marshalling of torch tensors: it makes a call only when every argument is of the plain
form, and otherwise leaves the matter, and the error, to binding.py's own checks."""
import os
import subprocess
import sys

import pytest

from paper_2603_13420_amd import binding as pk, build


def tensors(device, dtype=None, D=128):
    import torch
    dtype = dtype or torch.bfloat16
    t = lambda *s: torch.randn(s, device=device, dtype=dtype)     # noqa: E731
    return dict(q=t(2, 5, 4, D), k_suf=t(2, 5, 2, D), v_suf=t(2, 5, 2, D), k_pre=t(7, 2, D), v_pre=t(7, 2, D))


def test_what_is_not_plain_is_left_alone():
    d = tensors("cpu")
    m = pk._native()
    a = [d[k] for k in ("q", "k_suf", "v_suf", "k_pre", "v_pre")]
    assert m.fwd(*a, None, None, None, "auto", 0.0, None) is None          # tensors on the CPU
    assert m.fwd(*a, None, None, None, "auto", 0.0) is None                # arguments missing
    assert m.fwd(*a[:4], 3, None, None, None, "auto", 0.0, None) is None   # not a tensor
    with pytest.raises(ValueError, match="GPU"):
        pk.pskv_attn_fwd(*a)


# Tensors without storage (inside torch.vmap and torch.func.grad they are of the exact type Tensor) through a build of
# the marshalling that takes CPU tensors, its entry points bound to one that answers "ok".
WITHOUT_STORAGE = """
import ctypes, importlib.util, sys, torch
spec = importlib.util.spec_from_file_location("_pskv_torch", sys.argv[1])
m = importlib.util.module_from_spec(spec)
spec.loader.exec_module(m)
calls = []
ok = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: calls.append(1) or 0)
need = ctypes.CFUNCTYPE(ctypes.c_size_t)(lambda: 64)
m.bind(*[ctypes.cast(ok, ctypes.c_void_p).value] * 5, ctypes.cast(need, ctypes.c_void_p).value, lambda index: 0)
t = lambda *s: torch.zeros(s)
rest = t(2, 5, 2, 64), t(2, 5, 2, 64), t(7, 2, 64), t(7, 2, 64)
q, lse = t(2, 5, 4, 64), t(2, 4, 5)
fwd = lambda q: m.fwd(q, *rest, None, None, None, "auto", 0.0, None)
multi = lambda q: m.fwd_multi(q, *rest[:2], rest[2][None], rest[3][None], None, None, None, None, "auto", 0.0, None)
bwd = lambda q: m.bwd(q, *rest, None, q, lse, q, None, None, None, "auto", 0.0, None, None)[0]
assert fwd(q).shape == multi(q).shape == bwd(q).shape == q.shape and len(calls) == 3
for f in (fwd, multi, bwd):
    for under, x in ((torch.vmap(f), torch.stack([q, q])), (torch.func.grad(lambda q: f(q).sum()), q)):
        try:
            under(x)
        except RuntimeError as e:
            assert "storage" in str(e), e
        else:
            raise AssertionError("no error")
assert len(calls) == 3
print("done")
"""


def test_tensors_without_storage_give_an_error_and_not_a_crash(tmp_path):
    with open(os.path.join(build.CSRC, build.TORCH_SOURCE)) as f:
        text = f.read()
    assert "is_cuda()" in text
    src, lib = str(tmp_path / "m.cpp"), str(tmp_path / "_pskv_torch.so")
    with open(src, "w") as f:
        f.write(text.replace("is_cuda()", "is_cpu()").replace("../../include", os.path.join(os.path.dirname(build.HERE), "include")))
    cmd = [{build.TORCH_LIB: lib, os.path.join(build.CSRC, build.TORCH_SOURCE): src, "-O2": "-O0"}.get(x, x) for x in build.torch_command()]
    subprocess.run(cmd, check=True)
    res = subprocess.run([sys.executable, "-c", WITHOUT_STORAGE, lib], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0 and res.stdout.strip().endswith("done"), (res.returncode, res.stdout)


@pytest.mark.gpu
def test_native_calls_and_what_they_refuse():
    import torch
    d = tensors("cuda:0")
    a = [d[k] for k in ("q", "k_suf", "v_suf", "k_pre", "v_pre")]
    out, lse = torch.empty_like(d["q"]), torch.empty((2, 4, 5), device="cuda:0")
    m = pk._native()
    assert m.fwd(*a, None, out, lse, "auto", 0.0, None) is out
    assert torch.equal(pk.pskv_attn_fwd(*a), out)
    # the same through the parameters that the Python side fills in
    again = torch.empty_like(out)
    pk.PreparedCall(*a, None, again, impl="auto")()
    torch.cuda.synchronize()
    assert torch.equal(again, out)
    dout = torch.randn_like(out)
    grads = m.bwd(*a, None, out, lse, dout, None, None, None, "auto", 0.0, None, None)
    given = [torch.empty_like(g) for g in grads]
    assert all(x is y for x, y in zip(m.bwd_noalloc(*a, None, out, lse, dout, *given, "auto", 0.0, None), given))
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(grads, given))
    assert m.fwd(*a, None, out, lse, "nonsense", 0.0, None) is None
    assert m.fwd(d["q"].float(), *a[1:], None, None, None, "auto", 0.0, None) is None       # types differ
    class Own(torch.Tensor):                                                                   # may have its own empty_like
        pass
    assert m.fwd(d["q"].as_subclass(Own), *a[1:], None, None, None, "auto", 0.0, None) is None
    assert type(pk.pskv_attn_fwd(d["q"].as_subclass(Own), *a[1:])) is Own
    wide = d["k_pre"][:1].expand(7, 2, 128)                                                    # stride 0
    assert m.fwd(*a[:3], wide, wide, None, None, None, "auto", 0.0, None) is None
    with pytest.raises(ValueError, match="stride 0"):
        pk.pskv_attn_fwd(*a[:3], wide, wide)
    assert m.fwd(*a, None, d["q"], None, "auto", 0.0, None) == pk.PSKV_ERR_INVALID_ARG       # the library's own word
    with pytest.raises(pk.PskvError, match="out overlaps q"):
        pk.pskv_attn_fwd(*a, out=d["q"])
