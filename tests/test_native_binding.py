"""The native marshalling of torch tensors: it makes a call only when every argument is of the plain
form, and otherwise leaves the matter, and the error, to binding.py's own checks."""
import pytest

from paper_2603_13420_amd import binding as pk


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
