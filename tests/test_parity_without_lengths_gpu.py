"""Calls that bring no suffix lengths, against the oracle, one problem and more for every kernel that serves them; that a problem takes the
kernel is checked as well.  Results stand between guard values."""
import numpy as np
import pytest

import launch_notes as notes
import parity_util as pu
from paper_2603_13420_amd import inputs as gen

pytestmark = pytest.mark.gpu

GUARD = 7.5


@pytest.fixture(scope="module")
def pk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_13420_amd import binding
    binding.load()
    return binding


def takes(tmp_path, call, kernel, w):
    (rc, got), = notes.launches(tmp_path, [notes.case(call, "bf16", 128, w.B, w.P, w.S, w.Hq, w.Hkv)])
    assert rc == 0 and notes.named(got[0][2], kernel), got


def guarded(shape, dtype):
    import torch
    n = int(np.prod(shape))
    flat = torch.full((n + 8192,), GUARD, device="cuda:0", dtype=dtype)
    flat[4096:-4096] = float("nan")
    return flat, flat[4096:-4096].view(shape)


def forward(pk, inp):
    import torch
    w, d = inp.w, pu.to_device(inp)
    print(f"[case] no lengths B={w.B} P={w.P} S={w.S} Hq={w.Hq} Hkv={w.Hkv} seed={w.seed}", flush=True)
    (flat, out), (flat_lse, lse) = guarded(d["q"].shape, torch.bfloat16), guarded((w.B, w.Hq, w.S), torch.float32)
    pk.pskv_attn_fwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], None, out=out, lse=lse, scale=inp.scale)
    torch.cuda.synchronize()
    assert all((t == GUARD).all().item() for f in (flat, flat_lse) for t in (f[:4096], f[-4096:]))
    ref, ref_lse = pu.oracle_out(inp, want_lse=True)
    pu.compare_lse(lse.cpu().numpy().astype(np.float64), ref_lse, inp.suf_len, "bf16", w.name)
    pu.compare(pu.out_to_f64(out), ref, inp.suf_len, "bf16", w.name)
    return d, out, lse


@pytest.mark.parametrize("kernel,B,P,S,Hq,Hkv", [
    ("resident_general", 12, 70, 19, 4, 4),          # blocks across candidates, a ragged third tile
    ("resident_general", 20, 40, 20, 8, 2),
    ("resident_pipelined<true>", 40, 100, 32, 8, 8),
    ("resident_pipelined<true>", 33, 256, 24, 8, 2),
    ("resident_pipelined<false>", 10, 151, 27, 32, 32),
    ("resident_pipelined<false>", 9, 130, 30, 8, 4),
    ("stream_pipelined<true,true>", 20, 300, 32, 8, 2),
    ("stream_pipelined<true,false>", 20, 300, 30, 8, 8),
    ("stream_pipelined<false,true>", 65, 257, 64, 8, 8),
    ("stream_pipelined<false,false>", 65, 300, 60, 8, 8),
    ("stream_general", 20, 300, 19, 4, 4),
    ("stream_candidate<false>", 17, 300, 60, 32, 8),
    ("stream_candidate4", 4, 200, 40, 32, 4),
])
def test_forward(pk, tmp_path, kernel, B, P, S, Hq, Hkv):
    w = gen.custom_workload(f"nolen_{B}_{P}_{S}", B, P, S, S, S, Hq, Hkv, 128, "bf16", index=3700 + B + P + S)
    takes(tmp_path, "fwd", kernel, w)
    forward(pk, gen.make_inputs(w, pad="nan"))


@pytest.mark.parametrize("kernel,B,P,S,Hq,Hkv", [
    ("resident_pipelined<true>", 40, 100, 32, 8, 8), ("resident_pipelined<false>", 10, 151, 27, 32, 32),
    ("stream_pipelined<true,false>", 20, 300, 30, 8, 8), ("stream_pipelined<false,true>", 65, 257, 64, 8, 8),
])
def test_scores_far_above_the_first_tile(pk, tmp_path, kernel, B, P, S, Hq, Hkv):
    """A late key of 130 and more above everything before it: the general path takes over."""
    w = gen.custom_workload(f"nolen_spike_{P}_{S}", B, P, S, S, S, Hq, Hkv, 128, "bf16", index=3750 + P + S)
    takes(tmp_path, "fwd", kernel, w)
    inp = gen.make_inputs(w, pad="nan")
    inp.q[1] = 0x3F80           # one
    inp.k_pre[P - 3] = 0x4140   # twelve
    forward(pk, inp)


@pytest.mark.parametrize("kernel,B,P,S,Hq,Hkv", [
    ("bwd_dq_resident", 64, 256, 20, 8, 2),
    ("bwd_dq_resident", 64, 200, 30, 4, 4),
    ("bwd_dq_mfma", 40, 300, 20, 8, 2),
    ("bwd_dq_mfma", 300, 96, 8, 4, 4),
    ("bwd_dq_unit", 17, 100, 32, 8, 2),
])
def test_backward(pk, tmp_path, kernel, B, P, S, Hq, Hkv):
    import torch
    w = gen.custom_workload(f"nolen_bwd_{B}_{P}_{S}", B, P, S, S, S, Hq, Hkv, 128, "bf16", index=3800 + B + P + S)
    takes(tmp_path, "bwd", kernel, w)
    inp = gen.make_inputs(w, pad="nan")
    d, out, lse = forward(pk, inp)
    dout_host, dout64 = pu.make_dout(inp, w.seed + 7)
    dout = torch.from_numpy(dout_host).view(torch.bfloat16).to("cuda:0")
    (flat, dq), (flat_k, dk), (flat_v, dv) = (guarded(d[n].shape, torch.bfloat16) for n in ("q", "k_suf", "v_suf"))
    pk.pskv_attn_bwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], None, out, lse, dout, dq=dq, dk_suf=dk, dv_suf=dv, scale=inp.scale)
    torch.cuda.synchronize()
    assert all((t == GUARD).all().item() for f in (flat, flat_k, flat_v) for t in (f[:4096], f[-4096:]))
    valid = np.ones((B, S), dtype=bool)
    for name, got, r in zip(("dq", "dk_suf", "dv_suf"), (dq, dk, dv), pu.oracle_bwd(inp, dout64)):
        pu.compare_grad(pu.out_to_f64(got), r, valid, "bf16", f"{w.name} {name}")
