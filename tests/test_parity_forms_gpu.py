"""GPU parity of the fp32 kernels (heads of 64 and 128 columns) and of the bf16 kernels for heads of 64
columns on the forms that calls take: views into fused buffers, several instructions, random shapes;
forward and backward, against the oracle."""
import numpy as np
import pytest

from paper_2603_13420_amd import inputs as gen
import parity_util as pu

pytestmark = pytest.mark.gpu
KINDS = [("f32", 64), ("f32", 128), ("bf16", 64)]


@pytest.fixture(scope="module")
def pk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_13420_amd import binding
    binding.load()
    return binding


def check(pk, inp, fused=False):
    import torch
    w, multi = inp.w, hasattr(inp, "pre_len")
    d = (pu.to_device_multi if multi else pu.to_device)(inp)
    B, S, Hq, Hkv, D = w.Np * w.C if multi else w.B, w.S, w.Hq, w.Hkv, w.D
    print(f"[case] {w.name} {w.dtype} D={D} B={B} P={w.P} S={S} Hq={Hq} Hkv={Hkv} seed={w.seed}"
          + (f" pre_len={inp.pre_len.tolist()[:8]}" if multi else ""), flush=True)
    q, ks, vs, kp, vp = (d[n] for n in ("q", "k_suf", "v_suf", "k_pre", "v_pre"))
    dout_host, dout64 = pu.make_dout(inp, w.seed + 7)
    t = torch.from_numpy(dout_host)
    dout = (t.view(torch.bfloat16) if w.dtype == "bf16" else t).to("cuda:0")
    nan = float("nan")
    if fused:       # column slices of [B,S,(Hq+2Hkv),D], out and dout with a padded head stride, the prefix as [P,Hkv,2,D]
        buf, grads = (torch.full((B, S, Hq + 2 * Hkv, D), nan, dtype=q.dtype, device="cuda:0") for _ in range(2))
        buf[:, :, :Hq], buf[:, :, Hq:Hq + Hkv], buf[:, :, Hq + Hkv:] = q, ks, vs
        q, ks, vs = buf[:, :, :Hq], buf[:, :, Hq:Hq + Hkv], buf[:, :, Hq + Hkv:]
        dq, dk, dv = grads[:, :, :Hq], grads[:, :, Hq:Hq + Hkv], grads[:, :, Hq + Hkv:]
        both = torch.stack([kp, vp], dim=2)
        kp, vp = both[:, :, 0], both[:, :, 1]
        obuf, dbuf = (torch.full((B, S, Hq, 2 * D), nan, dtype=q.dtype, device="cuda:0") for _ in range(2))
        out = obuf[..., :D]
        dbuf[..., :D] = dout
        dout = dbuf[..., :D]
    else:
        out, dq, dk, dv = (torch.full_like(x, nan) for x in (q, q, ks, ks))
    lse = torch.full((B, Hq, S), 123.0, device="cuda:0")
    args = (q, ks, vs, kp, vp) + ((d["pre_len"],) if multi else ()) + (d["suf_len"],)
    (pk.pskv_attn_fwd_multi if multi else pk.pskv_attn_fwd)(*args, out=out, lse=lse, scale=inp.scale)
    (pk.pskv_attn_bwd_multi if multi else pk.pskv_attn_bwd)(*args, out, lse, dout, dq=dq, dk_suf=dk, dv_suf=dv, scale=inp.scale)
    torch.cuda.synchronize()
    ref, ref_lse = (pu.oracle_out_multi if multi else pu.oracle_out)(inp, want_lse=True)
    pu.compare_lse(lse.cpu().numpy().astype(np.float64), ref_lse, inp.suf_len, w.dtype, w.name)
    pu.compare(pu.out_to_f64(out.contiguous()), ref, inp.suf_len, w.dtype, w.name)
    valid = np.arange(S)[None, :] < inp.suf_len[:, None]
    for name, got, r in zip(("dq", "dk_suf", "dv_suf"), (dq, dk, dv), (pu.oracle_bwd_multi if multi else pu.oracle_bwd)(inp, dout64)):
        pu.compare_grad(pu.out_to_f64(got.contiguous()), r, valid, w.dtype, f"{w.name} {name}")
    if fused:
        assert torch.isnan(obuf[..., D:]).all()         # nothing written outside the view


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("B,P,S,lo,Hq,Hkv", [(5, 40, 11, 3, 8, 2), (3, 250, 33, 5, 14, 2), (4, 530, 20, 20, 4, 4)])
def test_views_of_fused_buffers(pk, dtype, D, B, P, S, lo, Hq, Hkv):
    w = gen.custom_workload(f"fused_{dtype}_{D}_{P}", B, P, S, lo, S, Hq, Hkv, D, dtype, index=2200 + P + D)
    check(pk, gen.make_inputs(w, pad="nan"), fused=True)


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("Np,C,P,S,Hq,Hkv", [
    (5, 4, 70, 19, 6, 2),
    (4, 3, 600, 21, 14, 2),      # 64 columns: some prefixes stay in LDS, others go through it in chunks
    (70, 1, 530, 4, 8, 8),       # ... in the same workgroup: more (instruction, KV head) pairs than can be served at a time
])
def test_several_instructions(pk, dtype, D, Np, C, P, S, Hq, Hkv):
    w = gen.custom_multi_workload(f"forms_multi_{dtype}_{D}_{P}", Np, C, P, P, P, S, 0, S, Hq, Hkv, D, dtype, index=2300 + P + D)
    inp = gen.make_multi_inputs(w, pad="nan")
    inp.pre_len[:] = np.random.default_rng(w.seed).integers(0, P + 1, Np)
    inp.pre_len[:3] = P, 0, 1
    for n in range(Np):
        inp.k_pre[n, :P - inp.pre_len[n]] = inp.v_pre[n, :P - inp.pre_len[n]] = 0x7FC0 if dtype == "bf16" else np.nan
    check(pk, inp)


@pytest.mark.parametrize("case", range(24))
def test_random_shapes(pk, case):
    rng = np.random.default_rng(4977 + case)
    dtype, D = KINDS[case % 3]
    G, Hkv = int(rng.choice([1, 2, 4, 7, 8])), int(rng.choice([1, 2, 4]))
    P = int(rng.choice([0, rng.integers(1, 64), rng.integers(64, 200), rng.integers(200, 700)]))
    S, B = int(rng.choice([rng.integers(1, 33), rng.integers(33, 80)])), int(rng.integers(1, 9))
    w = gen.custom_workload(f"forms_rand{case}", B, P, S, int(rng.integers(0, S + 1)), S, G * Hkv, Hkv, D, dtype, index=2400 + case)
    check(pk, gen.make_inputs(w, pad="nan"))
