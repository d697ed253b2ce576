"""GPU: what a row does not see does not reach it, whatever it holds.  Infinities and NaN are planted in
VALID rows of some candidates - keys and values that the rows of neighbouring candidates and the earlier
rows of the same one do not see, query rows that later keys do not see - and in the last row of a
ragged prefix.  The result has to be what the same definition gives in double precision with every row
taken over its visible keys only: the same elements not finite, the others as close as ever (the bars
of oracle/parity.py at a magnitude of one or so: 1e-5 for fp32 tensors, 2e-2 for bf16 ones)."""
import numpy as np
import pytest

from paper_2603_13420_amd import inputs as gen
import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_13420_amd import binding
    binding.load()
    return binding


def visible_only(q, ks, vs, kp, vp, lens, dout, scale):
    """out, dq, dk, dv by the definition, one query row at a time over its visible keys (float64)."""
    B, S, Hq, D = q.shape
    G, P = Hq // ks.shape[2], kp.shape[0]
    out, dq, dk, dv = np.zeros_like(q), np.zeros_like(q), np.zeros_like(ks), np.zeros_like(vs)
    for b in range(B):
        for i in range(lens[b]):
            for h in range(Hq):
                k = h // G
                K, V = np.concatenate([kp[:, k], ks[b, :i + 1, k]]), np.concatenate([vp[:, k], vs[b, :i + 1, k]])
                s = K @ q[b, i, h] * scale
                p = np.exp(s - s.max())
                p /= p.sum()
                o = out[b, i, h] = p @ V
                ds = p * (V @ dout[b, i, h] - dout[b, i, h] @ o)
                dq[b, i, h] = scale * (ds @ K)
                dk[b, :i + 1, k] += scale * ds[P:, None] * q[b, i, h]
                dv[b, :i + 1, k] += p[P:, None] * dout[b, i, h]
    return out, dq, dk, dv


def agree(got, ref, tol, what):
    """The same elements not finite; the others within tol of the reference, relative to its own scale."""
    bad = ~np.isfinite(ref)
    assert np.array_equal(~np.isfinite(got), bad), f"{what}: {(~np.isfinite(got) & ~bad).sum()} elements reached, " \
                                                  f"{(np.isfinite(got) & bad).sum()} of {bad.sum()} missed"
    scale = np.sqrt(np.mean(ref[~bad] ** 2))
    err = np.abs(got[~bad] - ref[~bad])
    assert err.max() <= tol * max(scale, np.abs(ref[~bad]).max()), f"{what}: {err.max():.3e} at rms {scale:.3e}"


@pytest.mark.parametrize("impl", ["simple", "auto"])
@pytest.mark.parametrize("dtype,D,P,S,lo,Hq,Hkv,B", [
    ("f32", 64, 19, 5, 3, 4, 4, 12),     # three candidates and more in a block of 16 rows
    ("f32", 128, 16, 18, 9, 4, 2, 4),    # blocks that straddle two candidates, two key tiles each
    ("f32", 64, 0, 3, 1, 14, 2, 9),
    ("bf16", 64, 40, 7, 3, 4, 4, 12),    # five candidates in a block of 32 rows, their keys in one step; ragged prefix
    ("bf16", 64, 32, 37, 33, 4, 2, 4),   # blocks that straddle two candidates, two own steps each
    ("bf16", 64, 0, 3, 1, 14, 2, 9),
])
def test_hidden_values_stay_hidden(pk, impl, dtype, D, P, S, lo, Hq, Hkv, B):
    import torch
    w = gen.custom_workload(f"hidden_{dtype}_{D}_{S}", B, P, S, lo, S, Hq, Hkv, D, dtype, index=1900 + B + S)
    inp = gen.make_inputs(w, pad="nan")
    inp.suf_len[1], inp.suf_len[2] = S, S
    rng = np.random.default_rng(w.seed)
    inp.q[1:3], inp.k_suf[1:3], inp.v_suf[1:3] = [      # (two candidates without padding)
        gen.f32_to_bf16_bits(x) if dtype == "bf16" else x
        for x in (rng.standard_normal(s, dtype=np.float32) for s in (inp.q[1:3].shape, inp.k_suf[1:3].shape, inp.k_suf[1:3].shape))]
    dout_host, _ = pu.make_dout(inp, w.seed + 7)
    inf, nan = (np.uint16(0x7F80), np.uint16(0x7FC0)) if dtype == "bf16" else (np.inf, np.nan)
    widen = (lambda x: gen.bf16_bits_to_f32(x).astype(np.float64)) if dtype == "bf16" else (lambda x: x.astype(np.float64))
    torch_type = torch.bfloat16 if dtype == "bf16" else torch.float32

    plants = {
        "values of a neighbour": lambda: inp.v_suf.__setitem__((1, 0, 0, 3), inf),
        "values of a late position": lambda: inp.v_suf.__setitem__((2, S - 1, Hkv - 1, D - 1), nan),
        "keys of a late position": lambda: inp.k_suf.__setitem__((1, S - 1, 0, 7), inf),
        "a query row": lambda: inp.q.__setitem__((2, 0, 0, 5), inf),
        "an incoming gradient": lambda: dout_host.__setitem__((1, 0, Hq - 1, 9), inf),
        "the last prefix row": lambda: inp.v_pre.__setitem__((P - 1, 0, 11), inf) if P else None,
    }
    for name, plant in plants.items():
        kept = {n: getattr(inp, n).copy() for n in ("q", "k_suf", "v_suf", "v_pre")}
        kept_dout = dout_host.copy()
        plant()
        d = pu.to_device(inp)
        dout = (torch.from_numpy(dout_host).view(torch_type) if dtype == "bf16" else torch.from_numpy(dout_host)).to("cuda:0")
        print(f"[case] hidden {dtype} D={D} P={P} S={S} Hq={Hq} Hkv={Hkv} B={B} {impl}: {name}", flush=True)
        lse = torch.empty((B, Hq, S), device="cuda:0")
        out = pk.pskv_attn_fwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], lse=lse, impl=impl, scale=inp.scale)
        grads = pk.pskv_attn_bwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], out, lse, dout, impl=impl,
                                 scale=inp.scale)
        torch.cuda.synchronize()
        with np.errstate(all="ignore"):
            refs = visible_only(*(widen(getattr(inp, n)) for n in ("q", "k_suf", "v_suf", "k_pre", "v_pre")), inp.suf_len,
                                widen(dout_host), inp.scale)
        for what, got, ref in zip(("out", "dq", "dk_suf", "dv_suf"), (out, *grads), refs):
            agree(pu.out_to_f64(got), ref, 2e-2 if dtype == "bf16" else 1e-5, f"{name}: {what}")
        for n, v in kept.items():
            getattr(inp, n)[...] = v
        dout_host[...] = kept_dout
