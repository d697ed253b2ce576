"""Forward calls of candidates whose rows fill no whole number of 32-row blocks, against the oracle.  They bring
lengths; test_parity_without_lengths_gpu.py has calls without."""
import numpy as np
import pytest

import parity_util as pu
from paper_2603_13420_amd import inputs as gen

pytestmark = pytest.mark.gpu

BF16_ONE, BF16_TWELVE = 0x3F80, 0x4140


@pytest.fixture(scope="module")
def pk():
    from paper_2603_13420_amd import binding
    return binding


def check(pk, inp):
    import torch
    w, d = inp.w, pu.to_device(inp)
    print(f"[case] B={w.B} P={w.P} S={w.S} len={w.len_lo}..{w.len_hi} Hq={w.Hq} Hkv={w.Hkv} seed={w.seed}", flush=True)
    guard = 7.5   # in front of and behind the tensors: nothing outside of them is written
    flat = torch.full((d["q"].numel() + 8192,), guard, device="cuda:0", dtype=torch.bfloat16)
    out = flat[4096:-4096].view(d["q"].shape)
    out.fill_(float("nan"))
    lse = torch.full((w.B * w.Hq * w.S + 128,), guard, device="cuda:0")
    pk.pskv_attn_fwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], out=out,
                     lse=lse[64:-64].view(w.B, w.Hq, w.S), scale=inp.scale)
    torch.cuda.synchronize()
    assert all((t == guard).all().item() for t in (flat[:4096], flat[-4096:], lse[:64], lse[-64:]))
    ref, ref_lse = pu.oracle_out(inp, want_lse=True)
    pu.compare_lse(lse[64:-64].view(w.B, w.Hq, w.S).cpu().numpy().astype(np.float64), ref_lse, inp.suf_len, "bf16", w.name)
    pu.compare(pu.out_to_f64(out), ref, inp.suf_len, "bf16", w.name)


@pytest.mark.parametrize("B,P,S,lo,hi,Hq,Hkv", [
    (5, 65, 31, 0, 31, 2, 2),       # one block, one row short; candidates may be empty; a ragged third tile
    (600, 96, 26, 26, 26, 4, 4),    # 26 of 32 rows, the least that can take this path; here a wavefront would have two blocks for one
    (1200, 96, 26, 26, 26, 4, 4),   # ... and takes it: three blocks for two
    (600, 96, 25, 25, 25, 4, 4),    # one row less: the general kernel
    (3, 256, 19, 1, 19, 6, 2),      # 57 rows, the whole prefix
    (4, 129, 31, 0, 31, 7, 1),      # 217 rows, group 7: blocks of pure padding in between
    (1, 200, 9, 9, 9, 28, 4),       # 63 rows
    (3, 257, 27, 0, 27, 4, 2),      # streamed prefix; 54 rows
    (40, 350, 30, 30, 30, 32, 8),   # ... 120 rows, more passes than compute units for some heads
    (2, 300, 53, 0, 53, 4, 4),      # ... two suffix steps
    (300, 300, 13, 0, 13, 32, 8),   # ... the general kernel: own blocks would take a round more
    (5, 130, 91, 20, 91, 32, 32),   # long suffix, prefix resident: the general kernel, its passes being 3/8 full
    (3, 130, 71, 20, 71, 7, 1),     # a candidate's passes, its own keys staged like the prefix; 497 rows
    (5, 70, 65, 0, 65, 28, 4),      # ... 455 rows, the third own tile holds one key; empty candidates
    (2, 700, 35, 1, 35, 28, 4),     # ... behind a long prefix
])
def test_own_blocks(pk, B, P, S, lo, hi, Hq, Hkv):
    w = gen.custom_workload(f"own_{B}_{P}_{S}", B, P, S, lo, hi, Hq, Hkv, 128, "bf16", index=1900 + B + P)
    check(pk, gen.make_inputs(w, pad="nan"))


@pytest.mark.parametrize("P,S,lo,Hq,Hkv", [(100, 27, 20, 4, 2), (300, 27, 20, 4, 2), (300, 53, 40, 4, 4), (130, 71, 60, 7, 1)])
def test_own_blocks_scores_far_above_the_first_tile(pk, P, S, lo, Hq, Hkv):
    """A late key of 130 and more above everything before it: the general path takes over."""
    w = gen.custom_workload(f"own_spike_{P}_{S}", 6, P, S, lo, S, Hq, Hkv, 128, "bf16", index=1950 + P + S)
    inp = gen.make_inputs(w, pad="nan")
    inp.q[1, :inp.suf_len[1]] = BF16_ONE
    inp.k_pre[P - 3] = BF16_TWELVE
    check(pk, inp)


@pytest.mark.parametrize("P,S", [(100, 13), (130, 29), (300, 13), (300, 53), (100, 71)])
def test_own_blocks_multi_instruction(pk, P, S):
    """Prefixes of their own lengths, some too short for the pipeline, one empty."""
    import torch
    w = gen.custom_multi_workload(f"own_multi_{P}_{S}", 5, 7, P, 0, P, S, 0, S, 8, 2, 128, "bf16", index=2000 + P + S)
    inp = gen.make_multi_inputs(w, pad="nan")
    inp.pre_len[:2] = 0, min(40, inp.pre_len[1])
    inp.k_pre[0] = inp.v_pre[0] = 0x7FC0
    inp.k_pre[1, :P - 40] = inp.v_pre[1, :P - 40] = 0x7FC0
    d = pu.to_device_multi(inp)
    out = pk.pskv_attn_fwd_multi(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["pre_len"], d["suf_len"],
                                 scale=inp.scale)
    torch.cuda.synchronize()
    pu.compare(pu.out_to_f64(out), pu.oracle_out_multi(inp), inp.suf_len, "bf16", w.name)
