"""Forward candidate passes of four blocks against the oracle, at the edges of their rings, pairs of steps and
passes; that a problem takes them is checked as well."""
import numpy as np
import pytest

import launch_notes as notes
import parity_util as pu
from paper_2603_13420_amd import inputs as gen

pytestmark = pytest.mark.gpu

BF16_ONE, BF16_TWELVE = 0x3F80, 0x4140


@pytest.fixture(scope="module")
def pk():
    from paper_2603_13420_amd import binding
    return binding


def takes_four(tmp_path, w, Np=1):
    (rc, got), = notes.launches(tmp_path, [notes.case("fwd", "bf16", 128, w.B, w.P, w.S, w.Hq, w.Hkv, Np, lens=True)])
    assert rc == 0 and "stream_candidate4" in got[0][2], got


def check(pk, inp):
    import torch
    w, d = inp.w, pu.to_device(inp)
    print(f"[case] B={w.B} P={w.P} S={w.S} len={w.len_lo}..{w.len_hi} Hq={w.Hq} Hkv={w.Hkv} seed={w.seed}", flush=True)
    out = torch.full_like(d["q"], float("nan"))
    lse = torch.full((w.B, w.Hq, w.S), 7.5, device="cuda:0")
    pk.pskv_attn_fwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], out=out, lse=lse, scale=inp.scale)
    torch.cuda.synchronize()
    ref, ref_lse = pu.oracle_out(inp, want_lse=True)
    pu.compare_lse(lse.cpu().numpy().astype(np.float64), ref_lse, inp.suf_len, "bf16", w.name)
    pu.compare(pu.out_to_f64(out), ref, inp.suf_len, "bf16", w.name)


@pytest.mark.parametrize("B,P,S,lo,Hq,Hkv", [
    (3, 65, 64, 0, 8, 2),       # the shortest prefix: three tiles, the last one of one key; four or five tiles in all
    (3, 96, 64, 33, 8, 2),      # four and five tiles, one more than the rings hold after the first step
    (4, 200, 40, 0, 32, 4),     # passes of four and of two blocks; the own keys end in their second tile
    (2, 256, 96, 1, 4, 1),      # whole prefix tiles, an odd number of tiles in the last pass
    (3, 300, 128, 97, 2, 2),    # one pass for all of a candidate's rows
    (3, 70, 160, 0, 8, 2),      # blocks that see one to five own tiles in one pass
    (2, 640, 80, 80, 8, 2),     # a longer prefix
    (2, 130, 59, 20, 32, 4),    # rows that fill no whole number of blocks
    (70, 128, 64, 0, 32, 8),    # several passes for a workgroup, some of them nothing but padding
])
def test_candidate4(pk, tmp_path, B, P, S, lo, Hq, Hkv):
    w = gen.custom_workload(f"cand4_{B}_{P}_{S}", B, P, S, lo, S, Hq, Hkv, 128, "bf16", index=2100 + B + P)
    takes_four(tmp_path, w)
    check(pk, gen.make_inputs(w, pad="nan"))


@pytest.mark.parametrize("P,S", [(100, 96), (130, 59)])
def test_candidate4_scores_far_above_the_first_tile(pk, tmp_path, P, S):
    """A late key of 130 and more above everything before it: the general path, with 256 threads."""
    w = gen.custom_workload(f"cand4_spike_{P}_{S}", 3, P, S, S - 10, S, 32, 4, 128, "bf16", index=2200 + P + S)
    takes_four(tmp_path, w)
    inp = gen.make_inputs(w, pad="nan")
    inp.q[1, :inp.suf_len[1]] = BF16_ONE
    inp.k_pre[P - 3] = BF16_TWELVE
    check(pk, inp)


def test_candidate4_multi_instruction(pk, tmp_path):
    """Prefixes of their own lengths, one too short for the pipeline, one empty."""
    import torch
    w = gen.custom_multi_workload("cand4_multi", 3, 2, 100, 66, 100, 96, 0, 96, 8, 2, 128, "bf16", index=2300)
    takes_four(tmp_path, w, 3)
    inp = gen.make_multi_inputs(w, pad="nan")
    inp.pre_len[:2] = 0, 40
    inp.k_pre[0] = inp.v_pre[0] = 0x7FC0
    inp.k_pre[1, :60] = inp.v_pre[1, :60] = 0x7FC0
    d = pu.to_device_multi(inp)
    out = pk.pskv_attn_fwd_multi(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["pre_len"], d["suf_len"],
                                 scale=inp.scale)
    torch.cuda.synchronize()
    pu.compare(pu.out_to_f64(out), pu.oracle_out_multi(inp), inp.suf_len, "bf16", w.name)
