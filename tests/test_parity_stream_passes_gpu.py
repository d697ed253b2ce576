"""Forward candidate passes of eight blocks, pipelined passes with three own steps and passes over packed rows with two and three
window steps against the oracle, at the edges of their rings, blocks and passes; that a problem takes the kernel is checked as well."""
import numpy as np
import pytest

import launch_notes as notes
import parity_util as pu
from paper_2603_13420_amd import inputs as gen
from test_parity_candidate4_gpu import BF16_ONE, BF16_TWELVE, check, pk  # noqa: F401 (pk is a fixture)

pytestmark = pytest.mark.gpu


def takes(tmp_path, kernel, w, Np=1):
    (rc, got), = notes.launches(tmp_path, [notes.case("fwd", "bf16", 128, w.B, w.P, w.S, w.Hq, w.Hkv, Np, lens=True)])
    assert rc == 0 and notes.named(got[0][2], kernel), got


@pytest.mark.parametrize("kernel,B,P,S,lo,hi,Hq,Hkv", [
    ("stream_candidate<true>", 17, 97, 64, 0, 64, 32, 8),      # four prefix tiles, the last one of one key; one pass of eight blocks
    ("stream_candidate<true>", 17, 128, 64, 33, 64, 32, 8),    # whole prefix tiles
    ("stream_candidate<true>", 9, 640, 128, 65, 128, 32, 8),   # a long prefix, two passes, up to four own tiles
    ("stream_candidate<true>", 64, 120, 64, 0, 20, 32, 8),     # several passes for a workgroup, most blocks nothing but padding
    ("stream_candidate<false>", 17, 128, 44, 0, 44, 32, 8),    # one pass of six blocks, the last one half full
    ("stream_candidate<false>", 17, 256, 60, 1, 60, 32, 8),    # the longest resident prefix
    ("stream_candidate<false>", 12, 200, 90, 5, 90, 32, 8),    # passes of eight and of four blocks, three own tiles
    ("stream_candidate<false>", 9, 130, 150, 0, 150, 32, 8),   # passes of eight, eight and three, five own tiles
    ("stream_candidate<false>", 17, 300, 60, 33, 60, 32, 8),   # a long prefix
    ("stream_packed<3>", 65, 200, 64, 0, 64, 8, 8),
    ("stream_packed<3>", 65, 257, 64, 33, 64, 8, 8),
    ("stream_packed<3>", 65, 257, 54, 0, 54, 8, 8),
    ("stream_packed<3>", 65, 300, 60, 30, 60, 8, 8),
    ("stream_pipelined<false,true>", 33, 288, 40, 0, 40, 32, 8),    # two own steps, whole blocks of grouped heads
    ("stream_pipelined<false,false>", 33, 288, 92, 0, 92, 16, 16),  # three own steps
])
def test_stream_passes(pk, tmp_path, kernel, B, P, S, lo, hi, Hq, Hkv):  # noqa: F811
    w = gen.custom_workload(f"passes_{B}_{P}_{S}", B, P, S, lo, hi, Hq, Hkv, 128, "bf16", index=2400 + B + P + S)
    takes(tmp_path, kernel, w)
    check(pk, gen.make_inputs(w, pad="nan"))


@pytest.mark.parametrize("kernel,B,P,S,Hq,Hkv", [
    ("stream_candidate<true>", 17, 100, 64, 32, 8), ("stream_candidate<false>", 17, 130, 44, 32, 8),
    ("stream_packed<3>", 65, 200, 64, 8, 8), ("stream_packed<3>", 65, 260, 60, 8, 8),
])
def test_scores_far_above_the_first_tile(pk, tmp_path, kernel, B, P, S, Hq, Hkv):  # noqa: F811
    """A late key of 130 and more above everything before it: the workgroup's passes once more on the general path."""
    w = gen.custom_workload(f"passes_spike_{P}_{S}", B, P, S, S - 10, S, Hq, Hkv, 128, "bf16", index=2500 + P + S)
    takes(tmp_path, kernel, w)
    inp = gen.make_inputs(w, pad="nan")
    inp.q[1, :inp.suf_len[1]] = BF16_ONE
    inp.k_pre[P - 3] = BF16_TWELVE
    check(pk, inp)


@pytest.mark.parametrize("kernel,P,S", [("stream_candidate<true>", 128, 64), ("stream_candidate<false>", 160, 44)])
def test_multi_instruction(pk, tmp_path, kernel, P, S):  # noqa: F811
    """Prefixes of their own lengths, one empty, one too short for the pipeline."""
    import torch
    w = gen.custom_multi_workload(f"passes_multi_{P}", 3, 6, P, 66, P, S, 0, S, 32, 8, 128, "bf16", index=2600 + P)
    takes(tmp_path, kernel, w, 3)
    inp = gen.make_multi_inputs(w, pad="nan")
    inp.pre_len[:2] = 0, 40
    inp.k_pre[0] = inp.v_pre[0] = 0x7FC0
    inp.k_pre[1, :P - 40] = inp.v_pre[1, :P - 40] = 0x7FC0
    d = pu.to_device_multi(inp)
    print(f"[case] {w.name} seed={w.seed}", flush=True)
    out = pk.pskv_attn_fwd_multi(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["pre_len"], d["suf_len"],
                                 scale=inp.scale)
    torch.cuda.synchronize()
    assert not np.isnan(pu.out_to_f64(out)).any()
    pu.compare(pu.out_to_f64(out), pu.oracle_out_multi(inp), inp.suf_len, "bf16", w.name)
