"""GPU parity of the matrix-core kernels whose 32-row blocks lie inside one candidate (bf16, heads of 128
columns) against the CPU oracle, at the sizes where the split of the work changes: rows per candidate
around the block and pass sizes, prefixes around the tile and the resident limit.  The bars are those of every
bf16 comparison (oracle/parity.py)."""
import numpy as np
import pytest

from paper_2603_13420_amd import inputs as gen
import parity_util as pu
from test_parity_hd64_gpu import check, pk  # noqa: F401 (pk is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,P,S,lo,hi,Hq,Hkv", [
    (5, 0, 1, 0, 1, 1, 1),          # no prefix, one row
    (9, 32, 11, 0, 11, 2, 2),       # the most rows a candidate can have without a block of its own ...
    (9, 33, 12, 1, 12, 2, 2),       # ... and the fewest with one
    (7, 31, 33, 1, 33, 2, 2),       # a second block of one row, a second own step
    (4, 256, 24, 0, 24, 8, 2),      # whole blocks, the longest resident prefix
    (3, 257, 24, 1, 24, 8, 2),      # ... one row more
    (3, 64, 25, 20, 25, 8, 2),      # four blocks, the last one of four rows: one pass
    (3, 1, 129, 100, 129, 2, 2),    # five blocks of five own steps
    (2, 65, 31, 0, 31, 14, 2),      # group of seven, seven blocks in two passes
    (2, 300, 65, 40, 65, 7, 1),     # long prefix, fifteen blocks
    (200, 40, 32, 5, 32, 8, 2),     # more passes than workgroups
])
def test_blocks_of_one_candidate(pk, B, P, S, lo, hi, Hq, Hkv):  # noqa: F811
    w = gen.custom_workload(f"cand_{B}_{P}_{S}", B, P, S, lo, hi, Hq, Hkv, 128, "bf16", index=2100 + B + P)
    check(pk, gen.make_inputs(w, pad="nan"), w.name)


def test_blocks_multi_instruction_backward(pk):  # noqa: F811
    """Prefixes of their own lengths, one empty: 9 and 40 positions of 4 heads (two blocks; five, four in a pass
    and one over)."""
    import torch
    for S in (9, 40, 56):
        w = gen.custom_multi_workload(f"cand_multi_{S}", 3, 4, 70, 0, 70, S, 0, S, 8, 2, 128, "bf16", index=2150 + S)
        inp = gen.make_multi_inputs(w, pad="nan")
        inp.pre_len[1] = 0
        inp.k_pre[1] = inp.v_pre[1] = 0x7FC0
        d = pu.to_device_multi(inp)
        lse = torch.full((w.Np * w.C, w.Hq, w.S), 123.0, device="cuda:0")
        out = pk.pskv_attn_fwd_multi(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["pre_len"], d["suf_len"],
                                     lse=lse, scale=inp.scale)
        torch.cuda.synchronize()
        pu.compare(pu.out_to_f64(out), pu.oracle_out_multi(inp), inp.suf_len, "bf16", w.name)
        dout_host, dout64 = pu.make_dout(inp, w.seed + 7)
        dout = torch.from_numpy(dout_host).view(torch.bfloat16).to("cuda:0")
        dq, dk, dv = pk.pskv_attn_bwd_multi(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["pre_len"],
                                            d["suf_len"], out, lse, dout, scale=inp.scale)
        torch.cuda.synchronize()
        refs = pu.oracle_bwd_multi(inp, dout64)
        valid = np.arange(w.S)[None, :] < inp.suf_len[:, None]
        for name, got, r in zip(("dq", "dk_suf", "dv_suf"), (dq, dk, dv), refs):
            pu.compare_grad(pu.out_to_f64(got), r, valid, "bf16", f"{w.name} {name}")


def test_rows_too_far_apart_for_32_bit_offsets(pk):  # noqa: F811
    """A candidate whose query rows span more than 2^31 bytes: the kernels that address rows by 64-bit offsets."""
    import torch
    w = gen.custom_workload("cand_far", 1, 40, 33, 33, 33, 4, 2, 128, "bf16", index=2170)
    inp = gen.make_inputs(w, pad="nan")
    d = pu.to_device(inp)
    far = (2 ** 30 // 32 + 127) // 128 * 128
    def spread():
        return torch.empty(w.S * far, device="cuda:0", dtype=torch.bfloat16).as_strided((1, w.S, w.Hq, 128), (w.S * far, far, 128, 1))
    q, dq = spread(), spread()
    q.copy_(d["q"])
    lse = torch.empty((1, w.Hq, w.S), device="cuda:0")
    out = torch.full_like(d["q"], float("nan"))
    pk.pskv_attn_fwd(q, d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], out=out, lse=lse, scale=inp.scale)
    torch.cuda.synchronize()
    pu.compare(pu.out_to_f64(out), pu.oracle_out(inp), inp.suf_len, "bf16", w.name)
    dout_host, dout64 = pu.make_dout(inp, w.seed + 7)
    dout = torch.from_numpy(dout_host).view(torch.bfloat16).to("cuda:0")
    dk, dv = torch.empty_like(d["k_suf"]), torch.empty_like(d["k_suf"])
    pk.pskv_attn_bwd(q, d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], out, lse, dout, dq=dq, dk_suf=dk,
                     dv_suf=dv, scale=inp.scale)
    torch.cuda.synchronize()
    valid = np.ones((1, w.S), dtype=bool)
    for name, got, r in zip(("dq", "dk_suf", "dv_suf"), (dq.contiguous(), dk, dv), pu.oracle_bwd(inp, dout64)):
        pu.compare_grad(pu.out_to_f64(got), r, valid, "bf16", f"{w.name} {name}")
