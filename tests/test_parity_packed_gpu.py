"""GPU parity of the kernels over packed rows, where they can go wrong: blocks across candidates and inside them, in ranges and in
turn, windows of one step and of two, more candidates than threads, empty candidates, candidates far apart in memory, prefixes too
short for the pipeline, rows that need rescaling.  Padded rows hold NaN; results start as NaN.  Which list a problem makes is asked of
the kernels' own function (test_packed_lists.py) where a test is about that."""
import numpy as np
import pytest

from paper_2603_13420_amd import inputs as gen
import parity_util as pu
from test_packed_lists import lib as lists, packed  # noqa: F401 (lists is a fixture)
from test_parity_own_blocks_gpu import check as check_guarded

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_13420_amd import binding
    binding.load()
    return binding


def put_lengths(inp, lens):
    """Other lengths than the drawn ones, with the padding they mean."""
    inp.suf_len[:] = lens
    pad = np.arange(inp.w.S)[None, :] >= inp.suf_len[:, None]
    rng = np.random.default_rng(inp.w.seed + 1)
    for x in (inp.q, inp.k_suf, inp.v_suf):
        x[...] = gen.f32_to_bf16_bits(rng.standard_normal(x.shape, dtype=np.float32))
        x[pad] = 0x7FC0


def check(pk, inp, q_batch_stride=0, backward=True):
    import torch
    w, multi = inp.w, hasattr(inp, "pre_len")
    d = (pu.to_device_multi if multi else pu.to_device)(inp)
    print(f"[case] {w.name} P={w.P} S={w.S} Hq={w.Hq} Hkv={w.Hkv} lens={inp.suf_len.tolist()[:12]} seed={w.seed}", flush=True)
    q = d["q"]
    B, S, Hq, D = q.shape
    if q_batch_stride:
        far = torch.empty(B * q_batch_stride, dtype=q.dtype, device="cuda:0").as_strided(q.shape, (q_batch_stride, Hq * D, D, 1))
        far.copy_(q)
        q = far
    out = torch.full((B, S, Hq, D), float("nan"), dtype=q.dtype, device="cuda:0")
    lse = torch.full((B, Hq, S), 123.0, device="cuda:0")
    args = (q, d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"]) + ((d["pre_len"],) if multi else ()) + (d["suf_len"],)
    (pk.pskv_attn_fwd_multi if multi else pk.pskv_attn_fwd)(*args, out=out, lse=lse, scale=inp.scale)
    torch.cuda.synchronize()
    ref, ref_lse = (pu.oracle_out_multi if multi else pu.oracle_out)(inp, want_lse=True)
    pu.compare_lse(lse.cpu().numpy().astype(np.float64), ref_lse, inp.suf_len, w.dtype, w.name)
    pu.compare(pu.out_to_f64(out), ref, inp.suf_len, w.dtype, w.name)
    if not backward:
        return
    dout_host, dout64 = pu.make_dout(inp, w.seed + 7)
    dout = torch.from_numpy(dout_host).view(torch.bfloat16).to("cuda:0")
    grads = [torch.empty_strided(x.shape, x.stride(), dtype=x.dtype, device="cuda:0").fill_(float("nan")) for x in (q, d["k_suf"], d["v_suf"])]
    (pk.pskv_attn_bwd_multi if multi else pk.pskv_attn_bwd)(*args, out, lse, dout, dq=grads[0], dk_suf=grads[1], dv_suf=grads[2], scale=inp.scale)
    torch.cuda.synchronize()
    valid = np.arange(S)[None, :] < inp.suf_len[:, None]
    for name, got, r in zip(("dq", "dk_suf", "dv_suf"), grads, (pu.oracle_bwd_multi if multi else pu.oracle_bwd)(inp, dout64)):
        got = pu.out_to_f64(got.contiguous())
        assert not got[~valid].any(), f"{name}: padded rows must be exactly 0"
        pu.compare_grad(got, r, valid, w.dtype, f"{w.name} {name}")


@pytest.mark.parametrize("B,P,S,lo,Hq,Hkv", [
    (7, 96, 20, 1, 4, 4),        # two-step windows, three prefix tiles
    (40, 97, 5, 0, 2, 2),        # many candidates in a block, ragged prefix
    (9, 256, 25, 17, 8, 2),      # one-step windows across candidates, the longest resident prefix
    (9, 255, 26, 20, 8, 2),      # ... the first suffix length whose windows go on
    (6, 130, 32, 32, 4, 4),      # whole blocks, nothing padded
    (6, 130, 32, 1, 4, 4),       # ... mostly padded
    (11, 100, 19, 3, 7, 1),      # heads that do not divide a block
    (3, 128, 31, 9, 40, 1),      # more heads than rows in a block
    (1, 96, 1, 1, 1, 1),
    (9, 1, 20, 1, 4, 4),         # one prefix tile: a single row, all but full, full
    (9, 31, 24, 1, 8, 2),
    (9, 32, 19, 4, 7, 1),
    (9, 33, 20, 1, 4, 4),        # two: the second with one row, full
    (30, 64, 24, 8, 8, 2),
    (1300, 128, 3, 0, 2, 1),     # six candidates per thread of those that add the lengths up
    (2200, 96, 2, 0, 1, 1),      # more lengths than it holds at a time
    (7, 40, 40, 33, 8, 2),       # (backward) one prefix tile, windows of up to 48 positions
    (6, 0, 64, 1, 4, 4),         # ... no prefix, the longest suffix
    (5, 256, 57, 20, 14, 2),
])
def test_packed_rows(pk, B, P, S, lo, Hq, Hkv):
    w = gen.custom_workload(f"packed_{B}_{P}_{S}", B, P, S, lo, S, Hq, Hkv, 128, "bf16", index=3100 + B + P + S)
    check(pk, gen.make_inputs(w, pad="nan"))


@pytest.mark.parametrize("B,P,S,lo,Hq,Hkv", [
    (7, 257, 20, 1, 4, 4),       # streamed prefixes: a ragged last tile, two-step windows, one block per pass
    (40, 288, 9, 0, 2, 2),
    (12, 512, 64, 32, 4, 4),     # windows of three steps
    (9, 300, 64, 64, 2, 2),      # ... nothing padded
    (10, 400, 25, 3, 14, 2),     # one-step windows
    (300, 320, 21, 1, 10, 10),   # several blocks per pass, some passes with fewer
    (2200, 260, 2, 0, 1, 1),     # more lengths than are held at a time
    (4200, 260, 2, 0, 3, 3),     # ... and than a search takes at once; heads that no XCD has alone
])
def test_packed_rows_streamed(pk, B, P, S, lo, Hq, Hkv):
    w = gen.custom_workload(f"packed_stream_{B}_{P}_{S}", B, P, S, lo, S, Hq, Hkv, 128, "bf16", index=3500 + B + P + S)
    check(pk, gen.make_inputs(w, pad="nan"), backward=False)


@pytest.mark.parametrize("P", [120, 300])
@pytest.mark.parametrize("name", ["none", "first", "last", "middle", "one", "alternate"])
def test_empty_candidates(pk, name, P):
    B, S = 70, 24
    lens = {"none": [0] * B, "first": [0] * 40 + [S] * 30, "last": [9] * 30 + [0] * 40, "middle": [S] * 5 + [0] * 60 + [7] * 5,
            "one": [0] * 33 + [13] + [0] * 36, "alternate": [(i % 2) * (i % S + 1) for i in range(B)]}[name]
    w = gen.custom_workload(f"packed_empty_{name}_{P}", B, P, S, 0, S, 14, 2, 128, "bf16", index=3200 + P)
    inp = gen.make_inputs(w, pad="nan")
    put_lengths(inp, lens)
    check(pk, inp)


@pytest.mark.parametrize("P", [100, 300])
def test_candidates_far_apart(pk, P):
    # 150 empty candidates between two that share a block, query rows of consecutive ones 16 MB apart: beyond 32-bit offsets
    B, S = 300, 8
    w = gen.custom_workload(f"packed_far_{P}", B, P, S, 0, S, 2, 1, 128, "bf16", index=3201)
    inp = gen.make_inputs(w, pad="nan")
    put_lengths(inp, [3] + [0] * 150 + [8] * 20 + [0] * 128 + [5])
    check(pk, inp, q_batch_stride=(1 << 23) - 8)


def alignment(lists, w, lens, streamed=False, P=None):
    """(window steps, alignment) of the list that the kernel makes of these lengths on this card."""
    import torch
    cus, heads, G = torch.cuda.get_device_properties(0).multi_processor_count, getattr(w, "Np", 1) * w.Hkv, w.Hq // w.Hkv
    C = w.B // getattr(w, "Np", 1)
    wavefronts = 0 if streamed else 8 * min(cus // min(heads, cus), C * ((w.S * G + 31) // 32))
    steps, _, align, _ = packed(lists, [int(x) for x in lens], w.S, w.Hq, w.Hkv, 3 if streamed else 2, w.P if P is None else P, wavefronts)
    return steps, align


@pytest.mark.parametrize("Hq,Hkv,P", [(32, 32, 100), (64, 32, 100), (96, 32, 50), (32, 32, 20)])
def test_candidates_far_apart_in_one_block(pk, lists, Hq, Hkv, P):
    # the same where blocks go across candidates in the resident kernels, dq among them: they end early, at an empty candidate
    B, S = 330, 8
    lens = [3] + [0] * 140 + [8] * 90 + [0] * 98 + [5]
    w = gen.custom_workload(f"packed_far_{P}_{Hq}", B, P, S, 0, S, Hq, Hkv, 128, "bf16", index=3202 + Hq)
    assert alignment(lists, w, lens)[1] == 1
    inp = gen.make_inputs(w, pad="nan")
    put_lengths(inp, lens)
    check(pk, inp, q_batch_stride=(1 << 23) - 8)


# More blocks than wavefronts: 32 key heads have eight workgroups, 64 wavefronts, each.
@pytest.mark.parametrize("B,P,S,lo,Hq,Hkv,steps,align", [
    (140, 20, 10, 1, 32, 32, 2, 1),      # across candidates: one prefix tile, two, and more; two window steps
    (140, 50, 12, 1, 32, 32, 2, 1),
    (140, 200, 20, 1, 32, 32, 2, 1),
    (300, 130, 9, 0, 32, 32, 2, 1),      # ... empty candidates in blocks
    (60, 130, 20, 5, 128, 32, 1, 1),     # ... one step
    (60, 40, 24, 9, 128, 32, 1, 1),
    (40, 100, 19, 3, 224, 32, 1, 1),     # ... groups of seven
    (150, 128, 20, 20, 32, 32, 2, 32),   # a block for each candidate, in turn
    (150, 128, 20, 12, 32, 32, 2, 32),   # ... lengths differ, blocks do not
    (200, 31, 32, 2, 32, 32, 2, 32),
    (130, 64, 32, 32, 32, 32, 2, 32),
    (150, 40, 32, 30, 32, 32, 2, 32),    # ... some blocks of two rows less
    (70, 150, 32, 32, 64, 32, 2, 32),    # ... two blocks for each
    (40, 33, 28, 28, 128, 32, 2, 32),    # ... four, the last one half full
    (130, 100, 32, 0, 32, 32, 2, 32),    # candidates without rows: blocks in ranges again
])
def test_lists_of_more_blocks_than_wavefronts(pk, lists, B, P, S, lo, Hq, Hkv, steps, align):
    w = gen.custom_workload(f"packed_many_{B}_{P}_{S}_{lo}", B, P, S, lo, S, Hq, Hkv, 128, "bf16", index=3650 + B + P + S + lo)
    inp = gen.make_inputs(w, pad="nan")
    assert alignment(lists, w, inp.suf_len) == (steps, align)
    check(pk, inp)


@pytest.mark.parametrize("Np,C,P,S,lo,Hq,Hkv,align", [
    (4, 80, 200, 20, 2, 8, 8, 1), (4, 80, 100, 20, 20, 8, 8, 32), (2, 60, 64, 20, 4, 64, 16, 1),
])
def test_such_lists_of_several_instructions(pk, lists, Np, C, P, S, lo, Hq, Hkv, align):
    w = gen.custom_multi_workload(f"packed_many_multi_{P}_{lo}", Np, C, P, P, P, S, lo, S, Hq, Hkv, 128, "bf16", index=3850 + P + lo)
    inp = gen.make_multi_inputs(w, pad="nan")
    inp.pre_len[:2] = P, P // 3         # (the second one goes the general way, or has fewer tiles)
    inp.k_pre[1, :P - P // 3] = inp.v_pre[1, :P - P // 3] = 0x7FC0
    for n in range(Np):
        assert alignment(lists, w, inp.suf_len[n * C:(n + 1) * C], P=int(inp.pre_len[n]))[1] == align
    check(pk, inp)


@pytest.mark.parametrize("B,P,S,lo,Hq,Hkv,align", [
    (140, 200, 20, 1, 32, 32, 1), (60, 130, 20, 5, 128, 32, 1), (150, 128, 20, 12, 32, 32, 32), (70, 150, 32, 32, 64, 32, 32), (140, 60, 10, 1, 32, 32, 1),
])
def test_such_lists_with_rows_that_need_rescaling(pk, lists, B, P, S, lo, Hq, Hkv, align):
    w = gen.custom_workload(f"packed_many_rescale_{P}_{S}_{lo}", B, P, S, lo, S, Hq, Hkv, 128, "bf16", index=3900 + P + S + lo)
    inp = gen.make_inputs(w, pad="nan")
    assert alignment(lists, w, inp.suf_len)[1] == align
    inp.k_pre[P - 5] = gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(inp.k_pre[P - 5]) * 8)
    for b in (0, B // 2, B - 1):
        inp.q[b] = gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(inp.q[b]) * 8)
    for x in (inp.v_pre, inp.v_suf):    # (values as in test_rows_that_need_rescaling)
        x[...] = gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(x) * np.float32(0.25))
    check(pk, inp, backward=False)


@pytest.mark.parametrize("Np,C,P,S,lo,Hq,Hkv", [(6, 9, 128, 20, 1, 4, 4), (5, 30, 200, 24, 12, 8, 2), (40, 3, 100, 11, 0, 14, 2)])
def test_several_instructions(pk, Np, C, P, S, lo, Hq, Hkv):
    w = gen.custom_multi_workload(f"packed_multi_{Np}", Np, C, P, P, P, S, lo, S, Hq, Hkv, 128, "bf16", index=3300 + P)
    inp = gen.make_multi_inputs(w, pad="nan")
    inp.pre_len[:] = np.random.default_rng(w.seed).integers(0, P + 1, Np)
    inp.pre_len[:4] = P, 0, 1, 65
    for n in range(Np):
        inp.k_pre[n, :P - inp.pre_len[n]] = inp.v_pre[n, :P - inp.pre_len[n]] = 0x7FC0
    check(pk, inp)


@pytest.mark.parametrize("S,Hq,Hkv,P", [(20, 4, 4, 200), (24, 8, 2, 200), (20, 4, 4, 300), (50, 2, 2, 300)])
def test_rows_that_need_rescaling(pk, S, Hq, Hkv, P):
    # scores some 100 above the first tile's maximum, in a prefix tile for some rows and among the own keys for others
    w = gen.custom_workload(f"packed_rescale_{S}_{P}", 12, P, S, 5, S, Hq, Hkv, 128, "bf16", index=3400 + S)
    inp = gen.make_inputs(w, pad="nan")
    loud = lambda x: gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(x) * 8)
    inp.k_pre[150] = loud(inp.k_pre[150])
    inp.q[2:4] = loud(inp.q[2:4])
    inp.k_suf[7, 1] = loud(inp.k_suf[7, 1])
    inp.q[7] = loud(inp.q[7])
    # one key may carry a whole row: its error is up to 2 * 2^-8 |v| (weight and result rounded once each), and the absolute
    # bar of 2e-2 is for |v| < 2.5: values of standard deviation 1/4, whose largest here is below 1.4
    for x in (inp.v_pre, inp.v_suf):
        x[...] = gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(x) * np.float32(0.25))
    check(pk, inp, backward=False)


@pytest.mark.parametrize("S,lo", [(20, 20), (20, 3), (40, 30)])
def test_some_passes_need_rescaling(pk, S, lo):
    # several passes for a workgroup, of which few are repeated (values as above)
    w = gen.custom_workload(f"packed_repeat_{S}_{lo}", 300, 300, S, lo, S, 24, 24, 128, "bf16", index=3450 + S + lo)
    inp = gen.make_inputs(w, pad="nan")
    inp.k_pre[290] = gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(inp.k_pre[290]) * 8)
    for b in (0, 131, 299):
        inp.q[b, :, ::5] = gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(inp.q[b, :, ::5]) * 8)
    for x in (inp.v_pre, inp.v_suf):
        x[...] = gen.f32_to_bf16_bits(gen.bf16_bits_to_f32(x) * np.float32(0.25))
    check(pk, inp, backward=False)


@pytest.mark.parametrize("lens,S,Hq,Hkv,P", [
    ([38, 30, 30, 30], 40, 4, 4, 257),       # lengths whose rows, each filled up to whole blocks, are as many as B*S*G: not a full batch
    ([40, 32, 32, 32], 40, 4, 4, 300),
    ([32, 32, 48, 48] * 3, 48, 2, 2, 260),
    ([40, 32], 40, 4, 2, 320),
    ([59, 59, 41, 59, 55, 57, 60, 48], 60, 4, 2, 300),
    ([40] * 9, 40, 4, 4, 300),               # full ones
    ([64] * 5 + [33, 40], 64, 4, 4, 300),
])
def test_lengths_that_add_up_like_full_ones(pk, lens, S, Hq, Hkv, P):
    w = gen.custom_workload(f"packed_sum_{S}_{P}", len(lens), P, S, 0, S, Hq, Hkv, 128, "bf16", index=3600 + S + P)
    inp = gen.make_inputs(w, pad="nan")
    put_lengths(inp, lens)
    check_guarded(pk, inp)
