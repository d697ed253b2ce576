"""GPU parity of the matrix-core kernels for bf16 tensors with heads of 64 columns against the CPU
oracle, forward and backward, at the edges of their tiles, blocks and prefix chunks.  The bars are those
of every bf16 comparison (oracle/parity.py)."""
import numpy as np
import pytest

from paper_2603_13420_amd import inputs as gen
import parity_util as pu

pytestmark = pytest.mark.gpu
BF16_ONE, BF16_TWELVE = 0x3F80, 0x4140


@pytest.fixture(scope="module")
def pk():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_13420_amd import binding
    binding.load()
    return binding


def check(pk, inp, what, backward=True):
    import torch
    w, d = inp.w, pu.to_device(inp)
    print(f"[case] {what} B={w.B} P={w.P} S={w.S} len={w.len_lo}..{w.len_hi} Hq={w.Hq} Hkv={w.Hkv} seed={w.seed}", flush=True)
    lse = torch.full((w.B, w.Hq, w.S), 123.0, device="cuda:0")
    out = torch.full_like(d["q"], float("nan"))
    pk.pskv_attn_fwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], out=out, lse=lse, scale=inp.scale)
    torch.cuda.synchronize()
    ref, ref_lse = pu.oracle_out(inp, want_lse=True)
    pu.compare_lse(lse.cpu().numpy().astype(np.float64), ref_lse, inp.suf_len, "bf16", what)
    pu.compare(pu.out_to_f64(out), ref, inp.suf_len, "bf16", what)
    if not backward:
        return
    dout_host, dout64 = pu.make_dout(inp, w.seed + 7)
    dout = torch.from_numpy(dout_host).view(torch.bfloat16).to("cuda:0")
    nan = float("nan")
    dq, dk, dv = torch.full_like(d["q"], nan), torch.full_like(d["k_suf"], nan), torch.full_like(d["k_suf"], nan)
    pk.pskv_attn_bwd(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["suf_len"], out, lse, dout, dq=dq,
                     dk_suf=dk, dv_suf=dv, scale=inp.scale)
    torch.cuda.synchronize()
    rq, rk, rv = pu.oracle_bwd(inp, dout64)
    valid = np.arange(w.S)[None, :] < inp.suf_len[:, None]
    for name, got, r in (("dq", dq, rq), ("dk_suf", dk, rk), ("dv_suf", dv, rv)):
        pu.compare_grad(pu.out_to_f64(got), r, valid, "bf16", f"{what} {name}")


@pytest.mark.parametrize("B,P,S,lo,hi,Hq,Hkv", [
    (1, 0, 1, 1, 1, 1, 1),          # one row, one key
    (3, 32, 32, 0, 32, 4, 2),       # whole tiles; candidates may be empty
    (5, 33, 33, 1, 33, 14, 2),      # one past a tile everywhere, group 7
    (40, 20, 3, 0, 3, 2, 2),        # ten short candidates in a block: their keys share a step
    (9, 192, 10, 1, 10, 4, 4),      # the longest prefix that leaves room for two workgroups
    (4, 193, 70, 30, 70, 4, 1),     # ... one row more; three steps of own keys
    (3, 513, 20, 4, 20, 6, 2),      # prefix in chunks, forward and backward
    (300, 40, 24, 12, 24, 16, 16),  # one round of blocks, the last slots empty
    (400, 40, 24, 12, 24, 16, 16),  # more blocks than wavefronts
    (3, 512, 20, 4, 20, 6, 2),      # the longest prefix that stays in LDS
    (2, 1, 40, 0, 40, 4, 4),        # a prefix of one row, which stands in for the rest of its tile
])
def test_hd64(pk, B, P, S, lo, hi, Hq, Hkv):
    w = gen.custom_workload(f"hd64_{B}_{P}_{S}", B, P, S, lo, hi, Hq, Hkv, 64, "bf16", index=1800 + B + P)
    check(pk, gen.make_inputs(w, pad="nan"), w.name)


def test_hd64_scores_far_above_the_first_tile(pk):
    """A late prefix key and a late own key 90 and more above everything before them: rescaling.  Forward
    only: every other weight of such a row is exp(-90) = 2^-130 and less, under fp32's smallest normal number
    2^-126, and the gradients' bounds are relative ones (|err| <= const * p_j ...), which hold down to there."""
    w = gen.custom_workload("hd64_spike", 4, 200, 40, 33, 40, 4, 2, 64, "bf16", index=1850)
    inp = gen.make_inputs(w, pad="nan")
    inp.q[1, :inp.suf_len[1]] = BF16_ONE
    inp.k_pre[197] = BF16_TWELVE
    inp.q[2, :inp.suf_len[2]] = BF16_ONE
    inp.k_suf[2, inp.suf_len[2] - 1] = BF16_TWELVE
    check(pk, inp, w.name, backward=False)


def test_hd64_multi_instruction(pk):
    """Left-padded prefixes of their own lengths (one empty), NaN in the padding."""
    import torch
    w = gen.custom_multi_workload("hd64_multi", 4, 5, 70, 0, 70, 11, 0, 11, 6, 2, 64, "bf16", index=1860)
    inp = gen.make_multi_inputs(w, pad="nan")
    inp.pre_len[1] = 0
    inp.k_pre[1] = inp.v_pre[1] = 0x7FC0
    d = pu.to_device_multi(inp)
    out = pk.pskv_attn_fwd_multi(d["q"], d["k_suf"], d["v_suf"], d["k_pre"], d["v_pre"], d["pre_len"], d["suf_len"],
                                 scale=inp.scale)
    torch.cuda.synchronize()
    pu.compare(pu.out_to_f64(out), pu.oracle_out_multi(inp), inp.suf_len, "bf16", w.name)


@pytest.mark.parametrize("impl", ["simple", "auto"])
def test_hd64_weights_in_full(pk, impl):
    """Weights and score gradients enter the sums over keys and rows with the 24 bits that they are computed to.
    Every sum here is over three terms whose weights are known beforehand and whose other factors are
    chosen, one after the other, to cancel what is there so far: the result is some 2^-17 of the terms, which an
    error of 2^-17 in a weight (16 bits) changes entirely.  The bound: 2^-20 of the terms' magnitudes - an
    exponential to one unit (2^-23), its argument from a 32-term fp32 sum (2^-22 together with the scale), three
    fp32 additions (2^-24 each) - and the result's own rounding to bf16."""
    import torch
    rng = np.random.default_rng(1890)
    n, D, half, G = 32, 64, 32, 4
    bf16 = lambda x: gen.bf16_bits_to_f32(gen.f32_to_bf16_bits(np.asarray(x, np.float32))).astype(np.float64)

    def cancelling(w):
        """[n,3,D] bf16 values whose sums weighted by w [n,3] nearly vanish, column by column."""
        x = np.zeros((n, 3, D))
        x[:, 0] = bf16(256 * rng.uniform(1, 2, (n, D)))
        for t in (1, 2):
            x[:, t] = bf16(-np.einsum("nt,ntd->nd", w, x) / w[:, t, None])
        return x

    # one candidate of one row and a prefix of two for each of n instructions, four query heads; scores are made by the
    # first half of the columns, the other half of q and of K is zero or free
    q, K = bf16(rng.standard_normal((n, G, D))), bf16(rng.standard_normal((n, 3, D)))
    q[:, :, half:] = K[:, :, half:] = 0
    scale = float(np.float32(D ** -0.5))
    s = np.einsum("ngd,ntd->ngt", q, K) * scale
    lse = np.log(np.exp(s).sum(-1))
    p = np.exp(s - lse[..., None])                                          # [n,G,3]

    def dev(x):
        return torch.from_numpy(gen.f32_to_bf16_bits(x.astype(np.float32))).view(torch.bfloat16).to("cuda:0")

    def call(q, K, V, dout=None):
        args = (dev(q[:, None]), dev(K[:, 2:, None]), dev(V[:, 2:, None]), dev(K[:, :2, None]), dev(V[:, :2, None]))
        if dout is None:
            return pk.pskv_attn_fwd_multi(*args, impl=impl, scale=scale)
        # (a result of zeros: <dout,out> is zero, and a score gradient the weight times <dout,V>)
        return pk.pskv_attn_bwd_multi(*args, None, None, torch.zeros_like(args[0]),
                                      torch.from_numpy(lse.astype(np.float32)[..., None]).to("cuda:0"), dev(dout[:, None]), impl=impl,
                                      scale=scale)

    def check(got, ref, mag, what):
        err, bound = np.abs(pu.out_to_f64(got).reshape(ref.shape) - ref), 2.0 ** -20 * mag + 2.0 ** -8 * np.abs(ref)
        print(f"[case] weights in full {impl} {what}: {(err / bound).max():.3f} of the bound", flush=True)
        assert (err <= bound).all(), f"{what}: {(err / bound).max():.2f} times the bound"

    V = cancelling(p[:, 0])
    check(call(q, K, V), np.einsum("ngt,ntd->ngd", p, V), np.einsum("ngt,ntd->ngd", p, np.abs(V)), "out")
    # dv of the own key: over three of the query heads
    dout = np.concatenate([cancelling(p[:, :3, 2]), np.zeros((n, 1, D))], axis=1)
    check(call(q, K, V, dout)[2], np.einsum("ng,ngd->nd", p[..., 2], dout), np.einsum("ng,ngd->nd", p[..., 2], np.abs(dout)), "dv")
    # dq and dk: score gradients p <dout,V> of small whole numbers, exact in fp32
    V, dout = rng.integers(1, 4, (n, 3, D)).astype(np.float64), rng.integers(1, 4, (n, G, D)).astype(np.float64)
    ds = p * np.einsum("ngd,ntd->ngt", dout, V)
    K2 = K.copy()
    K2[:, :, half:] = cancelling(ds[:, 0])[:, :, half:]
    check(call(q, K2, V, dout)[0], scale * np.einsum("ngt,ntd->ngd", ds, K2), scale * np.einsum("ngt,ntd->ngd", ds, np.abs(K2)), "dq")
    q2 = q.copy()
    q2[:, :3, half:] = cancelling(ds[:, :3, 2])[:, :, half:]
    check(call(q2, K, V, dout)[1], scale * np.einsum("ng,ngd->nd", ds[..., 2], q2), scale * np.einsum("ng,ngd->nd", ds[..., 2], np.abs(q2)), "dk")


def test_a_key_weighs_the_same_as_prefix_and_as_own_key(pk):
    """The gradient of a row that sees 32 prefix keys (a whole tile) and one own key, and of one that sees the same 33 as
    its own: the same numbers in the same order, so the same bits (two million of them: one product in some hundred
    thousand shows in a bf16 result when it is rounded at another place)."""
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(11)
    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda:0", dtype=torch.bfloat16)
    B, H, D = 1024, 32, 64                               # one KV head: a block of rows is one position
    q, k1, v1, dout = normal(B, 1, H, D), normal(B, 1, 1, D), normal(B, 1, 1, D), normal(B, 1, H, D)
    kp, vp = normal(32, 1, D), normal(32, 1, D)
    one = torch.full((B,), 1, dtype=torch.int32, device="cuda:0")
    lse = torch.empty((B, H, 1), device="cuda:0")
    out = pk.pskv_attn_fwd(q, k1, v1, kp, vp, one, lse=lse)
    dq, _, _ = pk.pskv_attn_bwd(q, k1, v1, kp, vp, one, out, lse, dout)
    # the same 33 keys as a candidate's own; the row is its last
    def last(x):
        return torch.cat([x.new_zeros((B, 32) + x.shape[2:]), x], 1).contiguous()
    def own(x, pre):
        return torch.cat([pre[None].expand(B, 32, 1, D), x], 1).contiguous()
    lse_own = torch.cat([torch.zeros((B, H, 32), device="cuda:0"), lse], 2).contiguous()
    none = torch.empty((0, 1, D), dtype=torch.bfloat16, device="cuda:0")
    dq_own, _, _ = pk.pskv_attn_bwd(last(q), own(k1, kp), own(v1, vp), none, none, one + 32, last(out), lse_own, last(dout))
    torch.cuda.synchronize()
    assert torch.equal(dq_own[:, 32:], dq)
