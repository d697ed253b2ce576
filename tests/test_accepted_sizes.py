"""What sizes are accepted does not depend on whether the vector or the matrix-core kernels take a problem
(fp32 tensors, bf16 heads of 64 columns): the vector kernels' limits on either side of their edges."""
import ctypes

import pytest

from paper_2603_13420_amd import binding as pk

KINDS = [("f32", 64), ("f32", 128), ("bf16", 64)]


def params(**kw):
    return pk.make_params(**{**dict(B=2, S=16, P=48, Hq=4, Hkv=4), **kw})


@pytest.mark.parametrize("dtype,D", KINDS)
def test_forward_limit(dtype, D):
    most = 64 * 1024 // (8 if dtype == "f32" else 4) - D - 16      # prefix rows beside D and S values in 64 KB
    for P, status in ((most, pk.PSKV_OK), (most + 1, pk.PSKV_ERR_UNSUPPORTED)):
        for impl in ("auto", "simple"):
            assert pk.pskv_attn_validate(params(P=P, D=D, dtype=dtype, impl=impl)) == status


@pytest.mark.parametrize("dtype,D", KINDS)
def test_backward_limits(dtype, D):
    size = 8 if dtype == "f32" else 4
    row = 64 * 1024 // size - 2 * D - 16                            # P + S + 2 D values: the dq kernel's
    group = (64 * 1024 // size - 2 * D) // 2 // 8                   # 2 (D + G S) values: the dk/dv kernel's, G = 8
    null = [None] * 12
    for kw, refused in ((dict(P=row), False), (dict(P=row + 1), True), (dict(S=group, Hq=8, Hkv=1), False),
                        (dict(S=group + 1, Hq=8, Hkv=1), True)):
        for impl in ("auto", "simple"):
            p = params(**{**dict(D=D, dtype=dtype, impl=impl), **kw})
            rc = pk.load().pskv_attn_bwd(ctypes.byref(p), *null, None, 0, None)
            # (sizes that are accepted get as far as the missing pointers)
            assert rc == (pk.PSKV_ERR_UNSUPPORTED if refused else pk.PSKV_ERR_INVALID_ARG), (kw, impl, pk.pskv_last_error())
