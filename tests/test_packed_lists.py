"""The lists of packed rows, on the host: the functions that the kernels call, compiled for the CPU, against a plain
enumeration of the rows."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
BLOCK = 32


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("lists") / "lists.so")
    res = subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-x", "hip",
                          f"-I{ROOT}/paper_2603_13420_amd/csrc", "-o", out, f"{ROOT}/tests/packed_lists/lists.hip"],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-4000:]
    return ctypes.CDLL(out)


def packed(lib, lens, S, Hq, Hkv, most, P, waves):
    """(window steps, rows, alignment, whether candidates are found by division) of the list of these lengths."""
    out = [ctypes.c_int() for _ in range(3)]
    arr = (ctypes.c_int * len(lens))(*lens)
    steps = lib.packed_list(len(lens), S, Hq, Hkv, arr, most, (P + 31) // 32, waves, *map(ctypes.byref, out))
    return (steps, *(x.value for x in out))


def rows_of(lens, G, align):
    """(candidate, its first row) of every row of the list."""
    rows, first = [], 0
    for b, n in enumerate(lens):
        run = (n * G + align - 1) // align * align
        rows += [(b, first)] * run
        first += run
    return rows


def lengths(rng, kind, B, S):
    if kind == "two":       # two lengths, as a batch of two templates has
        a, b = rng.integers(0, S + 1, 2)
        return np.where(rng.random(B) < rng.random(), a, b)
    if kind == "full":
        return np.full(B, S)
    lens = rng.integers(rng.integers(0, S + 1), S + 1, B)
    return np.where(rng.random(B) < 0.5, 0, lens) if kind == "holes" else lens


@pytest.mark.parametrize("lens,S,Hq,Hkv,P", [
    ([38, 30, 30, 30], 40, 4, 4, 257),       # runs of 64, 32, 32, 32 rows: as many as 4 x 40
    ([40, 32, 32, 32], 40, 4, 4, 300),
    ([32, 32, 48, 48], 48, 2, 2, 260),
    ([40, 32], 40, 4, 2, 320),
    ([59, 59, 41, 59, 55, 57, 60, 48], 60, 4, 2, 300),
])
def test_mixed_lengths_that_add_up_like_full_ones(lib, lens, S, Hq, Hkv, P):
    G, most = Hq // Hkv, 3
    _, total, align, division = packed(lib, lens, S, Hq, Hkv, most, P, 0)
    rows = rows_of(lens, G, align)
    assert total == len(rows)
    assert not division or all(rows[r] == (r // (S * G), r // (S * G) * S * G) for r in range(total))


@pytest.mark.parametrize("kind", ["uniform", "two", "full", "holes"])
@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (4, 2), (3, 1), (8, 2), (5, 1), (7, 1), (8, 1), (40, 1)])
def test_candidates_found_by_division(lib, kind, Hq, Hkv):
    rng = np.random.default_rng(Hq * 10 + Hkv)
    G, found, b, first = Hq // Hkv, 0, ctypes.c_int(), ctypes.c_int()
    for _ in range(150):
        B, S, P = int(rng.integers(1, 40)), int(rng.integers(1, 65)), int(rng.integers(65, 1100))
        lens = [int(x) for x in lengths(rng, kind, B, S)]
        for most, waves in ((3, 0), (2, 8)):
            _, total, align, division = packed(lib, lens, S, Hq, Hkv, most, P, waves)
            rows = rows_of(lens, G, align)
            assert total == len(rows)
            if division:
                found += 1
                for r0 in range(0, total, BLOCK):
                    lib.packed_place(B, S, Hq, Hkv, r0, ctypes.byref(b), ctypes.byref(first))
                    assert (b.value, first.value) == rows[r0], (lens, S, G, P, align, r0)
    assert found or kind != "full"
