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
    """(window steps, rows, alignment, whether every run is a full candidate's) of the list of these lengths."""
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
    G = Hq // Hkv
    _, total, align, even = packed(lib, lens, S, Hq, Hkv, 3, P, 0)
    assert (total, align, even) == (len(lens) * S * G, BLOCK, 0)
    assert total == len(rows_of(lens, G, align))


@pytest.mark.parametrize("kind", ["uniform", "two", "full", "holes"])
@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (4, 2), (3, 1), (8, 2), (5, 1), (7, 1), (8, 1), (40, 1)])
def test_candidates_found_by_division(lib, kind, Hq, Hkv):
    rng = np.random.default_rng(Hq * 10 + Hkv)
    G, found, b, first = Hq // Hkv, 0, ctypes.c_int(), ctypes.c_int()
    for _ in range(150):
        B, S, P = int(rng.integers(1, 40)), int(rng.integers(1, 65)), int(rng.integers(65, 1100))
        lens = [int(x) for x in lengths(rng, kind, B, S)]
        for most, waves in ((3, 0), (2, 8)):
            _, total, align, even = packed(lib, lens, S, Hq, Hkv, most, P, waves)
            rows = rows_of(lens, G, align)
            assert total == len(rows)
            if even:
                found += 1
                for r0 in range(0, total, BLOCK):
                    lib.packed_place(B, S, Hq, Hkv, align, r0, ctypes.byref(b), ctypes.byref(first))
                    assert (b.value, first.value) == rows[r0], (lens, S, G, P, align, r0)
    assert found or kind != "full"


def walk_all(lib, lens, S, Hq, Hkv, total, align, span):
    """(first row, last row, wide, window as (candidate, position)) of every block, one after the other."""
    B = len(lens)
    arr, walk, out, window = (ctypes.c_int * B)(*lens), (ctypes.c_int * 3)(0, 0, lens[0]), (ctypes.c_int * 5)(), (ctypes.c_uint * 96)()
    r0 = 0
    while r0 < total:
        lib.packed_walk(B, S, Hq, Hkv, arr, r0, total, align, span, walk, out, window)
        b, _, last, width, wide = out
        assert r0 <= last < r0 + BLOCK and width >= 1
        yield r0, last, bool(wide), width, [(b + (e >> 6), e & 63) for e in window], out[1]
        r0 = last + 1 if wide else r0 + BLOCK


@pytest.mark.parametrize("span", [2, 3, 128, 1 << 20])
@pytest.mark.parametrize("kind", ["uniform", "two", "holes", "apart"])
@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (4, 2), (3, 1), (8, 2), (7, 1), (8, 1), (40, 1)])
def test_blocks_and_windows(lib, kind, Hq, Hkv, span):
    rng = np.random.default_rng(Hq * 10 + Hkv + span)
    G, early = Hq // Hkv, 0
    for _ in range(8):
        B, S = int(rng.integers(1, 60)), int(rng.integers(1, 65))
        lens = [int(x) for x in lengths(rng, "uniform" if kind == "apart" else kind, B, S)]
        if kind == "apart":     # long runs of empty candidates
            lens = [x for n in lens for x in (n, *[0] * int(rng.integers(0, 200)))]
        own = [(b, i) for b, n in enumerate(lens) for i in range(n)]     # the list's positions
        start = np.concatenate([[0], np.cumsum(lens)])
        for align in (1, BLOCK):
            rows, seen = rows_of(lens, G, align), []
            for r0, last, wide, width, window, first in walk_all(lib, lens, S, Hq, Hkv, len(rows), align, span):
                b = rows[r0][0]
                assert first == rows[r0][1]
                seen += range(r0, last + 1)
                early += wide
                assert wide or last == min(r0 + BLOCK, len(rows)) - 1
                # positions from the first candidate's first to the last row's own (the last valid one's, where the row is padding)
                c, f = rows[last]
                end = start[c] + min((last - f) // G + 1, lens[c])
                assert width == end - start[b]
                shown = own[start[b]:end]
                assert window == (shown + [shown[-1]] * 96)[:96]
                assert window[0][0] == b and all(x - b < span or not wide for x, _ in shown)
            assert seen == list(range(len(rows)))
    assert early or span > 128 or kind != "apart"


def test_walk_ends_at_the_last_candidate(lib):
    """Lengths that are not those the list was added up from: every candidate and position exists all the same."""
    rng = np.random.default_rng(5)
    for _ in range(300):
        B, S, Hq = int(rng.integers(1, 40)), int(rng.integers(1, 65)), int(rng.integers(1, 9))
        now = [int(x) for x in rng.integers(0, S + 1, B)]
        for align in (1, BLOCK):
            total = len(rows_of([int(x) for x in rng.integers(0, S + 1, B)], Hq, align))
            for *_, window, _ in walk_all(lib, now, S, Hq, 1, total, align, 1 << 20):
                assert all(0 <= b < B and 0 <= i < S for b, i in window)
