"""The lane tier's bit-plane arithmetic on the CPU: one extension at a time
against the oracle, over every shape the tier accepts (band within the
window): X at both ends of each plane count, walls, empty sides, homopolymers
and tandem repeats, unrelated sequences, both walking directions, the
complemented strand, reads that start and end at every chunk offset."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
from helpers import mutate_codes, rand_codes

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIMIT = {5: 14, 6: 30, 7: 62}  # largest X of each plane count


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("lane") / "liblane.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wno-unknown-pragmas",
                           "-I" + os.path.join(ROOT, "paper_2001_10049_amd", "csrc"),
                           "-o", so, os.path.join(ROOT, "tests", "lane_shim.cpp")])
    return ctypes.CDLL(so)


def run(lib, planes, a, b, X, back_a=False, back_b=False, comp=False, pad=(0, 0), chain=False):
    """Lane result of extending a against b, stored in reads as the flags say
    (backwards, complemented), `pad` foreign bases before and after.  chain:
    what outgrows the window goes on in the 96-row one; whether it did comes
    last."""
    rng = np.random.default_rng(1)

    def store(s, back, comp):
        s = s[::-1] if back else s
        s = (3 - s) if comp else s
        r = np.concatenate([rand_codes(rng, pad[0]), s, rand_codes(rng, pad[1])])
        return np.ascontiguousarray(r, np.uint8), pad[0] + (len(s) - 1 if back else 0)
    A, oa = store(a, back_a, False)
    B, ob = store(b, back_b, comp)
    out = (ctypes.c_int64 * 6)()
    flags = (1 if back_a else 0) | (2 if back_b else 0) | (4 if comp else 0)
    p = lambda v: v.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    ok = lib.lane_extend(planes, int(chain), p(A), len(A), p(B), len(B), oa, ob, len(a), len(b), X, flags, out)
    if ok == 0:
        return None
    return tuple(out[:4]) + ((out[5],) if chain else ())


def want(a, b, X):
    return tuple(int(v) for v in oracle.extend(a, b, X)[:4])


def sequences(rng, kind):
    n = int(rng.integers(0, 700))
    a = rand_codes(rng, n)
    if kind == "overlap":
        b = mutate_codes(rng, a, float(rng.choice([0.0, 0.05, 0.15, 0.3])))
        b = np.concatenate([b, rand_codes(rng, int(rng.integers(0, 60)))])
    elif kind == "tail":  # an overlap that ends inside both
        k = int(rng.integers(0, n + 1))
        b = np.concatenate([mutate_codes(rng, a[:k], 0.15), rand_codes(rng, n - k)])
    elif kind == "random":
        b = rand_codes(rng, int(rng.integers(0, 700)))
    elif kind == "homopolymer":
        a = np.zeros(n, np.uint8)
        b = np.zeros(int(rng.integers(0, 300)), np.uint8)
    else:  # tandem repeats: many ties
        u = rand_codes(rng, int(rng.integers(1, 4)))
        a = np.resize(u, n)
        b = mutate_codes(rng, np.resize(u, n), 0.1)
    return a.astype(np.uint8), b.astype(np.uint8)


@pytest.mark.parametrize("planes", [5, 6, 7])
@pytest.mark.parametrize("kind", ["overlap", "tail", "random", "homopolymer", "repeat"])
def test_against_oracle(lib, planes, kind):
    rng = np.random.default_rng(planes * 100 + len(kind))
    done = 0
    for _ in range(250):
        a, b = sequences(rng, kind)
        lim = LIMIT[planes]
        X = int(rng.choice([0, 1, 2, 7, lim // 2, lim - 1, lim]))
        back_a, back_b, comp = (bool(v) for v in rng.integers(0, 2, 3))
        pad = tuple(int(v) for v in rng.integers(0, 200, 2))
        got = run(lib, planes, a, b, X, back_a, back_b, comp, pad)
        if got is None:
            continue
        done += 1
        assert got == want(a, b, X), (planes, kind, len(a), len(b), X, back_a, back_b, comp, pad)
    assert done >= (20 if kind in ("homopolymer", "repeat", "random") else 100), done


def test_long_overlap(lib):
    """Many refills and window moves: 30 kbp at 15 % errors."""
    rng = np.random.default_rng(5)
    a = rand_codes(rng, 30_000)
    b = mutate_codes(rng, a, 0.15)
    for planes, X in ((5, 7), (6, 25), (7, 50)):
        assert run(lib, planes, a, b, X, pad=(13, 7)) == want(a, b, X)


@pytest.mark.parametrize("planes", [5, 6, 7])
def test_every_small_shape(lib, planes):
    """Every pair of lengths up to 4, and each wall near a word's edge."""
    rng = np.random.default_rng(3)
    shapes = [(m, n) for m in range(5) for n in range(5)]
    shapes += [(m, n) for m in (30, 31, 32, 33, 63, 64, 65, 96) for n in (0, 1, 31, 32, 33, 64, 97)]
    for m, n in shapes:
        a = rand_codes(rng, m)
        b = np.resize(a, n).astype(np.uint8) if m else rand_codes(rng, n)
        for X in (0, 3, LIMIT[planes]):
            got = run(lib, planes, a, b, X, pad=(int(rng.integers(0, 70)), 0))
            if got is not None:
                assert got == want(a, b, X), (planes, m, n, X)


@pytest.mark.parametrize("planes", [5, 6])
def test_wider_window_resumes(lib, planes):
    """A band that outgrows 32 or 64 rows goes on in 96 from the state it left."""
    rng = np.random.default_rng(planes)
    moved = 0
    for _ in range(1200):
        n = int(rng.integers(100, 900))
        a = np.resize(rand_codes(rng, int(rng.integers(1, 5))), n)
        a = mutate_codes(rng, a, 0.1)
        b = mutate_codes(rng, a, 0.2) if rng.integers(2) else mutate_codes(rng, np.roll(a, 7), 0.1)
        X = int(rng.integers(LIMIT[planes] // 2, LIMIT[planes] + 1))
        got = run(lib, planes, a, b, X, back_a=bool(rng.integers(2)), chain=True)
        if got is None or not got[4]:
            continue
        moved += 1
        assert got[:4] == want(a, b, X), (planes, n, len(b), X)
    assert moved >= 20, moved
