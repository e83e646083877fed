"""The pair a residual layer's kernels use for the residual term, against the one the caller gave (host code, compiled here): the
same term for every residual value, and the 24-bit form's conditions wherever it differs."""
import ctypes
import subprocess

import numpy as np
import pytest

from paper_2207_01405_amd import build


@pytest.fixture(scope="module")
def pair_of(tmp_path_factory):
    d = tmp_path_factory.mktemp("pair")
    (d / "p.cpp").write_text('#include "residual_pair.hpp"\nextern "C" int64_t pair(int b, int c, int r) { auto p = ivit::residual_pair(b, c, r); return ((int64_t)p.c << 32) | p.b; }\n')
    subprocess.run(["g++", "-std=c++20", "-shared", "-fPIC", "-I", build.CSRC, str(d / "p.cpp"), "-o", str(d / "p.so")], check=True)
    f = ctypes.CDLL(str(d / "p.so")).pair
    f.restype, f.argtypes = ctypes.c_int64, [ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return lambda b, c, rnd: (f(b, c, rnd) & 0xffffffff, f(b, c, rnd) >> 32)


def _term(b, c, rnd):
    return [(v * b + (rnd << (c - 1))) >> c for v in range(-128, 128)]


@pytest.mark.parametrize("rnd", [0, 1])
def test_same_terms(pair_of, rnd):
    rng = np.random.default_rng(rnd)
    pairs = [(b, c) for c in range(1, 47) for b in (1, 2, 3, 20011, 2 ** 23 - 1, 2 ** 23, 2 ** 23 + 1, 2 ** 24 - 1, 2 ** 30, 2 ** 31 - 1) + tuple(2 ** k for k in range(c - 2, c + 1) if 0 <= k < 31)]
    pairs += list(zip(np.exp(rng.uniform(0, np.log(2 ** 31 - 1), 20000)).astype(int).tolist(), rng.integers(1, 47, 20000).tolist()))
    found = asked = 0
    for b, c in pairs:
        got = pair_of(b, c, rnd)
        if b < 2 ** 23 and c <= 30:
            assert got == (b, c)
            continue
        assert _term(*got, rnd) == _term(b, c, rnd), (b, c, got)
        if got != (b, c):
            assert 1 <= got[0] < 2 ** 23 and 1 <= got[1] <= 30 and got[1] < c
        if c <= 31 and 2 ** (c - 8) <= b <= 2 ** c:
            asked, found = asked + 1, found + (got != (b, c))
    assert asked > 300 and found > 0.97 * asked                  # (a term within 2^-16 of a step for one value in 2^9 pairs)
