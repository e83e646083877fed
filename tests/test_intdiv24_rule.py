"""Which Shiftmax parameters take the 24-bit IntDiv of the attention kernel, and that it is IntDiv there: the rule (host code, compiled
here) and the arithmetic that stands on it, on the CPU."""
import ctypes
import subprocess

import numpy as np
import pytest

from paper_2207_01405_amd import build


@pytest.fixture(scope="module")
def up_of(tmp_path_factory):
    d = tmp_path_factory.mktemp("intdiv")
    (d / "r.cpp").write_text('#include "attention_form.hpp"\nextern "C" int up(int64_t i, int n, int m, int k) { return ivit::intdiv24_up(i, n, m, k); }\n')
    subprocess.run(["g++", "-std=c++20", "-shared", "-fPIC", "-I", build.CSRC, str(d / "r.cpp"), "-o", str(d / "r.so")], check=True)
    f = ctypes.CDLL(str(d / "r.so")).up
    f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return f


def test_what_the_rule_takes(up_of):
    """Everything whose reciprocal has 24 bits: as before table entries were scaled, I_0 << N = 2^15 and more without a scale."""
    for i0, n in ((32, 10), (32, 9), (63, 9), (32, 3), (1, 8), (1, 15), (65535, 0)):
        assert up_of(i0, n, 31, 8) >= 0, (i0, n)
    assert up_of(1, 15, 31, 8) == up_of(65535, 0, 31, 8) == 0 and up_of(32, 9, 31, 8) == 1
    for i0, n, m, k in ((32, 2, 31, 8), (1, 7, 31, 8), (32, 10, 30, 8), (32, 10, 31, 7), (65536, 0, 31, 8)):
        assert up_of(i0, n, m, k) == -1, (i0, n, m, k)


@pytest.mark.parametrize("k_out", range(2, 9))
def test_the_product_is_intdiv(up_of, k_out):
    M, top = 23 + k_out, 2 ** (k_out - 1)
    rng = np.random.default_rng(k_out)
    e0s = {2 ** j + d for j in range(1, 17) for d in (-1, 0, 1)} | set(rng.integers(2, 65536, size=60).tolist())
    for e0 in sorted(v for v in e0s if top < v <= 65535):
        up = up_of(e0, 0, M, k_out)
        assert 0 <= up <= 8 and e0 << up <= 65535
        sums = np.unique(np.concatenate([np.arange(e0, e0 + 50), rng.integers(e0, 256 * e0 + 1, size=200), [2 * e0 - 1, 2 * e0, 256 * e0]]))
        e = np.unique(np.concatenate([np.arange(0, min(e0, 40) + 1), rng.integers(0, e0 + 1, size=60), [e0 - 1, e0]]))
        s, v = (a.astype(np.uint64) for a in np.meshgrid(sums, e))
        alone = s == e0                                          # one key has the whole sum: the others' entries are 0
        keep = ~alone | (v == 0) | (v == e0)
        s, v, alone = s[keep], v[keep], alone[keep]
        inv = np.uint64(2 ** M) // s
        f = (inv - alone) << np.uint64(8 - up)
        assert f.max() < 2 ** 24
        got = (f * (v << np.uint64(up))) >> np.uint64(32)
        assert np.array_equal(got, np.minimum((inv * v) >> np.uint64(24), np.uint64(top - 1))), e0


@pytest.mark.parametrize("k_out", range(2, 9))
@pytest.mark.parametrize("ulp", [-1, 0, 1])
def test_the_reciprocal_of_a_row(up_of, k_out, ulp):
    """floor(2^M / sum) from single precision as div_factor forms it, with a hardware reciprocal one unit off either way."""
    M, f32, f64 = 23 + k_out, np.float32, np.float64
    rng = np.random.default_rng(k_out)
    for e0 in sorted({2 ** (k_out - 1) + 1, 2 ** k_out, 2 ** k_out + 1, 300, 511, 512, 4095, 32767, 32768, 65535}):
        if e0 <= 2 ** (k_out - 1):
            continue
        up = up_of(e0, 0, M, k_out)
        sums = np.unique(np.concatenate([np.arange(e0, min(256 * e0, e0 + 70000) + 1), rng.integers(e0, 256 * e0 + 1, size=30000), [256 * e0]]))
        scaled = sums.astype(np.int64) << up
        s, num = scaled.astype(f32), f32(2.0 ** (M + up))
        r = (f32(1) / s).astype(f32)
        if ulp:
            r = np.nextafter(r, f32(ulp) * f32(np.inf))
        q = (num * r).astype(f32)
        fma = lambda a, b, c: (a.astype(f64) * b.astype(f64) + np.asarray(c, f64)).astype(f32)     # (48-bit products: exact but for the last rounding)
        inv = fma(fma(-q, s, num), r, q).astype(np.int64)
        rem = ((2 ** (M + up) - inv * scaled + 2 ** 31) % 2 ** 32) - 2 ** 31
        assert np.array_equal(inv + (rem >= scaled) - (rem < 0), 2 ** M // sums)
