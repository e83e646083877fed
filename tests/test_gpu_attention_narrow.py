"""Attention with 24-bit requantisations (sub-word instructions, 16-bit table entries, quotients written byte by byte), at the edges
of its key tiles and of its parameters, against the oracle: equality."""
import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import synth

pytestmark = pytest.mark.gpu


def _run(ivit, B, T, H, d_head, sm, qk, pv=(20011, 22), bias=False, mask=None, sigma=32.0, rounding="nearest", table=False, one_key=False):
    import torch
    rng = np.random.default_rng(T + 1000 * H + d_head + sm["i0"])
    C = H * d_head
    qkv = np.clip(np.rint(rng.normal(0, sigma, size=(B * T, 3 * C))), -128, 127).astype(np.int8)
    qkv[0] = -128
    if one_key:                                                  # key 2 of every image collects everything
        qkv[:, :C] = 100
        qkv[2::T, C:2 * C] = 127
    rb = rng.integers(-128, 128, size=(H, T, T)).astype(np.int8) if bias else None
    m = None
    if mask is not None:
        m = np.zeros((2, T, T), np.int8)
        m[rng.random(m.shape) < 0.4] = 1
        m[rng.random(m.shape) < 0.1] = -128
        if mask == "whole rows":
            m[:, ::3] = 1
    d = dict(B=B, T=T, C=C, H=H, F=C)
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    index = np.arange(T, dtype=np.int32)[None, ::-1].copy() if table else None
    o = torch.empty((B * T, C), dtype=torch.int8, device="cuda")
    ivit.ivit_window_attention(dev(qkv), o, d, qk, sm, pv, dev(rb), dev(index), mask=dev(m), rounding=rounding)
    if table:
        qkv = qkv.reshape(B, T, -1)[:, ::-1].reshape(B * T, -1)
    want = orc.attention(qkv, d, qk, sm, pv, rb, mask=m, floor_shift=rounding == "floor")
    want = want[0] if isinstance(want, tuple) else want
    if table:
        want = want.reshape(B, T, -1)[:, ::-1].reshape(B * T, -1)
    got = o.cpu().numpy()
    assert np.array_equal(got, want), "%d of %d differ" % ((got != want).sum(), got.size)


@pytest.mark.parametrize("T", [1, 2, 15, 16, 17, 48, 49, 63, 64, 65, 127, 128, 129, 197, 207, 208, 209, 255, 256])
@pytest.mark.parametrize("d_head", [32, 64])
@pytest.mark.parametrize("extra", ["none", "bias", "mask", "bias and mask"])
def test_tokens(ivit, T, d_head, extra):
    _run(ivit, 2, T, 2, d_head, synth.shift_params(32), (20011, 24 if d_head == 64 else 23), bias="bias" in extra,
         mask="some" if "mask" in extra else None, table="bias" in extra and T % 2 == 1)


# I_0 and N: ShiftExp(0) a power of two or not, at the smallest that takes this path (2^15 for k_out = 8) and below it; scores
# spread so that rows have one key, a few or all of them
@pytest.mark.parametrize("i0,n", [(1, 15), (4, 13), (5, 13), (16, 11), (32, 10), (32, 9), (63, 9), (64, 9), (127, 9), (7, 3)])
@pytest.mark.parametrize("c", [16, 20, 24])
@pytest.mark.parametrize("one_key", [False, True])
def test_exponent_parameters(ivit, i0, n, c, one_key):
    for k_out in (8, 4):
        sm = dict(i0=i0, n_shift=n, m_bits=24 + k_out - 1, k_out=k_out)
        _run(ivit, 1, 65, 1, 64, sm, (20011, c), one_key=one_key)
        _run(ivit, 2, 49, 1, 32, sm, (20011, c), bias=True, one_key=one_key, rounding="floor")


# more than 208 tokens and 64 features take the 24-bit requantisations with the 32-bit IntDiv where there is a mask
@pytest.mark.parametrize("i0,n", [(32, 10), (32, 9), (7, 3)])
@pytest.mark.parametrize("k_out", [8, 4])
@pytest.mark.parametrize("extra", ["bias", "mask", "bias and mask"])
def test_exponent_parameters_of_long_rows(ivit, i0, n, k_out, extra):
    sm = dict(i0=i0, n_shift=n, m_bits=24 + k_out - 1, k_out=k_out)
    for d_head, T in ((64, 250), (32, 250), (64, 200)):
        _run(ivit, 1, T, 1, d_head, sm, (20011, 24), bias="bias" in extra, mask="some" if "mask" in extra else None)


@pytest.mark.parametrize("i0", [1, 6, 7, 15, 16, 64])
@pytest.mark.parametrize("T", [49, 65])
def test_rows_with_every_key_masked(ivit, i0, T):
    _run(ivit, 2, T, 1, 32, synth.shift_params(i0), (20011, 23), bias=i0 % 2 == 0, mask="whole rows")


# bounds of the limits: b just inside the 24-bit form, multipliers whose limits are near 2^23
@pytest.mark.parametrize("qk", [(2 ** 14 - 1, 15), (2 ** 23 - 1, 24), (300, 24), (255, 24), (1, 2)])
@pytest.mark.parametrize("rounding", ["nearest", "floor"])
def test_multipliers(ivit, qk, rounding):
    _run(ivit, 1, 197, 2, 64, synth.shift_params(32), qk, pv=qk, sigma=60.0, rounding=rounding)
    _run(ivit, 1, 49, 2, 32, synth.shift_params(32), qk, pv=qk, bias=True, sigma=60.0, rounding=rounding)


# ShiftExp(0) over the range whose tables are scaled: ends of every octave, the smallest of each k_out (2^(k_out-1) + 1), odd values
@pytest.mark.parametrize("e0", [129, 255, 256, 257, 511, 512, 513, 1023, 1024, 4095, 4096, 9999, 16383, 16384, 32767, 32768, 65535])
@pytest.mark.parametrize("one_key", [False, True])
def test_exponent_scales(ivit, e0, one_key):
    sm = dict(i0=e0, n_shift=0, m_bits=31, k_out=8)
    while sm["i0"] > 40 and sm["i0"] % 2 == 0:
        sm = dict(sm, i0=sm["i0"] // 2, n_shift=sm["n_shift"] + 1)
    _run(ivit, 1, 197, 1, 64, sm, (20011, 24), one_key=one_key)
    _run(ivit, 2, 49, 1, 32, sm, (20011, 23), bias=True, mask="some", one_key=one_key)
    _run(ivit, 1, 145, 1, 32, sm, (20011, 22), bias=True, one_key=one_key)


@pytest.mark.parametrize("k_out", range(2, 8))
@pytest.mark.parametrize("one_key", [False, True])
def test_fewer_bits_of_probability(ivit, k_out, one_key):
    for i0, n in ((2 ** (k_out - 1) + 1, 0), (5, k_out), (33, 10)):
        _run(ivit, 1, 65, 1, 64, dict(i0=i0, n_shift=n, m_bits=23 + k_out, k_out=k_out), (20011, 24), one_key=one_key)
