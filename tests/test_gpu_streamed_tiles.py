"""The Dense kernel for any shape (gemm_st.hip) at the edges of its tiles, stages and stores, against the oracle.

Shapes: one row or one channel up to a few tiles; K from one 16-byte piece over partial stages to more stages than buffers;
N that is no multiple of 16, 8 or 4 (stores at any alignment, byte stores at the end of a row).  The smallest tile is reached with
more 32 x 32 tiles than the kernel for few rows takes (_smallest_tile looks), the two larger ones through shapes with enough
64 x 64 tiles that no other kernel takes (N % 16 != 0).  Results are whole numbers.
"""
import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import synth

pytestmark = pytest.mark.gpu

SMALL = [(16500, 1, 16), (17001, 7, 32), (1, 16500, 48), (63, 9000, 64), (5500, 72, 112), (17000, 15, 128), (4100, 130, 144), (2000, 280, 256),
         (200, 2500, 400), (1030, 513, 512), (67, 2900, 784), (197, 1200, 1552), (300, 900, 3072)]
LARGE = [(5000, 601, 144), (2600, 1400, 1040), (13001, 520, 112), (7000, 1017, 528)]


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def _smallest_tile(M, N, K):
    """More 32 x 32 tiles than gemm_kq.hip takes, few enough 64 x 64 tiles for the smallest tile of this kernel."""
    cus = _cus()
    return -(-M // 32) * -(-N // 32) > cus * (1 if K > 768 else 2) and 2 * (-(-M // 64) * -(-N // 64)) <= 5 * cus


def _rows_of(M, step):
    """Rows the oracle is asked for: the first and last tiles and some between."""
    return np.unique(np.concatenate([np.arange(min(M, 140)), np.arange(max(M - 140, 0), M), np.arange(0, M, step)]))


def _case(M, N, K, epi, regime):
    import torch
    x = synth.make_rows(M + N + K, M, K, "normal", 32.0)
    x[0, :7] = -128
    w, bias, rq_b, rq_c = synth.make_linear(M * 7 + N, N, K)
    w[0, :5] = -128
    if regime == "general":                                  # the same ratios with shifts beyond the 32-bit form, in some channels
        rq_b[::3] <<= 12
        rq_c[::3] += 12
    if regime == "no bias":
        bias = None
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    kw_o, kw_g = {}, {}
    if epi == "residual":
        res = synth.make_rows(N + 1, M, N, "uniform")
        res[-1, ::3] = -128
        kw_o = dict(residual=res, res_rq=(23456, 15)); kw_g = dict(residual=dev(res), res_rq=(23456, 15))
    elif epi == "gelu":
        kw_o = dict(gelu=synth.shift_params(32), gelu_rq=(24171, 21)); kw_g = dict(kw_o)
    return (x, w, bias, rq_b, rq_c), kw_o, tuple(dev(a) for a in (x, w, bias, rq_b, rq_c)), kw_g


def _run(ivit, args, kw, M, N, **more):
    import torch
    room = torch.full((M * N + 64,), 77, dtype=torch.int8, device="cuda")        # results leave the bytes behind them alone
    y = room[:M * N].view(M, N)
    ivit.ivit_linear_requant(*args, y, **kw, **more)
    torch.cuda.synchronize()
    assert bool((room[M * N:] == 77).all())
    return y.cpu().numpy()


@pytest.mark.parametrize("M,N,K", SMALL)
@pytest.mark.parametrize("epi", ["plain", "residual", "gelu"])
@pytest.mark.parametrize("regime,rounding", [("as drawn", "nearest"), ("general", "floor"), ("no bias", "floor")])
def test_edges(ivit, M, N, K, epi, regime, rounding):
    assert _smallest_tile(M, N, K)
    host, kw_o, dev, kw_g = _case(M, N, K, epi, regime)
    got = _run(ivit, dev, kw_g, M, N, rounding=rounding)
    rows = _rows_of(M, 61)
    if epi == "residual":
        kw_o["residual"] = kw_o["residual"][rows]
    assert np.array_equal(got[rows], orc.linear_requant(host[0][rows], *host[1:], floor_shift=(rounding == "floor"), **kw_o))


# sums up to the ends of int32 at pairs up to b = 2^c: with ShiftGELU a result is an index of 0 .. 255
@pytest.mark.parametrize("pair", [(1, 1), (2 ** 19 - 1, 20), (2 ** 19, 20), (2 ** 20, 20), (2 ** 30 - 1, 31), (2 ** 31 - 1, 31), (20011, 40)])
@pytest.mark.parametrize("epi", ["plain", "gelu"])
@pytest.mark.parametrize("rounding", ["nearest", "floor"])
def test_largest_sums(ivit, pair, epi, rounding):
    import torch
    M, N, K = 1030, 520, 144
    assert _smallest_tile(M, N, K)
    rng = np.random.default_rng(pair[1])
    x, w = rng.integers(-128, 128, size=(M, K)).astype(np.int8), rng.integers(0, 3, size=(N, K)).astype(np.int8)
    x[0], x[1] = 127, -128                                   # no negative weight: the extremes of every channel
    total = w.astype(np.int64).sum(axis=1)
    bias = np.where(np.arange(N) % 2, 128 * total - 2 ** 31, 2 ** 31 - 1 - 127 * total).astype(np.int32)
    bias[::3] = rng.integers(-2 ** 12, 2 ** 12, size=len(bias[::3]))
    bias[1::6], bias[4::6] = 0x3fffff00, -0x3fffff00
    b, c = np.full(N, pair[0], np.int32), np.full(N, pair[1], np.int32)
    kw = dict(gelu=synth.shift_params(32), gelu_rq=(24171, 21)) if epi == "gelu" else {}
    got = _run(ivit, tuple(torch.from_numpy(a).cuda() for a in (x, w, bias, b, c)), kw, M, N, rounding=rounding)
    rows = _rows_of(M, 7)
    assert np.array_equal(got[rows], orc.linear_requant(x[rows], w, bias, b, c, floor_shift=rounding == "floor", **kw))


@pytest.mark.parametrize("M,N,K", LARGE)
@pytest.mark.parametrize("epi", ["plain", "residual", "gelu"])
@pytest.mark.parametrize("regime", ["as drawn", "general"])
def test_larger_tiles(ivit, M, N, K, epi, regime):
    host, kw_o, dev, kw_g = _case(M, N, K, epi, regime)
    got = _run(ivit, dev, kw_g, M, N)
    rows = _rows_of(M, 61)
    if epi == "residual":
        kw_o["residual"] = kw_o["residual"][rows]
    assert np.array_equal(got[rows], orc.linear_requant(host[0][rows], *host[1:], **kw_o))


# 256 x 256 tiles: a row or a channel beyond a tile, N at any alignment, last stages of 16 bytes to whole ones, more channels than rows, more
# tiles than CUs.  Every result against the 128 x 128 tiles or the weight slab, which take the shape when asked to.
@pytest.mark.parametrize("M,N,K", [(7937, 1793, 144), (8191, 2047, 272), (8000, 2000, 640), (49999, 200, 400), (24001, 391, 304), (1793, 7937, 160),
                                   (40000, 1001, 336), (12000, 1040, 400), (16000, 1600, 1008)])
@pytest.mark.parametrize("epi", ["plain", "gelu"])
@pytest.mark.parametrize("regime,rounding", [("as drawn", "nearest"), ("general", "floor"), ("no bias", "nearest")])
def test_largest_tiles(ivit, M, N, K, epi, regime, rounding):
    cus = _cus()
    rounds = lambda t, per_cu: -(-(-(-M // t) * -(-N // t)) // (per_cu * cus))
    if cus == 256:
        assert 10 * rounds(256, 1) <= 6 * rounds(128, 2) and -(-M // 64) * -(-N // 64) > 7 * cus
    host, kw_o, dev, kw_g = _case(M, N, K, epi, regime)
    got = _run(ivit, dev, kw_g, M, N, rounding=rounding)
    assert np.array_equal(got, _run(ivit, dev, kw_g, M, N, rounding=rounding, kernel="many_rows"))
    rows = np.unique(np.concatenate([np.arange(0, 256, 5), np.arange(M - 40, M), np.arange(0, M, 251)]))
    assert np.array_equal(got[rows], orc.linear_requant(host[0][rows], *host[1:], floor_shift=rounding == "floor", **kw_o))


# Rows of 768 bytes and more and at most one tile a CU: 64 x 64 (more 32 x 32 tiles than gemm_kq.hip takes), 128 x 64, 128 x 128; last
# stages of 16 to 128 bytes, fewer stages than buffers cannot be
@pytest.mark.parametrize("M,N,K,tile", [(500, 1000, 784, (64, 64)), (449, 1009, 3072, (64, 64)), (1500, 760, 896, (128, 64)), (1665, 701, 1552, (128, 64)),
                                        (129, 7300, 768, (128, 64)), (1500, 2290, 784, (128, 128)), (1409, 2177, 1024, (128, 128))])
@pytest.mark.parametrize("epi", ["plain", "residual", "gelu"])
@pytest.mark.parametrize("regime", ["as drawn", "general"])
def test_one_tile_a_compute_unit(ivit, M, N, K, tile, epi, regime):
    fits = [t for t in ((64, 64), (128, 64), (128, 128)) if -(-M // t[0]) * -(-N // t[1]) <= _cus()]
    if _cus() == 256:
        assert fits[0] == tile and -(-M // 32) * -(-N // 32) > (256 if K > 768 else 512)
    host, kw_o, dev, kw_g = _case(M, N, K, epi, regime)
    got = _run(ivit, dev, kw_g, M, N)
    rows = _rows_of(M, 61)
    if epi == "residual":
        kw_o["residual"] = kw_o["residual"][rows]
    assert np.array_equal(got[rows], orc.linear_requant(host[0][rows], *host[1:], **kw_o))


# 192 x 128 tiles: a row or a channel beyond a tile or just a whole one, last stages of 16 to 128 bytes, shapes that gemm_ks.hip and gemm_tl.hip
# took before
@pytest.mark.parametrize("M,N,K", [(6145, 801, 1040), (4033, 1281, 1552), (12200, 384, 1536), (2304, 2561, 1024), (24300, 129, 1136), (6272, 768, 3072)])
@pytest.mark.parametrize("epi", ["plain", "residual", "gelu"])
@pytest.mark.parametrize("regime", ["as drawn", "general"])
def test_tiles_of_192_rows(ivit, M, N, K, epi, regime):
    if _cus() == 256:
        assert -(-M // 128) * -(-N // 128) > 256 >= -(-M // 192) * -(-N // 128)
    host, kw_o, dev, kw_g = _case(M, N, K, epi, regime)
    got = _run(ivit, dev, kw_g, M, N)
    assert np.array_equal(got, _run(ivit, dev, kw_g, M, N, kernel="many_rows"))
    rows = np.unique(np.concatenate([np.arange(0, 193, 3), np.arange(M - 40, M), np.arange(0, M, 251)]))
    if epi == "residual":
        kw_o["residual"] = kw_o["residual"][rows]
    assert np.array_equal(got[rows], orc.linear_requant(host[0][rows], *host[1:], **kw_o))


# QKV, or QKV and the first MLP layer, past the kernel for few rows; widths of both forms (to 384 and to 768 bytes a row)
@pytest.mark.parametrize("C,H,F,B,T", [(64, 2, 256, 43, 65), (128, 4, 400, 56, 25), (160, 5, 464, 18, 65), (384, 6, 1536, 8, 59), (416, 13, 1232, 7, 65),
                                       (736, 23, 2000, 4, 65), (768, 12, 3072, 2, 130)])
def test_layernorm_inside_the_dense_kernel(ivit, C, H, F, B, T):
    """A block whose I-LayerNorms run in the kernels of the QKV and the first MLP layer, against the oracle."""
    for n in (3 * C, F):
        assert _smallest_tile(B * T, n, C) and -(-B * T // 32) * -(-n // 128) <= 2 * _cus(), n      # (tiles of 32 x 128 there)
    import torch
    d = dict(B=B, T=T, C=C, H=H, F=F)
    p = synth.make_block(dict(T=T, C=C, H=H, F=F, seed=C + F, i0="fixed", rel_bias=False), 0)
    x = synth.make_rows(17 + C, B * T, C)
    x[0] = 5                                                 # a constant row: variance 0
    x[-1, ::2] = -128                                        # the largest variance
    x[-1, 1::2] = 127
    xd, y = torch.from_numpy(x).cuda(), torch.empty((B * T, C), dtype=torch.int8, device="cuda")
    ivit.ivit_encoder_block(xd, y, ivit.to_device(p), d, torch.empty(ivit.ivit_workspace_bytes(d), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), orc.encoder_block(x, p, d))
