"""The Dense kernel for any shape (gemm_st.hip) at the edges of its tiles, stages and stores, against the oracle.

Shapes: one row and one channel up to a few tiles; K from one 16-byte piece over partial stages to more stages than buffers;
N that is no multiple of 16, 8 or 4 (stores at any alignment, byte stores at the end of a row).  The two larger tiles are
reached through shapes with enough 64 x 64 tiles that no other kernel takes (N % 16 != 0).  Results are whole numbers.
"""
import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import synth

pytestmark = pytest.mark.gpu

SMALL = [(1, 1, 16), (63, 7, 32), (64, 64, 48), (65, 72, 112), (129, 15, 128), (130, 130, 144), (67, 24, 256), (200, 1000, 400),
         (31, 65, 512), (197, 250, 1552), (300, 128, 3072)]
LARGE = [(5000, 601, 144), (2600, 1400, 1040), (13001, 520, 112), (7000, 1017, 528)]


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
    host, kw_o, dev, kw_g = _case(M, N, K, epi, regime)
    got = _run(ivit, dev, kw_g, M, N, rounding=rounding)
    assert np.array_equal(got, orc.linear_requant(*host, floor_shift=(rounding == "floor"), **kw_o))


@pytest.mark.parametrize("M,N,K", LARGE)
@pytest.mark.parametrize("epi", ["plain", "residual", "gelu"])
@pytest.mark.parametrize("regime", ["as drawn", "general"])
def test_larger_tiles(ivit, M, N, K, epi, regime):
    host, kw_o, dev, kw_g = _case(M, N, K, epi, regime)
    got = _run(ivit, dev, kw_g, M, N)
    # the oracle on the first and last tiles and on rows spread over the rest
    rows = np.unique(np.concatenate([np.arange(0, 140), np.arange(M - 140, M), np.arange(0, M, 61)]))
    if epi == "residual":
        kw_o["residual"] = kw_o["residual"][rows]
    assert np.array_equal(got[rows], orc.linear_requant(host[0][rows], *host[1:], **kw_o))


@pytest.mark.parametrize("C,H,F", [(64, 2, 256), (96, 3, 144), (128, 4, 208), (160, 5, 64), (384, 6, 1536), (416, 13, 400), (736, 23, 272), (768, 12, 3072)])
@pytest.mark.parametrize("B,T", [(1, 1), (3, 21), (5, 13), (2, 65)])
def test_layernorm_inside_the_dense_kernel(ivit, C, H, F, B, T):
    """A block whose I-LayerNorms run in the kernels of the QKV and the first MLP layer, against the oracle."""
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
