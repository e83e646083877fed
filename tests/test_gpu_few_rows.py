"""The Dense kernel for few rows (gemm_kq.hip) at the edges of its tiles, of its split of K and of its range, against the oracle;
the same shapes with an I-LayerNorm in front run inside blocks.  Whole numbers, compared for equality."""
import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import synth

pytestmark = pytest.mark.gpu


def _dense(ivit, M, N, K, epilogue, rounding, wide=False, seed=0):
    import torch
    rng = np.random.default_rng(seed + M + 7 * N + 13 * K)
    x, w, res = (rng.integers(-128, 128, size=s).astype(np.int8) for s in ((M, K), (N, K), (M, N)))
    b = rng.integers(2 ** 14, 2 ** 15, size=N).astype(np.int32)
    c = np.full(N, 24, np.int32)
    if wide:                                                     # channels beyond the 32-bit form
        b[N // 2:] <<= 8
        c[N // 2:] += 8
    bias = rng.integers(-2 ** 20, 2 ** 20, size=N).astype(np.int32)
    kw, okw = {}, {}
    if epilogue == "residual":
        kw = okw = dict(res_rq=(20011, 15))
    elif epilogue == "gelu":
        kw = okw = dict(gelu=synth.shift_params(32), gelu_rq=(20011, 20))
    dev = lambda a: torch.from_numpy(a).cuda()
    y = torch.empty((M, N), dtype=torch.int8, device="cuda")
    more = dict(residual=dev(res)) if epilogue == "residual" else {}
    ivit.ivit_linear_requant(dev(x), dev(w), dev(bias) if seed == 0 else None, dev(b), dev(c), y, rounding=rounding, **kw, **more)
    omore = dict(residual=res) if epilogue == "residual" else {}
    want = orc.linear_requant(x, w, bias if seed == 0 else None, b, c, floor_shift=rounding == "floor", **okw, **omore)
    got = y.cpu().numpy()
    assert np.array_equal(got, want), "%d of %d differ" % ((got != want).sum(), got.size)


# K: one to 24 k-steps of 32 bytes in every remainder of four and with a half step at the end, then two, three and more parts
@pytest.mark.parametrize("K", [16, 32, 48, 112, 128, 144, 192, 272, 384, 400, 512, 640, 752, 768, 784, 1536, 1552, 2304, 3072, 3088, 4112])
@pytest.mark.parametrize("epilogue", ["plain", "residual", "gelu"])
def test_split_of_k(ivit, K, epilogue):
    _dense(ivit, 37, 72, K, epilogue, "floor" if K % 64 == 16 else "nearest", wide=K == 400)


# edges of the 32 x 32 tiles, odd widths, and both sides of the range (256 CUs: 512 tiles, 256 beyond K = 768)
@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (1, 1000, 384), (31, 33, 96), (32, 32, 192), (33, 30, 384), (65, 62, 64), (197, 1151, 192), (512, 1024, 48),
                                   (513, 1024, 48), (512, 512, 800), (512, 513, 800), (3000, 5, 80)])
@pytest.mark.parametrize("epilogue", ["plain", "residual", "gelu"])
def test_tiles(ivit, M, N, K, epilogue):
    _dense(ivit, M, N, K, epilogue, "nearest", seed=M % 2)


@pytest.mark.parametrize("C,H,F", [(32, 1, 64), (96, 3, 144), (64, 2, 256), (192, 3, 768), (384, 6, 1536), (640, 10, 2000), (768, 12, 3072), (800, 25, 160)])
@pytest.mark.parametrize("B,T", [(1, 1), (1, 33), (3, 65)])
def test_block_with_layernorm(ivit, C, H, F, B, T):
    import torch
    cfg = dict(T=T, C=C, H=H, F=F, seed=C + T, i0="fixed", rel_bias=False)
    p = synth.make_block(cfg, 0)
    d = dict(B=B, T=T, C=C, H=H, F=F)
    x = synth.make_rows(C + T, B * T, C)
    x[0] = 77                                                     # a constant row: variance 0
    xd = torch.from_numpy(x).cuda()
    y = torch.empty_like(xd)
    ws = torch.empty(ivit.ivit_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    ivit.ivit_encoder_block(xd, y, ivit.to_device(p), d, ws)
    want, _ = orc.encoder_block(x, p, d, want_taps=True)
    got = y.cpu().numpy()
    assert np.array_equal(got, want), "%d of %d differ" % ((got != want).sum(), got.size)
