"""7 x 7 windows in numbers that give every wavefront whole windows, against the same windows in parts too small for that form and,
some of them, against the oracle: odd and even heads, windows that leave the last pass partly empty, tables with entries
outside the image, masks with and without a bias, rows with everything masked, one key that has the whole sum.  Equality."""
import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import synth

pytestmark = pytest.mark.gpu
T = 49


@pytest.mark.parametrize("H", [1, 2, 3, 6, 9, 32])
@pytest.mark.parametrize("more", [0, 5])
@pytest.mark.parametrize("kind", ["bias", "table", "mask", "bias and mask", "table and mask"])
@pytest.mark.parametrize("i0,sigma", [(32, 32.0), (1, 60.0)])
def test_parts_equal_whole(ivit, H, more, kind, i0, sigma):
    import torch
    n_win = 4
    B = -(-9 * torch.cuda.get_device_properties(0).multi_processor_count // (H * n_win)) * n_win + more * n_win
    C, rng = 32 * H, np.random.default_rng(100 * H + more + i0)
    qkv = np.clip(np.rint(rng.normal(0, sigma, size=(B * T, 3 * C))), -128, 127).astype(np.int8)
    qkv[:T, :C] = 100                                            # the first window: key 2 collects everything
    qkv[2, C:2 * C] = 127
    bias = rng.integers(-128, 128, size=(H, T, T)).astype(np.int8) if "bias" in kind or "table" in kind else None
    index = mask = None
    if "table" in kind:
        index = rng.permutation(n_win * T).astype(np.int32).reshape(n_win, T)
        index[1, 48], index[2, 0] = n_win * T + 7, 2 ** 31 - 1   # (limited to the image's last token)
    if "mask" in kind:
        mask = (rng.random((n_win, T, T)) < 0.4).astype(np.int8)
        mask[0] = 0
        mask[1, ::3] = 1
        mask[2] = np.where(np.arange(T) == T - 1, -128, 0)       # the last key alone
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    x, b, ix, m = dev(qkv), dev(bias), dev(index), dev(mask)
    out = [torch.full((B * T, C), 99, dtype=torch.int8, device="cuda") for _ in range(2)]
    for o, part in ((out[0], B), (out[1], max(n_win, B // 8 // n_win * n_win))):
        for at in range(0, B, part):
            n = min(part, B - at)
            ivit.ivit_window_attention(x[at * T:(at + n) * T], o[at * T:(at + n) * T], dict(B=n, T=T, C=C, H=H, F=C), (20011, 23),
                                       synth.shift_params(i0), (20011, 22), b, ix, mask=m, rounding="floor" if more else "nearest")
    # the oracle, window by window: those of the first image and of the last, and some between
    got, last = out[0].cpu().numpy(), n_win * T - 1
    for w in sorted({0, 1, 2, 3, B - 1, B - 2, B - 3, *range(5, B, max(B // 6, 1))}):
        rows = np.arange(w * T, (w + 1) * T) if index is None else w // n_win * n_win * T + np.minimum(index[w % n_win].astype(np.int64), last)
        want = orc.attention(qkv[rows], dict(B=1, T=T, C=C, H=H, F=C), (20011, 23), synth.shift_params(i0), (20011, 22), bias,
                             mask=None if mask is None else mask[w % n_win:w % n_win + 1], floor_shift=bool(more))
        sure = rows % (n_win * T) != last if index is not None else np.ones(T, bool)       # (several tokens of a table write the last row)
        assert np.array_equal(got[rows][sure], want[sure]), "window %d" % w
    if index is not None:                                        # (several tokens write the last row, some rows are written by none)
        rows = [r for r in range(B * T) if r % (n_win * T) not in (n_win * T - 1,)]
        out = [o[rows] for o in out]
    assert torch.equal(out[0], out[1]), "%d of %d differ" % ((out[0] != out[1]).sum(), out[0].numel())
    assert len(torch.unique(out[0])) > 20                        # (not all alike; flat rows average 49 values of spread 32)
