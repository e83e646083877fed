"""The tiled I-LayerNorm where its workgroups change: every number of lanes that share a row's sums, widths at which rows do not fill the
workgroup, rows past the end, the widest rows; rows of extremes and constant rows among them.  Against the oracle: equality."""
import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [64, 80, 96, 176, 256, 384, 528, 768, 1008, 1024, 1040, 1536, 2032, 2048])
@pytest.mark.parametrize("rows", [1, 4, 63, 1037, 9001, 40003])
def test_rows(ivit, C, rows):
    import torch
    rng = np.random.default_rng(C + rows)
    x = np.clip(np.rint(rng.normal(rng.integers(-60, 61, size=(rows, 1)), rng.integers(1, 90, size=(rows, 1)), size=(rows, C))), -128, 127).astype(np.int8)
    x[0] = np.where(np.arange(C) % 2, 127, -128)
    x[rows // 2] = 5
    x[-1, -1] = -128
    g, b = synth._ln(rng, C)
    prm = synth.LN_F_BITS, synth.LN_C_SHIFT
    dev = lambda a: torch.from_numpy(a).cuda()
    y = torch.empty((rows, C), dtype=torch.int8, device="cuda")
    ivit.ivit_ilayernorm(dev(x), dev(g), dev(b), y, *prm)
    want = orc.ilayernorm(x, g, b, *prm)
    got = y.cpu().numpy()
    assert np.array_equal(got, want), "%d of %d differ" % ((got != want).sum(), got.size)
    assert rows < 63 or len(np.unique(got)) > 100
