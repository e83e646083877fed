"""The I-LayerNorm of patch merging that reads the tokens where they lie, inside the windowed forward pass without blocks, against the
oracle: its narrowest and widest rows, odd widths, rows that leave the last workgroup partly empty, and parameters off their 16 bytes,
which it does not take (gather, then I-LayerNorm).  Whole numbers, compared for equality."""
import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("C,grid,window,stages,B", [(32, 2, 1, 2, 1), (32, 40, 5, 4, 3), (96, 12, 3, 3, 3), (160, 10, 5, 2, 5), (256, 12, 3, 3, 1),
                                                    (288, 40, 2, 2, 2), (512, 2, 1, 2, 1), (512, 12, 6, 2, 7)])
def test_merge(ivit, C, grid, window, stages, B, off):
    import torch
    cfg = dict(grid=grid, window=window, C=C, heads=tuple((C << s) // 32 for s in range(stages)), depths=(0,) * stages, patch_dim=48,
               n_classes=64, seed=C + grid)
    model, patches = synth.make_swin_model(cfg), synth.make_swin_patches(cfg, B)
    want = orc.swin_forward(patches, model)
    m = ivit.swin_to_device(model)
    for st in m["stages"][1:]:
        g = st["merge"]["ln_gamma"]
        st["merge"]["ln_gamma"] = torch.cat([g[:off], g])[off:]
    sp, keep = ivit.swin_params(m)
    ws = torch.empty(ivit.ivit_swin_workspace_bytes(sp, B), dtype=torch.uint8, device="cuda")
    logits = torch.empty((B, 64), dtype=torch.int8, device="cuda")
    ivit.ivit_forward_swin(torch.from_numpy(patches).cuda(), logits, sp, B, ws)
    got = logits.cpu().numpy()
    assert want.std() > 5 and np.array_equal(got, want), "%d of %d differ" % ((got != want).sum(), got.size)
