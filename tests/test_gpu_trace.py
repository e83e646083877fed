"""The per-launch trace: one record for every kernel launch, in launch order, with the work of that launch."""
import pytest

from paper_2207_01405_amd import synth

pytestmark = pytest.mark.gpu

LN, GEMM, RES, GELU, ATT, BLOCK, TABLES = 1, 2, 3, 4, 5, 11, 12


def _records(ivit, R, C, H, F, L):
    import torch
    d = dict(B=R, T=1, C=C, H=H, F=F)
    cfg = dict(T=1, C=C, H=H, F=F, seed=1, i0="fixed", rel_bias=False)
    blocks = [ivit.to_device(synth.make_block(cfg, l % 2)) for l in range(L)]
    x = torch.zeros((R, C), dtype=torch.int8, device="cuda")
    ws = torch.empty(ivit.ivit_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    ivit.ivit_trace_begin(200)
    ivit.ivit_forward(x, torch.empty_like(x), blocks, d, ws)
    rec = ivit.ivit_trace_end(200)
    assert all(r[0] > 0 and r[3] > 0 for r in rec)
    # every multiply-accumulate of the Dense layers is in exactly one record
    assert sum(r[2] for r in rec if r[1] != ATT) == 2 * L * R * (4 * C * C + 2 * C * F)
    return [r[1] for r in rec]


def test_block_kernels_and_their_constants(ivit):
    assert _records(ivit, 500, 192, 3, 768, 2) == [TABLES, BLOCK, ATT, BLOCK, ATT, BLOCK]


def test_constants_of_more_layers_than_one_launch_takes(ivit):
    kinds = _records(ivit, 4000, 96, 3, 256, 20)
    assert kinds.count(TABLES) == 2 and kinds.count(BLOCK) == 21 and kinds.count(ATT) == 20


def test_rows_beyond_full_rounds_are_a_launch_of_their_own(ivit):
    import torch
    R = 128 * torch.cuda.get_device_properties(0).multi_processor_count + 5
    assert _records(ivit, R, 192, 3, 768, 1) == [TABLES, BLOCK, BLOCK, ATT, BLOCK, BLOCK]


def test_separate_kernels(ivit):
    assert _records(ivit, 40000, 128, 2, 512, 1) == [LN, GEMM, ATT, RES, LN, GELU, RES]
