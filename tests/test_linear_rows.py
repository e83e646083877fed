"""Dense layers over rows that lie far apart (the classifier head reads one row of every image through a row stride).

The kernel they run on addresses the rows of a tile by 32-bit offsets: the rule that keeps a launch within them is checked
on the CPU over strides up to the largest the interface allows, and on the GPU the head against the oracle at strides
where the last offsets of a tile, and the stride itself, are beyond 32 bits.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import build, synth


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    src = d / "rows.cpp"
    src.write_text('#include "linear_rows.hpp"\nextern "C" int64_t rows_of(int64_t ldx, int64_t K) { return ivit::linear_rows_per_launch(ldx, K); }\n'
                   'extern "C" int64_t tile_rows() { return ivit::kTileRows; }\n')
    subprocess.run(["g++", "-std=c++20", "-shared", "-fPIC", "-I", build.CSRC, str(src), "-o", str(d / "rows.so")], check=True)
    lib = ctypes.CDLL(str(d / "rows.so"))
    lib.rows_of.restype = lib.tile_rows.restype = ctypes.c_int64
    lib.rows_of.argtypes = [ctypes.c_int64, ctypes.c_int64]
    return lib


@pytest.mark.parametrize("C", [16, 768, 65536])
def test_offsets_of_a_launch_fit(rule, C):
    tile = rule.tile_rows()
    strides = {C * t for t in (1, 197, 256, 1041, 65537, 2 ** 31 - 1)}
    strides |= {s // 16 * 16 + e for e in (-16, 0, 16) for n in (1, 2, 3, 63, 126, 127, 128) for s in (2 ** 31 // n, 2 ** 32 // n)}
    for ldx in sorted(s for s in strides if s >= C):
        rows = rule.rows_of(ldx, C)
        assert rows >= 1
        last = min(rows, tile) - 1                           # the last row of a tile of such a launch
        assert last * ldx + C <= 2 ** 31, (ldx, C, rows)
        assert rows >= tile or (last + 1) * ldx + C > 2 ** 31          # and no launch more than it takes
    assert rule.rows_of(256 * 1024, 1024) > 2 ** 40          # what the model forwards use: a single launch


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,C,N", [(64, 1041, 65536, 24), (3, 65552, 65536, 17), (131, 2200000, 16, 48), (5, 262144, 8192, 250)])
def test_head_over_images_far_apart(ivit, B, T, C, N):
    import torch
    assert (min(B, 64) - 1) * T * C >= 2 ** 31
    x = synth.make_rows(B + N, B, C, "uniform")
    w, bias, rq_b, rq_c = synth.make_linear(N, N, C)
    dev = lambda a: torch.from_numpy(a).cuda()
    tokens = torch.empty(B * T * C, dtype=torch.int8, device="cuda")
    tokens.view(B, T * C)[:, :C] = dev(x)
    room = torch.full((B * N + 64,), 77, dtype=torch.int8, device="cuda")
    ivit.ivit_classifier_head(tokens.view(B * T, C), T, dev(w), dev(bias), dev(rq_b), dev(rq_c), room[:B * N].view(B, N))
    got = room.cpu().numpy()
    assert np.array_equal(got[:B * N].reshape(B, N), orc.linear_requant(x, w, bias, rq_b, rq_c)) and (got[B * N:] == 77).all()


@pytest.mark.gpu
@pytest.mark.parametrize("B,C", [(2, 16), (2, 1024), (64, 8192)])
def test_a_launch_that_ends_where_its_offsets_do(ivit, B, C):
    """The last row ends at byte 2^31 of a tile exactly, and there are more classes than the kernel for few rows takes."""
    import torch
    T = (2 ** 31 // C - 1) // (B - 1)
    assert (B - 1) * T * C + C == 2 ** 31
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    N = 32 * (cus * (1 if C > 768 else 2) // -(-B // 32)) + 40
    x = synth.make_rows(B + C, B, C, "uniform")
    x[-1] = np.where(x[-1] == 0, 77, x[-1])
    w, bias, rq_b, rq_c = synth.make_linear(N, N, C)
    dev = lambda a: torch.from_numpy(a).cuda()
    tokens = torch.empty(B * T * C, dtype=torch.int8, device="cuda")
    tokens.view(B, T * C)[:, :C] = dev(x)
    room = torch.full((B * N + 64,), 77, dtype=torch.int8, device="cuda")
    ivit.ivit_classifier_head(tokens.view(B * T, C), T, dev(w), dev(bias), dev(rq_b), dev(rq_c), room[:B * N].view(B, N))
    got = room.cpu().numpy()
    assert np.array_equal(got[:B * N].reshape(B, N), orc.linear_requant(x, w, bias, rq_b, rq_c)) and (got[B * N:] == 77).all()
