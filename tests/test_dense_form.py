"""Which form of the Dense kernels a shape takes: the rules (host code, compiled here) on both sides of their lines, on the CPU, and on
the GPU that the forms agree there."""
import ctypes
import subprocess

import numpy as np
import pytest

import oracle as orc
from paper_2207_01405_amd import build, synth

I64, INT = ctypes.c_int64, ctypes.c_int


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("dense")
    (d / "r.cpp").write_text('#include "dense_form.hpp"\n'
                             'extern "C" int before_slab(int64_t M, int64_t N, int64_t K, int slab) { return ivit::tiles_before_slab(M, N, K, slab, 256); }\n'
                             'extern "C" int of_192(int64_t M, int64_t N, int64_t K, int residual) { return ivit::one_round_of_192(M, N, K, residual, 256); }\n'
                             'extern "C" int of_128(int64_t M, int64_t N, int64_t K, int residual) { return ivit::one_round_of_128(M, N, K, residual, 256); }\n')
    subprocess.run(["g++", "-std=c++20", "-shared", "-fPIC", "-I", build.CSRC, str(d / "r.cpp"), "-o", str(d / "r.so")], check=True)
    lib = ctypes.CDLL(str(d / "r.so"))
    lib.before_slab.argtypes = [I64, I64, I64, INT]
    lib.of_192.argtypes = lib.of_128.argtypes = [I64, I64, I64, INT]
    return lib


@pytest.mark.parametrize("M,N,K,slab,tiles", [
    # few channels over very many rows stay on the slab: both sides are measured at the rule
    (200000, 16, 400, 64, False), (262144, 64, 640, 64, False), (200000, 64, 1152, 64, False), (50000, 64, 896, 64, False),
    (131072, 96, 640, 96, True), (200000, 96, 400, 96, False), (200000, 128, 400, 128, False), (262144, 96, 896, 96, False), (200000, 128, 1152, 128, True),
    # channels that tiles pad by a third and slabs do not
    (50000, 144, 896, 64, True), (131072, 192, 896, 96, True), (200000, 144, 1152, 96, False), (90000, 272, 896, 96, False), (262144, 272, 1152, 96, False),
    (262144, 272, 1664, 64, True),
    # rows of up to 768 bytes: four rounds of tiles, 768 itself among them
    (131072, 256, 400, 128, True), (131073, 256, 400, 128, False), (90000, 640, 640, 128, False), (90000, 400, 896, 96, True), (90000, 208, 768, 128, True),
    (200000, 208, 768, 128, False), (50000, 528, 768, 96, True), (200000, 272, 768, 96, False),
    (50000, 1008, 352, 128, False), (20000, 208, 1024, 64, False), (12000, 1040, 400, 128, True), (4000, 3008, 1152, 128, True)])
def test_tiles_or_the_slab(rules, M, N, K, slab, tiles):
    assert bool(rules.before_slab(M, N, K, slab)) == tiles


@pytest.mark.parametrize("M,N,K,residual,taken", [
    (40000, 16, 1024, False, False), (49000, 64, 1536, False, False), (33000, 64, 2048, False, False), (33000, 64, 3072, False, True), (49000, 48, 2560, False, True),
    (40000, 16, 3072, True, False), (33000, 64, 2048, True, False), (40000, 48, 3072, True, False), (49000, 64, 2560, True, True),
    # 1024 bytes a row: two tiles of 128 x 64 a CU are the line, one column of tiles stays off without a residual
    (20000, 192, 1024, False, False), (20000, 192, 1024, True, False), (24500, 192, 1024, False, True), (24500, 192, 1024, True, True), (20000, 192, 1040, False, True),
    (12000, 272, 1024, True, False), (14000, 272, 1024, True, True), (40900, 128, 1024, False, True), (41000, 128, 1024, False, False), (49000, 128, 1024, False, False), (49000, 128, 1024, True, True), (49000, 80, 1040, False, True),
    (7000, 528, 1024, False, False), (8000, 528, 1024, False, True),
    (4000, 1536, 1024, False, True), (6272, 768, 3072, True, True), (8064, 768, 2048, False, True), (8065, 768, 2048, False, False), (6272, 768, 1008, False, False)])
def test_one_round_of_192_rows(rules, M, N, K, residual, taken):
    assert bool(rules.of_192(M, N, K, residual)) == taken


@pytest.mark.parametrize("M,N,K,residual,taken", [
    # two 64 x 64 tiles a CU; two and a half, with a residual and rows of less than 2048 bytes; one 128 x 128 tile a CU
    (129, 10736, 1536, False, False), (257, 6384, 2048, True, False), (1341, 1520, 3072, False, False), (1341, 1536, 2048, True, False),
    (20000, 80, 768, True, False), (20000, 80, 768, False, True), (21245, 80, 768, True, True), (8957, 256, 1024, True, False), (8957, 256, 2048, True, True),
    (1469, 1536, 768, True, False), (1725, 1536, 768, True, True), (1576, 2304, 768, False, True), (4000, 768, 3072, True, True), (32768, 128, 768, True, True),
    (32769, 128, 768, True, False)])
def test_one_round_of_128_rows(rules, M, N, K, residual, taken):
    assert bool(rules.of_128(M, N, K, residual)) == taken
    assert not rules.of_192(M, N, K, residual) or M > 32768       # (what is left to smaller tiles is not for the larger ones)


def _agree(ivit, M, N, K, epi):
    """The form of the shape against the kernel for many rows, and some rows against the oracle."""
    import torch
    x = synth.make_rows(M + N + K, M, K)
    w, bias, rq_b, rq_c = synth.make_linear(N + K, N, K)
    kw_o, kw_g = {}, {}
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    rows = np.unique(np.concatenate([np.arange(0, min(M, 200), 3), np.arange(M - 40, M), np.arange(0, M, 997)]))
    if epi == "residual":
        res = synth.make_rows(7, M, N)
        kw_o, kw_g = dict(residual=res[rows], res_rq=(20011, 15)), dict(residual=dev(res), res_rq=(20011, 15))
    d, out = [dev(a) for a in (x, w, bias, rq_b, rq_c)], []
    for kernel in ("auto", "many_rows"):
        y = torch.full((M, N), 55, dtype=torch.int8, device="cuda")
        ivit.ivit_linear_requant(*d, y, kernel=kernel, **kw_g)
        out.append(y.cpu().numpy())
    assert np.array_equal(*out)
    assert np.array_equal(out[0][rows], orc.linear_requant(x[rows], w, bias, rq_b, rq_c, **kw_o))


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(66001, 48, 400), (66001, 64, 1152), (131080, 80, 400), (200001, 96, 400), (66003, 144, 896), (90001, 272, 896), (33001, 208, 768)])
def test_tiles_and_the_slab_agree(ivit, M, N, K):
    _agree(ivit, M, N, K, "plain")


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(33001, 64, 2048), (33001, 64, 2560), (40001, 17, 1040), (20001, 192, 1024), (24501, 192, 1024), (12001, 272, 1024), (49001, 128, 1024),
                                   (129, 8699, 1536), (257, 6384, 784), (20001, 80, 768), (1469, 1537, 1040)])
@pytest.mark.parametrize("epi", ["plain", "residual"])
def test_few_channels_and_long_rows(ivit, M, N, K, epi):
    _agree(ivit, M, N, K, epi)
