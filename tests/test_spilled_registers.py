"""No Dense or block kernel keeps vector registers in scratch memory.

Those kernels have requests of weights in flight, and a reload from scratch memory waits for all that were made before it; and their
matrix instructions are written in asm, so that the compiler does not know how long a result takes to be there for a store of its own
making.  The figures are those that the compiler writes into the library's notes, read without a GPU."""
import os
import re

import pytest

from paper_2207_01405_amd import binding


def _number(b, i):
    """A msgpack unsigned integer."""
    return b[i] if b[i] < 0x80 else int.from_bytes(b[i + 1:i + 1 + {0xcc: 1, 0xcd: 2, 0xce: 4}[b[i]]], "big")


def _spills():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2207_01405_amd import build
        build.build_lib()
    b, out, key = open(binding.LIB_PATH, "rb").read(), {}, b".vgpr_spill_count"
    for m in re.finditer(rb"\.symbol[\xa0-\xbf\xd9\xda][\x00-\xff]{0,2}?(_Z\w+)\.kd", b):
        out[m.group(1).decode()] = _number(b, b.index(key, m.end()) + len(key))
    return out


@pytest.mark.parametrize("kernel", ["token_block_kernel", "token_stream_kernel", "gemm_st_kernel", "gemm_tl_kernel", "gemm_rs_kernel", "gemm_ks_kernel",
                                    "gemm_kq_kernel", "gemm_ws_kernel"])
def test_no_vector_register_is_spilled(kernel):
    of = {name: n for name, n in _spills().items() if re.search(r"\d" + kernel, name)}
    assert of and not [(name, n) for name, n in of.items() if n]
