"""bench.py's accounting of the kernels: every attention kernel has a timing slot, and the executed
products are those of the kernels that ran."""
import os
import re

import bench
from paper_2607_01701_amd import _lib
from paper_2607_01701_amd import build as B


def test_every_attention_kernel_has_a_slot():
    names = set()
    for src in B.HIP_SOURCES:
        text = open(os.path.join(B.CSRC, src)).read()
        names |= set(re.findall(r"__global__[^;{]*?\b(attn_\w+_kernel)\s*\(", text))
    assert len(names) >= 6
    assert {n: bench._slot(n) in _lib.KERNEL_SLOTS for n in names} == dict.fromkeys(names, True)


def test_executed_products():
    """Two products forward; backward S, dP, dV, dK, dQ, with S and dP once more for dQ unless it is one pass."""
    assert sum(bench.kernel_flops(3, 128, 1000).values()) == (2 + 5 + 2) * 2 * 3 * 128 * 1000
    assert sum(bench.kernel_flops(3, 128, 1000, one_pass=True).values()) == (2 + 5) * 2 * 3 * 128 * 1000
