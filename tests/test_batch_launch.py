"""Workgroups of the batched multiply, on the host: a product of few block rows takes
exactly as many as it has 64x64 blocks of C, a larger one whole rounds of the 8
XCDs with no more than a round of strips to spare."""

from __future__ import annotations

import ctypes


def test_a_small_product_takes_one_workgroup_per_block():
    from paper_2103_13042_amd import binding

    blocks = binding.library()._ZN5spamm12batch_blocksEl
    blocks.argtypes, blocks.restype = [ctypes.c_int64], ctypes.c_int64
    for n in (1, 48, 64, 65, 100, 128, 129, 200, 300, 512, 700, 832):
        assert blocks(n) == (-(-n // 64)) ** 2, n
    for n in (833, 1000, 2048, 4097, 8192, 65536):
        nb = -(-n // 64)
        assert blocks(n) % 8 == 0 and nb * nb <= blocks(n) <= nb * (nb + 2) + 8, n
