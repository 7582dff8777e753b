"""Batches of many small products: every product's blocks are found, whatever the
sizes around it.  Whole-number matrices with zero tiles, so C is exact in any
order of sums and the kept pairs are the nonzero ones."""

from __future__ import annotations

import pytest
import torch

from paper_2103_13042_amd import binding as sp

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def _matrix(n, leaf, gen):
    x = torch.randint(-3, 4, (n, n), generator=gen).float()
    b = -(-n // leaf)
    keep = torch.rand((b, b), generator=gen) < 0.6
    x *= keep.repeat_interleave(leaf, 0)[:n].repeat_interleave(leaf, 1)[:, :n]
    x[0, 0] = 1.0
    return x


@pytest.mark.parametrize("leaf", [32, 64, 128])
def test_batches_of_small_products(leaf):
    gen = torch.Generator().manual_seed(leaf)
    # one block, 13 and 14 block rows (the last taken in launch order and the first in strips)
    sizes = [1, 2, 3, 5, 17, 31, 32, 33, 48, 63, 64, 65, 100, 128, 129, 191, 257, 300, 832, 833, 900, 1024] + [40] * 300
    order = torch.randperm(len(sizes), generator=gen).tolist()
    sizes = [sizes[i] for i in order]
    a = [_matrix(n, leaf, gen) for n in sizes]
    b = [_matrix(n, leaf, gen) for n in sizes]
    batch = sp.Batch([x.to(DEV) for x in a], [x.to(DEV) for x in b], [leaf] * len(sizes), [0.5] * len(sizes))
    for c in batch.c:
        c.fill_(float("nan"))
    for _ in range(2):
        batch.run()
    torch.cuda.synchronize()
    pairs = batch.pairs.tolist()
    for n, x, y, c, got in zip(sizes, a, b, batch.c, pairs):
        t = -(-n // leaf)

        def nonzero(m):
            p = torch.zeros(t * leaf, t * leaf)
            p[:n, :n] = m
            return (p.view(t, leaf, t, leaf).abs().sum(dim=(1, 3)) > 0).double()

        assert got == int((nonzero(x) @ nonzero(y)).sum().item()), n
        assert torch.equal(c.cpu(), (x.double() @ y.double()).float()), n
