"""The plan, macro tiles and LDS-DMA multiply at leaf 64 and 128, at sizes whose
one-call product runs on other kernels and at those where it runs on these."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2103_13042_amd import binding as sp
from paper_2103_13042_amd import inputs

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)
U = 2.0**-24


def gamma32(k: int) -> float:
    return k * U / (1 - k * U)


def staged(a, b, tau, leaf, *, scheduled, c=None):
    """C and the kept pairs by the plan and the LDS-DMA multiply."""
    offsets, klist, pairs = sp.prepare(a, b, tau, leaf, schedule=scheduled)
    run = sp.execute_scheduled if scheduled else sp.execute
    return run(a, b, leaf, offsets, klist, c=c), int(pairs.item())


@pytest.mark.parametrize("leaf", [64, 128])
@pytest.mark.parametrize("n", [2176, 2688, 3968])
def test_one_call_between_the_block_ranges_runs_on_macro_tiles(n, leaf):
    """Multiples of 128 between 2048 and 4096: one call is the staged calls, sum
    for sum, at a narrow band and with every pair kept."""
    for alpha, tau in ((0.05, 1e-6), (0.01, 0.0)):
        a, b = (inputs.exp_decay_torch(n, alpha, s, DEV) for s in (21, 22))
        c, pairs = sp.multiply(a, b, tau, leaf)
        want, kept = staged(a, b, tau, leaf, scheduled=True)
        assert pairs == kept and torch.equal(c, want)
        if tau == 0.0:
            ref = a.double() @ b.double()
            assert pairs == sp.bdim(n, leaf) ** 3
            assert bool(((c.double() - ref).abs() <= gamma32(n) * ref).all())
