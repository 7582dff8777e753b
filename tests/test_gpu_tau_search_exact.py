"""The search for an error target decides by spamm_error_for_tau's error, whatever
thresholds it tried before: err_out is that number to the rounding of E's FP32
sums, a target equal to it finds the same threshold again, and one unit below
it a smaller one."""

from __future__ import annotations

import math

import numpy as np
import pytest
import torch

from paper_2103_13042_amd import binding as sp
from paper_2103_13042_amd import inputs

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def _problem(n, leaf, alpha, signed):
    a, b = (inputs.exp_decay_torch(n, alpha, s, DEV) for s in (11, 12))
    if signed:
        gen = torch.Generator(device=DEV).manual_seed(n)
        a, b = (x * (1.0 - 2.0 * torch.randint(0, 2, (n, n), device=DEV, generator=gen)) for x in (a, b))
    c, _ = sp.multiply(a, b, 0.0, leaf)
    return a, b, sp.pyramid(a, leaf), sp.pyramid(b, leaf), float(sp.sumsq(c).item())


# 5 tiles per side (n = 300 at leaf 64, 70 at leaf 16), one tile, several blocks
@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("n,leaf,alpha", [(300, 64, 0.02), (70, 16, 0.1), (100, 128, 0.1), (777, 32, 0.05),
                                          (1024, 64, 0.03), (1000, 128, 0.02), (1024, 16, 0.1)])
def test_error_of_the_search_is_error_for_tau(n, leaf, alpha, signed):
    a, b, pa, pb, ab = _problem(n, leaf, alpha, signed)
    ladder = np.sort(np.unique((sp.pyramid_levels(pa, n, leaf)[-1].cpu().numpy()[:, :, None]
                                * sp.pyramid_levels(pb, n, leaf)[-1].cpu().numpy()[None, :, :]))) if n <= 300 else None
    for target in (0.3, 1e-2, 1e-4):
        tau, err, pairs, _ = sp.search_tau_for_error(a, b, leaf, target, pa, pb, ab)
        if err == 0.0:  # the smallest product, where nothing but zeros is dropped
            continue
        same, dropped = sp.error_for_tau(a, b, tau, leaf, pa, pb, ab)
        # two FP32 sums of the same products, of their magnitudes where signs differ
        size = sp.error_for_tau(a.abs(), b.abs(), tau, leaf, pa, pb, ab)[0]
        assert abs(err - same) <= 2 * n * 2.0**-24 / (1 - n * 2.0**-24) * size
        assert err <= target and same <= target
        assert pairs + dropped == sp.bdim(n, leaf) ** 3
        if signed:
            continue  # the error need not grow with tau
        again = sp.search_tau_for_error(a, b, leaf, same, pa, pb, ab)
        assert again[:3] == (tau, same, pairs)
        seeded = sp.search_tau_for_error(a, b, leaf, same, pa, pb, ab, guess=3.0 * tau)
        assert seeded[:3] == (tau, same, pairs)
        below = sp.search_tau_for_error(a, b, leaf, math.nextafter(same, 0.0), pa, pb, ab)
        assert below[0] < tau and below[1] < same
        if ladder is not None:  # every product, tried one by one
            above = ladder[ladder > tau]
            assert above.size == 0 or sp.error_for_tau(a, b, float(above[0]), leaf, pa, pb, ab)[0] > target
