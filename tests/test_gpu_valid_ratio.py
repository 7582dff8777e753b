"""Valid-ratio search (section 3.5.2) on the GPU, through the C ABI.

The GPU search takes the oracle's steps (mean norm product, upper bound grown
in steps of the mean, bisection) with counts from the plan kernels; it must
return the oracle's tau (relative 1e-12: only the summation order of the mean
differs), the same number of kept triples and the same number of bisections.
At the sizes the oracle is slow for, it must reproduce the tau Table 1 prints.
"""

from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2103_13042_amd import binding as sp
from paper_2103_13042_amd import inputs

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def gpu(x: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(DEV)


def toeplitz_on_device(n: int) -> torch.Tensor:
    """paper_algebraic(n) built on the device (inputs.paper_algebraic_torch)."""
    return inputs.paper_algebraic_torch(n, DEV)


def test_device_toeplitz_matches_host_generator():
    n = 777
    assert torch.equal(toeplitz_on_device(n).cpu(), torch.from_numpy(inputs.paper_algebraic(n)))


@pytest.mark.parametrize(
    "n,leaf,kind,target",
    [
        (1024, 32, "paper", 0.30),
        (2048, 32, "paper", 0.05),
        (1000, 32, "exp", 0.20),
        (1100, 64, "alg", 0.10),
        (300, 32, "exp", 0.50),
        (4096, 128, "alg", 0.02),
    ],
)
def test_search_matches_oracle(n, leaf, kind, target):
    if kind == "paper":
        a = b = inputs.paper_algebraic(n)
    elif kind == "exp":
        a, b = inputs.exp_decay(n, 0.05, 40), inputs.exp_decay(n, 0.05, 41)
    else:
        a, b = inputs.algebraic_decay_signed(n, 42), inputs.algebraic_decay_signed(n, 43)
    tau_o, cnt_o, it_o = oracle.search_tau_for_valid_ratio(a, b, leaf, target, 0.01, 20)
    pa, pb = sp.pyramid(gpu(a), leaf), sp.pyramid(gpu(b), leaf)
    tau, cnt, it = sp.search_valid_ratio(pa, pb, n, leaf, target, 0.01, 20)
    assert tau == pytest.approx(tau_o, rel=1e-12, abs=0.0)
    assert (cnt, it) == (cnt_o, it_o)
    # the count reported is the plan's count at that tau
    _, _, pairs = sp.plan(pa, pb, n, leaf, tau)
    assert int(pairs.item()) == cnt


def test_search_zero_matrix_and_bad_arguments():
    n, leaf = 256, 32
    z = torch.zeros(n, n, dtype=torch.float32, device=DEV)
    pz = sp.pyramid(z, leaf)
    # every product is 0 and the mean is 0: tau stays 0 and every triple is kept
    tau, cnt, it = sp.search_valid_ratio(pz, pz, n, leaf, 0.5, 0.01, 5)
    assert tau == 0.0 and cnt == (n // leaf) ** 3 and it == 5
    for target in (0.0, -0.1, 1.5, float("nan")):
        with pytest.raises(sp.SpammError):
            sp.search_valid_ratio(pz, pz, n, leaf, target)
    with pytest.raises(sp.SpammError):
        sp.search_valid_ratio(pz, pz, n, leaf, 0.5, -1.0)
    with pytest.raises(ValueError):
        sp.search_valid_ratio(pz[:-1], pz[:-1], n, leaf, 0.5)


def _golden_rows(golden, n):
    return [(t, tau) for t, nn, tau in golden("table1_tau.txt") if int(nn) == n]


@pytest.mark.parametrize("n", [8192, 16384, 32768])
def test_search_reproduces_table1(golden, n):
    leaf = 32
    x = toeplitz_on_device(n)
    p = sp.pyramid(x, leaf)
    del x
    torch.cuda.synchronize()
    bd = n // leaf
    for target, tau_paper in _golden_rows(golden, n):
        tau, cnt, it = sp.search_valid_ratio(p, p, n, leaf, target / 100.0, 0.01, 20)
        assert abs(tau - tau_paper) <= 1.5e-6, (n, target, tau, tau_paper)
        assert abs(cnt / bd**3 - target / 100.0) <= 0.01
        assert 1 <= it < 20


@pytest.mark.parametrize("n,alpha,target", [(20, 0.05, 0.5), (64, 0.2, 0.3), (2080, 0.3, 0.004), (2049, 0.02, 0.1),
                                            (4200, 0.5, 0.002)])
def test_search_matches_brute_force_at_grid_edges(n, alpha, target):
    """1, 2, 65 and 132 tiles per side, and bounds that grow well past the 15
    multiples of the mean that one round tries: tau, count and bisections of
    the paper's search written out over the plain list of products."""
    leaf, tol, max_iters = 32, 0.0005, 20
    a, b = inputs.exp_decay_torch(n, alpha, 40, DEV), inputs.exp_decay_torch(n, alpha, 41, DEV)
    pa, pb = sp.pyramid(a, leaf), sp.pyramid(b, leaf)
    tau, pairs, iters = sp.search_valid_ratio(pa, pb, n, leaf, target, tol, max_iters)
    bd = sp.bdim(n, leaf)
    na = sp.pyramid_levels(pa, n, leaf)[-1][:bd, :bd].cpu().numpy()
    nb = sp.pyramid_levels(pb, n, leaf)[-1][:bd, :bd].cpu().numpy()
    prods = np.sort((na[:, :, None] * nb[None, :, :]).ravel())
    count = lambda t: prods.size - int(np.searchsorted(prods, t, side="left"))
    ave = float(np.sum(na.sum(axis=0) * nb.sum(axis=1))) / bd**3
    k, hi = 1, ave
    while count(hi) / bd**3 > target + tol and k < 1024:
        k += 1
        hi = k * ave
    lo, want, steps = 0.0, hi, 0
    while abs(count(want) / bd**3 - target) > tol and steps < max_iters:
        want = 0.5 * (lo + hi)
        steps += 1
        if count(want) / bd**3 > target:
            lo = want
        else:
            hi = want
    assert (pairs, iters) == (count(want), steps) and tau == pytest.approx(want, rel=1e-12)


def test_search_counts_as_the_plan_with_infinite_and_zero_norms():
    """A zero norm against an infinite one gives a NaN product, which the plan
    drops: the search's count is the plan's at the threshold it returns."""
    n, leaf = 256, 32
    a, b = torch.zeros(n, n, device=DEV), torch.rand(n, n, device=DEV)
    a[:64] = 1.0
    b[32, 200] = float("inf")
    pa, pb = sp.pyramid(a, leaf), sp.pyramid(b, leaf)
    tau, pairs, _ = sp.search_valid_ratio(pa, pb, n, leaf, 0.3)
    if tau == tau:  # the mean of products with an infinity may be NaN: then nothing is kept
        assert int(sp.plan(pa, pb, n, leaf, tau)[2].item()) == pairs
    else:
        assert pairs == 0
