"""The plan, macro tiles and LDS-DMA multiply at leaf 64 and 128, at sizes whose
one-call product runs on other kernels and at those where it runs on these."""

from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2103_13042_amd import binding as sp
from paper_2103_13042_amd import inputs

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)
U = 2.0**-24


def gamma32(k: int) -> float:
    return k * U / (1 - k * U)


def gpu(x: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(DEV)


def offset_view(x: np.ndarray, offset: int) -> torch.Tensor:
    """x on the GPU as a view that starts `offset` floats into its buffer."""
    n = x.shape[0]
    buf = torch.zeros(n * n + offset, dtype=torch.float32, device=DEV)
    buf[offset:] = gpu(x).reshape(-1)
    return buf[offset:].view(n, n)


def check_oracle(c: torch.Tensor, pairs: int, a, b, tau, leaf):
    """C within the FP32 accumulation bound of the oracle's, the same pairs."""
    ref, count, _ = oracle.spamm(a, b, tau, leaf)
    mag, _, _ = oracle.spamm(np.abs(a), np.abs(b), tau, leaf)
    assert pairs == count
    worst = float(np.max(np.abs(c.cpu().numpy().astype(np.float64) - ref) - gamma32(a.shape[0]) * mag - 1e-38))
    assert worst <= 0.0, worst


def middle_product(a, b, leaf) -> float:
    """A threshold that about half of the products reach, on none of them."""
    na, nb = oracle.leaf_norms(a, leaf), oracle.leaf_norms(b, leaf)
    return float(np.quantile(na[:, None, :] * nb.T[None, :, :], 0.5)) * (1.0 + 1e-9)


def staged(a, b, tau, leaf, *, scheduled, c=None):
    """C and the kept pairs by the plan and the LDS-DMA multiply."""
    offsets, klist, pairs = sp.prepare(a, b, tau, leaf, schedule=scheduled)
    run = sp.execute_scheduled if scheduled else sp.execute
    return run(a, b, leaf, offsets, klist, c=c), int(pairs.item())


@pytest.mark.parametrize("n,leaf", [(2176, 64), (2688, 64), (3968, 64), (2176, 128), (3968, 128), (4096, 128),
                                    (5120, 128)])
def test_one_call_between_the_block_ranges_runs_on_macro_tiles(n, leaf):
    """Multiples of 128 above 2048 (leaf 64: to 3968): one call is the staged calls,
    sum for sum, at a narrow band and with every pair kept."""
    for alpha, tau in ((0.05, 1e-6), (0.01, 0.0)):
        a, b = (inputs.exp_decay_torch(n, alpha, s, DEV) for s in (21, 22))
        c, pairs = sp.multiply(a, b, tau, leaf)
        want, kept = staged(a, b, tau, leaf, scheduled=True)
        assert pairs == kept and torch.equal(c, want)
        if tau == 0.0:
            ref = a.double() @ b.double()
            assert pairs == sp.bdim(n, leaf) ** 3
            assert bool(((c.double() - ref).abs() <= gamma32(n) * ref).all())


@pytest.mark.parametrize("leaf", [64, 128])
@pytest.mark.parametrize("kind", ["one_block", "scattered"])
@pytest.mark.parametrize("n", [1024, 961, 1000, 1090])
def test_staged_macro_tiles_shared_between_workgroups(n, kind, leaf):
    """Macro tiles split between workgroups, whose partial sums the fixup kernel
    adds: one_block: all products in one 128x128 block of C, shared by as many
    workgroups as it has items; scattered: blocks split between two.  At ragged n
    the block is the last one, past whose edge the fixup must not store."""
    rng = np.random.default_rng(n)
    a, b = inputs.uniform_pm1(n, 41), inputs.uniform_pm1(n, 42)
    if kind == "one_block":
        first = (n - 1) // 128 * 128
        a[:first], b[:, :first] = 0.0, 0.0
    else:
        t = -(-n // leaf)
        for x in (a, b):
            keep = np.kron(rng.random((t, t)) < 0.15, np.ones((leaf, leaf), dtype=bool))
            x[~keep[:n, :n]] = 0.0
    ga, gb = gpu(a), gpu(b)
    first_c = None
    for scheduled in (True, False, True):
        guard = torch.full((n * n + 4096,), float("nan"), device=DEV)  # nothing past C is written
        c, pairs = staged(ga, gb, 1e-6, leaf, scheduled=scheduled, c=guard[: n * n].view(n, n))
        assert bool(guard[n * n :].isnan().all())
        check_oracle(c, pairs, a, b, 1e-6, leaf)
        first_c = c if first_c is None else first_c
        assert torch.equal(c, first_c)  # the partials are added in a fixed order


@pytest.mark.parametrize("leaf", [64, 128])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 65, 127, 129, 190, 193, 255, 320, 1023, 1090])
def test_staged_multiply_at_ragged_edges(n, leaf):
    """N no multiple of 128 on the LDS-DMA multiply: macro tiles, k-chunks and
    16-byte copies that cross the matrix's edge, one tile row in the last macro
    row, N below the copy's four floats.  C starts as NaN: all of it is written."""
    a, b = inputs.uniform_pm1(n, 51), inputs.uniform_pm1(n, 52)
    for tau in (0.0, middle_product(a, b, leaf)):
        for scheduled in (True, False):
            c = torch.full((n, n), float("nan"), device=DEV)
            c, pairs = staged(gpu(a), gpu(b), tau, leaf, scheduled=scheduled, c=c)
            check_oracle(c, pairs, a, b, tau, leaf)


@pytest.mark.parametrize("leaf", [64, 128])
@pytest.mark.parametrize("n", [130, 131, 189, 250])
def test_staged_values_past_a_row_stay_out_of_it(n, leaf):
    """Copies reach past a ragged row into the next one, and in the last row back
    from its end: infinities there must not enter other rows' products."""
    a, b = inputs.uniform_pm1(n, 53), inputs.uniform_pm1(n, 54)
    a[7, :5] = np.inf
    b[9, 2] = b[n - 1, n - 4] = np.inf
    c, pairs = staged(gpu(a), gpu(b), 0.0, leaf, scheduled=True)
    assert pairs == sp.bdim(n, leaf) ** 3
    got = c.cpu().numpy()
    with np.errstate(invalid="ignore"):
        want = a.astype(np.float64) @ b.astype(np.float64)
        ok = np.isfinite(want)
        assert np.array_equal(np.isfinite(got), ok)
        a0, b0 = np.where(np.isfinite(a), a, 0.0), np.where(np.isfinite(b), b, 0.0)
        bound = gamma32(n) * (np.abs(a0).astype(np.float64) @ np.abs(b0).astype(np.float64))
        assert np.all(np.abs(got - want)[ok] <= bound[ok])


@pytest.mark.parametrize("n,leaf,offset", [(1024, 64, 1), (1024, 128, 3), (1000, 64, 1), (1000, 128, 2), (1023, 128, 1)])
def test_staged_multiply_on_views_that_are_only_4_byte_aligned(n, leaf, offset):
    a, b = inputs.exp_decay(n, 0.02, 8), inputs.exp_decay(n, 0.02, 9)
    tau = middle_product(a, b, leaf)
    ga, gb = offset_view(a, offset), offset_view(b, offset)
    assert ga.data_ptr() % 16 != 0 and gb.data_ptr() % 16 != 0
    c, pairs = staged(ga, gb, tau, leaf, scheduled=True)
    check_oracle(c, pairs, a, b, tau, leaf)
    aligned, kept = staged(gpu(a), gpu(b), tau, leaf, scheduled=True)
    assert kept == pairs and torch.equal(aligned, c)


@pytest.mark.parametrize("n,leaf", [(1000, 64), (1024, 64), (1024, 128), (1100, 128)])
def test_staged_graph_replays_equal_eager_run(n, leaf):
    """Plan, schedule, LDS-DMA multiply and fixup captured and replayed with eager
    work in between: the plan's state is cleared by a kernel on every replay."""
    a, b = (inputs.exp_decay_torch(n, 0.02, s, DEV) for s in (28, 29))
    ws = torch.empty(sp.workspace_bytes(n, leaf), dtype=torch.uint8, device=DEV)
    bufs = sp.plan_buffers(n, leaf, DEV)
    c = torch.empty((n, n), device=DEV)

    def call():
        sp.prepare(a, b, 1e-6, leaf, bufs=bufs, ws=ws, schedule=True)
        sp.execute_scheduled(a, b, leaf, bufs[0], bufs[1], c=c, ws=ws)

    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        call()
    torch.cuda.synchronize()
    eager, kept = c.clone(), int(bufs[2].item())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        c.fill_(7.0)
        bufs[2].fill_(-5)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(bufs[2].item()) == kept and torch.equal(c, eager)


@pytest.mark.parametrize("leaf", [64, 128])
@pytest.mark.parametrize("n", [5121, 5187])
def test_one_call_at_odd_sizes_above_the_blocks(n, leaf):
    a, b = (inputs.exp_decay_torch(n, 0.003, s, DEV) for s in (61, 62))
    c = torch.full((n, n), float("nan"), device=DEV)
    _, pairs = sp.multiply(a, b, 0.0, leaf, c=c)
    assert pairs == sp.bdim(n, leaf) ** 3
    ref = a.double() @ b.double()
    excess = float(((c.double() - ref).abs() - gamma32(n) * ref).max())
    assert excess <= 0.0, excess
