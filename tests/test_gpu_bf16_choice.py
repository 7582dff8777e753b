"""BF16 in one call, with room for the planes: the device writes and multiplies the
planes where many pairs are kept and reads the FP32 inputs where few are, with the
same C and pairs as without room."""

from __future__ import annotations

import pytest
import torch

from paper_2103_13042_amd import binding as sp
from paper_2103_13042_amd import inputs

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda", 0)


def _untouched(buf):
    return bool((buf == 0xA5).all())


def _scattered(n, share, seed):
    """Random 64x64 tiles, the others zero."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    keep = torch.rand((n // 64, n // 64), device=DEV, generator=gen) < share
    return torch.rand((n, n), device=DEV, generator=gen) * keep.repeat_interleave(64, 0).repeat_interleave(64, 1)


def _pair(n, alpha):
    """Decaying matrices, or for a negative alpha that share of scattered tiles."""
    return [inputs.exp_decay_torch(n, alpha, s, DEV) if alpha > 0 else _scattered(n, -alpha, s) for s in (31, 32)]


# (n, decay, tau, planes): either form in each range of the weight, none below the
# smallest size with a choice (4224), with every pair kept where strips come out
# even (8192) and where not (11008), beyond the one-launch plan's 256 tiles a side
@pytest.mark.parametrize("n,alpha,tau,planes", [
    (4224, -0.6, 1e-6, False), (4352, -0.6, 1e-6, True), (4352, -0.2, 1e-6, False), (4352, 0.0035, 1e-6, False),
    (5504, 0.005, 1e-6, False), (5632, 0.003, 1e-6, True), (6272, 0.008, 1e-6, False), (6400, 0.005, 1e-6, True), (6400, 0.05, 1e-6, False), (6400, 0.008, 1e-6, False),
    (8192, -0.3, 1e-6, True), (8192, -0.08, 1e-6, False),
    (8192, 0.0035, 1e-6, True), (8192, 0.02, 1e-6, False), (8192, 0.01, 0.0, False), (11008, 0.01, 0.0, True),
    (11008, 0.01, 1e-6, False), (16512, 0.0035, 1e-6, True), (16512, 0.03, 1e-6, False),
])
def test_form_is_picked_on_the_device(n, alpha, tau, planes):
    a, b = _pair(n, alpha)
    ws = sp.workspace(n, 64, DEV)
    small = torch.empty(256, dtype=torch.uint8, device=DEV)
    want, kept = sp.multiply_precision(a, b, tau, 64, "bf16", split_buf=small, ws=ws)
    buf = sp.split_buffer(n, "bf16", DEV)
    buf.fill_(0xA5)
    ws.fill_(0xFF)
    c = torch.full((n, n), float("nan"), device=DEV)
    _, views = sp.split_views(buf, n, "bf16")
    for _ in range(2):
        _, pairs = sp.multiply_precision(a, b, tau, 64, "bf16", c=c, split_buf=buf, ws=ws)
        assert pairs == kept
        assert torch.equal(c, want)
    if planes:
        assert torch.equal(views[0], a.bfloat16().view(torch.int16))
        assert torch.equal(views[1], b.t().contiguous().bfloat16().view(torch.int16))
    else:
        assert _untouched(buf)


def test_unaligned_room_is_not_used():
    n = 6400
    a, b = (inputs.exp_decay_torch(n, 0.005, s, DEV) for s in (31, 32))
    want, kept = sp.multiply_precision(a, b, 1e-6, 64, "bf16", split_buf=torch.empty(256, dtype=torch.uint8, device=DEV))
    buf = torch.full((sp.split_bytes(n, "bf16") + 64,), 0xA5, dtype=torch.uint8, device=DEV)
    c, pairs = sp.multiply_precision(a, b, 1e-6, 64, "bf16", split_buf=buf[16:])
    assert pairs == kept and torch.equal(c, want) and _untouched(buf)


def test_choice_in_a_graph_follows_the_inputs():
    """Replays take the form that the matrices then call for."""
    n = 6400
    narrow = [inputs.exp_decay_torch(n, 0.05, s, DEV) for s in (31, 32)]
    wide = [inputs.exp_decay_torch(n, 0.005, s, DEV) for s in (33, 34)]
    want = [sp.multiply(*p, 1e-6, 64)[1] for p in (narrow, wide)]
    a, b = (x.clone() for x in narrow)
    c, pairs = torch.empty_like(a), torch.empty(1, dtype=torch.int64, device=DEV)
    ws = torch.empty(sp.workspace_bytes(n, 64), dtype=torch.uint8, device=DEV)
    buf = sp.split_buffer(n, "bf16", DEV)

    def call():
        sp.multiply_precision(a, b, 1e-6, 64, "bf16", c=c, pairs=pairs, split_buf=buf, ws=ws, sync=False)

    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    for turn in (0, 1, 0, 1):
        for x, y in zip((a, b), (narrow, wide)[turn]):
            x.copy_(y)
        c.fill_(float("nan"))
        buf.fill_(0xA5)
        graph.replay()
        torch.cuda.synchronize()
        assert int(pairs.item()) == want[turn]
        assert _untouched(buf) == (turn == 0)
        got = c.clone()
        call()
        assert torch.equal(got, c)
