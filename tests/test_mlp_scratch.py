"""The threshold network's scratch: what a gradient step keeps of a batch (both
hidden layers' outputs and gradients, the predictions and their residuals) and
no more."""

from __future__ import annotations

import pytest


@pytest.mark.parametrize("batch", [1, 2, 256, 1000])
def test_scratch_holds_the_arrays_in_use(batch):
    from paper_2103_13042_amd import binding

    assert binding.library().spamm_mlp_acts_floats(batch) == batch * (4 * 128 + 2)
