"""Every multiply kernel that the library launches is checked to use no scratch
memory before its first launch (check_no_scratch), in the file that launches it."""

from __future__ import annotations

import re
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2103_13042_amd" / "csrc"


def test_every_launched_multiply_kernel_is_checked():
    launched = 0
    for src in sorted(CSRC.glob("*.hip")):
        text = src.read_text()
        kernels = set(re.findall(r"\b(multiply_\w*kernel)(?:<[^;<>]*>)?\s*<<<", text))
        checked = set(re.findall(r"check_no_scratch\(\s*(multiply_\w*kernel)\b", text))
        assert kernels <= checked, (src.name, kernels - checked)
        launched += len(kernels)
    assert launched >= 9
