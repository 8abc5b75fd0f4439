"""Scratch of a small system's plan: steps of merged launches hold their partial
sums, the steps with launches of their own share one buffer."""
import re

import pytest


def _listing(o, v):
    from paper_2409_06759_amd import _lib as L
    return L.load().cc_plan_describe_dry(o, v, 1, 0).decode()


# dense CCSD from the smallest to the largest systems that are merged
@pytest.mark.parametrize("o,v", [(2, 3), (4, 20), (13, 61), (20, 100), (20, 140), (32, 90), (50, 57), (10, 200)])
def test_split_buffers(o, v):
    text = _listing(o, v)
    held = sum(int(re.search(r"dims=(\d+)", line).group(1)) for line in text.splitlines() if line.startswith("splitk_ws"))
    need = 0
    for line in text.splitlines():
        if line.startswith("GEMM") and " tile=32x32" in line:
            M, N, split = (int(re.search(rf" {k}=(\d+)", line).group(1)) for k in ("M", "N", "split"))
            need += M * N * split if split > 1 else 0
    # one shared buffer: the partial sums of a launch's K-split tail take at most 2^25 elements
    assert held <= need + 2 ** 25
