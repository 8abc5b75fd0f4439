"""Names of an op list's own tensors against those of the buffers the planner
makes for it: the list keeps its meaning whatever its tensors are called."""
import numpy as np
import pytest

from plan_interp import execute, triples
from test_triples_merge import BASE, INPUTS, LISTS, O_, V_, _literal

from paper_2409_06759_amd import _lib as L


def _listing(text):
    return L.load().cc_plan_describe_ops_dry(O_, V_, 1, 0, text.encode()).decode()


def _inputs(seed):
    rng = np.random.default_rng(seed)
    return {k: rng.normal(size=[O_ if c == "o" else V_ for c in sp]) for k, sp in INPUTS.items()}


@pytest.mark.parametrize("name", ["Y3w0", "Y3w1", "Y3_w0", "scratch", "splitk_ws"])
def test_caller_tensor_named_like_a_merged_sum(name):
    """Terms with a shared factor are summed into a buffer of the planner's."""
    text = (BASE + LISTS["intermediates"]).replace("G ", name + " ")
    inputs = _inputs(3)
    listing = _listing(text)
    assert not listing.startswith("error"), listing
    got, want = execute(listing, inputs, O_, V_, False, 1), _literal(text, inputs, False)
    r3 = triples(got, O_, V_)
    ref = triples(lambda k: want[k].ravel(), O_, V_)
    assert np.abs(r3 - ref).max() < 1e-12 * np.abs(ref).max()


def test_caller_tensor_named_like_a_gemm_buffer():
    """Small systems give every GEMM whose output is permuted a buffer of its own,
    numbered by its place among the plan's tensors."""
    body = BASE + "op w Xr ijab 1.0 t2 ikac ovvo kbcj\nop g {0} klij 1.0 oovv klcd t2 ijcd\n"
    body += "op c XP ijab 1.0 {0} klij t2 klab\nop x XP ijab 0.5 {0} ijkl oovv klab\n"
    inputs = _inputs(4)
    want = _literal("work G oooo\nwork Xr oovv\n" + body.format("G"), inputs, False)
    for n in range(24, 48):
        name = f"scratch_{n}"
        listing = _listing(f"work {name} oooo\n" + body.format(name))
        assert not listing.startswith("error"), listing
        got = execute(listing, inputs, O_, V_, False, 1)
        for x in ("XP", "Xr"):
            assert np.abs(got(x) - want[x].ravel()).max() < 1e-12 * np.abs(want[x]).max(), (name, x)
