"""Op lists that the planner refuses stay refused when they also hold triples
terms that it would merge, whether or not the faulty line is one of them."""
import numpy as np
import pytest

from plan_interp import execute, triples
from test_triples_merge import BASE, INPUTS, O_, V_

from paper_2409_06759_amd import _lib as L

# two terms with the factor ooov in the same canonical labels
PAIR = "op a Y3 ijkabc 0.5 G lmij t3 lmkabc\nop b Y3 jkiabc -0.5 K lmjk t3 lmiabc\n"
MAKE = "work G oooo\nwork K oooo\nop g G klij 1.0 oovv klcd t2 ijcd\nop k K klij 1.0 oooo klij - -\n"

MALFORMED = {
    "declared twice": ("work G oooo\n" + MAKE + PAIR, "tensor G already exists"),
    "space not o or v": (MAKE.replace("G oooo", "G ooox") + PAIR, "spaces of G must be o/v"),
    "written with too few indices": (MAKE.replace("G oooo", "G ooooo") + PAIR, "rank mismatch for G"),
    "written with too many indices": (MAKE.replace("G oooo", "G ooo") + PAIR, "rank mismatch for G"),
    "read with too few indices": (MAKE + PAIR.replace("G lmij", "G lij"), ""),
    "unknown tensor": (MAKE + PAIR.replace("G lmij", "H lmij"), "unknown tensor H"),
    "index label out of range": (MAKE + PAIR.replace("lmkabc", "lmkabz").replace("lmiabc", "lmiabz")
                                 .replace("ijkabc", "ijkabz").replace("jkiabc", "jkiabz"), "bad index label z"),
}


def _listing(text):
    return L.load().cc_plan_describe_ops_dry(O_, V_, 1, 0, text.encode()).decode()


@pytest.mark.parametrize("name", sorted(MALFORMED))
def test_malformed_lists_are_refused(name):
    text, why = MALFORMED[name]
    listing = _listing(BASE + text)
    assert listing.startswith("error: op list: ") and why in listing, listing


def test_the_same_list_without_the_fault_is_merged():
    listing = _listing(BASE + MAKE + PAIR)
    assert not listing.startswith("error"), listing
    assert sum(line.startswith("GEMM Y3_") for line in listing.splitlines()) == 1


def test_second_factor_of_rank_eight():
    """A factor of more indices than a permutation takes is multiplied as it stands."""
    o, v = 3, 56
    text = BASE + """work w ooovvooo
op g w ijkablmn 1.0 t3 ijkabd ooov lmnd
op a Y3 ijkabc 0.5 w ijkablmn ooov lmnc
op b Y3 kijabc 0.25 w kijablmn ooov lmnc
"""
    rng = np.random.default_rng(8)
    inputs = {k: rng.normal(size=[o if c == "o" else v for c in sp]) for k, sp in INPUTS.items()}
    listing = L.load().cc_plan_describe_ops_dry(o, v, 1, 0, text.encode()).decode()
    assert not listing.startswith("error"), listing
    r3 = triples(execute(listing, inputs, o, v, False, 1), o, v)
    g = np.tensordot(inputs["t3"], inputs["ooov"], axes=([5], [3]))
    y = np.tensordot(g, inputs["ooov"], axes=([5, 6, 7], [0, 1, 2]))
    y = 0.5 * y + 0.25 * y.transpose(1, 2, 0, 3, 4, 5)
    ref = triples(lambda _: y.ravel(), o, v)
    assert np.abs(r3 - ref).max() < 1e-12 * np.abs(y).max()
