"""Triples contributions that share a factor are summed before they are
multiplied: the planner's listing, run on NumPy buffers, against the op list
taken line by line."""
import numpy as np
import pytest

from plan_interp import execute, triples

O_, V_ = 3, 4
SP = {**{c: O_ for c in "ijklmn"}, **{c: V_ for c in "abcdefgh"}}
INPUTS = {"foo": "oo", "fov": "ov", "fvv": "vv", "oooo": "oooo", "ooov": "ooov", "oovv": "oovv", "ovvo": "ovvo",
          "ovvv": "ovvv", "vvvv": "vvvv", "t1": "ov", "t2": "oovv", "t3": "ooovvv"}


def _literal(text, inputs, cplx):
    dt = np.complex128 if cplx else np.float64
    t = dict(inputs)
    shape = lambda sp: tuple(O_ if c == "o" else V_ for c in sp)  # noqa: E731
    t["Y3"] = np.zeros(shape("ooovvv"), dtype=dt)
    t["R1"] = np.zeros(shape("ov"), dtype=dt)
    t["XP"] = np.zeros(shape("oovv"), dtype=dt)
    for line in text.splitlines():
        w = line.split()
        if w[0] == "work":
            t[w[1]] = np.zeros(shape(w[2]), dtype=dt)
            continue
        _, _, C, cl, alpha, A, al, B, bl = w[:9]
        f = w[9:]
        a = t[A].conj() if "conjA" in f else t[A]
        if B == "-":
            t[C] = t[C] + float(alpha) * np.einsum(f"{al}->{cl}", a)
        else:
            b = t[B].conj() if "conjB" in f else t[B]
            t[C] = t[C] + float(alpha) * np.einsum(f"{al},{bl}->{cl}", a, b)
    return t


BASE = "op r R1 ia 1.0 fov ia - -\n"
LISTS = {
    # relabelled external and summed indices, both orders of the factors
    "relabelled": """op a Y3 ijkabc 0.5 t2 lica ooov jklb
op b Y3 jikbac -0.25 t2 ljcb ooov ikla
op c Y3 kijcab 0.125 ooov ijmb t2 mkac
""",
    # intermediates: made for one term alone, made for two, written again later
    "intermediates": """work G oooo
work H oooo
work K oooo
op g G klij 1.0 oovv klcd t2 ijcd
op a Y3 ijkabc 0.5 G lmij t3 lmkabc
op h H klij 2.0 oovv klcd t2 ijcd
op b Y3 kijabc 0.5 H mlki t3 mljabc
op c XP ijab 1.0 H klij t2 klab
op k K klij 1.0 oooo klij - -
op d Y3 jkibca -0.5 K lmjk t3 lmibca
op k2 K klij 1.0 oovv klcd t2 ijcd
op e Y3 ijkabc 0.75 K lmij t3 lmkabc
op f Y3 ijkabc 0.3 oooo lmij t3 lmkabc
""",
    # the shared factor is written between two of its terms
    "factor_rewritten": """work G oovo
op g G ijal 1.0 ooov ijla - -
op a Y3 ijkabc 1.0 G ijal t2 lkbc
op g2 G ijal 1.0 oooo ijml t1 ma
op b Y3 jkibca 0.5 G jkbl oovv lica
op c Y3 ijkabc 0.25 G ijal oovv lkbc
op d Y3 kijcab 0.5 G kicl t2 ljab
""",
    "reads_y3": """op a Y3 ijkabc 1.0 oooo lmij t3 lmkabc
op b Y3 ijkabc 0.5 oooo lmjk t3 lmiabc
op c XP ijab 1.0 fov me Y3 mijeab
op d Y3 ijkabc 0.1 t3 ijkabc - -
""",
    "conjugated": """work G oooo
op g G klij 1.0 oovv klcd t2 ijcd conjA
op a Y3 ijkabc 0.5 oooo lmij t3 lmkabc conjA
op b Y3 jikabc 0.5 G lmji t3 lmkabc conjA
op c Y3 kijabc 0.5 oooo lmki t3 lmjabc
op d Y3 ijkabc 0.25 oooo lmij t3 lmkabc conjB
op e Y3 ijkabc 0.25 ooov ijla t2 lkbc conjA conjB
op f Y3 jkiabc 0.5 ooov jkla t2 libc conjA conjB
""",
}


@pytest.mark.parametrize("name", sorted(LISTS))
@pytest.mark.parametrize("cplx", [False, True])
def test_merged_triples_equal_the_list(name, cplx):
    from paper_2409_06759_amd import _lib as L
    text = BASE + LISTS[name]  # (every list writes R1)
    rng = np.random.default_rng(len(name))
    inputs = {}
    for k, sp in INPUTS.items():
        x = rng.normal(size=[O_ if c == "o" else V_ for c in sp])
        inputs[k] = x + 1j * rng.normal(size=x.shape) if cplx else x
    listing = L.load().cc_plan_describe_ops_dry(O_, V_, 1, 1 if cplx else 0, text.encode()).decode()
    assert not listing.startswith("error"), listing
    got = execute(listing, inputs, O_, V_, cplx, 1)
    want = _literal(text, inputs, cplx)
    ref = triples(lambda k: want[k].ravel(), O_, V_)
    r3 = triples(got, O_, V_)
    assert np.abs(r3 - ref).max() < 1e-12 * np.abs(ref).max()
