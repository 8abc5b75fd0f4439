"""The triples kernel (antisymmetriser, update, norm) at the edges of its
8-wide tiles, for any Y3, against NumPy."""
import itertools

import numpy as np
import pytest

from ccinputs.synth import make_system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def E():
    from paper_2409_06759_amd import engine
    return engine


@pytest.fixture(scope="module")
def ctx(E):
    c = E.Context(0)
    yield c
    c.close()


def _antisymmetriser(y):
    out = np.zeros_like(y)
    for ph in itertools.permutations(range(3)):
        for pp in itertools.permutations(range(3)):
            sg = round(np.linalg.det(np.eye(3)[list(ph)]) * np.linalg.det(np.eye(3)[list(pp)]))
            out += sg * np.transpose(y, list(ph) + [3 + q for q in pp])
    return out


@pytest.mark.parametrize("o,v,cplx", [(3, 7, False), (3, 8, False), (4, 9, False), (5, 16, False), (3, 17, True),
                                      (2, 4, False), (3, 2, False), (1, 9, False)])
def test_triples_antisymmetriser_update_and_norm(E, ctx, o, v, cplx):
    print(f"triples o={o} v={v} complex={cplx}", flush=True)
    s = make_system(o, v, 3, is_complex=cplx)
    d = E.DeviceSystem(s)
    rng = np.random.default_rng(o * 100 + v)
    y = rng.normal(size=(o,) * 3 + (v,) * 3)
    if cplx:
        y = y + 1j * rng.normal(size=y.shape)
    t1, t2 = E.zeros_amps(d, E.CCSD)
    t3 = torch.from_numpy(y).cuda()
    r3 = torch.full_like(t3, float("nan"))
    with E.Plan(ctx, d, E.CCSD, ops="op zero R1 ia 1.0 fov ia - -\nop copy Y3 ijkabc 1.0 t3 ijkabc - -\n") as p:
        p.set_triples(t3, r3)
        _, _, rn = p.residual(t1, t2)
        ref = _antisymmetriser(y)
        eps = 36 * np.finfo(float).eps * np.abs(y).max() * 6
        assert np.abs(r3.cpu().numpy() - ref).max() <= eps
        assert abs(rn - np.linalg.norm(ref)) <= 1e-13 * max(1.0, np.linalg.norm(ref))
        assert np.array_equal(t3.cpu().numpy(), y)  # a residual leaves the amplitudes
        p.step(t1, t2)
        torch.cuda.synchronize()
    eo, ev = np.diag(s.f_oo).real, np.diag(s.f_vv).real
    D = eo[:, None, None] + eo[None, :, None] + eo[None, None, :]
    D = D[:, :, :, None, None, None] - (ev[:, None, None] + ev[None, :, None] + ev[None, None, :])
    want = y + ref / D
    i, j, k, a, b, c = np.indices(y.shape)
    want[(i == j) | (j == k) | (i == k) | (a == b) | (b == c) | (a == c)] = 0.0
    got = t3.cpu().numpy()
    assert np.abs(got - want).max() <= eps + 4 * np.finfo(float).eps * np.abs(y).max()
