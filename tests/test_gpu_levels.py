"""Small systems run an iteration as merged launches, one per dependency level;
profiling runs the same steps one by one.  Both run the same bodies on the same
tiles and split-K factors, so they may differ only in how a multiply and an add
were contracted: a few units in the last place of the largest term."""
import numpy as np
import pytest

from ccinputs.synth import make_system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = 1e-13  # times the largest element


@pytest.fixture(scope="module")
def E():
    from paper_2409_06759_amd import engine
    return engine


@pytest.fixture(scope="module")
def ctx(E):
    c = E.Context(0)
    yield c
    c.close()


def _amps(o, v, seed):
    rng = np.random.default_rng(seed)
    t1 = rng.normal(size=(o, v)) * 0.03
    t2 = rng.normal(size=(o, o, v, v)) * 0.03
    t2 = t2 - t2.transpose(1, 0, 2, 3)
    t2 = t2 - t2.transpose(0, 1, 3, 2)
    return torch.from_numpy(t1).cuda(), torch.from_numpy(t2).cuda()


def _close(a, b):
    scale = max(float(b.abs().max()), 1e-300)
    assert float((a - b).abs().max()) <= TOL * scale


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("method", ["ccd", "ccsd"])
@pytest.mark.parametrize("o,v", [(1, 1), (1, 5), (2, 3), (3, 33), (4, 20), (9, 31), (16, 64), (6, 140)])
def test_levels_equal_single_steps(E, ctx, o, v, method, packed):
    print(f"levels {method} o={o} v={v} packed={packed}", flush=True)
    d = E.DeviceSystem(make_system(o, v, 7 + v))
    m = E.METHODS[method]
    with E.Plan(ctx, d, m, packed=packed) as p:
        for seed in (1, 2):  # new buffers on the second pass
            t1, t2 = _amps(o, v, seed)
            t1 = t1 if m == E.METHODS["ccsd"] else None
            r1, r2, n = p.residual(t1, t2)
            u1, u2 = (None if t1 is None else t1.clone()), t2.clone()
            p.step(u1, u2, 0.1)
            su = p.scalars()
            p.profile(True)
            q1, q2, nq = p.residual(t1, t2)
            w1, w2 = (None if t1 is None else t1.clone()), t2.clone()
            p.step(w1, w2, 0.1)
            sw = p.scalars()
            p.profile(False)
            _close(r2, q2)
            _close(u2, w2)
            if t1 is not None:
                _close(r1, q1)
                _close(u1, w1)
            assert abs(n - nq) <= TOL * max(nq, 1e-300)
            for x, y in zip(su, sw):
                assert abs(x - y) <= TOL * max(abs(y), 1.0)
