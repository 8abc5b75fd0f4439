"""The fused FP32 training passes at the edges of their row blocks and
slices, against the FP64 NumPy network."""
import numpy as np
import pytest

from oracle import mlp as ref

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

STATS = {"sx": 1.0, "mD": 0.0, "sD": 1.0, "me": 0.0, "se": 1.0, "st": 1.0}


@pytest.fixture(scope="module")
def E():
    from paper_2409_06759_amd import engine
    return engine


@pytest.fixture(scope="module")
def ctx(E):
    c = E.Context(0)
    yield c
    c.close()


def _data(n, seed):
    rng = np.random.default_rng(seed)
    return ref.init_params(5), rng.normal(size=(n, 3)), rng.normal(size=n) * 0.5


# samples: less than one 16-row block, the two branches in one block, whole
# and ragged 64-row blocks, one and two slices (rows 2n = 512, 514), slices of
# 272 and 288 rows (no whole number of 64-row blocks), the largest minibatch
# of equal slices, one whose slices do not fit (layer by layer), two vector
# slices per weight slice
@pytest.mark.parametrize("n", [1, 5, 8, 31, 32, 33, 256, 257, 1001, 4111, 32768, 33001, 65536])
def test_fused_gradient_matches_oracle(E, ctx, n):
    print(f"fused gradient n={n}", flush=True)
    p, z, y = _data(n, 3 + n)
    net = E.MLP(ctx, torch.from_numpy(ref.flatten(p)).cuda(), STATS, E.F32)
    loss, g = net.loss_grad(torch.from_numpy(z).cuda(), torch.from_numpy(y).cuda())
    l_ref, g_ref = ref.loss_and_grad(p, z, y)
    g_ref = ref.flatten(g_ref)
    assert abs(loss - l_ref) < 2e-5 * max(1.0, l_ref)
    assert np.abs(g.cpu().numpy() - g_ref).max() < 2e-5 * max(1.0, np.abs(g_ref).max())


@pytest.mark.parametrize("n,batch,ordered", [(3000, 1024, True), (2500, 1250, False)])
def test_fused_minibatches_in_the_order_given(E, ctx, n, batch, ordered):
    """Adam's first moments after one epoch at a negligible learning rate: the
    running mean of the minibatch gradients, a ragged last minibatch included."""
    print(f"fused minibatches n={n} batch={batch} ordered={ordered}", flush=True)
    p, z, y = _data(n, 11)
    order = np.random.default_rng(1).permutation(n)[:n - 7] if ordered else np.arange(n)
    net = E.MLP(ctx, torch.from_numpy(ref.flatten(p)).cuda(), STATS, E.F32)
    loss = net.train(torch.from_numpy(z).cuda(), torch.from_numpy(y).cuda(), batch=batch, lr=1e-14,
                     order=torch.from_numpy(order).cuda() if ordered else None)
    m, losses = 0.0, []
    for a in range(0, order.size, batch):
        rows = order[a:a + batch]
        lv, g = ref.loss_and_grad(p, z[rows], y[rows])
        m = 0.9 * m + 0.1 * ref.flatten(g)
        losses.append(lv)
    assert abs(loss[0] - np.mean(losses)) < 2e-5
    assert np.abs(net.m.cpu().numpy() - m).max() < 2e-5 * max(1.0, np.abs(m).max())


# pairs i < j and a < b at the edges of the 32-wide tiles, of the 256-thread
# strides of the pair sums, and at the smallest sizes
@pytest.mark.parametrize("o,v", [(2, 2), (2, 3), (3, 23), (2, 31), (5, 32), (3, 33), (2, 64), (4, 65), (7, 100)])
def test_features_and_guess_at_tile_edges(E, ctx, o, v):
    from ccinputs.synth import make_system
    print(f"features and guess o={o} v={v}", flush=True)
    s = make_system(o, v, 50 + v)
    d = E.DeviceSystem(s)
    oovv = d.t["oovv"].cpu().numpy()
    eo, ev = np.diag(d.t["f_oo"].cpu().numpy()).real, np.diag(d.t["f_vv"].cpu().numpy()).real
    io, jo = np.triu_indices(o, 1)
    av, bv = np.triu_indices(v, 1)
    x = oovv[io, jo][:, av, bv]
    D = (eo[io] + eo[jo])[:, None] - (ev[av] + ev[bv])[None, :]
    e = (x * x / D).sum(1)
    raw = E.MLP.raw_features(ctx, d)
    z = raw.cpu().numpy().reshape(len(io), len(av), 3)
    assert np.array_equal(z[..., 0], x)
    assert np.allclose(z[..., 1], D, rtol=1e-15, atol=0)
    # at most nab rounding errors of terms of one sign
    assert np.all(np.abs(z[..., 2] - e[:, None]) <= (len(av) + 4) * np.finfo(np.float64).eps * np.abs(e)[:, None])
    net = E.MLP(ctx, E.MLP.init_params(3), STATS | {"st": 0.37}, E.F32)
    zs, _ = net.standardise(raw)
    f = net.forward(zs).cpu().numpy().reshape(len(io), len(av))
    want = np.zeros((o, o, v, v))
    for p, (i, j) in enumerate(zip(io, jo)):
        m = np.zeros((v, v))
        m[av, bv] = 0.37 * f[p]
        want[i, j] = m - m.T
        want[j, i] = m.T - m
    t1, t2 = E.zeros_amps(d, E.CCSD)
    t1.fill_(1.0)
    t2.fill_(1.0)
    net.guess(d, t1, t2)
    assert np.array_equal(t2.cpu().numpy(), want) and torch.all(t1 == 0)
    assert np.array_equal(E.MLP.targets(ctx, o, v, t2).cpu().numpy(), want[io, jo][:, av, bv].ravel())
