"""Work that programs have this engine do, as timed cases.

Each case goes through the public front end (``paper_2409_06759_amd.engine``)
with what such a program keeps between calls: the system resident in device
memory and the plan, batch or network made from it.  Plans run on the
library's own tile choice; none is tuned by timing first.

``listed()`` gives the fixed cases, ``draw(rng)`` more of the same ranges,
``prepare``/``run`` one pass, ``work`` the bytes and operations that a pass
cannot do without, and ``exact`` the same results in plain 64-bit PyTorch.
"""
import math

import numpy as np
import torch

from paper_2409_06759_amd import engine as E
from paper_2409_06759_amd.codegen.emit import op_list

DEV = "cuda"
SIGMA = 0.01
MLP_HIDDEN = 128


def listed():
    return [
        # ten bare Jacobi iterations of spin-orbital CCD on a small system, the whole solve
        # with its plan: the call that scans over geometries or parameters make by the thousand
        {"name": "solve_ccd_o8_v24", "kind": "solve", "o": 8, "v": 24, "method": "ccd", "iters": 10},
        # one residual of the smallest system: launches and latency
        {"name": "residual_o4_v20", "kind": "residual", "o": 4, "v": 20, "prec": "f64", "packed": False,
         "complex": False},
        # odd sizes in the range of the small systems: ragged tiles everywhere
        {"name": "residual_o13_v61", "kind": "residual", "o": 13, "v": 61, "prec": "f64", "packed": False,
         "complex": False},
        # an ordinary system of the training range, ladder over packed pairs
        {"name": "residual_o20_v100_packed", "kind": "residual", "o": 20, "v": 100, "prec": "f64", "packed": True,
         "complex": False},
        # the benchmark's system, dense pairs
        {"name": "residual_o32_v160", "kind": "residual", "o": 32, "v": 160, "prec": "f64", "packed": False,
         "complex": False},
        # the same over packed pairs
        {"name": "residual_o32_v160_packed", "kind": "residual", "o": 32, "v": 160, "prec": "f64", "packed": True,
         "complex": False},
        # the reduced-precision phase of a mixed-precision solve (split bf16 contractions)
        {"name": "residual_o24_v120_bf16x3", "kind": "residual", "o": 24, "v": 120, "prec": "bf16x3",
         "packed": False, "complex": False},
        # complex Hermitian integrals (relativistic Hamiltonians)
        {"name": "residual_o16_v80_complex", "kind": "residual", "o": 16, "v": 80, "prec": "f64", "packed": False,
         "complex": True},
        # one Jacobi step of 64 uneven systems iterated together
        {"name": "batch_step_64", "kind": "batch", "systems": 64, "o_min": 4, "o_max": 16, "v_min": 20, "v_max": 60,
         "shapes": 1000},
        # starting amplitudes from the trained kind of network for the benchmark's system
        {"name": "guess_o32_v160", "kind": "guess", "o": 32, "v": 160},
        # one pass of Adam over a training set, minibatches of the default size
        {"name": "train_1m", "kind": "train", "samples": 1 << 20, "batch": 65536},
        # CCSDT residual from the generated contraction list
        {"name": "ccsdt_o10_v40", "kind": "ccsdt", "o": 10, "v": 40},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "residual", "residual", "residual", "residual", "batch", "guess", "train", "ccsdt"])
    if kind == "solve":
        return {"kind": kind, "o": rng.randint(4, 12), "v": rng.randint(16, 48), "method": rng.choice(["ccd", "ccsd"]),
                "iters": rng.randint(5, 20)}
    if kind == "residual":
        form = rng.choice(["f64", "f64", "packed", "packed", "bf16x3", "f32", "complex"])
        o, v = _log_int(rng, 3, 30), _log_int(rng, 16, 150)
        if form == "complex":
            o, v = min(o, 20), min(v, 90)
        return {"kind": kind, "o": o, "v": v, "prec": form if form in ("bf16x3", "f32") else "f64",
                "packed": form == "packed", "complex": form == "complex"}
    if kind == "batch":
        v0 = rng.randint(16, 36)
        return {"kind": kind, "systems": rng.randint(8, 63), "o_min": rng.randint(3, 6), "o_max": rng.randint(8, 16),
                "v_min": v0, "v_max": v0 + rng.randint(4, 24), "shapes": rng.randint(1, 1 << 20)}
    if kind == "guess":
        return {"kind": kind, "o": rng.randint(8, 30), "v": rng.randint(40, 150)}
    if kind == "train":
        return {"kind": kind, "samples": _log_int(rng, 1 << 14, 1 << 20), "batch": rng.choice([65536, 65536, 16384, 8192])}
    return {"kind": kind, "o": rng.randint(4, 9), "v": rng.randint(12, 38)}


# ------------------------------------------------------------------ inputs --
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(shape, g, cplx):
    if not cplx:
        return torch.randn(shape, generator=g, dtype=torch.float64, device=DEV)
    return torch.complex(*(torch.randn(shape, generator=g, dtype=torch.float64, device=DEV) / math.sqrt(2)
                           for _ in range(2)))


def _pairs(n):
    """(n*n) index of the unordered pair and its sign (0 on the diagonal)."""
    p = torch.arange(n, device=DEV)
    lo, hi = torch.minimum(p[:, None], p[None, :]), torch.maximum(p[:, None], p[None, :])
    idx = (lo * n - lo * (lo + 1) // 2 + hi - lo - 1).clamp_(min=0, max=max(n * (n - 1) // 2 - 1, 0))
    sign = torch.sign(p[None, :] - p[:, None]).to(torch.float64)
    return idx.reshape(-1), sign.reshape(-1)


def _hermitian(n, g, cplx):
    """Hermitian with independent N(0, sigma^2) elements on and above the diagonal."""
    x = SIGMA * _randn((n, n), g, cplx)
    up = torch.triu(x, 1)
    d = torch.diagonal(x).real if cplx else torch.diagonal(x)
    x = up + up.conj().T if cplx else up + up.T
    x.diagonal().copy_(d)
    return x


def _spread(m, rows, cols):
    """Pair matrix -> block over ordered indices; rows/cols are (index, sign) or None (all used once)."""
    if rows is not None:
        m = m[rows[0]] * rows[1][:, None]
    if cols is not None:
        m = m[:, cols[0]]
        m *= cols[1][None, :]
    return m


def _system(o, v, seed, cplx=False):
    """Fock and antisymmetrised integral blocks: N(0, 0.01^2) canonical elements, orbital
    energies uniform in [-2, -0.5] and [0.5, 3], diagonal Fock operator."""
    g = _generator(seed)
    dt = torch.complex128 if cplx else torch.float64
    eo = (-2.0 + 1.5 * torch.rand(o, generator=g, dtype=torch.float64, device=DEV)).sort().values
    ev = (0.5 + 2.5 * torch.rand(v, generator=g, dtype=torch.float64, device=DEV)).sort().values
    po, pv = _pairs(o), _pairs(v)
    no, nv, nov = max(o * (o - 1) // 2, 1), max(v * (v - 1) // 2, 1), o * v
    t = {"f_oo": torch.diag(eo).to(dt), "f_ov": torch.zeros((o, v), dtype=dt, device=DEV),
         "f_vv": torch.diag(ev).to(dt)}
    t["oooo"] = _spread(_hermitian(no, g, cplx), po, po).reshape(o, o, o, o)
    t["ooov"] = _spread(SIGMA * _randn((no, nov), g, cplx), po, None).reshape(o, o, o, v)
    t["oovv"] = _spread(SIGMA * _randn((no, nv), g, cplx), po, pv).reshape(o, o, v, v)
    # <ia||bj> = -<ia||jb>, Hermitian in (ia), (jb)
    t["ovvo"] = (-_hermitian(nov, g, cplx)).reshape(o, v, o, v).transpose(2, 3).contiguous()
    t["ovvv"] = _spread(SIGMA * _randn((nov, nv), g, cplx), None, pv).reshape(o, v, v, v)
    t["vvvv"] = _spread(_hermitian(nv, g, cplx), pv, pv).reshape(v, v, v, v)
    return t, eo, ev


def _denominators(eo, ev):
    d1 = eo[:, None] - ev[None, :]
    return d1, d1[:, None, :, None] + d1[None, :, None, :]


def _amplitudes(t, eo, ev, seed):
    """Amplitudes as they are some steps into a solve: t2 near the MP2 ones, a small t1."""
    cplx = t["oovv"].is_complex()
    g = _generator(seed + 1)
    d2 = _denominators(eo, ev)[1]
    t2 = t["oovv"].conj().resolve_conj() * (0.8 / d2)
    t1 = 1e-3 * _randn(t["f_ov"].shape, g, cplx)
    return t1, t2.contiguous()


def _antisymmetric_t3(o, v, seed):
    g = _generator(seed + 2)
    x = 1e-4 * torch.randn((o, o, o, v, v, v), generator=g, dtype=torch.float64, device=DEV)
    for a in (0, 3):
        x = x - x.transpose(a, a + 1)
        x = x - x.transpose(a, a + 2) - x.transpose(a + 1, a + 2)
    return x.contiguous()


def _batch_shapes(case):
    r = np.random.Generator(np.random.PCG64(case["shapes"]))
    os_ = r.integers(case["o_min"], case["o_max"] + 1, size=case["systems"])
    vs_ = r.integers(case["v_min"], case["v_max"] + 1, size=case["systems"])
    return [(int(a), int(b)) for a, b in zip(os_, vs_)]


def _network(seed):
    """Parameters (He-normal, small biases) in the library's order."""
    r = np.random.default_rng(seed)
    h = MLP_HIDDEN
    parts = [r.normal(size=(h, 3)) * math.sqrt(2 / 3), 0.05 * r.normal(size=h), r.normal(size=(h, h)) * math.sqrt(2 / h),
             0.05 * r.normal(size=h), r.normal(size=(1, h)) * math.sqrt(2 / h), np.zeros(1)]
    return torch.from_numpy(np.concatenate([p.ravel() for p in parts])).to(DEV)


GUESS_STATS = {"sx": SIGMA, "mD": -6.0, "sD": 1.2, "me": -0.1, "se": 0.05, "st": 0.002}


def _training_rows(n, seed):
    """Standardised features of n amplitudes and their targets (shuffled already)."""
    g = _generator(seed)
    z = torch.randn((n, 3), generator=g, dtype=torch.float64, device=DEV)
    y = z[:, 0] / (1.0 - 0.2 * z[:, 1]).clamp_(min=0.3) * (1.0 + 0.1 * z[:, 2])
    y = y + 0.15 * torch.randn(n, generator=g, dtype=torch.float64, device=DEV)
    return z, y


# ---------------------------------------------------------------- one pass --
class _State:
    """What the program keeps; plans and batches go with it."""

    def __init__(self, case):
        self.case = case
        self.ctx = E.Context(0)
        self.own = []

    def __del__(self):
        for x in self.own:
            x.close()
        self.ctx.close()


def prepare(case, seed):
    s = _State(case)
    kind = case["kind"]
    if kind == "train":
        s.z, s.y = _training_rows(case["samples"], seed)
        s.net = E.MLP(s.ctx, _network(seed), GUESS_STATS)
        return s
    if kind == "batch":
        shapes = _batch_shapes(case)
        # one buffer for all amplitudes, each array on a 16-byte boundary
        sizes = [(o * v + o * v % 2, o * o * v * v + o * o * v * v % 2) for o, v in shapes]
        s.flat = torch.zeros(sum(a + b for a, b in sizes), dtype=torch.float64, device=DEV)
        at, amps, systems = 0, [], []
        for (o, v), (n1, n2) in zip(shapes, sizes):
            t, eo, ev = _system(o, v, seed * 1009 + at)
            t1, t2 = _amplitudes(t, eo, ev, seed * 1009 + at)
            a1 = s.flat[at:at + o * v].view(o, v)
            a2 = s.flat[at + n1:at + n1 + o * o * v * v].view(o, o, v, v)
            a1.copy_(t1)
            a2.copy_(t2)
            at += n1 + n2
            amps.append((a1, a2))
            systems.append(E.DeviceSystem.from_tensors(o, v, t))
        s.batch = E.Batch(s.ctx, systems, E.CCSD, amps=amps)
        s.own.append(s.batch)
        return s
    o, v = case["o"], case["v"]
    t, eo, ev = _system(o, v, seed, case.get("complex", False))
    s.sys = E.DeviceSystem.from_tensors(o, v, t)
    if kind == "solve":
        s.method = E.METHODS[case["method"]]
        s.t1, s.t2 = E.zeros_amps(s.sys, s.method)
    elif kind == "guess":
        s.net = E.MLP(s.ctx, _network(seed), GUESS_STATS)
        s.t1, s.t2 = E.zeros_amps(s.sys, E.CCSD)
    else:
        s.t1, s.t2 = _amplitudes(t, eo, ev, seed)
        if kind == "ccsdt":
            s.t3 = _antisymmetric_t3(o, v, seed)
            s.r3 = torch.empty_like(s.t3)
            s.plan = E.Plan(s.ctx, s.sys, E.CCSD, ops=op_list("ccsdt", o, v))
            s.plan.set_triples(s.t3, s.r3)
        else:
            s.plan = E.Plan(s.ctx, s.sys, E.CCSD, prec=E.PRECS[case["prec"]], packed=case["packed"])
        s.own.append(s.plan)
    return s


def run(s):
    kind = s.case["kind"]
    if kind == "solve":
        s.t2.zero_()
        if s.t1 is not None:
            s.t1.zero_()
        r = E.iterate(s.ctx, s.sys, s.method, s.t1, s.t2, tol=1e-13, max_iter=s.case["iters"])
        return {"t1": s.t1, "t2": s.t2, "energies": np.array(r["hist_e"])}
    if kind == "residual":
        r1, r2, rn = s.plan.residual(s.t1, s.t2)
        return {"r1": r1, "r2": r2, "norm": rn}
    if kind == "batch":
        s.batch.step(dressed=True)
        # later work of the program on its own stream waits for the step
        torch.cuda.current_stream().wait_stream(s.ctx.stream)
        return s.flat
    if kind == "guess":
        s.net.guess(s.sys, s.t1, s.t2)
        return {"t1": s.t1, "t2": s.t2}
    if kind == "train":
        losses = s.net.train(s.z, s.y, epochs=1, batch=s.case["batch"])
        return {"params": s.net.params, "loss": losses[0]}
    r1, r2, rn = s.plan.residual(s.t1, s.t2)
    return {"r1": r1, "r2": r2, "r3": s.r3, "norm": rn}


# -------------------------------------------------------------------- work --
def _ccsd_flops(o, v, packed, ccd=False):
    """Multiply-adds (x2) of the factorised equations, the ladders over all ordered
    pairs or over canonical ones."""
    no, nv = o * (o - 1) / 2, v * (v - 1) / 2
    big = 2 * 2 * o ** 3 * v ** 3                                     # both ring terms
    big += 2 * o ** 4 * v * v                                         # W_mnij
    if packed:
        big += 2 * no * nv * nv + 2 * no * no * nv + (0 if ccd else 2 * no * nv * o * v)
    else:
        big += 2 * o * o * v ** 4 + 2 * o ** 4 * v * v + (0 if ccd else 2 * o ** 3 * v ** 3)
    small = 2 * (2 * o ** 3 * v * v + 2 * o * o * v ** 3)             # F terms and their products with t2
    if not ccd:
        small += 2 * (4 * o * o * v ** 3 + 6 * o ** 3 * v * v)        # t1 contractions
    return big + small


def _ccsd_bytes(o, v, size, ccd=False):
    ints = o ** 4 + 2 * o * o * v * v + v ** 4 + (0 if ccd else o ** 3 * v + o * v ** 3)
    return size * (ints + 2 * (o * o * v * v + o * v))


def work(case):
    kind = case["kind"]
    if kind == "solve":
        ccd = case["method"] == "ccd"
        n = case["iters"]
        return {"bytes": n * _ccsd_bytes(case["o"], case["v"], 8, ccd),
                "flops": n * _ccsd_flops(case["o"], case["v"], False, ccd)}
    if kind == "residual":
        size, fac = (16, 4) if case["complex"] else (8, 1)
        return {"bytes": _ccsd_bytes(case["o"], case["v"], size),
                "flops": fac * _ccsd_flops(case["o"], case["v"], case["packed"])}
    if kind == "batch":
        sh = _batch_shapes(case)
        return {"bytes": sum(_ccsd_bytes(o, v, 8) for o, v in sh), "flops": sum(_ccsd_flops(o, v, True) for o, v in sh)}
    if kind == "guess":
        o, v = case["o"], case["v"]
        n = (o * (o - 1) // 2) * (v * (v - 1) // 2)
        return {"bytes": 8 * (n + o * o * v * v), "flops": n * 2 * 2 * (3 * MLP_HIDDEN + MLP_HIDDEN ** 2 + MLP_HIDDEN)}
    if kind == "train":
        n = case["samples"]
        return {"bytes": n * 32, "flops": n * 3 * 2 * 2 * (3 * MLP_HIDDEN + MLP_HIDDEN ** 2 + MLP_HIDDEN)}
    o, v = case["o"], case["v"]
    n3 = o ** 3 * v ** 3
    return {"bytes": _ccsd_bytes(o, v, 8) + 16 * n3,
            "flops": _ccsd_flops(o, v, False) + 2 * n3 * (v * v + o * o + 2 * o * v + 2 * v + 2 * o)}


# ------------------------------------------------------------------- exact --
def _ccsd_residual(t, t1, t2, dressed=False):
    """Spin-orbital CCSD (t1 None: CCD) residual in the Stanton-Gauss intermediates, complex
    Hermitian integrals allowed; also the diagonals of the dressed one-body operators."""
    es = torch.einsum
    fo, fov, fv = t["f_oo"], t["f_ov"], t["f_vv"]
    oooo, ooov, oovv, ovvo, ovvv, vvvv = (t[k] for k in ("oooo", "ooov", "oovv", "ovvo", "ovvv", "vvvv"))
    ccsd = t1 is not None
    if not ccsd:
        t1 = torch.zeros_like(fov)
    x = es("ia,jb->ijab", t1, t1)
    x = x - x.transpose(2, 3)
    tau, taut = t2 + x, t2 + 0.5 * x
    fme = fov + es("nf,mnef->me", t1, oovv)
    fae = fv - 0.5 * es("ma,me->ae", t1, fov) + es("mf,mafe->ae", t1, ovvv) - 0.5 * es("mnaf,mnef->ae", taut, oovv)
    fmi = fo + 0.5 * es("me,ie->mi", fov, t1) + es("mnie,ne->mi", ooov, t1) + 0.5 * es("mnef,inef->mi", oovv, taut)
    w = es("mnie,je->mnij", ooov, t1)
    wmnij = oooo + w - w.transpose(2, 3) + 0.5 * es("mnef,ijef->mnij", oovv, tau)
    wmbej = (ovvo + es("mbef,jf->mbej", ovvv, t1) + es("mnje,nb->mbej", ooov, t1)
             - es("mnef,jnfb->mbej", oovv, 0.5 * t2 + es("jf,nb->jnfb", t1, t1)))
    ff = fae - 0.5 * es("mb,me->be", t1, fme)
    gg = fmi + 0.5 * es("me,je->mj", fme, t1)
    r2 = oovv.conj() + 0.5 * es("mnij,mnab->ijab", wmnij, tau) + 0.5 * es("ijef,abef->ijab", tau, vvvv)
    y = es("ijae,be->ijab", t2, ff) - es("ma,ijmb->ijab", t1, ooov.conj())
    y = y - 0.5 * es("mb,ijam->ijab", t1, -es("ijef,maef->ijam", tau, ovvv))
    r2 = r2 + y - y.transpose(2, 3)
    y = -es("imab,mj->ijab", t2, gg) - es("ie,jeab->ijab", t1, ovvv.conj())
    r2 = r2 + y - y.transpose(0, 1)
    y = es("imae,mbej->ijab", t2, wmbej) - es("imbj,ma->ijab", es("ie,mbej->imbj", t1, ovvo), t1)
    y = y - y.transpose(0, 1)
    r2 = r2 + y - y.transpose(2, 3)
    r1 = None
    if ccsd:
        r1 = (fov.conj() + es("ie,ae->ia", t1, fae) - es("mi,ma->ia", fmi, t1) + es("imae,me->ia", t2, fme)
              + es("nafi,nf->ia", ovvo, t1) - 0.5 * es("imef,maef->ia", t2, ovvv) - 0.5 * es("mnae,mnie->ia", t2, ooov))
    if dressed:
        return r1, r2, [torch.diagonal(q).real for q in (fmi, fae, gg, ff)]
    return r1, r2


def _norm(*rs):
    return float(torch.sqrt(sum((r.abs() ** 2).sum() for r in rs)))


def _mlp_weights(p):
    h = MLP_HIDDEN
    sizes = [3 * h, h, h * h, h, h, 1]
    w1, b1, w2, b2, w3, b3 = torch.split(p, sizes)
    return w1.view(h, 3), b1, w2.view(h, h), b2, w3, b3


def _mlp_odd(p, z):
    """f(z) = (g(z) - g(z with its first component negated)) / 2."""
    w1, b1, w2, b2, w3, _ = _mlp_weights(p)
    flip = torch.tensor([-1.0, 1.0, 1.0], dtype=torch.float64, device=z.device)
    g = [torch.relu(torch.relu(q @ w1.T + b1) @ w2.T + b2) @ w3 for q in (z, z * flip)]
    return 0.5 * (g[0] - g[1])


def exact(case, seed):
    kind = case["kind"]
    if kind == "ccsdt":
        return None
    if kind == "train":
        z, y = _training_rows(case["samples"], seed)
        p = _network(seed)
        m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
        for k, r0 in enumerate(range(0, case["samples"], case["batch"])):
            p.requires_grad_(True)
            loss = ((_mlp_odd(p, z[r0:r0 + case["batch"]]) - y[r0:r0 + case["batch"]]) ** 2).mean()
            grad, = torch.autograd.grad(loss, p)
            p = p.detach()
            losses.append(float(loss.detach()))
            m = 0.9 * m + 0.1 * grad
            v = 0.999 * v + 0.001 * grad * grad
            p = p - 1e-3 * (m / (1 - 0.9 ** (k + 1))) / (torch.sqrt(v / (1 - 0.999 ** (k + 1))) + 1e-8)
        return {"params": p, "loss": sum(losses) / len(losses)}
    if kind == "batch":
        shapes = _batch_shapes(case)
        parts, at = [], 0
        for o, v in shapes:
            t, eo, ev = _system(o, v, seed * 1009 + at)
            t1, t2 = _amplitudes(t, eo, ev, seed * 1009 + at)
            r1, r2, (fi, fa, gi, ga) = _ccsd_residual(t, t1, t2, dressed=True)
            t1 = t1 + r1 / (fi[:, None] - fa[None, :])
            d = gi[:, None, None, None] + gi[None, :, None, None] - ga[None, None, :, None] - ga[None, None, None, :]
            t2 = t2 + r2 / d
            for q in (t1, t2):
                q = q.reshape(-1)
                parts.append(torch.cat([q, q.new_zeros(q.numel() % 2)]))
                at += parts[-1].numel()
        return torch.cat(parts)
    o, v = case["o"], case["v"]
    t, eo, ev = _system(o, v, seed, case.get("complex", False))
    if kind == "solve":
        d1, d2 = _denominators(eo, ev)
        ccsd = case["method"] == "ccsd"
        t1, t2 = (torch.zeros_like(t["f_ov"]) if ccsd else None), torch.zeros_like(t["oovv"])
        es = []
        for _ in range(case["iters"]):
            x = torch.einsum("ia,jb->ijab", t1, t1) if ccsd else None
            tau = t2 + x - x.transpose(2, 3) if ccsd else t2
            es.append(float(0.25 * (t["oovv"] * tau).sum()))
            r1, r2 = _ccsd_residual(t, t1, t2)
            t2 = t2 + r2 / d2
            t1 = t1 + r1 / d1 if ccsd else None
        return {"t1": t1, "t2": t2, "energies": np.array(es)}
    if kind == "guess":
        ij, ab = torch.triu_indices(o, o, 1, device=DEV), torch.triu_indices(v, v, 1, device=DEV)
        x = t["oovv"][ij[0], ij[1]][:, ab[0], ab[1]]
        d = (eo[ij[0]] + eo[ij[1]])[:, None] - (ev[ab[0]] + ev[ab[1]])[None, :]
        e = (x * x / d).sum(1, keepdim=True).expand_as(x)
        st, p = GUESS_STATS, _network(seed)
        t2 = torch.zeros((o, o, v, v), dtype=torch.float64, device=DEV)
        for k in range(x.shape[0]):
            z = torch.stack([x[k] / st["sx"], (d[k] - st["mD"]) / st["sD"], (e[k] - st["me"]) / st["se"]], 1)
            f = st["st"] * _mlp_odd(p, z)
            i, j = ij[0][k], ij[1][k]
            t2[i, j, ab[0], ab[1]] = f
            t2[j, i, ab[1], ab[0]] = f
            t2[i, j, ab[1], ab[0]] = -f
            t2[j, i, ab[0], ab[1]] = -f
        return {"t1": torch.zeros((o, v), dtype=torch.float64, device=DEV), "t2": t2}
    t1, t2 = _amplitudes(t, eo, ev, seed)
    r1, r2 = _ccsd_residual(t, t1, t2)
    return {"r1": r1, "r2": r2, "norm": _norm(r1, r2)}
