"""Autotuned choices kept per shape: plans that may use different tiles do not
share them, a kept choice is the one that was timed, and a file of choices from
a library with other configurations is no harm."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from ccinputs.synth import make_system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _amps(o, v):
    rng = np.random.default_rng(o + v)
    t2 = rng.normal(size=(o, o, v, v)) * 0.03
    t2 = t2 - t2.transpose(1, 0, 2, 3)
    return (torch.from_numpy(rng.normal(size=(o, v)) * 0.03).cuda(),
            torch.from_numpy(t2 - t2.transpose(0, 1, 3, 2)).cuda())


def _choices(plan):
    """(shape and operand forms, split, tile) of every GEMM of the iteration."""
    out = []
    for line in plan.describe().split("# iteration\n")[1].splitlines():
        if line.startswith("GEMM "):
            kv = dict(re.findall(r"(\w+)=([^ ]+)", line))
            out.append((tuple(kv[k] for k in ("M", "N", "K", "sak", "sbk")), int(kv["split"]), kv["tile"]))
    return out


# sizes of no other test: the cache lives as long as the process
@pytest.mark.parametrize("first", ["merged", "single"])
def test_merged_and_single_plans_tune_apart(first, monkeypatch, tmp_path):
    from paper_2409_06759_amd import engine as E
    o, v = (9, 53) if first == "merged" else (9, 59)
    print(f"tuned apart o={o} v={v} first {first}", flush=True)
    path = tmp_path / "choices"
    monkeypatch.setenv("CC_AUTOTUNE_CACHE", str(path))
    t1, t2 = _amps(o, v)
    with E.Context(0) as ctx:
        d = E.DeviceSystem(make_system(o, v, 5))
        want = E.residual(ctx, d, E.CCSD, t1, t2)[1]
        keys, chosen = {}, {}
        for kind in (("merged", "single") if first == "merged" else ("single", "merged")):
            before = len(path.read_text().splitlines()) if path.exists() else 0
            for again in (False, True):
                # a plan of every contraction in one precision has no merged launches
                with E.Plan(ctx, d, E.CCSD, lowp_all=kind == "single") as p:
                    p.autotune(t1, t2, reps=1)
                    if again:
                        assert _choices(p) == chosen[kind]
                    chosen[kind] = _choices(p)
                    r2 = p.residual(t1, t2)[1]
                    assert float((r2 - want).abs().max()) <= 1e-12 * float(want.abs().max())
            keys[kind] = [line.split()[0].split("/")[0] for line in path.read_text().splitlines()[before:]]
        # each kind timed every one of its shapes (distinct in M, N, K and forms)
        for kind in keys:
            assert len(set(keys[kind])) == len(set(c[0] for c in chosen[kind])) > 10
        assert not set(keys["merged"]) & set(keys["single"])


FOREIGN = """
import sys
sys.path.insert(0, {root!r})
import numpy as np, torch
from ccinputs.synth import make_system
from paper_2409_06759_amd import engine as E
o, v = 5, 23
rng = np.random.default_rng(1)
t1, t2 = (torch.from_numpy(rng.normal(size=s) * 0.03).cuda() for s in ((o, v), (o, o, v, v)))
with E.Context(0) as ctx:
    d = E.DeviceSystem(make_system(o, v, 5))
    for lowp_all in (False, True):
        with E.Plan(ctx, d, E.CCSD, lowp_all=lowp_all) as p:
            a = p.residual(t1, t2)[1]
            p.autotune(t1, t2, reps=1)
            b = p.residual(t1, t2)[1]
            assert float((a - b).abs().max()) <= 1e-12 * float(a.abs().max())
print("foreign choices ok", flush=True)
"""


def test_choices_of_another_library(tmp_path):
    """Tiles this library does not have, and factors that no workspace holds."""
    path = tmp_path / "choices"
    dims = sorted({a * b for a in (1, 5, 23, 25, 115, 529) for b in (1, 5, 23, 25, 115, 529)})
    with open(path, "w") as f:
        for i, M in enumerate(dims):
            for j, N in enumerate(dims):
                for k, K in enumerate(dims):
                    for form in ("kk", "kn", "mk", "mn", "kkg", "kng", "mkg", "mng"):
                        f.write(f"0:{M}x{N}x{K}{form}{(' 999', '/100000 3')[(i + j + k) % 2]}\n")
    r = subprocess.run([sys.executable, "-c", FOREIGN.format(root=ROOT)], capture_output=True, text=True, timeout=100,
                       env={**os.environ, "CC_AUTOTUNE_CACHE": str(path)})
    assert r.returncode == 0 and "foreign choices ok" in r.stdout, r.stderr[-2000:]


@pytest.mark.parametrize("prec", ["F64", "F32", "BF16X3"])
def test_tuning_a_new_plan_only_reads_the_amplitudes(prec):
    """The tiles are timed on the intermediates at t: t stays as it is, and the
    residuals that follow, at t and at other amplitudes, are the untuned plan's
    (same products in other tiles: rounding of the plan's type)."""
    from paper_2409_06759_amd import engine as E
    o, v = 6, 31
    t1, t2 = _amps(o, v)
    k1, k2 = t1.clone(), t2.clone()
    rel = {"F64": 1e-12, "F32": 1e-4, "BF16X3": 1e-3}[prec]
    with E.Context(0) as ctx:
        d = E.DeviceSystem(make_system(o, v, 5))
        with E.Plan(ctx, d, E.CCSD, prec=getattr(E, prec)) as p, E.Plan(ctx, d, E.CCSD, prec=getattr(E, prec)) as q:
            p.autotune(t1, t2, reps=1)
            assert torch.equal(t1, k1) and torch.equal(t2, k2)
            for scale in (1.0, 0.5):
                got, want = p.residual(scale * t1, scale * t2)[1], q.residual(scale * t1, scale * t2)[1]
                assert float((got - want).abs().max()) <= rel * float(want.abs().max())


@pytest.mark.parametrize("packed,prec", [(False, "F64"), (True, "F64"), (True, "BF16X3")])
def test_tuning_at_unset_amplitudes_leaves_nothing_behind(packed, prec):
    """A solve may tune before its amplitudes are formed: what the workspace
    holds afterwards must not reach the iterations that follow."""
    from paper_2409_06759_amd import engine as E
    o, v = 7, 37
    t1, t2 = _amps(o, v)
    rel = {"F64": 1e-12, "BF16X3": 1e-3}[prec]
    with E.Context(0) as ctx:
        d = E.DeviceSystem(make_system(o, v, 5))
        with E.Plan(ctx, d, E.CCSD, prec=getattr(E, prec), packed=packed) as p, \
                E.Plan(ctx, d, E.CCSD, prec=getattr(E, prec), packed=packed) as q:
            p.autotune(torch.full_like(t1, float("nan")), torch.full_like(t2, float("nan")), reps=1)
            got, want = p.residual(t1, t2), q.residual(t1, t2)
            for a, b in zip(got[:2], want[:2]):
                assert float((a - b).abs().max()) <= rel * float(b.abs().max())
