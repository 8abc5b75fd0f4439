"""A step of a small system captured into the caller's own graph, replayed
after the plan was tuned: the merged launches' tables live as long as the plan."""
import numpy as np
import pytest

from ccinputs.synth import make_system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("o,v", [(4, 20), (7, 45)])
def test_captured_step_outlives_autotune(o, v):
    from paper_2409_06759_amd import engine as E
    print(f"captured step o={o} v={v}", flush=True)
    rng = np.random.default_rng(o + v)
    a1 = torch.from_numpy(rng.normal(size=(o, v)) * 0.03).cuda()
    t2 = rng.normal(size=(o, o, v, v)) * 0.03
    t2 = t2 - t2.transpose(1, 0, 2, 3)
    a2 = torch.from_numpy(t2 - t2.transpose(0, 1, 3, 2)).cuda()
    with E.Context(0) as ctx:
        d = E.DeviceSystem(make_system(o, v, 5))
        with E.Plan(ctx, d, E.CCSD) as p:
            t1, t2 = a1.clone(), a2.clone()
            want = []
            for _ in range(3):
                p.step(t1, t2, 0.1)
                torch.cuda.synchronize()
                want.append((t1.clone(), t2.clone()))
            t1.copy_(a1)
            t2.copy_(a2)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=ctx.stream):
                p.step(t1, t2, 0.1)
            p.autotune(t1, t2, reps=1)
            filler = [torch.full((1 << 16,), float("nan"), device="cuda") for _ in range(8)]
            for w1, w2 in want:
                g.replay()
                torch.cuda.synchronize()
                assert torch.equal(t1, w1) and torch.equal(t2, w2)
                t1.add_(0.0)  # eager work between the replays
                p.residual(t1, t2)
            del filler, g
