"""Op lists that write the caller's amplitudes, through merged launches: cleared,
copied into, added to by an outer product and by a GEMM, against the same steps
run one by one.  The tables hold no pointer to the amplitudes, so the steps must
find them at the launch, and in new buffers at the next one."""
import numpy as np
import pytest

from ccinputs.synth import make_system

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BASE = "op r R1 ia 1.0 fov ia - -\nop x XP ijab 1.0 oovv ijab - -\n"
LISTS = {
    # zeroed (a fill), then an outer product; read by the ops behind it
    "fill_outer_t2": "op a t2 ijab 0.5 t1 ia fov jb\nop b Xr ijab 1.0 t2 ikac ovvo kbcj\n",
    # overwritten by a copy
    "copy_t2": "op a t2 ijab 0.25 oovv jiab - -\nop b XP ijab 0.5 t2 ijcd vvvv abcd\n",
    # written by a GEMM, directly and through a permutation
    "gemm_t2": "op a t2 ijab 0.5 oooo ijkl oovv klab\nop b Xij ijab 1.0 t2 ikab foo jk\n",
    "gemm_permuted_t2": "op a t2 ijab 0.5 t2 ikac ovvo kbcj\nop b XP ijab 0.5 t2 ijcd vvvv abcd\n",
    "gemm_split_t1": "op a t1 ia 0.5 t2 ijbc ovvv jabc\nop b R1 ia 1.0 t2 ijab t1 jb\n",
    "gemm_t1": "op a t1 ia 1.0 oovv ijab fov jb\nop b R1 ia 1.0 t2 ijab t1 jb\n",
    "gemm_t3": "op a t3 ijkabc 0.5 ooov ijla t2 lkbc\nop b Y3 ijkabc 1.0 t3 ijkdbc fvv ad\nop c XP ijab 0.5 t3 ijkabc fov kc\n",
}


@pytest.mark.parametrize("name", sorted(LISTS))
@pytest.mark.parametrize("o,v", [(3, 5), (4, 17)])
def test_lists_that_write_amplitudes(name, o, v):
    from paper_2409_06759_amd import engine as E
    print(f"amplitudes written: {name} o={o} v={v}", flush=True)
    rng = np.random.default_rng(o + v)
    triples = "t3" in LISTS[name]
    shapes = [(o, v), (o, o, v, v)] + ([(o,) * 3 + (v,) * 3] if triples else [])
    with E.Context(0) as ctx:
        d = E.DeviceSystem(make_system(o, v, 5))
        with E.Plan(ctx, d, E.CCSD, ops=BASE + LISTS[name]) as p:
            for _ in range(2):  # new buffers on the second pass
                amps = [torch.from_numpy(0.1 * rng.normal(size=s)).cuda() for s in shapes]
                got = []
                for single in (False, True):
                    p.profile(single)
                    for step in (False, True):
                        t = [x.clone() for x in amps]
                        r3 = torch.empty_like(t[2]) if triples else None
                        if triples:
                            p.set_triples(t[2], r3)
                        if step:
                            p.step(t[0], t[1], 0.1)
                            out = []
                        else:
                            r1, r2, _ = p.residual(t[0], t[1])
                            out = [r1, r2] + ([r3] if triples else [])
                        torch.cuda.synchronize()
                        got.append(out + t)
                p.profile(False)
                assert any(not torch.equal(a, b) for a, b in zip(got[0][-len(amps):], amps))  # written
                for merged, one in zip(got[:2], got[2:]):
                    for a, b in zip(merged, one):
                        assert float((a - b).abs().max()) <= 1e-13 * max(float(b.abs().max()), 1e-300)
