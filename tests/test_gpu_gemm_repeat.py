"""cc_gemm's choice of tile and split-K factor follows the call's sizes alone:
the same bits whatever the context ran before, and from cc_gemm_noalloc."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# few output tiles and a long K (split along K), few and many partial sums
@pytest.mark.parametrize("M,N,K", [(9, 76, 17951), (129, 8, 679), (21, 768, 5749), (365, 47, 3469), (10, 960, 2832),
                                   (133, 8, 3009), (700, 900, 9000), (1024, 1000, 4100)])
def test_gemm_bits_do_not_depend_on_earlier_calls(M, N, K):
    from paper_2409_06759_amd import engine as E
    print(f"gemm repeated M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    A, B, X = (torch.randn(s, generator=g, dtype=torch.float64, device="cuda") for s in ((M, K), (N, K), (1024, 20000)))

    def run(f):
        C = torch.empty((M, N), dtype=torch.float64, device="cuda")
        f(ctx, A, B, C, 1.0, 0.0)
        torch.cuda.synchronize()
        return C

    with E.Context(0) as ctx:
        first = run(E.gemm)
        E.gemm(ctx, X, X, torch.empty((1024, 1024), dtype=torch.float64, device="cuda"), 1.0, 0.0)
        assert torch.equal(run(E.gemm), first)
        assert torch.equal(run(E.gemm_noalloc), first)
