"""FP64 GEMM configurations with LDS-direct loads at the edges of their
tiles, against the register-staged kernels (bitwise) and NumPy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    from paper_2409_06759_amd import engine as E
    c = E.Context(0)
    yield c
    c.close()


# (LDS-direct configuration, staged configuration): 256x128, 64x128 (two
# stages) and 32x32
PAIRS = [(16, 4), (17, 13), (18, 3)]


@pytest.mark.parametrize("direct,staged", PAIRS)
# K: one partial chunk, partial last chunks behind one to three whole ones,
# whole chunks, an odd K (staged kernel); rows longer than K hold NaN behind it
@pytest.mark.parametrize("M,N,K,pad", [(1, 1, 2, 0), (33, 130, 14, 2), (64, 128, 18, 4), (70, 257, 34, 0),
                                       (257, 31, 48, 2), (129, 64, 62, 6), (31, 33, 45, 0), (300, 270, 1030, 2)])
def test_gemm_f64_direct_partial_chunks(ctx, monkeypatch, direct, staged, M, N, K, pad):
    print(f"direct tile {direct} M={M} N={N} K={K} pad={pad}", flush=True)
    import ctypes as C
    monkeypatch.setenv("CC_GEMM_TAIL", "0")  # one launch, no split-K
    rng = np.random.default_rng(M + 5 * N + K)
    A, B, C0 = rng.normal(size=(M, K)), rng.normal(size=(N, K)), rng.normal(size=(M, N))
    ld = K + pad
    Ap, Bp = np.full((M, ld), np.nan), np.full((N, ld), np.nan)
    Ap[:, :K], Bp[:, :K] = A, B
    Ad, Bd = torch.from_numpy(Ap).cuda(), torch.from_numpy(Bp).cuda()
    out = []
    for t in (staged, direct):
        monkeypatch.setenv("CC_GEMM_TILE", str(t))
        Cd = torch.from_numpy(C0).cuda()
        ctx.enter()
        ctx.check(ctx.lib.cc_gemm(ctx.h, 0, 0, M, N, K, 0.5, C.c_void_p(Ad.data_ptr()), ld, 1,
                                  C.c_void_p(Bd.data_ptr()), ld, 1, -1.25, C.c_void_p(Cd.data_ptr()), N))
        torch.cuda.synchronize()
        out.append(Cd.cpu().numpy())
    assert np.array_equal(out[0], out[1])
    ref = 0.5 * (A @ B.T) - 1.25 * C0
    bound = 2 * K * np.finfo(np.float64).eps * (0.5 * (np.abs(A) @ np.abs(B).T) + 1.25 * np.abs(C0))
    assert np.all(np.abs(out[1] - ref) <= bound + 1e-300)
