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


# (and 64x64, against the staged tile of that size)
@pytest.mark.parametrize("direct,staged", PAIRS + [(19, 2)])
# the last k on its own, at every place of a chunk it can have; rows of odd
# length (8-byte aligned) with an even K
@pytest.mark.parametrize("M,N,K,pad", [(1, 1, 1, 0), (33, 130, 15, 0), (64, 128, 17, 1), (70, 65, 35, 2), (65, 129, 37, 0),
                                       (31, 257, 39, 4), (257, 31, 41, 3), (128, 64, 59, 1), (129, 64, 62, 3),
                                       (300, 270, 1031, 0)])
def test_gemm_f64_direct_odd_rows(ctx, monkeypatch, direct, staged, M, N, K, pad):
    test_gemm_f64_direct_partial_chunks(ctx, monkeypatch, direct, staged, M, N, K, pad)


@pytest.mark.parametrize("prec,staged,direct", [("bf16x3", 6, 9), ("bf16x3", 6, 12), ("bf16x3", 6, 13),
                                                ("f32", 7, 10), ("f32", 7, 11), ("f32", 7, 12), ("bf16x3", 6, -1),
                                                ("f32", 7, -1)])
# partial last chunks of 4, 8, 16 and 24, whole chunks; sizes below, at and
# over a tile's edge.  K % 8 == 4 goes to the staged kernel in split bf16.
@pytest.mark.parametrize("M,N,K", [(1, 1, 8), (63, 130, 40), (128, 128, 32), (130, 257, 72), (257, 64, 100),
                                   (300, 270, 1000), (65, 700, 2016)])
def test_gemm_lowp_direct_partial_chunks(ctx, monkeypatch, prec, staged, direct, M, N, K):
    """Every reduced-precision kernel, and the library's own choice, adds the
    same products in the same order: bit-identical results."""
    from paper_2409_06759_amd import engine as E
    print(f"direct {prec} tile {direct} M={M} N={N} K={K}", flush=True)
    monkeypatch.setenv("CC_GEMM_TAIL", "0")
    monkeypatch.setenv("CC_GEMM_BLOCKED", "0")
    rng = np.random.default_rng(M + 5 * N + K)
    A, B, C0 = rng.normal(size=(M, K)), rng.normal(size=(N, K)), rng.normal(size=(M, N))
    Ad, Bd = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    out = []
    for t in (staged, direct):
        if t >= 0:
            monkeypatch.setenv("CC_GEMM_TILE", str(t))
        else:
            monkeypatch.delenv("CC_GEMM_TILE")
        Cd = torch.from_numpy(C0).cuda()
        E.gemm(ctx, Ad, Bd, Cd, 0.5, -1.25, prec=E.PRECS[prec])
        out.append(Cd.cpu().numpy())
    assert np.array_equal(out[0], out[1])
    ref = 0.5 * (A @ B.T) - 1.25 * C0
    eps = (K + 2) * 2.0 ** -24 + (3 * 2.0 ** -17 if prec == "bf16x3" else 0.0)
    bound = 2 * eps * 0.5 * (np.abs(A) @ np.abs(B).T) + 4 * np.finfo(float).eps * np.abs(1.25 * C0)
    assert np.all(np.abs(out[1] - ref) <= bound)


@pytest.mark.parametrize("direct", [4, 5, 6])
# any K: below, at and over a chunk; sizes below, at and over a tile's edge
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 130, 13), (64, 64, 16), (65, 31, 17), (32, 129, 47), (130, 70, 500)])
def test_gemm_c128_direct_partial_chunks(ctx, monkeypatch, direct, M, N, K):
    from paper_2409_06759_amd import engine as E
    print(f"direct c128 tile {direct} M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(M + 5 * N + K)
    A, B, C0 = (rng.normal(size=s) + 1j * rng.normal(size=s) for s in ((M, K), (N, K), (M, N)))
    Ad, Bd = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    out = []
    for t in (0, direct):
        monkeypatch.setenv("CC_GEMM_TILE", str(t))
        Cd = torch.from_numpy(C0).cuda()
        E.gemm(ctx, Ad, Bd, Cd, 0.5, -1.25)
        out.append(Cd.cpu().numpy())
    assert np.array_equal(out[0], out[1])
    ref = 0.5 * (A @ B.T) - 1.25 * C0
    bound = 8 * K * np.finfo(np.float64).eps * (0.5 * (np.abs(A) @ np.abs(B).T) + 1.25 * np.abs(C0))
    assert np.all(np.abs(out[1] - ref) <= bound)
