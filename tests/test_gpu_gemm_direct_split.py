"""LDS-direct GEMM configurations split along K: slices that begin inside the
rows, a last slice with a partial chunk and an odd last element, and slices left
empty because a slice is a whole number of chunks.  Against the register-staged
configuration at the same factor (bitwise) and NumPy."""
import ctypes as C

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


def _both(ctx, monkeypatch, prec, tiles, M, N, K, pad):
    """cc_gemm on each tile; few output tiles, so that it splits K into 256-long parts."""
    monkeypatch.delenv("CC_GEMM_TAIL", raising=False)
    monkeypatch.setenv("CC_GEMM_BLOCKED", "0")
    rng = np.random.default_rng(M + 5 * N + K)
    A, B, C0 = rng.normal(size=(M, K)), rng.normal(size=(N, K)), rng.normal(size=(M, N))
    ld = K + pad
    Ap, Bp = np.full((M, ld), np.nan), np.full((N, ld), np.nan)
    Ap[:, :K], Bp[:, :K] = A, B
    Ad, Bd = torch.from_numpy(Ap).cuda(), torch.from_numpy(Bp).cuda()
    out = []
    for t in tiles:
        monkeypatch.setenv("CC_GEMM_TILE", str(t))
        Cd = torch.from_numpy(C0).cuda()
        ctx.enter()
        ctx.check(ctx.lib.cc_gemm(ctx.h, prec, 0, M, N, K, 0.5, C.c_void_p(Ad.data_ptr()), ld, 1,
                                  C.c_void_p(Bd.data_ptr()), ld, 1, -1.25, C.c_void_p(Cd.data_ptr()), N))
        torch.cuda.synchronize()
        out.append(Cd.cpu().numpy())
    ref = 0.5 * (A @ B.T) - 1.25 * C0
    size = 0.5 * (np.abs(A) @ np.abs(B).T)
    return out, ref, size, 1.25 * np.abs(C0)


@pytest.mark.parametrize("direct,staged", [(16, 4), (17, 13), (18, 3), (19, 2)])
# factors 2, 4, 16 and 32; in the last two rows the last slice (of 272) is empty
@pytest.mark.parametrize("M,N,K,pad", [(33, 130, 515, 0), (65, 31, 1031, 1), (1, 1, 1040, 3), (70, 65, 4099, 2),
                                       (129, 64, 4111, 0), (31, 33, 8193, 0), (257, 30, 8202, 5)])
def test_gemm_f64_direct_split(ctx, monkeypatch, direct, staged, M, N, K, pad):
    print(f"direct split tile {direct} M={M} N={N} K={K} pad={pad}", flush=True)
    out, ref, size, c0 = _both(ctx, monkeypatch, 0, (staged, direct), M, N, K, pad)
    assert np.array_equal(out[0], out[1])
    assert np.all(np.abs(out[1] - ref) <= 2 * K * np.finfo(np.float64).eps * (size + c0))


@pytest.mark.parametrize("prec,staged,direct", [("bf16x3", 6, 9), ("bf16x3", 6, 12), ("bf16x3", 6, 13),
                                                ("f32", 7, 10), ("f32", 7, 11), ("f32", 7, 12)])
# slices of 288: partial last ones, and the last three of 32 empty
@pytest.mark.parametrize("M,N,K", [(33, 130, 520), (65, 31, 1040), (129, 64, 4104), (31, 257, 8200)])
def test_gemm_lowp_direct_split(ctx, monkeypatch, prec, staged, direct, M, N, K):
    from paper_2409_06759_amd import engine as E
    print(f"direct split {prec} tile {direct} M={M} N={N} K={K}", flush=True)
    out, ref, size, c0 = _both(ctx, monkeypatch, E.PRECS[prec], (staged, direct), M, N, K, 0)
    assert np.array_equal(out[0], out[1])
    eps = (K + 2) * 2.0 ** -24 + (3 * 2.0 ** -17 if prec == "bf16x3" else 0.0)
    assert np.all(np.abs(out[1] - ref) <= 2 * eps * size + 4 * np.finfo(float).eps * c0)
