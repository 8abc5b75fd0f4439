"""The fused FP32 training passes give the bits of the layer-by-layer ones: the
same FP32 products in the same order, the same FP64 bias, ReLU and output
gradient.  The layers are put together here from the library's FP32 GEMM and
FP64 elementwise operations."""
import numpy as np
import pytest

from oracle import mlp as ref

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

STATS = {"sx": 1.0, "mD": 0.0, "sD": 1.0, "me": 0.0, "se": 1.0, "st": 1.0}
HID = 128


def _layers(E, ctx, params, z, y):
    def gemm(A, B, M, N, ak=True, bk=True):
        C = torch.empty((M, N), dtype=torch.float64, device="cuda")
        E.gemm(ctx, A, B, C, a_kcontig=ak, b_kcontig=bk, prec=E.F32)
        return C

    n = z.shape[0]
    sizes = [HID * 3, HID, HID * HID, HID, HID, 1]
    w1, b1, w2, b2, w3, _ = (x.contiguous() for x in torch.split(params, sizes))
    w1, w2, w3 = w1.view(HID, 3), w2.view(HID, HID), w3.view(1, HID)
    z2 = torch.cat([z, z * torch.tensor([-1.0, 1.0, 1.0], dtype=torch.float64, device="cuda")]).contiguous()
    zero = torch.zeros((), dtype=torch.float64, device="cuda")
    h1 = gemm(z2, w1, 2 * n, HID) + b1
    h1 = torch.where(h1 > 0, h1, zero)
    h2 = gemm(h1, w2, 2 * n, HID) + b2
    h2 = torch.where(h2 > 0, h2, zero)
    g = gemm(h2, w3, 2 * n, 1).view(-1)
    res = 0.5 * (g[:n] - g[n:]) - y
    dg = (torch.cat([res, -res]) / n).view(1, -1).contiguous()
    ones = torch.ones_like(dg)
    gw3, gb3 = gemm(dg, h2, 1, HID, bk=False), gemm(dg, ones, 1, 1)
    da2 = torch.where(h2 > 0, dg.view(-1, 1) * w3, zero)
    gw2, gb2 = gemm(da2, h1, HID, HID, ak=False, bk=False), gemm(ones, da2, 1, HID, bk=False)
    da1 = gemm(da2, w2, 2 * n, HID, bk=False)
    da1 = torch.where(h1 > 0, da1, zero)
    gw1, gb1 = gemm(da1, z2, HID, 3, ak=False, bk=False), gemm(ones, da1, 1, HID, bk=False)
    return torch.cat([x.reshape(-1) for x in (gw1, gb1, gw2, gb2, gw3, gb3)]).cpu().numpy()


# one row block and less, ragged ones, two slices, slices of 272 and 288 rows,
# two vector slices per weight slice, the largest whose slices the library's
# GEMM has too (above, its workspace would hold more of them than training's)
@pytest.mark.parametrize("n", [1, 5, 32, 33, 257, 1001, 4111, 20000, 32768])
def test_fused_gradient_equals_the_layers(monkeypatch, n):
    from paper_2409_06759_amd import engine as E
    print(f"fused against layers n={n}", flush=True)
    monkeypatch.setenv("CC_GEMM_LPIN", "0")  # FP64 operands rounded while staging, as the layers' are
    monkeypatch.delenv("CC_GEMM_TAIL", raising=False)
    monkeypatch.delenv("CC_GEMM_TILE", raising=False)
    rng = np.random.default_rng(n)
    params = torch.from_numpy(ref.flatten(ref.init_params(5))).cuda()
    params += 0.05 * torch.from_numpy(rng.normal(size=params.numel())).cuda()
    z, y = torch.from_numpy(rng.normal(size=(n, 3))).cuda(), torch.from_numpy(0.5 * rng.normal(size=n)).cuda()
    with E.Context(0) as ctx:
        _, grad = E.MLP(ctx, params, STATS, E.F32).loss_grad(z, y)
        assert np.array_equal(grad.cpu().numpy(), _layers(E, ctx, params, z, y))
