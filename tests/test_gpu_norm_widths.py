"""RMSNorm + quantisation and its backward around every row width where the
kernel changes (512, 1024, 2048 and 4096 elements held in registers, longer
rows read again): the forward equal to the oracle, the backward's dX and every
block's partial gamma gradient against float64.  A row's dX is bounded by its
bf16 rounding and the fp32 rounding of the K-term dot product; a partial sum
by the fp32 rounding of its terms."""
import numpy as np
import pytest
import torch

from oracle import dqt_oracle as O
from paper_2412_04787_amd import dqt, workloads as W
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

WIDTHS = [16, 512, 528, 1024, 1040, 2048, 2064, 4096, 4112, 8192]


@pytest.mark.parametrize("K", WIDTHS)
@pytest.mark.parametrize("xdt,act", [("bf16", "i8"), ("f32", "e4m3")])
def test_forward(K, xdt, act):
    M = 7
    G.log(f"norm fwd K={K} {xdt} {act}")
    X = W.draw_normal((M, K), 1.0, 31, K, 1)
    X[3] = 0.0
    g = (1.0 + 0.3 * W.draw_normal((K,), 1.0, 31, K, 2)).astype(np.float32)
    Xd, xv = G.to_dev(X, xdt)
    Xq = torch.empty((M, K), dtype=torch.int8 if act == "i8" else torch.uint8, device=G.DEV)
    xdq, rinv = torch.empty(M, device=G.DEV), torch.empty(M, device=G.DEV)
    dqt.dqt_rmsnorm_act_quant(Xd, torch.from_numpy(g).to(G.DEV), 1e-5, G.act_code(act), Xq, xdq, rinv)
    torch.cuda.synchronize()
    wq, wd, wr, _ = O.rmsnorm_act_quant(xv, g, 1e-5, act)
    assert np.array_equal(rinv.cpu().numpy(), wr) and np.array_equal(xdq.cpu().numpy(), wd)
    assert np.array_equal(Xq.cpu().numpy(), wq)


@pytest.mark.parametrize("K", WIDTHS)
@pytest.mark.parametrize("n_dy", [1, 2, 3, 4])
def test_backward(K, n_dy):
    M, blocks = 19, 3
    G.log(f"norm bwd K={K} n_dy={n_dy}")
    Xd, x = G.to_dev(W.draw_normal((M, K), 1.0, 32, K, 1), "bf16")
    dys = [G.to_dev(W.draw_normal((M, K), 1e-2, 32, K, 3, i), "bf16") for i in range(n_dy)]
    g = (1.0 + 0.3 * W.draw_normal((K,), 1.0, 32, K, 2)).astype(np.float32)
    r32 = (1.0 / np.sqrt((x.astype(np.float64) ** 2).mean(-1) + 1e-6)).astype(np.float32)
    dX = torch.empty_like(Xd)
    gpart = torch.empty((blocks, K), device=G.DEV)
    dqt.dqt_rmsnorm_backward([d for d, _ in dys], Xd, torch.from_numpy(g).to(G.DEV),
                             torch.from_numpy(r32).to(G.DEV), dX, gpart)
    torch.cuda.synchronize()
    x, r = x.astype(np.float64), r32.astype(np.float64)[:, None]
    dn = sum(v.astype(np.float64) for _, v in dys)
    gr = dn * g.astype(np.float64)
    c = (gr * x).mean(-1, keepdims=True)
    ref = r * gr - x * r ** 3 * c
    eps = 2.0 ** -23
    tol = np.abs(ref) * 2.0 ** -8 + eps * (K + 8) * np.abs(x) * r ** 3 * np.abs(gr * x).mean(-1, keepdims=True) \
        + 8 * eps * np.abs(r * gr)
    assert (np.abs(dX.float().cpu().numpy() - ref) <= tol).all()
    t = dn * x * r
    for b in range(blocks):
        rows = [m for m in range(M) if m // 4 % blocks == b]
        got = gpart[b].cpu().numpy()
        assert (np.abs(got - t[rows].sum(0)) <= (len(rows) + 8) * eps * np.abs(t[rows]).sum(0) + 1e-30).all()
