"""The persistent GEMM's main loops at the ends of their reduction: one to five
steps, whole and ragged (the two-phase loop keeps five half-tiles of copies in
flight and drains them over its last two or three steps; forward tiles of few
steps take the one-phase loop), for every operand layout: int8, e4m3 and FP4
forward, dX (K-contiguous), dW (K-major) unfused and with the SR update.  Rows and columns past one tile, ragged in both directions.
int8 is exact; the rest is bounded by fp32 sums of exact products, 1e-3 of
sum |terms|, as every product of the library."""
import numpy as np
import pytest
import torch

from oracle import dqt_oracle as O
from paper_2412_04787_amd import dqt, workloads as W
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

GRID = {"ternary": (-1, 1), "i3": (-4, 3), "i4": (-8, 7), "i8": (-127, 127)}


def _bf16(a):
    return torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16).float().numpy().astype(np.float64)


@pytest.mark.parametrize("d_in", [16, 128, 144, 256, 272, 384, 400, 512, 656])
@pytest.mark.parametrize("wfmt,act,M,d_out", [
    ("i8", "i8", 256 * 385 - 3, 16), ("ternary", "i8", 256 * 513 - 3, 16), ("i8", "i8", 256 * 193 - 3, 272),
    ("ternary", "i8", 256 * 257 - 3, 272), ("i4", "e4m3", 801, 272), ("i3", "e4m3", 1030, 48)])
def test_forward(wfmt, act, M, d_out, d_in):
    _forward(wfmt, act, M, d_out, d_in)


# more than 8 column tiles: bands of four row tiles, the last band of one
@pytest.mark.parametrize("wfmt,act,M,d_out,d_in", [
    ("i8", "i8", 256 * 41 - 3, 2320, 144), ("i4", "i8", 256 * 53 - 3, 2320, 272), ("ternary", "e4m3", 1030, 2320, 192)])
def test_forward_in_bands(wfmt, act, M, d_out, d_in):
    _forward(wfmt, act, M, d_out, d_in)


@pytest.mark.parametrize("d_in", [64, 128, 192, 256, 320, 384, 448])
def test_forward_fp4(d_in):
    _forward("ternary", "e4m3", 900, 272, d_in)


def _forward(wfmt, act, M, d_out, d_in):
    lo, hi = GRID[wfmt]
    q = W.draw_int((d_out, d_in), lo, hi, 5, M, d_in, d_out)
    X = W.draw_normal((M, d_in), 1.0, 5, M, d_in, 1)
    alpha = np.float32(0.017)
    G.log(f"fwd {wfmt} {act} M={M} {d_in}->{d_out}")
    Xd, Xv = G.to_dev(X, "bf16")
    w, Wq = G.make_weight(d_out, d_in, wfmt, lo, hi, alpha), G.weight_codes_dev(q, wfmt)
    Xq, xdq, Y = G.run_fwd(w, Wq, Xd, act, "f32")
    torch.cuda.synchronize()
    # beside a linear of 32 steps, whose mean takes the call to the two-phase
    # loop: the same bits
    K, N = 4096, max(272, d_out)
    g = torch.Generator(device=G.DEV)
    g.manual_seed(5)
    Wl = torch.randint(0, 127, (N * K // (4 if wfmt == "ternary" else 1),), generator=g, device=G.DEV, dtype=torch.uint8)
    if wfmt == "ternary":
        Wl &= 0x55                              # codes 0 and 1
    Xl = torch.randint(0, 127, (M, K), generator=g, device=G.DEV, dtype=torch.uint8)
    wl = G.make_weight(N, K, wfmt, lo, hi, alpha, 1)
    Y2 = torch.full_like(Y, -7.0)
    io = dqt.linear_io([dict(w=w, Wq=Wq, Xq=Xq, xdq=xdq, Y=Y2),
                        dict(w=wl, Wq=Wl, Xq=Xl, xdq=xdq, Y=torch.empty((M, N), device=G.DEV))])
    dqt.dqt_linear_fwd_batch(io, M, G.act_code(act), dqt.DQT_F32,
                             dqt.workspace(dqt.dqt_linear_fwd_batch_workspace(io)))
    torch.cuda.synchronize()
    assert torch.equal(Y2, Y)
    codes, d = O.act_quant(Xv, act)
    a = codes.astype(np.float64) if act == "i8" else O.e4m3_decode(codes).astype(np.float64)
    sc = (d.astype(np.float32) * alpha).astype(np.float32)[:, None]
    acc = a @ q.T.astype(np.float64)
    got = Y.cpu().numpy()
    if act == "i8":
        assert np.array_equal(got, acc.astype(np.float32) * sc)
    else:
        ok, bad, err = G.gemm_close(got, acc * sc, np.abs(a) @ np.abs(q.T.astype(np.float64)) * sc)
        assert ok, (bad, err)


# dX reduces over d_out, dW over M: both in steps of 64
@pytest.mark.parametrize("M", [1, 63, 64, 65, 128, 130, 193, 257, 320, 321])
@pytest.mark.parametrize("wfmt,act,d_in,d_out", [
    ("ternary", "i8", 272, 16), ("ternary", "e4m3", 48, 64), ("i8", "i8", 16, 80), ("i4", "i8", 288, 128),
    ("i3", "i8", 80, 144), ("i8", "i8", 272, 192), ("ternary", "i8", 64, 208), ("i4", "e4m3", 16, 336)])
def test_backward(wfmt, act, d_in, d_out, M):
    lo, hi = GRID[wfmt]
    q = W.draw_int((d_out, d_in), lo, hi, 6, M, d_in, d_out)
    X = W.draw_normal((M, d_in), 1.0, 6, M, d_in, 1)
    dY = W.draw_normal((M, d_out), 0.01, 6, M, d_in, 2)
    alpha = np.float32(0.011)
    w = G.make_weight(d_out, d_in, wfmt, lo, hi, alpha, 3)
    Wq = G.weight_codes_dev(q, wfmt)
    codes, d = O.act_quant(X, act)
    Xq = torch.from_numpy(np.ascontiguousarray(codes)).to(G.DEV)
    xdq = torch.from_numpy(d.astype(np.float32)).to(G.DEV)
    dYd, dYv = G.to_dev(dY, "bf16")
    G.log(f"bwd {wfmt} {act} M={M} {d_in}->{d_out}")
    dX, dW = G.run_bwd(w, Wq, Xq, act, xdq, dYd, "bf16")
    torch.cuda.synchronize()
    a = codes.astype(np.float32) if act == "i8" else O.e4m3_decode(codes).astype(np.float32)
    xt = _bf16(a * d.astype(np.float32)[:, None])
    g, qq = dYv.astype(np.float64), q.astype(np.float64)
    ok, bad, err = G.gemm_close(dX.cpu().numpy(), float(alpha) * (g @ qq), float(alpha) * (np.abs(g) @ np.abs(qq)))
    assert ok, ("dX", bad, err)
    ok, bad, err = G.gemm_close(dW.cpu().numpy(), g.T @ xt, np.abs(g.T) @ np.abs(xt))
    assert ok, ("dW", bad, err)
    # dX of the same call alone, and dW with the SR update: the same sums, so
    # the codes of the update of this dW
    dX1, _ = G.run_bwd(w, Wq, Xq, act, xdq, dYd, "bf16", want_dw=False)
    W2 = Wq.clone()
    dqt.dqt_sr_update(w, W2, dW, 0.05, 9, 4)
    dX2 = torch.empty_like(dX)
    io = dqt.linear_io([dict(w=w, Wq=Wq, Xq=Xq, xdq=xdq, dY=dYd, dX=dX2)])
    dqt.dqt_linear_bwd_sr_batch(io, M, G.act_code(act), dqt.DQT_BF16, dqt.DQT_BF16, dqt.DQT_F32, 0.05, 9, 4, None,
                                dqt.workspace(dqt.dqt_linear_bwd_batch_workspace(io, M)))
    torch.cuda.synchronize()
    assert torch.equal(dX1, dX) and torch.equal(dX2, dX)
    assert torch.equal(W2, Wq)


@pytest.mark.parametrize("M", [70, 1200, 9000])
def test_backward_batch_is_its_singles(M):
    """Both orders of the two products in one launch (dX's reductions longer
    than dW's at 70 tokens, shorter at 9000), with at most one tile per compute
    unit (70, 1200) and with several (9000): dX of the batch is that of each
    linear alone, bit for bit, and the fused update's codes and counts are
    those of the update of the batch's dW."""
    ents = []
    for tid, (d_in, d_out) in enumerate([(272, 1040), (1040, 272), (528, 528), (16, 16)]):
        q = W.draw_int((d_out, d_in), -1, 1, 12, M, tid)
        X = W.draw_normal((M, d_in), 1.0, 12, M, tid, 1)
        codes, d = O.act_quant(X, "i8")
        w = G.make_weight(d_out, d_in, "ternary", -1, 1, 0.015, tid)
        ents.append(dict(w=w, Wq=G.weight_codes_dev(q, "ternary"), Xq=torch.from_numpy(codes).to(G.DEV),
                         xdq=torch.from_numpy(d.astype(np.float32)).to(G.DEV),
                         dY=G.to_dev(W.draw_normal((M, d_out), 0.01, 12, M, tid, 2), "bf16")[0],
                         dX=torch.empty((M, d_in), dtype=torch.bfloat16, device=G.DEV),
                         dW=torch.empty((d_out, d_in), device=G.DEV)))
    io = dqt.linear_io(ents)
    ws = dqt.workspace(dqt.dqt_linear_bwd_batch_workspace(io, M))
    bf, i8 = dqt.DQT_BF16, dqt.DQT_I8
    dqt.dqt_linear_bwd_batch(io, M, i8, bf, bf, bf, ws)
    torch.cuda.synchronize()
    for e in ents:
        dX, _ = G.run_bwd(e["w"], e["Wq"], e["Xq"], "i8", e["xdq"], e["dY"], "bf16", "bf16", want_dw=False)
        torch.cuda.synchronize()
        assert torch.equal(dX, e["dX"])
    cnt, cnt2 = (torch.zeros(2, dtype=torch.int64, device=G.DEV) for _ in range(2))
    two = [dict(e, Wq=e["Wq"].clone()) for e in ents]
    dqt.dqt_sr_update_batch(dqt.linear_io(two), 0.02, 5, 3, cnt)
    fused = [dict(e, dW=None, dX=torch.empty_like(e["dX"])) for e in ents]
    dqt.dqt_linear_bwd_sr_batch(dqt.linear_io(fused), M, i8, bf, bf, bf, 0.02, 5, 3, cnt2, ws)
    torch.cuda.synchronize()
    for a, b, e in zip(two, fused, ents):
        assert torch.equal(a["Wq"], b["Wq"]) and torch.equal(b["dX"], e["dX"])
    assert torch.equal(cnt, cnt2)
