"""fp32-environment backward of small linears (32 x 32 tiles, both products in
one launch) and the line to the 128 x 128 kernels, against float64: reductions
inside one group of 16, one and several groups per wave and ragged tokens;
ragged outputs; every code format; dX or dW alone; bf16 dX; batches on both
sides of the line against their linears one by one.  The bound is
that of fp32 sums of R terms, |error| <= 2 (R + 2) 2^-24 sum |terms|, plus one
bf16 rounding where dX is bf16."""
import numpy as np
import pytest
import torch

from oracle import dqt_oracle as O
from paper_2412_04787_amd import dqt, workloads as W
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

GRID = {"ternary": (-1, 1), "i3": (-4, 3), "i4": (-8, 7), "i8": (-128, 127)}


def _close(got, ref, bound, R, bf16=False):
    tol = 2 * (R + 2) * 2.0 ** -24 * bound + (np.abs(ref) * 2.0 ** -8 if bf16 else 0.0) + 1e-30
    return bool((np.abs(got.astype(np.float64) - ref) <= tol).all())


def _case(M, d_in, d_out, wfmt, act, dx_out="f32", want_dw=True, want_dx=True):
    lo, hi = GRID[wfmt]
    q = W.draw_int((d_out, d_in), lo, hi, 8, M, d_in, d_out)
    X = W.draw_normal((M, d_in), 1.0, 8, M, d_in, 1)
    dY = W.draw_normal((M, d_out), 0.01, 8, M, d_in, 2)
    alpha = np.float32(0.019)
    codes, d = O.act_quant(X, act)
    G.log(f"f32 bwd M={M} {d_in}->{d_out} {wfmt} {act} {dx_out}")
    dX, dW = G.run_bwd(G.make_weight(d_out, d_in, wfmt, lo, hi, alpha), G.weight_codes_dev(q, wfmt),
                       torch.from_numpy(np.ascontiguousarray(codes)).to(G.DEV), act,
                       torch.from_numpy(d.astype(np.float32)).to(G.DEV), torch.from_numpy(dY).to(G.DEV), "f32",
                       dx_out if want_dx else None, want_dw)
    torch.cuda.synchronize()
    g, qq = dY.astype(np.float64), q.astype(np.float64) * float(alpha)
    if want_dx:
        assert _close(dX.float().cpu().numpy(), g @ qq, np.abs(g) @ np.abs(qq), d_out, dx_out == "bf16")
    if want_dw:
        a = codes.astype(np.float32) if act == "i8" else O.e4m3_decode(codes).astype(np.float32)
        xt = (a * d.astype(np.float32)[:, None]).astype(np.float64)
        assert _close(dW.cpu().numpy(), g.T @ xt, np.abs(g.T) @ np.abs(xt), M)


@pytest.mark.parametrize("wfmt,act", [(f, a) for f in GRID for a in ("i8", "e4m3") if (f, a) != ("i8", "e4m3")])
@pytest.mark.parametrize("M,d_in,d_out", [(1, 16, 16), (15, 48, 32), (17, 32, 80), (64, 80, 16), (100, 272, 144),
                                          (129, 16, 272), (512, 256, 256)])
def test_small(M, d_in, d_out, wfmt, act):
    _case(M, d_in, d_out, wfmt, act, "bf16" if M % 2 else "f32")


@pytest.mark.parametrize("wfmt", ["ternary", "i3"])
def test_one_product_alone(wfmt):
    _case(77, 144, 96, wfmt, "i8", want_dw=False)
    _case(77, 144, 96, wfmt, "i8", want_dx=False)


@pytest.mark.parametrize("M", [4096, 4097])
def test_line_in_tokens(M):
    _case(M, 48, 64, "ternary", "i8")


@pytest.mark.parametrize("d_out", [1024, 1088])     # 512 + 1024 and 512 + 1088 tiles of 64 x 64
def test_line_in_tiles(d_out):
    _case(512, 4096, d_out, "i4", "i8")


# the products' own lines: 256 tiles of dX with d_out = 16, then 258; 488 with
# d_out = 64, then 520; 256 of dW with 16 tokens, then 272; 256 tiles of dW that
# the 128 x 128 kernel splits, with 3072 tokens, then 3088
LINES = [(128, 8192, 16), (128, 8208, 16), (512, 3904, 64), (512, 4112, 64), (16, 1024, 1024), (16, 1024, 1040),
         (3072, 1024, 1024), (3088, 1024, 1024)]


@pytest.mark.parametrize("M,d_in,d_out", LINES)
def test_line_of_each_product(M, d_in, d_out):
    _case(M, d_in, d_out, "ternary", "i8")


# (M, shapes): all small; 2560 tiles in all, each linear 384 or 512 of them;
# one linear past the line (1600) among small ones; past the line in tokens;
# one product of a linear past its own line
BATCHES = [(50, [(64, 48), (272, 16), (32, 208)]),
           (512, [(1024, 1024)] * 4 + [(1024, 1536)] * 2),
           (512, [(64, 80), (4096, 1088), (272, 144)]),
           (4097, [(48, 64), (80, 32)]),
           (128, [(8208, 16), (48, 64), (64, 16)]),
           (16, [(1024, 1040), (64, 48)]),
           (3088, [(1024, 1024), (64, 48)])]


@pytest.mark.parametrize("M,shapes", BATCHES)
def test_batch_is_its_singles(M, shapes):
    """A batch gives the bits of its linears one by one, whichever of dX and
    dW each of them asks for."""
    g = np.random.default_rng(3)
    ents, ref = [], []
    for tid, (d_in, d_out) in enumerate(shapes):
        G.log(f"f32 batch M={M} {d_in}->{d_out}")
        q = g.integers(-8, 8, size=(d_out, d_in)).astype(np.int8)
        w = G.make_weight(d_out, d_in, "i4", -8, 7, 0.02, tid)
        e = dict(w=w, Wq=G.weight_codes_dev(q, "i4"),
                 Xq=torch.from_numpy(g.integers(-127, 128, size=(M, d_in)).astype(np.int8)).to(G.DEV),
                 xdq=torch.rand(M, device=G.DEV), dY=torch.randn((M, d_out), device=G.DEV),
                 dX=torch.empty((M, d_in), device=G.DEV), dW=torch.empty((d_out, d_in), device=G.DEV))
        ents.append(e)
        args = (w, e["Wq"], e["Xq"], "i8", e["xdq"], e["dY"], "f32")
        dX, dW = G.run_bwd(*args)
        dX1, _ = G.run_bwd(*args, want_dw=False)
        _, dW1 = G.run_bwd(*args, dx_out=None)
        torch.cuda.synchronize()
        assert torch.equal(dX1, dX) and torch.equal(dW1, dW)
        ref.append((dX, dW))

    def batch(ents):
        io = dqt.linear_io(ents)
        dqt.dqt_linear_bwd_batch(io, M, dqt.DQT_I8, dqt.DQT_F32, dqt.DQT_F32, dqt.DQT_F32,
                                 dqt.workspace(dqt.dqt_linear_bwd_batch_workspace(io, M)))
        torch.cuda.synchronize()

    batch(ents)
    for e, (dX, dW) in zip(ents, ref):
        assert torch.equal(e["dX"], dX) and torch.equal(e["dW"], dW)
    # every third linear dX alone, the next dW alone, the next neither
    part = [dict(e, dX=torch.full_like(e["dX"], 7.0) if i % 3 == 0 else None,
                 dW=torch.full_like(e["dW"], 7.0) if i % 3 == 1 else None) for i, e in enumerate(ents)]
    batch(part)
    for e, (dX, dW) in zip(part, ref):
        assert e["dX"] is None or torch.equal(e["dX"], dX)
        assert e["dW"] is None or torch.equal(e["dW"], dW)
