"""Forward for few tokens: the streaming and the 128 x 128 kernels and the
persistent GEMM on both sides of every line of the rule between them, against
the oracle: tokens around 16, 32, 48, 64 (streaming), 128, 256 (the reduction in
two halves) and the last few hundred; reductions that end inside a 16-, 64-
and 128-code step; outputs that end inside a tile.  int8 activations are
exact; e4m3 ones within the forward's bound (fp32 sums of exact products)."""
import numpy as np
import pytest
import torch

from oracle import dqt_oracle as O
from paper_2412_04787_amd import dqt, workloads as W
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

GRID = {"ternary": (-1, 1), "i3": (-4, 3), "i4": (-8, 7), "i8": (-128, 127)}
KINDS = [("ternary", "i8"), ("ternary", "e4m3"), ("i3", "i8"), ("i3", "e4m3"), ("i4", "i8"), ("i4", "e4m3"),
         ("i8", "i8")]
# (M, d_in, d_out)
SHAPES = [(1, 16, 16), (16, 272, 48), (17, 64, 32), (33, 1040, 80), (48, 704, 144), (49, 80, 272), (64, 320, 48),
          (65, 144, 80), (128, 192, 128),
          (129, 2064, 144), (256, 448, 160), (257, 400, 272), (513, 128, 16), (800, 336, 144), (801, 336, 144),
          (900, 320, 304)]


def _check(M, d_in, d_out, wfmt, act, y_out, seed=11):
    lo, hi = GRID[wfmt]
    q = W.draw_int((d_out, d_in), lo, hi, seed, M, d_in, d_out)
    X = W.draw_normal((M, d_in), 1.0, seed, M, d_in, 1)
    X[M // 2] = 0.0                                       # a zero row: scale from the floor
    alpha = np.float32(0.013)
    w = G.make_weight(d_out, d_in, wfmt, lo, hi, alpha)
    Xd, Xv = G.to_dev(X, "bf16")
    G.log(f"fwd M={M} d_in={d_in} d_out={d_out} {wfmt} {act} {y_out}")
    Xq, xdq, Y = G.run_fwd(w, G.weight_codes_dev(q, wfmt), Xd, act, y_out)
    torch.cuda.synchronize()
    codes, d = O.act_quant(Xv, act)
    a = codes.astype(np.float64) if act == "i8" else O.e4m3_decode(codes).astype(np.float64)
    acc = a @ q.T.astype(np.float64)
    sc = (d.astype(np.float32) * alpha).astype(np.float32)[:, None]
    got = Y.float().cpu().numpy()
    if act == "i8":
        ref = (acc.astype(np.float32) * sc).astype(np.float32)
        if y_out == "bf16":
            ref = torch.from_numpy(ref).to(torch.bfloat16).float().numpy()
        assert np.array_equal(got, ref)
    else:
        bound = np.abs(a) @ np.abs(q.T.astype(np.float64)) * sc
        ok, bad, err = G.gemm_close(got, acc * sc, bound, bf16_out=y_out == "bf16")
        assert ok, (bad, err)


@pytest.mark.parametrize("wfmt,act", KINDS)
@pytest.mark.parametrize("shape", SHAPES)
def test_shapes(shape, wfmt, act):
    _check(*shape, wfmt, act, "bf16" if (shape[0] + shape[1] // 16) % 2 else "f32")


@pytest.mark.parametrize("wfmt", list(GRID))
def test_int8_line_of_the_persistent_gemm(wfmt):
    """The rule for int8 activations counts 256 x 256 tiles: one row tile of
    tokens on each side of its lines (384 tiles for 8-bit codes, 512 else),
    with one column tile and with two."""
    line = 384 if wfmt == "i8" else 512
    for past in (0, 1):
        _check(256 * line + past, 80, 16, wfmt, "i8", "bf16")
        _check(128 * line + past, 48, 272, wfmt, "i8", "f32")


@pytest.mark.parametrize("M", [7, 60, 200, 300])
def test_batch_equals_singles_and_needs_only_the_counters(M):
    """Linears of different widths in one call, with the smallest workspace
    the call accepts and guard bytes after every output."""
    g = np.random.default_rng(M)
    ents, singles = [], []
    for tid, (d_in, d_out) in enumerate([(320, 48), (704, 144), (320, 272), (1024, 16)]):
        q = g.integers(-1, 2, size=(d_out, d_in)).astype(np.int8)
        w = G.make_weight(d_out, d_in, "ternary", -1, 1, 0.02, tid)
        Xd, _ = G.to_dev(g.standard_normal((M, d_in)).astype(np.float32), "bf16")
        Wq = G.weight_codes_dev(q, "ternary")
        Xq, xdq, Y = G.run_fwd(w, Wq, Xd, "e4m3", "bf16")
        buf = torch.full((M * d_out + 64,), -7.0, dtype=torch.bfloat16, device=G.DEV)
        ents.append(dict(w=w, Wq=Wq, Xq=Xq, xdq=xdq, Y=buf))
        singles.append(Y)
    io = dqt.linear_io(ents)
    dqt.dqt_linear_fwd_batch(io, M, dqt.DQT_FP8E4M3, dqt.DQT_BF16, dqt.workspace(256))
    torch.cuda.synchronize()
    for e, Y in zip(ents, singles):
        assert torch.equal(e["Y"][:Y.numel()].view_as(Y), Y)
        assert bool((e["Y"][Y.numel():] == -7.0).all())


# (M, wfmt, act, shapes): the first linear alone fills its rounds of tiles and
# takes the persistent GEMM (on FP4, e4m3 and int8 operands); the others alone
# take the 128 x 128 tiles, as does the batch with e4m3 activations, at 200 and
# 256 tokens with the reduction in two halves
ACROSS = [(800, "ternary", "e4m3", [(576, 32768), (704, 1040), (64, 48)]),
          (800, "i3", "e4m3", [(576, 32768), (272, 1040), (1040, 144)]),
          (800, "i8", "i8", [(1024, 32768), (272, 1040), (1040, 144)]),
          (200, "ternary", "e4m3", [(64, 65536), (192, 272)]),
          (256, "i4", "e4m3", [(16, 65536), (272, 16)])]


@pytest.mark.parametrize("M,wfmt,act,shapes", ACROSS)
def test_batch_is_its_singles_across_the_line(M, wfmt, act, shapes):
    """fp32 outputs, bit for bit, of inputs whose products span 12 powers of
    two; also with the 256 counter bytes alone, where the formats allow it."""
    g = torch.Generator(device=G.DEV)
    g.manual_seed(M + len(wfmt))
    lo, hi = GRID[wfmt]
    ents, singles = [], []
    for tid, (d_in, d_out) in enumerate(shapes):
        G.log(f"across the line M={M} {d_in}->{d_out} {wfmt} {act}")
        q = np.random.default_rng(tid).integers(lo, hi + 1, size=(d_out, d_in)).astype(np.int8)
        w = G.make_weight(d_out, d_in, wfmt, lo, hi, 0.02, tid)
        Wq = G.weight_codes_dev(q, wfmt)
        X = torch.randn((M, d_in), generator=g, device=G.DEV)
        X *= torch.exp2(torch.randint(-6, 7, (M, d_in), generator=g, device=G.DEV).float())
        Xq, xdq, Y = G.run_fwd(w, Wq, X, act, "f32")
        ents.append(dict(w=w, Wq=Wq, Xq=Xq, xdq=xdq, Y=torch.full_like(Y, -7.0)))
        singles.append(Y)
    io = dqt.linear_io(ents)
    sizes = [dqt.dqt_linear_fwd_batch_workspace(io)]
    if wfmt == "ternary":
        sizes.append(256)
    for nbytes in sizes:
        dqt.dqt_linear_fwd_batch(io, M, G.act_code(act), dqt.DQT_F32, dqt.workspace(nbytes))
        torch.cuda.synchronize()
        for e, Y in zip(ents, singles):
            assert torch.equal(e["Y"], Y)
            e["Y"].fill_(-7.0)
