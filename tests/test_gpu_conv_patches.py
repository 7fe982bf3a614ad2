"""The convolution source on both sides of the line between its two ways (patches of at most 448 16-byte pieces go by
lines, longer ones and images narrower than four pixels through register tiles): which kernel runs, codes and
scales against the oracle."""
import numpy as np
import pytest
import torch

from launches import launched
from oracle import capi
from paper_2310_03675_amd import binding as B
from test_gpu_conv import NE, ST, o_op, relu_act, step_params, unfold

pytestmark = pytest.mark.gpu

LINES, TILES = 1, 2
# (batch, C, H, W, kh, kw, way): the shortest and the longest patches beyond the line, narrow and wide images, one-row
# and one-column windows; the rest below it, the first, 440 and 448 pieces
PATCHES = [(1, 64, 16, 16, 3, 1, TILES), (1, 64, 16, 4, 1, 3, TILES), (2, 64, 32, 32, 3, 1, TILES),
           (1, 64, 32, 32, 13, 1, TILES), (1, 64, 2, 64, 5, 3, TILES), (1, 64, 3, 64, 15, 3, TILES),
           (1, 64, 2, 128, 9, 5, TILES), (1, 64, 32, 2, 3, 3, TILES), (1, 64, 128, 1, 3, 1, TILES),
           (1, 64, 16, 4, 3, 3, LINES), (1, 64, 16, 16, 5, 1, LINES), (1, 64, 8, 8, 1, 5, LINES), (1, 64, 1, 128, 1, 5, LINES)]


def way_of(call):
    names = launched(call)
    found = {w for w in (LINES, TILES) if f", {w}>" in names}
    assert len(found) == 1, names
    return found.pop()


@pytest.mark.parametrize("batch,C,H,W,kh,kw,way", PATCHES)
@pytest.mark.parametrize("b,n", [(4, 64), (4, 16), (8, 64)])
def test_patches(batch, C, H, W, kh, kw, way, b, n):
    rect = relu_act((batch, C, H, W), seed=C + H * 7 + W + kh)
    for act in (rect, rect - rect.flip(0, 1, 2, 3)):
        X = unfold(act, kh, kw)
        for r in (NE, ST):
            op1, op0 = B.Operand(b, r, 1.0, 3), B.Operand(b, r, 0.975, 9)
            print(f"act {tuple(act.shape)} window {kh}x{kw} n={n} b={b} rounding={r}", flush=True)
            c1, s1, c0, s0 = B.quantize_dual_im2col(act.to("cuda:0"), kh, kw, n, op1, op0, seed=5)
            torch.cuda.synchronize()
            for axis, got_c, got_s, op in ((1, c1, s1, op1), (0, c0, s0, op0)):
                codes, scale, _ = capi.quantize(X.numpy(), axis, n, o_op(op), 5)
                assert float(got_s) == float(scale)
                assert np.array_equal(got_c.cpu().numpy().reshape(-1).view(np.uint8),
                                      np.ascontiguousarray(capi.pack_codes(codes, b)).reshape(-1).view(np.uint8))


@pytest.mark.parametrize("batch,C,H,W,kh,kw,way", PATCHES)
def test_which_way(batch, C, H, W, kh, kw, way):
    act, op = relu_act((batch, C, H, W), seed=1).to("cuda:0"), B.Operand(4, NE, 1.0, 3)
    assert way_of(lambda: B.quantize_dual_im2col(act, kh, kw, 64, op, op)) == way


@pytest.mark.parametrize("batch,C,H,W,kh,kw,way", [PATCHES[2], PATCHES[4]])
@pytest.mark.parametrize("b,a", [(4, 8), (8, 16)])
def test_a_layer_with_weights_and_gradient_in_the_launch(batch, C, H, W, kh, kw, way, b, a):
    act = relu_act((batch, C, H, W), seed=11)
    X = unfold(act, kh, kw)
    (M, K), N = X.shape, 128
    g = torch.Generator().manual_seed(12)
    Wt, G = torch.randn((K, N), generator=g) * (2.0 / K) ** 0.5, torch.randn((M, N), generator=g) * 1e-2
    prm = step_params(layer_id=1, b=b, a=a)
    d = lambda t: t.contiguous().to("cuda:0")
    print(f"conv_step act {tuple(act.shape)} window {kh}x{kw} b={b}", flush=True)
    got, want = B.conv_step(d(act), kh, kw, d(Wt), d(G), *prm)[:3], B.layer_step(d(X), d(Wt), d(G), *prm)[:3]
    torch.cuda.synchronize()
    for u, v in zip(got, want):
        assert torch.equal(u, v)
