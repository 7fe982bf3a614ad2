"""The convolution source where its tiles are taken in several steps of one wave, end inside a
workgroup, or lie in images too narrow for whole pieces of a row."""
import numpy as np
import pytest
import torch

from oracle import capi
from paper_2310_03675_amd import binding as B
from test_gpu_conv import NE, ST, o_op, unfold

pytestmark = pytest.mark.gpu

# (batch, C, H, W, kh, kw, n): 1080 workgroups' tiles in two steps, 57 rows of tiles in groups of four;
# images two and one pixels wide
SHAPES = [(57, 512, 8, 8, 3, 3, 64), (2, 64, 32, 2, 3, 3, 32), (1, 64, 128, 1, 3, 1, 8)]


@pytest.mark.parametrize("batch,C,H,W,kh,kw,n", SHAPES)
@pytest.mark.parametrize("rounding,b", [("nearest", 4), ("stochastic", 4), ("nearest", 8)])
@pytest.mark.parametrize("signed", [False, True])
def test_quantize_dual_im2col_steps(batch, C, H, W, kh, kw, n, rounding, b, signed):
    g = torch.Generator().manual_seed(batch + 3 * C + H)
    act = torch.randn((batch, C, H, W), generator=g)
    act = act if signed else torch.relu(act)
    X = unfold(act, kh, kw)
    r = ST if rounding == "stochastic" else NE
    op1, op0 = B.Operand(b, r, 1.0, 3), B.Operand(b, r, 0.975, 9)
    print(f"im2col source: act {tuple(act.shape)} window {kh}x{kw}, n={n}, {rounding}, b={b}, signed={signed}", flush=True)
    c1, s1, c0, s0 = B.quantize_dual_im2col(act.to("cuda:0"), kh, kw, n, op1, op0, seed=5)
    torch.cuda.synchronize()
    for axis, got_c, got_s, op in ((1, c1, s1, op1), (0, c0, s0, op0)):
        codes, scale, _ = capi.quantize(X.numpy(), axis, n, o_op(op), 5)
        assert float(got_s) == float(scale)
        assert np.array_equal(got_c.cpu().numpy().reshape(-1).view(np.uint8),
                              np.ascontiguousarray(capi.pack_codes(codes, b)).reshape(-1).view(np.uint8))
