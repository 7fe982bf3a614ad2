"""The any-shape quantizer where a workgroup takes several pieces of a tensor: code and scale against
the oracle, the last pieces cut by both edges of the tensor."""
import numpy as np
import pytest
import torch

from oracle import capi
from paper_2310_03675_amd import binding as B

pytestmark = pytest.mark.gpu


# 2048 values to a piece: 3185 to 6500 pieces, two to four to a workgroup; orders above 64 along axis 0 go
# through LDS from one wave to another
@pytest.mark.parametrize("rows,cols,axis,n", [(5001, 1301, 0, 64), (5001, 1301, 1, 64), (5120, 1301, 0, 256),
                                              (1301, 5120, 1, 256), (100003, 61, 0, 64), (50001, 131, 1, 1)])
@pytest.mark.parametrize("b", [4, 8])
@pytest.mark.parametrize("rounding", [B.ROUND_NEAREST, B.ROUND_STOCHASTIC])
def test_quantize_in_steps(rows, cols, axis, n, b, rounding):
    print(f"quantize {rows}x{cols} axis={axis} n={n} b={b} rounding={rounding}", flush=True)
    T = torch.randn((rows, cols), generator=torch.Generator().manual_seed(rows + cols))
    op = B.Operand(b, rounding, 0.975, 5)
    got, scale = B.quantize(T.to("cuda:0"), axis, n, op, 9)
    torch.cuda.synchronize()
    codes, want_scale, _ = capi.quantize(T.numpy(), axis, n, capi.Operand(b=b, round_mode=rounding, clip=0.975, tensor_id=5), 9)
    assert float(scale) == float(want_scale)
    want = np.ascontiguousarray(capi.pack_codes(codes, b)).view(np.uint8).reshape(-1)
    assert np.array_equal(got.cpu().numpy().view(np.uint8).reshape(-1), want)
