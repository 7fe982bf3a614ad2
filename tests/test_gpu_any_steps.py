"""The any-shape quantizer where a workgroup takes several pieces of a tensor: code and scale against
the oracle, the last pieces cut by both edges of the tensor."""
import numpy as np
import pytest
import torch

from launches import launched
from oracle import capi
from paper_2310_03675_amd import binding as B

pytestmark = pytest.mark.gpu


def in_steps(call):
    """Whether the any-shape kernel takes a call's tensors in steps."""
    names = launched(call)
    found = [many for many in (False, True) if f"fwht_any_kernel<true, {str(many).lower()}>" in names]
    assert len(found) == 1, names
    return found[0]


# (pieces, of them along axis 0): from 3072 on, with half of them or more along axis 0
@pytest.mark.parametrize("kind,M,K,N,steps", [
    (B.GEMM_FWD, 20884, 301, 32, False),            # 3105, 5
    (B.GEMM_FWD, 53894, 301, 99, False),            # 8020, 20
    (B.GEMM_BWD_INPUT, 4003, 99, 2001, False),      # 4023, 0
    (B.GEMM_BWD_WEIGHT, 22513, 250, 32, True),      # 3168, all
    (B.GEMM_BWD_WEIGHT, 21021, 250, 32, False),     # 2961, all
    (B.GEMM_BWD_WEIGHT, 97001, 99, 35, True)])      # 9096, all: four to a workgroup
def test_which_products_go_in_steps(kind, M, K, N, steps):
    sizes = {B.GEMM_FWD: ((M, K), (K, N)), B.GEMM_BWD_INPUT: ((M, N), (K, N)), B.GEMM_BWD_WEIGHT: ((M, K), (M, N))}[kind]
    P, Q = (torch.ones(s, device="cuda:0") for s in sizes)
    op = B.Operand(4, B.ROUND_NEAREST, 1.0, 0)
    prm = B.Params(had_block=64, acc_bits=8, s=32, seed=0, A=op, B=op)
    assert in_steps(lambda: B.gemm(kind, P, Q, M, K, N, prm)) == steps


@pytest.mark.parametrize("rows,cols,axis,steps", [(20884, 301, 1, False), (5001, 1301, 0, True), (5001, 1229, 0, True),
                                                  (5001, 1209, 0, False), (100003, 601, 1, False)])
def test_which_tensors_go_in_steps(rows, cols, axis, steps):
    T = torch.ones((rows, cols), device="cuda:0")
    assert in_steps(lambda: B.quantize(T, axis, 64, B.Operand(4, B.ROUND_NEAREST, 1.0, 0), 0)) == steps


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
