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


def pieces(R, C, axis, n):
    """Of 2048 values, as the kernel cuts them."""
    if axis:
        return -(-R * -(-C // 8) // 256)
    wide = 1 if B.n_eff(R, n) > 64 or C <= 8 else 2 if C <= 16 else 4
    return -(-C // (8 * wide)) * -(-R // (64 * 4 // wide))


# orders used 1, 8, 64 and 256 (which goes through LDS from one wave to another), two to four pieces to a workgroup, the
# last ones cut by both edges of the tensor
@pytest.mark.parametrize("rows,cols,n,order,steps", [(5001, 1301, 64, 1, 2), (100003, 61, 64, 1, 2), (40008, 157, 64, 8, 2),
                                                     (4992, 1301, 64, 64, 2), (8000, 1301, 64, 64, 3), (12032, 1301, 64, 64, 4),
                                                     (5120, 1301, 256, 256, 2), (8192, 1301, 256, 256, 3), (10240, 1301, 256, 256, 4)])
@pytest.mark.parametrize("b", [4, 8])
@pytest.mark.parametrize("rounding", [B.ROUND_NEAREST, B.ROUND_STOCHASTIC])
def test_quantize_in_steps(rows, cols, n, order, steps, b, rounding):
    print(f"quantize {rows}x{cols} n={n} b={b} rounding={rounding}", flush=True)
    assert B.n_eff(rows, n) == order and min(pieces(rows, cols, 0, n) // 1536, 4) == steps
    T = torch.randn((rows, cols), generator=torch.Generator().manual_seed(rows + cols))
    op, on_device, got = B.Operand(b, rounding, 0.975, 5), T.to("cuda:0"), []
    assert in_steps(lambda: got.extend(B.quantize(on_device, 0, n, op, 9)))
    got, scale = got
    codes, want_scale, _ = capi.quantize(T.numpy(), 0, n, capi.Operand(b=b, round_mode=rounding, clip=0.975, tensor_id=5), 9)
    assert float(scale) == float(want_scale)
    want = np.ascontiguousarray(capi.pack_codes(codes, b)).view(np.uint8).reshape(-1)
    assert np.array_equal(got.cpu().numpy().view(np.uint8).reshape(-1), want)


# a layer's six tensors in one launch: (M, K, N, order asked for, pieces to a workgroup, maxima side by side): orders along the lines of 64
# and 256, along the columns up to 256
@pytest.mark.parametrize("M,K,N,n,steps,side_by_side", [
    (16380, 254, 18, 256, 2, True), (20000, 201, 64, 64, 3, True), (20000, 256, 100, 64, 4, True), (20000, 256, 100, 256, 4, True),
    (19968, 250, 100, 256, 4, True), (9000, 1023, 333, 64, 4, False)])
@pytest.mark.parametrize("b", [4, 8])
def test_a_layer_in_steps(M, K, N, n, steps, side_by_side, b):
    cut = [pieces(*t, n) for t in ((M, K, 1), (M, K, 0), (M, N, 1), (M, N, 0), (K, N, 0), (K, N, 1))]
    assert min(sum(cut) // 1536, 4) == steps and all(-(-c // steps) <= 1024 for c in cut) == side_by_side
    g = torch.Generator().manual_seed(M + K)
    host = [torch.randn(s, generator=g) for s in ((M, K), (K, N), (M, N))]
    X, W, G = (t.to("cuda:0") for t in host)
    op = lambda rounding, tid: B.Operand(b, rounding, 0.975, tid)
    NE, ST, acc = B.ROUND_NEAREST, B.ROUND_STOCHASTIC, 8 if b == 4 else 16
    prm = [B.Params(had_block=n, acc_bits=acc, s=32, seed=3, A=op(*i), B=op(*j))
           for i, j in (((NE, 0), (NE, 1)), ((ST, 6), (NE, 5)), ((NE, 8), (ST, 10)))]
    print(f"layer M={M} K={K} N={N} n={n} b={b}", flush=True)
    got = []
    assert in_steps(lambda: got.extend(B.layer_step(X, W, G, *prm)[:3]))
    for out, p, (A, axis_a, a), (Q, axis_q, q), D in ((got[0], prm[0], (X, 1, 0), (W, 0, 1), K), (got[1], prm[1], (G, 1, 2), (W, 1, 1), N),
                                                      (got[2], prm[2], (X, 0, 0), (G, 0, 2), M)):
        codes, scales = [], []
        for T, axis, o in ((host[a].numpy(), axis_a, p.A), (host[q].numpy(), axis_q, p.B)):
            c, scale, _ = capi.quantize(T, axis, n, capi.Operand(b=b, round_mode=o.round, clip=o.clip, tensor_id=o.tensor_id), 3)
            codes.append(torch.from_numpy(capi.pack_codes(c, b)).to("cuda:0"))
            scales.append(torch.tensor([float(scale)], device="cuda:0"))
        want = B.gemm_codes(*codes, b, b, *scales, D, B.n_eff(D, n), acc, 32, want_acc=False)[0]
        assert torch.equal(out, want)
