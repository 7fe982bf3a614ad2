"""GPU parity of the any-shape quantizer: shapes that are multiples of nothing, both ways of
collecting the maxima (side by side, and in slots that were cleared), and tensors that ride along
in a launch of the two-axis kernel."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import capi
from paper_2310_03675_amd import binding as B
from paper_2310_03675_amd import workloads
from test_gpu_parity import check_quantize, dev, host, o_operand

pytestmark = pytest.mark.gpu
NE, ST = B.ROUND_NEAREST, B.ROUND_STOCHASTIC


LEFT = 0x7F                  # every byte of a used workspace: as a maximum 3.4e38


def check_dirty(T, axis, n, op, seed):
    rows, cols = T.shape
    lines, D = (rows, cols) if axis else (cols, rows)
    x, lib, cop = dev(T), B.load(), op.c()
    codes = torch.empty((lines, B.codes_pitch(D, op.b)), dtype=torch.uint8, device="cuda:0")
    scale = torch.empty(1, device="cuda:0")
    ws = torch.full((lib.hdqt_quantize_workspace_size(),), LEFT, dtype=torch.uint8, device="cuda:0")
    rc = lib.hdqt_quantize(x.data_ptr(), rows, cols, axis, n, C.byref(cop), seed, codes.data_ptr(), scale.data_ptr(),
                           ws.data_ptr(), ws.numel(), B._stream(None))
    want, want_scale, _ = capi.quantize(T, axis, n, o_operand(op), seed)
    assert rc == 0 and host(scale)[0] == want_scale and np.array_equal(host(codes), capi.pack_codes(want, op.b))


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("b,rounding", [(4, NE), (4, ST), (3, ST), (8, ST), (7, NE)])
@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 9), (9, 1), (63, 17), (64, 8), (65, 33), (192, 31), (256, 30),
                                       (130, 12), (128, 561), (561, 11)])
def test_quantize_any_shape(rows, cols, axis, b, rounding):
    rng = np.random.default_rng(rows * 1009 + cols)
    T = (rng.standard_normal((rows, cols)) * 2.0).astype(np.float32)
    for n in (1, 8, 64, 128, 256):
        check_quantize(T, axis, n, B.Operand(b, rounding, 0.975, 5), seed=0x1_0000_0007)


@pytest.mark.parametrize("rows,cols,axis", [(3001, 1001, 0), (3001, 1001, 1), (4160, 770, 0)])
def test_quantize_many_workgroups(rows, cols, axis):
    """More workgroups than maxima that stand side by side; a workspace with leftovers in it."""
    T = np.random.default_rng(rows).standard_normal((rows, cols)).astype(np.float32)
    check_quantize(T, axis, 64, B.Operand(4, ST, 1.0, 2), seed=3)
    check_dirty(T, axis, 64, B.Operand(4, ST, 1.0, 2), 3)


@pytest.mark.parametrize("rows,cols,axis,n", [(64, 40, 0, 64), (2048, 1024, 1, 64), (4096, 1024, 1, 64), (4096, 1024, 0, 256)])
def test_workspace_with_leftovers(rows, cols, axis, n):
    """Maxima side by side, where nothing is cleared, and the tuned kernels' slots."""
    T = np.random.default_rng(rows).standard_normal((rows, cols)).astype(np.float32)
    check_dirty(T, axis, n, B.Operand(4, NE, 1.0, 2), 3)


def kernels_of(call):
    B.profile_enable(True)
    B.profile_collect()
    call()
    torch.cuda.synchronize()
    B.profile_enable(False)
    return {name for name, (launches, _) in B.profile_collect().items() if launches}


# a tensor without company on both sides of the lines between the any-shape kernel and the tuned ones
@pytest.mark.parametrize("rows,cols,axis,n,b,rounding,kernel", [
    (2048, 1024, 1, 64, 4, NE, "any"), (2056, 1024, 1, 64, 4, NE, "row"), (4096, 1024, 1, 64, 8, ST, "row"),
    (2048, 1024, 0, 64, 4, NE, "any"), (2112, 1024, 0, 64, 4, NE, "col"), (4096, 2048, 0, 256, 4, NE, "col"),
    (5632, 512, 0, 64, 4, ST, "any"), (5696, 512, 0, 64, 4, ST, "col"), (4096, 640, 0, 128, 4, ST, "any"),
    (2048, 512, 0, 256, 4, NE, "any"), (2304, 512, 0, 256, 4, NE, "col"), (4096, 768, 0, 256, 8, ST, "col"),
    (5000, 1000, 0, 64, 8, ST, "any"), (24640, 192, 0, 64, 4, ST, "any"), (24640, 128, 0, 64, 4, ST, "col")])
def test_lone_tensor_takes_the_faster_kernel(rows, cols, axis, n, b, rounding, kernel):
    op = B.Operand(b, rounding, 1.0, 4)
    T = np.random.default_rng(rows + cols).standard_normal((rows, cols)).astype(np.float32)
    x = dev(T)
    assert f"fwht_{kernel}_quant" in kernels_of(lambda: B.quantize(x, axis, n, op, 7))
    check_quantize(T, axis, n, op, seed=7)


@pytest.mark.parametrize("kind,M,K,N,n,kernels", [
    (B.GEMM_FWD, 2048, 2048, 2048, 64, {"any"}), (B.GEMM_FWD, 2048, 4608, 512, 256, {"row", "col"}),
    (B.GEMM_BWD_WEIGHT, 16384, 512, 64, 256, {"col", "any"}), (B.GEMM_BWD_WEIGHT, 2048, 1152, 128, 256, {"any"}),
    (B.GEMM_BWD_WEIGHT, 6144, 512, 768, 128, {"col"}), (B.GEMM_BWD_WEIGHT, 16384, 128, 192, 256, {"any"})])
def test_operands_of_a_product_share_launches_where_that_is_faster(kind, M, K, N, n, kernels):
    layer = workloads.fc_layer(M, K, N, seed=2)
    P, Q = {B.GEMM_FWD: (layer.X, layer.W), B.GEMM_BWD_WEIGHT: (layer.X, layer.G)}[kind]
    P, Q = dev(P), dev(Q)
    prm = B.Params(had_block=n, acc_bits=8, s=32, seed=9, A=B.Operand(4, NE, 1.0, 0), B=B.Operand(4, ST, 1.0, 1))
    used = kernels_of(lambda: B.gemm(kind, P, Q, M, K, N, prm))
    assert {k for k in ("any", "row", "col", "dual") if f"fwht_{k}_quant" in used} == kernels
    out, acc, _ = B.gemm(kind, P, Q, M, K, N, prm, want_acc=True)
    axis = (1, 0) if kind == B.GEMM_FWD else (0, 0)
    (qa, sa), (qb, sb) = (B.quantize(t, a, n, o, 9) for t, a, o in zip((P, Q), axis, (prm.A, prm.B)))
    D = K if kind == B.GEMM_FWD else M
    want, want_acc = B.gemm_codes(qa, qb, 4, 4, sa, sb, D, B.n_eff(D, n), 8, 32)
    assert torch.equal(acc, want_acc) and torch.equal(out, want)


def test_zeros_and_lone_values():
    for rows, cols in ((65, 33), (64, 64)):
        for axis in (0, 1):
            T = np.zeros((rows, cols), np.float32)
            check_quantize(T, axis, 16, B.Operand(4, ST, 1.0, 2))
            T[-1, -1] = -3.0
            check_quantize(T, axis, 16, B.Operand(4, NE, 1.0, 2))


def reference_codes(T, axis, n, b):
    """Nearest rounding of the oracle's transform, by the definition, where values are not finite: the maximum
    is that of the numbers among the values, and what is no number times the step's inverse (also an
    infinity, whose inverse is zero) takes the lowest code."""
    D = T.shape[1] if axis else T.shape[0]
    with np.errstate(all="ignore"):
        y = capi.hadamard_transform(T, axis, B.n_eff(D, n))
        amax = np.float32(np.nanmax(np.abs(y)))
        v = y * np.float32(np.float32(1 << (b - 1)) / amax)
        q = np.clip(np.rint(v), -(1 << (b - 1)), (1 << (b - 1)) - 1)
    q = np.where(np.isnan(v), -(1 << (b - 1)), q).astype(np.int8)
    return np.ascontiguousarray(q if axis else q.T), np.float32(amax / np.float32(1 << (b - 1)))


@pytest.mark.parametrize("rows,cols", [(65, 33), (64, 96), (256, 24), (130, 561), (2304, 1024)])
@pytest.mark.parametrize("values", [(np.nan,), (np.inf,), (-np.inf, np.nan), (np.inf, -np.inf)])
def test_values_that_are_not_finite(rows, cols, values):
    """The any-shape kernel, and (the largest) the tuned ones."""
    T = np.random.default_rng(rows).standard_normal((rows, cols)).astype(np.float32)
    for i, v in enumerate(values):
        T[rows // 2, cols // 3 + i] = T[rows // 2 + i, cols // 3] = v
    for axis in (0, 1):
        for n in (1, 8, 64, 256):
            for b in (4, 8):
                want, want_scale = reference_codes(T, axis, n, b)
                print(f"quantize {T.shape} with {values} axis={axis} n={n} b={b}", flush=True)
                codes, scale = B.quantize(dev(T), axis, n, B.Operand(b))
                assert host(scale)[0] == want_scale
                assert np.array_equal(host(codes), capi.pack_codes(want, b))


@pytest.mark.parametrize("rows,cols", [(3, 5), (65, 33), (561, 11)])
def test_pad_nibble_when_the_inverse_of_the_step_overflows(rows, cols):
    """A maximum below 2^-125: one over the step is infinite, and zero times it no number.  The half byte
    behind the last code of an odd line is zero all the same."""
    T = (np.random.default_rng(rows).standard_normal((rows, cols)) * 1e-39).astype(np.float32)
    T[0, 0] = 0.0
    for axis in (0, 1):
        want, want_scale = reference_codes(T, axis, 1, 4)
        codes, scale = B.quantize(dev(T), axis, 1, B.Operand(4))
        got = host(codes)
        assert not (got[:, -1] >> 4).any()
        assert host(scale)[0] == want_scale and np.array_equal(got, capi.pack_codes(want, 4))


@pytest.mark.parametrize("M,K,N,n,dx", [(200, 132, 70, 64, True), (64, 256, 128, 16, True), (128, 561, 11, 64, True),
                                        (131, 27, 64, 32, False), (1024, 1152, 100, 64, True),
                                        (2048, 640, 70, 64, False), (1088, 576, 24, 64, True), (512, 640, 384, 256, True)])
def test_step_equals_three_products(M, K, N, n, dx):
    """One call's sets, small enough for the any-shape kernel, against each product by itself, and the two
    calls of a training loop against both."""
    check_step(M, K, N, (n, n, n), dx, {"any"})


# (the orders of the three products; what the tensors of the one call go to, riders not seen by name)
@pytest.mark.parametrize("M,K,N,n,dx,route", [
    (4096, 640, 70, (64, 64, 64), True, {"dual"}),            # X in tiles, all of W and G riding
    (4096, 1152, 128, (64, 64, 64), True, {"dual"}),          # G leaves the tiles and rides with X and W
    (4096, 1152, 256, (64, 256, 32), True, {"dual"}),         # riders of order 256
    (4096, 640, 70, (64, 64, 64), False, {"dual"}),
    (32768, 640, 70, (64, 64, 64), True, {"dual"}),           # more workgroups than maxima side by side
    (33, 70001, 64, (64, 64, 64), True, {"any"}),             # ... of the any-shape kernel's launch
    (16384, 640, 64, (64, 64, 256), True, {"row", "col", "dual"})])
def test_riders_equal_three_products(M, K, N, n, dx, route):
    """Small tensors in the launches of the two-axis kernel, and sets that the kernels share."""
    check_step(M, K, N, n, dx, route)


def check_step(M, K, N, n, dx, route):
    layer = workloads.fc_layer(M, K, N, seed=7)
    X, W, G = (dev(t) for t in (layer.X, layer.W, layer.G))
    op = lambda rnd, tid: B.Operand(4, rnd, 1.0, tid)
    prm = [B.Params(had_block=order, acc_bits=8, s=32, seed=9, A=a, B=b)
           for order, (a, b) in zip(n, ((op(NE, 0), op(NE, 1)), (op(ST, 6), op(NE, 5)), (op(NE, 8), op(ST, 10))))]
    kinds = ((B.GEMM_FWD, X, W), (B.GEMM_BWD_INPUT, G, W), (B.GEMM_BWD_WEIGHT, X, G))
    want = [B.gemm(kind, P, Q, M, K, N, p)[0] for (kind, P, Q), p in zip(kinds, prm)]
    if not dx:
        prm[1] = None
    lib, ref = B.load(), [C.byref(p.c()) if p else None for p in prm]
    left = lambda size: torch.full((size,), LEFT, dtype=torch.uint8, device="cuda:0")
    out = (torch.empty_like(want[0]), torch.empty_like(X) if dx else None, torch.empty_like(W))
    used = kernels_of(lambda: B.layer_step(X, W, G, *prm, out=out,
                                           workspace=left(B.layer_step_workspace_size(M, K, N, *prm))))
    assert {k for k in ("any", "row", "col", "dual") if any(name.startswith(f"fwht_{k}_quant") for name in used)} == route
    Z, dX, dW = out
    assert torch.equal(Z, want[0]) and torch.equal(dW, want[2]) and (not dx or torch.equal(dX, want[1]))
    Z, saved = B.layer_fwd(X, W, prm[0], prm[2], workspace=left(lib.hdqt_layer_fwd_workspace_size(M, K, N, ref[0], ref[2])))
    dX, dW = B.layer_bwd(G, W, saved, K, prm[1], prm[2],
                         workspace=left(lib.hdqt_layer_bwd_workspace_size(M, K, N, ref[1], ref[2])))
    assert torch.equal(Z, want[0]) and torch.equal(dW, want[2]) and (not dx or torch.equal(dX, want[1]))
    codes, scale, _ = capi.quantize(layer.X.numpy(), 1, n[0], o_operand(prm[0].A), 9)
    got, got_scale = B.quantize(X, 1, n[0], prm[0].A, 9)
    assert host(got_scale)[0] == scale and np.array_equal(host(got), capi.pack_codes(codes, 4))
