"""Products of packed codes through the kernel that brings them straight to LDS: against the oracle on
sampled outputs, at the edges of its tiles and stages, in parts, behind a mask and written past the caches."""
import numpy as np
import pytest
import torch

from launches import launched
from oracle import capi
from paper_2310_03675_amd import binding as B

pytestmark = pytest.mark.gpu
SA, SB = np.float32(0.37), np.float32(0.0113)
DQ = np.float32(np.float32(SA * SB) * np.float32(1 / 8))


def codes(rng, R, D, kind, b):
    lo, hi = -(1 << (b - 1)), (1 << (b - 1)) - 1
    if kind == "lowest":
        return np.full((R, D), lo, dtype=np.int8)
    if kind == "uniform":
        return rng.integers(lo, hi + 1, (R, D), dtype=np.int8)
    return np.clip(np.rint(rng.standard_normal((R, D)) * 1.8), lo, hi).astype(np.int8)


# rows and columns that end inside a tile and a block of 32; contractions that end inside a stage of 128, a tile and 32 codes
# (8, 40, 136, 264), of one stage and of many; up to 64 columns, unsplit and in parts whose totals fit 16 bits (27 x 64,
# 300 x 64) and do not (tiles that cannot saturate); 512 columns in whole lines, 135 MB
@pytest.mark.parametrize("RA,RB,D", [(4100, 1290, 128), (30001, 130, 136), (12544, 700, 8), (2214, 10688, 40),
                                     (131001, 63, 264), (27, 64, 131072), (300, 64, 16456), (66000, 512, 96)])
@pytest.mark.parametrize("s,a", [(32, 8), (64, 8), (32, 32)])
@pytest.mark.parametrize("kind,b", [("gauss", 4), ("uniform", 3), ("lowest", 4)])
def test_gemm_codes_packed(RA, RB, D, s, a, kind, b):
    print(f"gemm_codes RA={RA} RB={RB} D={D} s={s} a={a} {kind} b={b}", flush=True)
    rng = np.random.default_rng(RA + D + s)
    cA, cB = codes(rng, RA, D, kind, b), codes(rng, RB, D, kind, b)
    qA, qB = (torch.from_numpy(capi.pack_codes(c, b)).to("cuda:0") for c in (cA, cB))
    sA, sB = torch.tensor([SA], device="cuda:0"), torch.tensor([SB], device="cuda:0")
    out, acc = torch.full((RA + 1, RB), -1.0, device="cuda:0"), torch.empty(RA, RB, dtype=torch.int32, device="cuda:0")
    ran = launched(lambda: B.gemm_codes(qA, qB, b, b, sA, sB, D, 8, a, s, out=out[:RA], acc=acc))
    torch.cuda.synchronize()
    assert "lines_gemm_i4_kernel" in ran, ran
    assert bool((out[RA] == -1.0).all())                 # nothing behind the output
    ii, jj = rng.integers(0, RA, 1024), rng.integers(0, RB, 1024)
    ii[:2], jj[:2] = (0, RA - 1), (0, RB - 1)
    want = capi.tiled_matmul_sampled(cA, cB, s, a, ii, jj)
    assert np.array_equal(acc.cpu().numpy()[ii, jj], want)
    assert np.array_equal(out.cpu().numpy()[ii, jj], want.astype(np.float32) * DQ)


@pytest.mark.parametrize("M,K,N", [(4099, 1153, 128), (131001, 60, 96), (66000, 512, 64)])
def test_masked_input_gradient(M, K, N):
    g = torch.Generator(device="cuda:0").manual_seed(5)
    G, W, X = (torch.randn(s, generator=g, device="cuda:0") for s in ((M, N), (K, N), (M, K)))
    X[:, ::7] = 0.0
    op = B.Operand(4, B.ROUND_NEAREST, 1.0, 0)
    prm = B.Params(had_block=32, acc_bits=8, s=32, seed=0, A=op, B=op)
    got, plain = [], []
    ran = launched(lambda: got.append(B.gemm(B.GEMM_BWD_INPUT, G, W, M, K, N, prm, mask=X)[0]))
    assert "lines_gemm_i4_kernel" in ran and "relu_mask" not in ran, ran
    plain.append(B.gemm(B.GEMM_BWD_INPUT, G, W, M, K, N, prm)[0])
    assert torch.equal(got[0], torch.where(X > 0, plain[0], torch.zeros_like(plain[0])))


# parts of tiles that divide no stage: one line in the last rows of tiles, slices of 16 bits that the lowest codes fill (480 codes
# of 64 each) and of 32
@pytest.mark.parametrize("RA,RB,D,s", [(64, 128, 15384, 96), (300, 512, 15416, 96), (129, 129, 100000, 96), (129, 129, 99968, 160),
                                       (129, 512, 131080, 96), (130, 385, 50056, 224)])
@pytest.mark.parametrize("kind", ["gauss", "lowest"])
def test_parts_of_no_whole_stages(RA, RB, D, s, kind):
    print(f"gemm_codes RA={RA} RB={RB} D={D} s={s} a=32 {kind}", flush=True)
    rng = np.random.default_rng(D + s)
    cA, cB = codes(rng, RA, D, kind, 4), codes(rng, RB, D, kind, 4)
    qA, qB = (torch.from_numpy(capi.pack_codes(c, 4)).to("cuda:0") for c in (cA, cB))
    sA, sB = torch.tensor([SA], device="cuda:0"), torch.tensor([SB], device="cuda:0")
    out, acc = B.gemm_codes(qA, qB, 4, 4, sA, sB, D, 8, 32, s)
    ii, jj = rng.integers(0, RA, 1024), rng.integers(0, RB, 1024)
    ii[:64], jj[64:128] = RA - 1, RB - 1
    want = capi.tiled_matmul_sampled(cA, cB, s, 32, ii, jj)
    assert np.array_equal(acc.cpu().numpy()[ii, jj], want)
    assert np.array_equal(out.cpu().numpy()[ii, jj], want.astype(np.float32) * DQ)


# split contractions, whose parts the pass behind them adds and masks, that end 8, 16 and 24 codes behind whole 32s
@pytest.mark.parametrize("M,K,N", [(1024, 2080, 1000), (5060, 412, 1360), (4096, 1024, 2040)])
@pytest.mark.parametrize("s", [32, 64])
def test_masked_input_gradient_in_parts(M, K, N, s):
    print(f"bwd_input M={M} K={K} N={N} s={s}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(M + N + s)
    G, W, X = (torch.randn(shape, generator=g, device="cuda:0") for shape in ((M, N), (K, N), (M, K)))
    X[:, ::7] = 0.0
    op = B.Operand(4, B.ROUND_NEAREST, 1.0, 0)
    prm = B.Params(had_block=8, acc_bits=8, s=s, seed=0, A=op, B=op)
    want, acc, _ = B.gemm(B.GEMM_BWD_INPUT, G, W, M, K, N, prm, want_acc=True)
    masked = torch.where(X > 0, want, torch.zeros_like(want))
    got = []
    ran = launched(lambda: got.append(B.gemm(B.GEMM_BWD_INPUT, G, W, M, K, N, prm, mask=X, want_acc=True)))
    assert "reduce" in ran and "relu_mask" not in ran, ran
    assert torch.equal(got[0][0], masked) and torch.equal(got[0][1], acc)
    _, saved = B.layer_fwd(X, W, prm, prm)
    dX, dW = B.layer_bwd(G, W, saved, K, prm, prm, mask=X)
    assert torch.equal(dX, masked)
    assert torch.equal(dW, B.gemm(B.GEMM_BWD_WEIGHT, X, G, M, K, N, prm)[0])


# Tiles asked whether they can saturate, where there are more than 512 workgroups of them: codes in patches that pass and that do
# not, the first stage passing (the test goes on) and failing (it is given up behind the first), every tile saturating upwards
# (255 of them), contractions that end inside a stage and a pair of tiles
KINDS = ["patches", "first passes", "first fails", "upwards"]


def asked_codes(rng, R, D, kind):
    if kind == "upwards":
        return np.full((R, D), 7, dtype=np.int8)
    full = rng.integers(-8, 8, (R, D), dtype=np.int8)
    small = rng.integers(-1, 2, (R, D), dtype=np.int8)
    which = rng.random((-(-R // 96), -(-D // 80))) < 0.3
    which = np.repeat(np.repeat(which, 96, 0), 80, 1)[:R, :D]
    if kind == "first fails":
        which[:, :128] = True
    else:
        which[:, :128] = False if kind == "first passes" else which[:, :128] & (rng.random() < 0.5)
    return np.where(which, full, small).astype(np.int8)


def multiply_and_compare(rng, cA, cB):
    """The kernels that ran; outputs drawn and those of the last rows against the oracle's."""
    (RA, D), RB = cA.shape, cB.shape[0]
    qA, qB = (torch.from_numpy(capi.pack_codes(c, 4)).to("cuda:0") for c in (cA, cB))
    sA, sB = torch.tensor([SA], device="cuda:0"), torch.tensor([SB], device="cuda:0")
    got = []
    ran = launched(lambda: got.append(B.gemm_codes(qA, qB, 4, 4, sA, sB, D, 8, 8, 32)))
    ii, jj = rng.integers(0, RA, 4096), rng.integers(0, RB, 4096)
    ii[:2], jj[:2] = (0, RA - 1), (0, RB - 1)
    ii[2:66] = RA - 1
    want = capi.tiled_matmul_sampled(cA, cB, 32, 8, ii, jj)
    out, acc = got[0]
    assert np.array_equal(acc.cpu().numpy()[ii, jj], want)
    assert np.array_equal(out.cpu().numpy()[ii, jj], want.astype(np.float32) * DQ)
    return ran


@pytest.mark.parametrize("RA,RB,D", [(66001, 128, 1152), (4100, 4130, 736), (3000, 3001, 544), (8300, 1030, 8160)])
@pytest.mark.parametrize("kind", KINDS)
def test_tiles_that_are_asked(RA, RB, D, kind):
    print(f"gemm_codes RA={RA} RB={RB} D={D} {kind}", flush=True)
    rng = np.random.default_rng(RA + D)
    assert "lines_gemm_i4_kernel<3" in multiply_and_compare(rng, asked_codes(rng, RA, D, kind), asked_codes(rng, RB, D, kind))


# The same with lines that end inside 32 codes, 8, 16 and 24 behind the last whole ones: the next line's first codes, in the
# same 16 bytes, are no part of the sums
@pytest.mark.parametrize("RA,RB,D", [(16384, 1024, 1000), (3000, 3001, 592), (66001, 128, 536), (4100, 4130, 760), (8300, 1030, 8152)])
@pytest.mark.parametrize("kind", KINDS)
def test_tiles_that_are_asked_in_lines_that_end_inside_32_codes(RA, RB, D, kind):
    print(f"gemm_codes RA={RA} RB={RB} D={D} {kind}", flush=True)
    rng = np.random.default_rng(RA + D)
    multiply_and_compare(rng, asked_codes(rng, RA, D, kind), asked_codes(rng, RB, D, kind))
