"""Large products of packed codes, which multiply through the 6-bit floating-point matrix instructions:
against the oracle on sampled outputs, and against the integer kernel (which runs where the workspace
does not hold the codes' other form) on all of them, bit for bit."""
import numpy as np
import pytest
import torch

from launches import launched
from oracle import capi
from paper_2310_03675_amd import binding as B

pytestmark = pytest.mark.gpu


def codes(rng, R, D, kind, b):
    lo, hi = -(1 << (b - 1)), (1 << (b - 1)) - 1
    if kind == "lowest":
        return np.full((R, D), lo, dtype=np.int8)
    if kind == "uniform":
        return rng.integers(lo, hi + 1, (R, D), dtype=np.int8)
    return np.clip(np.rint(rng.standard_normal((R, D)) * 1.8), lo, hi).astype(np.int8)


# rows that end inside a block of 32, contractions that end inside a stage of 128 and inside a tile of 64;
# tiles of 64 with 8-bit accumulators, and tiles that cannot saturate
@pytest.mark.parametrize("RA,RB,D", [(4096, 4096, 2048), (4137, 4005, 2080), (3969, 4100, 2240), (2100, 4200, 16384)])
@pytest.mark.parametrize("s,a", [(64, 8), (16, 16), (256, 32)])
@pytest.mark.parametrize("kind,b", [("gauss", 4), ("uniform", 4), ("lowest", 4), ("uniform", 3)])
def test_gemm_codes_expanded(RA, RB, D, s, a, kind, b):
    print(f"gemm_codes RA={RA} RB={RB} D={D} s={s} a={a} {kind} b={b}", flush=True)
    rng = np.random.default_rng(RA + D + s)
    cA, cB = codes(rng, RA, D, kind, b), codes(rng, RB, D, kind, b)
    qA, qB = (torch.from_numpy(capi.pack_codes(c, b)).to("cuda:0") for c in (cA, cB))
    sA, sB = torch.tensor([0.37], device="cuda:0"), torch.tensor([0.0113], device="cuda:0")
    got = {}
    room = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda:0")
    for name, ws in (("gemm_six_kernel", room(B.load().hdqt_gemm_codes_workspace_size(RA, RB, D, s))), ("gemm_i4_kernel", room(256))):
        ran = launched(lambda: got.update({name: B.gemm_codes(qA, qB, b, b, sA, sB, D, 32, a, s, workspace=ws)}))
        assert name in ran and (name == "gemm_six_kernel") == ("gemm_six_kernel" in ran), ran
    (out, acc), (out_i, acc_i) = got.values()
    torch.cuda.synchronize()
    assert torch.equal(acc, acc_i) and torch.equal(out, out_i)
    ii, jj = rng.integers(0, RA, 512), rng.integers(0, RB, 512)
    ii[:2], jj[:2] = (0, RA - 1), (0, RB - 1)
    assert np.array_equal(acc.cpu().numpy()[ii, jj], capi.tiled_matmul_sampled(cA, cB, s, a, ii, jj))


@pytest.mark.parametrize("s", [24, 33])
def test_unclamped_tiles_of_no_whole_32_codes(s):
    """Otherwise the generic kernel's."""
    RA, RB, D = 4137, 6005, 2080
    rng = np.random.default_rng(s)
    cA, cB = (rng.integers(-8, 8, (R, D), dtype=np.int8) for R in (RA, RB))
    qA, qB = (torch.from_numpy(capi.pack_codes(c, 4)).to("cuda:0") for c in (cA, cB))
    one, got = torch.full((1,), 0.5, device="cuda:0"), []
    for name, n in (("gemm_six_kernel", B.load().hdqt_gemm_codes_workspace_size(RA, RB, D, s)), ("gemm_tiled_kernel", 256)):
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        assert name in launched(lambda: got.append(B.gemm_codes(qA, qB, 4, 4, one, one, D, 32, 32, s, workspace=ws)))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    ii, jj = rng.integers(0, RA, 512), rng.integers(0, RB, 512)
    ii[:2], jj[:2] = (0, RA - 1), (0, RB - 1)
    assert np.array_equal(got[0][1].cpu().numpy()[ii, jj], capi.tiled_matmul_sampled(cA, cB, s, 32, ii, jj))


def test_gemm_takes_a_workspace_without_room_for_it():
    """A workspace as large as the layout's parts, without the codes' other form behind them."""
    M, K, N = 3105, 2080, 2979
    op = B.Operand(4, B.ROUND_NEAREST, 1.0, 0)
    prm = B.Params(had_block=32, acc_bits=8, s=64, seed=0, A=op, B=op)
    g = torch.Generator(device="cuda:0").manual_seed(3)
    X, W = (torch.randn(s, generator=g, device="cuda:0") for s in ((M, K), (K, N)))
    full = B.workspace_size(B.GEMM_FWD, M, K, N, prm)
    least = B.workspace_layout(B.GEMM_FWD, M, K, N, prm).acc + 256
    assert least < full
    outs = []
    for n, name in ((full, "gemm_six_kernel"), (least, "gemm_i4_kernel")):
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        assert name in launched(lambda: outs.append(B.gemm(B.GEMM_FWD, X, W, M, K, N, prm, workspace=ws)[0]))
    assert torch.equal(*outs)


def test_masked_and_narrow_calls_hold_only_what_they_use():
    M, K, N = 3105, 2979, 2080
    op = B.Operand(4, B.ROUND_NEAREST, 1.0, 0)
    prm = B.Params(had_block=32, acc_bits=8, s=64, seed=0, A=op, B=op)
    least = B.load().hdqt_workspace_least(B.GEMM_BWD_INPUT, M, K, N, prm.c())
    G, W, X = (torch.ones(s, device="cuda:0") for s in ((M, N), (K, N), (M, K)))
    held = lambda **how: B.gemm(B.GEMM_BWD_INPUT, G, W, M, K, N, prm, **how)[2].numel()
    assert held(mask=X) == held(bf16=True) == least < held() == B.workspace_size(B.GEMM_BWD_INPUT, M, K, N, prm)
