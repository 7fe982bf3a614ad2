"""Products of codes with a byte each through the kernel that brings them straight to LDS: against the
oracle on sampled outputs, at the edges of its tiles and stages and in parts."""
import numpy as np
import pytest
import torch

from launches import launched
from oracle import capi
from paper_2310_03675_amd import binding as B

pytestmark = pytest.mark.gpu


# rows inside a tile of 128 and a block of 32, contractions that end inside a stage of 128 and of one stage alone;
# tiles of one stage, of two and one tile; in one part and in several (512 x 4608, 448 x 610)
@pytest.mark.parametrize("RA,RB,D", [(4096, 1024, 128), (2081, 1935, 656), (2049, 4100, 144), (512, 4608, 2048),
                                     (448, 610, 14864)])
@pytest.mark.parametrize("s,a", [(128, 8), (256, 16), (128, 32), (40000, 12)])
@pytest.mark.parametrize("kind,b", [("gauss", 8), ("uniform", 5), ("lowest", 8)])
def test_gemm_codes_bytes(RA, RB, D, s, a, kind, b):
    print(f"gemm_codes RA={RA} RB={RB} D={D} s={s} a={a} {kind} b={b}", flush=True)
    rng = np.random.default_rng(RA + D + s)
    lo, hi = -(1 << (b - 1)), (1 << (b - 1)) - 1
    make = {"lowest": lambda R: np.full((R, D), lo, dtype=np.int8),
            "uniform": lambda R: rng.integers(lo, hi + 1, (R, D), dtype=np.int8),
            "gauss": lambda R: np.clip(np.rint(rng.standard_normal((R, D)) * 25), lo, hi).astype(np.int8)}[kind]
    cA, cB = make(RA), make(RB)
    qA, qB = (torch.from_numpy(capi.pack_codes(c, b)).to("cuda:0") for c in (cA, cB))
    sA, sB = torch.tensor([0.37], device="cuda:0"), torch.tensor([0.0113], device="cuda:0")
    out, acc = torch.full((2, RA, RB), -1.0, device="cuda:0"), torch.empty(RA, RB, dtype=torch.int32, device="cuda:0")
    ran = launched(lambda: B.gemm_codes(qA, qB, b, b, sA, sB, D, 16, a, s, out=out[0], acc=acc))
    torch.cuda.synchronize()
    # (one tile of 448 x 610 cannot be split, and goes to the small products)
    assert ("gemm_small_kernel" if (RA, s) == (448, 40000) else "gemm_bytes_kernel") in ran, ran
    assert bool((out[1] == -1.0).all())                  # nothing behind the output
    ii, jj = rng.integers(0, RA, 512), rng.integers(0, RB, 512)
    ii[:2], jj[:2] = (0, RA - 1), (0, RB - 1)
    want = capi.tiled_matmul_sampled(cA, cB, s, a, ii, jj)
    assert np.array_equal(acc.cpu().numpy()[ii, jj], want)
    dq = np.float32(np.float32(np.float32(0.37) * np.float32(0.0113)) * np.float32(1 / 16))
    assert np.array_equal(out[0].cpu().numpy()[ii, jj], want.astype(np.float32) * dq)
