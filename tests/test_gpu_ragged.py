"""GPU parity at sizes that are multiples of nothing: contraction lengths whose rows of codes are
no whole dwords (the feature counts of sensor data, a first convolution's 27, prime sizes), every
epilogue of the matrix-core kernel, and the outputs only its flexible instances write."""
import numpy as np
import pytest
import torch

from oracle import capi
from paper_2310_03675_amd import binding as B
from paper_2310_03675_amd import workloads
from test_gpu_parity import assert_close_f32, check_gemm_codes, dev, host, o_params, random_codes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [1, 27, 31, 33, 100, 127, 129, 243, 405, 561, 1148])
def test_gemm_codes_any_contraction_length(D):
    """Row pitches of every phase modulo 4; half the codes at the range ends, so that a code of the
    next row (or of the last row's slack) leaking in would change a saturating tile.  One tile,
    exact tiles, a short last tile; one column tile and two."""
    for bA, bB, settings in ((4, 4, ((32, 8), (64, 8), (16, 8), (32, 12), (64, 12), (16, 9), (16, 6), (96, 32), (128, 16),
                                     (256, 16), (2048, 32))),
                             (8, 8, ((32, 16), (64, 16), (16, 16), (16, 12), (96, 32), (128, 32), (32, 12)))):
        for s, a in settings:
            check_gemm_codes(131, 37, D, bA, bB, s, a, extreme=0.5)
            check_gemm_codes(65, 150, D, bA, bB, s, a, extreme=0.05)


def test_gemm_codes_any_contraction_length_split():
    check_gemm_codes(64, 70, 4099, 4, 4, 32, 8, extreme=0.3)
    check_gemm_codes(100, 60, 16387, 4, 4, 64, 12, extreme=0.3)
    check_gemm_codes(33, 40, 4097, 7, 8, 32, 16, extreme=0.3)
    check_gemm_codes(33, 40, 4098, 4, 4, 16, 8, extreme=0.3)


@pytest.mark.parametrize("D,b,s,a", [(96, 4, 16, 8), (96, 4, 32, 12), (96, 8, 32, 16), (96, 6, 96, 32), (97, 4, 32, 8),
                                     (27, 4, 32, 8), (99, 8, 16, 12)])
def test_outputs_of_the_flexible_instances(D, b, s, a):
    """bfloat16 and masked input gradients where an epilogue has no instance of its own for them."""
    M, K = 130, 67
    layer = workloads.fc_layer(M, K, D, seed=5)
    X = torch.relu(layer.X)
    prm = B.Params(had_block=32, acc_bits=a, s=s, seed=3, A=B.Operand(b, B.ROUND_STOCHASTIC, 1.0, 6), B=B.Operand(b))
    print(f"flexible outputs D={D} b={b} s={s} a={a}", flush=True)
    G, W = dev(layer.G), dev(layer.W)
    ref = capi.gemm(capi.BWD_INPUT, layer.G.numpy(), layer.W.numpy(), M, K, D, o_params(prm))
    out, acc, _ = B.gemm(B.GEMM_BWD_INPUT, G, W, M, K, D, prm, want_acc=True, mask=dev(X))
    assert np.array_equal(host(acc), ref["acc"])
    assert_close_f32(host(out), capi.relu_mask(ref["out"], X.numpy()))
    narrow, _, _ = B.gemm(B.GEMM_BWD_INPUT, G, W, M, K, D, prm, bf16=True)
    plain, _, _ = B.gemm(B.GEMM_BWD_INPUT, G, W, M, K, D, prm)
    assert torch.equal(narrow, plain.to(torch.bfloat16))
