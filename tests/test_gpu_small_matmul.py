"""GPU parity of the matmul on both sides of the line between its two kernels: small products (32 x 32
blocks, the contraction shared by a workgroup's waves) and those that an estimate gives to the large tiles:
long contractions, and outputs of many blocks.  Which kernel a case is for is checked with it."""
import pytest
import torch

from paper_2310_03675_amd import binding as B  # noqa: F401
from launches import launched
from test_gpu_parity import check_gemm_codes

pytestmark = pytest.mark.gpu

PACKED = ((32, 8), (64, 8), (16, 8), (32, 12), (16, 9), (16, 6), (96, 32), (128, 16), (256, 16), (8192, 32))
BYTES = ((32, 16), (64, 16), (64, 12), (64, 8), (16, 16), (16, 12), (96, 32), (32, 12), (256, 16))


def kernels(RA, RB, D, b, s, a):
    """What a product launches."""
    pitch = B.codes_pitch(D, b)
    qA, qB = (torch.zeros((n, pitch), dtype=torch.uint8, device="cuda") for n in (RA, RB))
    one = torch.ones(1, device="cuda")
    return launched(lambda: B.gemm_codes(qA, qB, b, b, one, one, D, 1, a, s, want_acc=False))


def both_kinds(RA, RB, D, extreme):
    for s, a in PACKED:
        check_gemm_codes(RA, RB, D, 4, 4, s, a, extreme=extreme)
    for s, a in BYTES:
        check_gemm_codes(RA, RB, D, 8, 7, s, a, extreme=extreme)


@pytest.mark.parametrize("D", [1, 8, 15, 16, 17, 31, 33, 64, 95, 250, 257, 561, 1000])
def test_small_products(D):
    """Contractions that end anywhere in a step, with more waves than steps and the other way
    round; blocks that end inside a row and a column block; one row."""
    both_kinds(33, 65, D, 0.4)
    both_kinds(1, 40, D, 0.1)


def test_small_products_of_long_contractions():
    both_kinds(40, 33, 4608, 0.3)
    both_kinds(33, 31, 4607, 0.05)


# (a single tile of packed codes stays with the small kernel at any length)
SINGLE = (8192, 32)


@pytest.mark.parametrize("D", [4640, 5003, 8200])
def test_contractions_on_either_kernel(D):
    both_kinds(131, 70, D, 0.3)


@pytest.mark.parametrize("D", [24008, 40003])
def test_long_contractions_on_large_tiles(D):
    """In parts, with rows that end inside a tile, a step and a dword."""
    for b, settings in ((4, PACKED), (7, BYTES)):
        for s, a in settings:
            assert ("gemm_small_kernel" in kernels(131, 70, D, b, s, a)) == ((s, a) == SINGLE)
    both_kinds(131, 70, D, 0.3)


@pytest.mark.parametrize("RA,RB,D", [(771, 1025, 6008), (515, 1027, 8203)])
@pytest.mark.parametrize("b,s,a", [(4, 64, 8), (4, 16, 9), (4, 96, 32), (4, 128, 16), (7, 32, 16), (7, 16, 12), (7, 64, 12)])
def test_many_large_tiles_in_parts(RA, RB, D, b, s, a):
    assert "gemm_small_kernel" not in kernels(RA, RB, D, b, s, a)
    check_gemm_codes(RA, RB, D, b, b, s, a, extreme=0.2)


@pytest.mark.parametrize("RA,RB,D,b,s,a", [(224, 256, 4480, 4, 16, 8), (2299, 128, 3712, 8, 64, 16), (288, 1024, 3456, 8, 128, 32),
                                           (224, 192, 4480, 4, 16, 8), (507, 512, 4240, 8, 16, 16), (1504, 192, 4480, 4, 256, 16),
                                           (539, 512, 3707, 8, 32, 16), (64, 192, 4235, 8, 256, 16)])
def test_long_chains_around_the_estimates(RA, RB, D, b, s, a):
    """Products inside the small kernel's lines, on both sides of what its estimate gives away."""
    check_gemm_codes(RA, RB, D, b, b, s, a, extreme=0.2)


@pytest.mark.parametrize("D", [27, 64, 100, 129, 520])
def test_many_blocks(D):
    both_kinds(1100, 1000, D, 0.2)


@pytest.mark.parametrize("D", [27, 64, 100, 129, 264])
def test_many_blocks_on_large_tiles(D):
    """Short contractions in one part, rows and columns that end inside a tile."""
    for b, settings in ((4, PACKED), (7, BYTES)):
        for s, a in settings:
            assert "gemm_small_kernel" not in kernels(4100, 2001, D, b, s, a)
    both_kinds(4100, 2001, D, 0.2)


@pytest.mark.parametrize("RB,D", [(37, 27), (64, 27), (64, 100), (50, 37), (64, 561)])
def test_narrow_outputs_with_ragged_rows(RB, D):
    for s, a in ((32, 8), (64, 8), (128, 16), (96, 32), (32, 32)):
        check_gemm_codes(17000, RB, D, 4, 4, s, a, extreme=0.3)


def test_tiles_of_64_bytes_streamed_output():
    """Outputs of 128 MB in whole lines take the instances with streaming stores, whose waves are one
    block high; in rows that end inside a line, the others."""
    for a in (8, 16):
        check_gemm_codes(8200, 4096, 192, 8, 8, 64, a, extreme=0.3)
        check_gemm_codes(8200, 4100, 192, 8, 8, 64, a, extreme=0.3)


@pytest.mark.parametrize("RA,RB", [(33000, 1024), (33000, 1025), (33000, 1040), (16400, 8208)])
@pytest.mark.parametrize("D,s,a", [(64, 32, 8), (48, 48, 8), (128, 64, 16), (27, 32, 8)])
def test_large_outputs_in_whole_and_broken_lines(RA, RB, D, s, a):
    """Either way of storing a large output against the same product in pieces that stay in the caches."""
    print(f"large outputs {RA}x{RB}x{D} s={s} a={a}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(RB)
    pitch = B.codes_pitch(D, 4)
    qA, qB = (torch.randint(0, 256, (n, pitch), dtype=torch.uint8, device="cuda", generator=g) for n in (RA, RB))
    one = torch.full((1,), 0.5, device="cuda")
    out, _ = B.gemm_codes(qA, qB, 4, 4, one, one, D, 1, a, s, want_acc=False)
    for r in range(0, RA, 8192):
        part, _ = B.gemm_codes(qA[r:r + 8192].contiguous(), qB, 4, 4, one, one, D, 1, a, s, want_acc=False)
        assert torch.equal(out[r:r + 8192], part)


@pytest.mark.parametrize("M,K,N,b,s,a", [
    (33000, 1040, 112, 4, 32, 8), (33000, 1032, 136, 4, 32, 8), (36000, 1168, 128, 4, 32, 8),
    (3564, 1152, 32, 8, 64, 16), (2058, 144, 64, 6, 32, 12), (4608, 1728, 16, 5, 16, 12), (3969, 144, 128, 4, 16, 12)])
def test_step_equals_its_products_where_they_take_other_routes(M, K, N, b, s, a):
    """A step streams Z and dX by lines of its own, and its small products keep a long chain in their
    launch; the same products by themselves give the same."""
    print(f"step {M}x{K}x{N} b={b} s={s} a={a}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K)
    X, W, G = (torch.randn(*n, device="cuda", generator=g) for n in ((M, K), (K, N), (M, N)))
    prm = [B.Params(had_block=64, acc_bits=a, s=s, seed=i, A=B.Operand(b, B.ROUND_NEAREST, 1.0, 2 * i),
                    B=B.Operand(b, B.ROUND_NEAREST, 1.0, 2 * i + 1)) for i in range(3)]
    step = B.layer_step(X, W, G, *prm)[:3]
    kinds = (B.GEMM_FWD, X, W), (B.GEMM_BWD_INPUT, G, W), (B.GEMM_BWD_WEIGHT, X, G)
    for got, (kind, P, Q), p in zip(step, kinds, prm):
        assert torch.equal(got, B.gemm(kind, P, Q, M, K, N, p)[0])


@pytest.mark.parametrize("s,a,b", [(32, 8, 4), (64, 12, 4), (16, 8, 4), (96, 10, 3), (32, 16, 8), (16, 12, 6), (64, 16, 5)])
def test_every_length_of_a_waves_chain(s, a, b):
    """Chains of no step to ten per wave, whole groups of loads and remainders, lines of every phase modulo
    four bytes, aligned and ragged, ends inside a step and inside a tile."""
    for D in [8 * k for k in (3, 5, 8, 9, 17, 33, 52, 63, 80, 129, 160)] + [k for k in (33, 65, 130, 199, 262, 325, 519, 645, 1034, 1282)]:
        check_gemm_codes(70, 45, D, b, b, s, a, extreme=0.2)


@pytest.mark.parametrize("RA,RB,D,b,s,a", [(481, 1001, 12312, 4, 32, 8), (600, 660, 4863, 4, 32, 8), (257, 640, 12287, 4, 32, 8),
                                           (320, 900, 2559, 4, 64, 12), (1000, 90, 3392, 8, 32, 16), (400, 130, 3391, 8, 16, 12)])
def test_products_with_less_work_than_lds_takes(RA, RB, D, b, s, a):
    assert "gemm_small_kernel<true>" not in kernels(RA, RB, D, b, s, a)
    check_gemm_codes(RA, RB, D, b, b, s, a, extreme=0.1)


@pytest.mark.parametrize("RA,RB,D,b,s,a", [
    (480, 1000, 12288, 4, 32, 8), (600, 900, 4863, 4, 32, 8), (520, 1001, 4735, 4, 32, 8), (480, 1000, 12287, 4, 32, 8), (512, 1024, 4736, 4, 32, 8),
    (700, 640, 6000, 4, 64, 12), (400, 900, 2559, 4, 64, 12), (400, 901, 2560, 4, 64, 12), (700, 641, 6000, 4, 96, 10), (500, 1000, 5184, 3, 96, 10),
    (1300, 500, 4120, 8, 32, 16), (1300, 501, 4100, 8, 32, 16), (500, 900, 4136, 8, 16, 16), (600, 600, 4160, 7, 16, 12),
    (1000, 300, 3392, 8, 32, 16), (601, 660, 4096, 8, 64, 12), (601, 661, 4108, 8, 64, 12)])
def test_products_through_lds(RA, RB, D, b, s, a):
    """Enough work for the chunks that go through LDS: whole chunks, what is left of one, an end inside a step."""
    assert "gemm_small_kernel<true>" in kernels(RA, RB, D, b, s, a)
    check_gemm_codes(RA, RB, D, b, b, s, a, extreme=0.1)


@pytest.mark.parametrize("M,K,N,b,s,a", [(517, 4736, 840, 4, 32, 8), (1032, 2504, 454, 4, 64, 12), (1156, 2052, 430, 7, 32, 12)])
def test_step_whose_products_share_a_launch_through_lds(M, K, N, b, s, a):
    """Lines in whole pieces, lines that are not, and lines off a dword beside each other: the same as one by one."""
    g = torch.Generator(device="cuda").manual_seed(M)
    X, W, G = (torch.randn(*n, device="cuda", generator=g) for n in ((M, K), (K, N), (M, N)))
    prm = [B.Params(had_block=64, acc_bits=a, s=s, seed=i, A=B.Operand(b, B.ROUND_NEAREST, 1.0, 2 * i),
                    B=B.Operand(b, B.ROUND_NEAREST, 1.0, 2 * i + 1)) for i in range(3)]
    step = []
    names = launched(lambda: step.extend(B.layer_step(X, W, G, *prm)[:3]))
    assert names.count("gemm_small_kernel<true>") == 1 and "gemm_i4" not in names, names
    kinds = (B.GEMM_FWD, X, W), (B.GEMM_BWD_INPUT, G, W), (B.GEMM_BWD_WEIGHT, X, G)
    for got, (kind, P, Q), p in zip(step, kinds, prm):
        assert torch.equal(got, B.gemm(kind, P, Q, M, K, N, p)[0])


@pytest.mark.parametrize("RA,RB,D,b,s,a,small", [(2304, 586, 16987, 6, 16960, 12, False), (1920, 600, 5632, 8, 5632, 16, False),
                                                 (64, 586, 16987, 6, 16960, 12, True), (800, 832, 8384, 4, 8384, 16, True)])
def test_which_kernel_has_a_few_long_tiles(RA, RB, D, b, s, a, small):
    """Bytes in fewer tiles than a workgroup has waves: many blocks of them are the large tiles' kernel's."""
    assert ("gemm_small_kernel" in kernels(RA, RB, D, b, s, a)) == small
