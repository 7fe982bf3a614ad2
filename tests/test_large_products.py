"""Which large products of packed codes multiply through the 6-bit matrix instructions, as far as the size of
their workspace tells (host code): it holds the codes' other form, for those and for no others."""
import ctypes as C

import pytest

from dispatch import dispatch
from paper_2310_03675_amd import binding as B

MOST_THREADS = 1 << 32          # of a grid


def other_form(RA, RB, D, s=64):
    return B.load().hdqt_gemm_codes_workspace_size(RA, RB, D, s)


# (RA, RB, D): on both sides of what a grid holds, of the kernel that writes the other form (256 threads for 32 rows
# of 256 codes) and of the product's (512 threads for 128 x 128 outputs)
@pytest.mark.parametrize("RA,RB,D,fits", [(1 << 20, 512, 1 << 17, False), ((1 << 20) - 1024, 512, 1 << 17, True),
                                          (1 << 19, 1 << 18, 1024, False), (1 << 19, (1 << 18) - 256, 1024, True)])
def test_products_whose_grids_cannot_be_launched_stay_with_the_integer_kernel(RA, RB, D, fits):
    threads = max(-(-RA // 128) * -(-RB // 128) * 512, (-(-RA // 128) + -(-RB // 128)) * 4 * (D // 256) * 256)
    assert (threads < MOST_THREADS) == fits
    assert (other_form(RA, RB, D) > 0) == fits


def has_other_form(RA, RB, D, acc, s):
    op = B.Operand(4, B.ROUND_NEAREST, 1.0, 0)
    prm = B.Params(had_block=64, acc_bits=acc, s=s, seed=0, A=op, B=op)
    return B.workspace_size(B.GEMM_FWD, RA, D, RB, prm) > B.load().hdqt_workspace_least(B.GEMM_FWD, RA, D, RB, C.byref(prm.c()))


# products timed with either kernel, on both sides of the line; those that fill half rounds of 512 tiles come later, and wide
# outputs of short contractions not at all (1536 x 24832 x 512, 32768 x 2048 x 512)
@pytest.mark.parametrize("RA,RB,D,acc,s,other", [
    (8192, 8192, 8192, 8, 64, True), (4096, 4096, 4096, 8, 64, True), (8192, 1024, 8192, 8, 64, True), (2304, 10368, 2048, 8, 64, True),
    (24576, 768, 768, 8, 64, False), (1536, 32768, 512, 8, 64, False), (1024, 32768, 512, 8, 64, False),
    (2048, 16384, 512, 8, 64, False), (2048, 4096, 2048, 8, 64, False), (1536, 24832, 512, 8, 64, False),
    (8192, 8192, 8192, 32, 256, True), (4096, 4096, 2048, 32, 256, True), (16384, 1024, 2048, 32, 256, False),
    (2048, 32768, 512, 32, 256, False), (32768, 2048, 512, 32, 256, False), (4096, 8192, 1024, 32, 256, False),
    (8192, 4096, 1024, 32, 256, False), (4096, 8192, 1536, 32, 256, True)])
def test_which_products_take_the_other_form(RA, RB, D, acc, s, other):
    (rc, kernels), = dispatch([("fwd", RA, D, RB, 4, acc, s, 0)])
    assert rc == 0 and any(k.startswith("gemm_six_kernel") for k in kernels) == other, kernels
    assert has_other_form(RA, RB, D, acc, s) == other



# tiles of no whole 32 codes, which the kernel that `pays` compares with does not take: the other form from where it beats
# the kernels that do
@pytest.mark.parametrize("RA,RB,D,s,other", [(6825, 2768, 1792, 33, True), (148480, 1664, 512, 24, True), (4096, 8192, 1536, 24, True),
                                             (8192, 4096, 1024, 33, True), (8192, 4096, 1024, 32, False), (16384, 1024, 2048, 33, False)])
def test_unclamped_tiles_of_no_whole_32_codes(RA, RB, D, s, other):
    (rc, kernels), = dispatch([("fwd", RA, D, RB, 4, 32, s, 0)])
    assert rc == 0 and any(k.startswith("gemm_six_kernel") for k in kernels) == other, kernels
    assert has_other_form(RA, RB, D, 32, s) == other

def test_only_calls_that_use_the_other_form_are_told_to_hold_it():
    lib, (RA, RB, D) = B.load(), (4096, 4096, 4096)
    size = lambda bA, bB, acc, bf16=0, s=64: lib.hdqt_gemm_codes_workspace_size_for(RA, RB, D, s, bA, bB, acc, bf16)
    other = (RA + RB) * D * 3 // 4
    assert size(4, 4, 8) == size(3, 2, 8) == size(4, 4, 32) == other == lib.hdqt_gemm_codes_workspace_size(RA, RB, D, 64)
    assert size(8, 8, 32) == size(4, 5, 32) == size(4, 4, 12) == size(4, 4, 8, s=32) == size(4, 4, 8, bf16=1) == 0
    assert size(9, 4, 8) == size(4, 4, 40) == 0 == lib.hdqt_gemm_codes_workspace_size_for(0, RB, D, 64, 4, 4, 8, 0)
    # a split contraction's slices, whatever the widths
    for args in ((4, 4, 8, 0), (8, 8, 16, 0), (4, 4, 8, 1)):
        assert lib.hdqt_gemm_codes_workspace_size_for(1152, 128, 65536, 32, *args) == \
            lib.hdqt_gemm_codes_workspace_size(1152, 128, 65536, 32) > 0
    op = B.Operand(4, B.ROUND_NEAREST, 1.0, 0)
    for M, K, N, more in ((RA, D, RB, other), (512, 576, 128, 0), (65536, 1152, 128, 0)):
        p = B.Params(had_block=64, acc_bits=8, s=64, seed=0, A=op, B=op).c()
        for kind in (B.GEMM_FWD, B.GEMM_BWD_INPUT, B.GEMM_BWD_WEIGHT):
            assert lib.hdqt_workspace_size(kind, M, K, N, C.byref(p)) - lib.hdqt_workspace_least(kind, M, K, N, C.byref(p)) == more
    assert lib.hdqt_workspace_least(7, 8, 8, 8, C.byref(p)) == 0
    assert 0 < lib.hdqt_workspace_least(B.GEMM_FWD, 2304, 2048, 4224, C.byref(p)) < lib.hdqt_gemm_fwd_static_max_bytes() < \
        lib.hdqt_workspace_size(B.GEMM_FWD, 2304, 2048, 4224, C.byref(p))
