"""Which large products of packed codes multiply through the 6-bit matrix instructions, as far as the size of
their workspace tells (host code): it holds the codes' other form."""
import pytest

from paper_2310_03675_amd import binding as B

MOST_THREADS = 1 << 32          # of a grid


def other_form(RA, RB, D, s=64):
    return B.load().hdqt_gemm_codes_workspace_size(RA, RB, D, s)


# (RA, RB, D): on both sides of what a grid holds, of the kernel that writes the other form (256 threads for 32 rows
# of 256 codes) and of the product's (512 threads for 128 x 128 outputs)
@pytest.mark.parametrize("RA,RB,D,fits", [(1 << 20, 512, 1 << 17, False), ((1 << 20) - 1024, 512, 1 << 17, True),
                                          (1 << 19, 1 << 18, 512, False), (1 << 19, (1 << 18) - 256, 512, True)])
def test_products_whose_grids_cannot_be_launched_stay_with_the_integer_kernel(RA, RB, D, fits):
    threads = max(-(-RA // 128) * -(-RB // 128) * 512, (-(-RA // 128) + -(-RB // 128)) * 4 * (D // 256) * 256)
    assert (threads < MOST_THREADS) == fits
    assert (other_form(RA, RB, D) > 0) == fits
