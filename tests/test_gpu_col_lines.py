"""GPU parity of the tuned axis-0 quantizer where lines of codes start at any byte: row counts of every
kind modulo 16, strips cut off by the last row and the last column, short strips and long ones."""
import numpy as np
import pytest

from paper_2310_03675_amd import binding as B
from test_gpu_parity import check_quantize

pytestmark = pytest.mark.gpu
NE, ST = B.ROUND_NEAREST, B.ROUND_STOCHASTIC


@pytest.mark.parametrize("b,rounding", [(4, NE), (3, ST), (8, NE), (5, ST)])
@pytest.mark.parametrize("rows,cols", [(8226, 1024), (8228, 1020), (8232, 1024), (8240, 1024), (8254, 1020), (8310, 1020)])
def test_quantize_lines_at_any_byte(rows, cols, b, rounding):
    T = np.random.default_rng(rows + cols).standard_normal((rows, cols)).astype(np.float32)
    check_quantize(T, 0, 64, B.Operand(b, rounding, 0.975, 5), seed=11)


@pytest.mark.parametrize("rows", [8194, 8388])
@pytest.mark.parametrize("b", [4, 8])
def test_quantize_long_strips_at_any_byte(rows, b):
    T = np.random.default_rng(rows).standard_normal((rows, 4096)).astype(np.float32)
    check_quantize(T, 0, 64, B.Operand(b, NE, 1.0, 5), seed=11)
