"""GPU parity of the folded input gradient where its kernel's pieces end: contractions with an odd
number of steps per tap and more or fewer codes than an LDS buffer, channel counts around a
workgroup's 64, pixel counts around its 256, both clamps, one tile per tap and short last tiles."""
import pytest

import test_gpu_fold as fold

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,C,H,W,kh,kw,N,s,a", [
    (3, 65, 8, 8, 3, 3, 96, 32, 8), (1, 1, 1, 2, 1, 1, 32, 32, 8), (5, 40, 16, 16, 3, 3, 128, 64, 8),
    (2, 130, 32, 32, 3, 3, 32, 32, 8), (3, 33, 4, 4, 1, 5, 288, 96, 10), (2, 64, 8, 8, 3, 3, 64, 32, 16),
    (1, 63, 16, 16, 3, 3, 160, 64, 7), (9, 31, 1, 32, 1, 7, 224, 224, 12), (1, 20, 16, 4, 5, 3, 544, 32, 8),
    (1, 7, 40, 8, 13, 1, 32, 32, 6)])
def test_fold_edges(batch, C, H, W, kh, kw, N, s, a):
    fold.test_gemm_codes_fold(batch, C, H, W, kh, kw, N, s, a)
