"""GPU parity of the folded input gradient where its kernel's pieces end: contractions with an odd
number of steps per tap and more or fewer codes than an LDS buffer, channel counts around a
workgroup's 64, pixel counts around its 256, both clamps, one tile per tap and short last tiles."""
import pytest
import torch

from paper_2310_03675_amd import binding as B
import test_gpu_fold as fold

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,C,H,W,kh,kw,N,s,a", [
    (3, 65, 8, 8, 3, 3, 96, 32, 8), (1, 1, 1, 2, 1, 1, 32, 32, 8), (5, 40, 16, 16, 3, 3, 128, 64, 8),
    (2, 130, 32, 32, 3, 3, 32, 32, 8), (3, 33, 4, 4, 1, 5, 288, 96, 10), (2, 64, 8, 8, 3, 3, 64, 32, 16),
    (1, 63, 16, 16, 3, 3, 160, 64, 7), (9, 31, 1, 32, 1, 7, 224, 224, 12), (1, 20, 16, 4, 5, 3, 544, 32, 8),
    (1, 7, 40, 8, 13, 1, 32, 32, 6)])
def test_fold_edges(batch, C, H, W, kh, kw, N, s, a):
    fold.test_gemm_codes_fold(batch, C, H, W, kh, kw, N, s, a)


@pytest.mark.parametrize("C,H,W,kh,kw,N,whole,part", [(64, 8, 8, 3, 3, 64, 800, 100), (96, 16, 16, 3, 3, 32, 130, 33), (48, 1, 128, 1, 5, 96, 400, 57),
                                                      (256, 4, 4, 3, 3, 128, 800, 7), (40, 2, 64, 3, 3, 64, 500, 1)])
@pytest.mark.parametrize("s,a", [(32, 8), (64, 12), (96, 10)])
def test_small_and_large_workgroups_agree(C, H, W, kh, kw, N, whole, part, s, a):
    """A batch whose workgroups have 64 channels against pieces of it, whose have 32: channel counts that
    end inside either, pixels that end inside a wave."""
    g = torch.Generator(device="cuda").manual_seed(C + N)
    qG, qW = (torch.randint(0, 256, (n, N // 2), dtype=torch.uint8, device="cuda", generator=g) for n in (whole * H * W, C * kh * kw))
    one = torch.full((1,), 0.5, device="cuda")
    gradient = lambda q, n: B.gemm_codes_fold(q, qW, 4, 4, one, one, (n, C, H, W), kh, kw, 1, a, s)
    out = gradient(qG, whole)
    for i in range(0, whole, part):
        n = min(part, whole - i)
        assert torch.equal(out[i:i + n], gradient(qG[i * H * W:(i + n) * H * W].contiguous(), n))
