"""Maxima of a convolution's unfolded input: the tiles without negative values are added up, the others
transformed.  An activation and its negative have the same maxima bit for bit, one through either way."""
import numpy as np
import pytest
import torch

from paper_2310_03675_amd import binding as B

pytestmark = pytest.mark.gpu


def _scales(act, kh, kw, n):
    op = B.Operand(4, B.ROUND_NEAREST, 0.975, 1)
    _, s1, _, s0 = B.quantize_dual_im2col(act, kh, kw, n, op, op)
    return torch.cat((s1, s0)).view(torch.int32).cpu().numpy()


@pytest.mark.parametrize("kind", ["rectified", "one negative", "minus zero", "tiny", "huge", "infinite", "nan", "large sums"])
@pytest.mark.parametrize("shape,kh,kw,ns", [((3, 64, 8, 8), 3, 3, (8, 16, 32, 64)), ((2, 64, 1, 128), 1, 5, (8, 32, 64)),
                                            ((2, 64, 32, 32), 3, 3, (64,)), ((1, 64, 2, 64), 3, 3, (4, 64)),
                                            ((1, 64, 16, 4), 3, 3, (16, 64))])
def test_sums_give_the_same_maxima(shape, kh, kw, ns, kind):
    rng = np.random.default_rng(sum(shape) + len(kind))
    a = np.maximum(rng.standard_normal(shape), 0).astype(np.float32)
    at = tuple(int(rng.integers(d)) for d in shape)
    if kind == "one negative": a[at] = -0.5
    elif kind == "minus zero": a[a == 0] = -0.0
    elif kind == "tiny": a *= np.float32(1e-39)
    elif kind == "huge": a *= np.float32(3e38) / a.max()
    elif kind == "infinite": a[at] = np.inf
    elif kind == "nan": a[at] = np.nan
    elif kind == "large sums": a *= (10.0 ** rng.integers(-6, 6, shape)).astype(np.float32)
    act = torch.from_numpy(a).cuda()
    for n in ns:
        assert np.array_equal(_scales(act, kh, kw, n), _scales(-act, kh, kw, n)), n
