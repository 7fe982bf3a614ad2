"""Which kernel multiplies, at the edges of the rules (host code: nothing is launched)."""
import pytest

from dispatch import dispatch


def instance(kernels, name):
    """The template arguments of the kernels of that name."""
    return [k[len(name) + 1:k.index(">")].split(", ") for k in kernels if k.startswith(name + "<")]


LINES, TEST_32 = "lines_gemm_i4_kernel", "3"      # (its first argument: the clamp)


# more than 512 tiles of 128 x 128, more than 512 codes to a part: whole 32 codes ask, in the kernel that brings lines to LDS,
# and what ends inside them does not come there
@pytest.mark.parametrize("M,K,N", [(65536, 992, 1024), (65536, 608, 256), (50000, 608, 512), (16384, 8160, 1000)])
def test_tiles_that_are_asked_lie_in_whole_32_codes(M, K, N):
    calls = [(kind, M, K + more, N, 4, 8, 32, 0) for more in range(0, 32, 8) for kind in ("fwd", "codes", "layer_fwd")]
    for call, (rc, kernels) in zip(calls, dispatch(calls)):
        asked = [k for k in instance(kernels, LINES) if k[0] == TEST_32]
        assert rc == 0
        assert len(asked) == (call[2] % 32 == 0), (call, kernels)
