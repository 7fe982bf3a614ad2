"""Which kernel multiplies, at the edges of the rules (host code: nothing is launched)."""
import math
import random

import pytest

from dispatch import dispatch


def instance(kernels, name):
    """The template arguments of the kernels of that name."""
    return [k[len(name) + 1:k.index(">")].split(", ") for k in kernels if k.startswith(name + "<")]


def field(kernel, name):
    return int(kernel.split(f" {name}=")[1].split()[0])


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


# masks behind contractions that are split (the pass that adds the parts masks) and that end inside 32 codes
@pytest.mark.parametrize("M,K,N", [(1024, 2080, 1000), (4096, 1024, 2040), (5060, 412, 1360), (128, 4096, 4008), (70, 640, 3992)])
def test_masked_gradients_in_parts_are_multiplied(M, K, N):
    calls = [(kind, M, K, N, b, 8, s, 1) for kind in ("bwd_input", "layer_bwd") for b in (4, 3) for s in (32, 64)]
    for call, (rc, kernels) in zip(calls, dispatch(calls)):
        assert rc == 0, (call, kernels)
        assert any("gemm" in k for k in kernels), (call, kernels)


def _size(rng, lo, hi):
    v, q = round(math.exp(rng.uniform(math.log(lo), math.log(hi)))), rng.choice((1, 8, 8, 32, 64))
    return max(q, v // q * q)


@pytest.mark.parametrize("seed", range(4))
def test_no_call_is_left_without_a_kernel(seed):
    """Layers and products at random, over every kind of call, width, accumulator and tile: arguments that are valid
    are multiplied."""
    rng, calls = random.Random(seed), []
    for _ in range(5000):
        kind, option = rng.choice((("fwd", 0), ("bwd_weight", 0), ("bwd_input", 0), ("bwd_input", 1), ("bwd_input", 1), ("bwd_input", 2),
                                   ("codes", 0), ("step", 0), ("step", 1), ("layer_fwd", 0), ("layer_bwd", 0), ("layer_bwd", 1)))
        b, acc = rng.choice(((4, 8),) * 6 + ((3, 8), (2, 8), (4, 12), (4, 16), (4, 32), (6, 12), (8, 16), (5, 12), (8, 8), (8, 24)))
        s = rng.choice((32, 32, 32, 64, 64, 16, 96, 128, 160, 192, 224, 256, 24, 4000))
        calls.append((kind, _size(rng, 1, 65536), _size(rng, 10, 4096), _size(rng, 10, 4096), b, acc, s, option))
    for call, (rc, kernels) in zip(calls, dispatch(calls)):
        assert rc == 0, (call, kernels)


# Tiles that divide no stage of 128 codes, in as many parts as the products of any size are split into: where lines go straight
# to LDS no part begins at or behind a line's end, and 16-bit slices hold what a part can add up to
@pytest.mark.parametrize("b,acc", [(4, 32), (3, 32), (2, 32), (4, 8), (3, 8), (8, 32), (8, 16)])
def test_parts_end_inside_their_lines(b, acc):
    rng, calls = random.Random(b + acc), [("codes", 129, 131080, 512, b, acc, 96, 0), ("codes", 129, 100000, 129, b, acc, 96, 0)]
    for _ in range(3000):
        calls.append(("codes", _size(rng, 1, 1500), _size(rng, 512, 300000), _size(rng, 1, 1500), b, acc,
                      rng.choice((32, 64, 128)) if acc == 8 else 32 * rng.choice((1, 2, 3, 3, 4, 5, 5, 6, 7, 8, 9, 10, 11, 20, 33)), 0))
    seen = 0
    for call, (rc, kernels) in zip(calls, dispatch(calls)):
        assert rc in (0, -5, -6), (call, kernels)            # (more than 32 bits hold)
        for k in kernels:
            if " parts=" not in k or field(k, "parts") == 1:
                continue
            parts, codes = field(k, "parts"), field(k, "part_codes")
            seen += 1
            assert (parts - 1) * codes < call[2], (call, k)
            if field(k, "slices16"):
                most = min(codes << 2 * (b - 1), -(-codes // call[6]) << (acc - 1))
                assert most < 1 << 15, (call, k)
    assert seen > 20


# Folded input gradients: whole steps of 32 codes a tap, odd widths no more than even ones (whose codes a call keeps in
# padded lines where nothing is folded)
@pytest.mark.parametrize("batch,C,side", [(8, 64, 8), (2, 64, 16), (2, 128, 32)])
def test_folded_gradients_take_whole_32_channels(batch, C, side):
    calls = [("conv_bwd", batch, C, N, 4, 8, 32, side) for N in (32, 64, 96, 33, 65, 31, 1, 63, 95, 97, 40, 48)]
    for call, (rc, kernels) in zip(calls, dispatch(calls)):
        assert rc == (0 if call[3] % 32 == 0 else -13), (call, kernels)
        assert (call[3] % 32 == 0) == any(k.startswith("gemm_fold_kernel") for k in kernels), (call, kernels)


# Odd contractions: a workspace with room for the codes alone is enough, the zeros behind them are not asked for
@pytest.mark.parametrize("M,K,N", [(1000001, 3, 64), (4097, 27, 64), (64000, 99, 99), (16384, 405, 243), (128, 561, 11), (1023, 64, 129)])
def test_codes_lie_without_padding_where_there_is_no_room(M, K, N):
    calls = [(kind + even, M, K, N, b, acc, s, 0) for kind in ("step", "layer_fwd", "layer_bwd") for even in ("", "_even")
             for b, acc, s in ((4, 8, 32), (4, 8, 1000), (8, 16, 32))]
    for call, (rc, kernels) in zip(calls, dispatch(calls)):
        assert rc == 0, (call, kernels)


# Masks behind padded contractions: in the epilogue of the kernel that brings lines to LDS, by a pass where gemm_i4_kernel
# multiplies and the output stays in the memory-side cache
@pytest.mark.parametrize("M,K,N,s,by_pass", [(24059, 1035, 79, 32, False), (24059, 1035, 79, 256, True), (198243, 67, 103, 128, True),
                                             (25344, 2298, 1719, 128, True), (25344, 2400, 1719, 128, False), (24059, 1035, 80, 256, False)])
def test_masks_behind_padded_contractions(M, K, N, s, by_pass):
    (rc, kernels), = dispatch([("layer_bwd", M, K, N, 4, 8, s, 1)])
    assert rc == 0 and ("relu_mask_kernel" in kernels) == by_pass, kernels
