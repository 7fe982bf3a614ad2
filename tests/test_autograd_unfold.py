"""The autograd functions around the layout kernels, on the CPU: the library's calls are replaced by
PyTorch's own unfold and fold, detached, as results of the library are, and with its alignment
and size checks."""
import pytest
import torch
import torch.nn.functional as F

from paper_2310_03675_amd import autograd as A
from paper_2310_03675_amd import binding as B


def _im2col(act, kh, kw, stride=1, pad_h=0, pad_w=0, stream=None):
    cols = F.unfold(act.detach(), (kh, kw), padding=(pad_h, pad_w), stride=stride)
    return cols.transpose(1, 2).reshape(-1, act.shape[1] * kh * kw)


def _col2im(dX, act_shape, kh, kw, stride=1, pad_h=0, pad_w=0, stream=None):
    b, c, h, w = act_shape
    assert dX.is_contiguous() and dX.data_ptr() % 16 == 0
    return F.fold(dX.detach().reshape(b, -1, c * kh * kw).transpose(1, 2), (h, w), (kh, kw), padding=(pad_h, pad_w),
                  stride=stride)


@pytest.fixture
def library(monkeypatch):
    monkeypatch.setattr(B, "im2col", _im2col)
    monkeypatch.setattr(B, "col2im", _col2im)


def _plain(act, k, stride, pad):
    return F.unfold(act, k, padding=pad, stride=stride).transpose(1, 2).reshape(-1, act.shape[1] * k * k)


GEOMETRIES = [(2, 32, 6, 6, 3, 1, 1), (3, 40, 7, 5, 3, 2, 1), (2, 5, 6, 6, 3, 1, 1)]


@pytest.mark.parametrize("b,c,h,w,k,stride,pad", GEOMETRIES)
def test_gradient_of_a_gradient(library, b, c, h, w, k, stride, pad):
    """create_graph: the gradient itself can be differentiated."""
    got = []
    for unfold in (A.Unfold.apply, _plain):
        act = torch.randn(b, c, h, w, generator=torch.Generator().manual_seed(1)).requires_grad_()
        first, = torch.autograd.grad((unfold(act, k, stride, pad) ** 3).sum(), act, create_graph=True)
        assert first.requires_grad
        second, = torch.autograd.grad((first ** 2).sum(), act)
        got.append((first, second))
    assert torch.equal(got[0][0], got[1][0])
    # (two binary32 sums of the same k * k terms a rounding apart)
    assert torch.allclose(got[0][1], got[1][1], rtol=1e-5, atol=1e-5 * float(got[1][1].abs().max()))


@pytest.mark.parametrize("b,c,h,w,k,stride,pad", GEOMETRIES)
def test_batched_gradients(library, b, c, h, w, k, stride, pad):
    """is_grads_batched: many gradients of the matrix in one backward pass."""
    act = torch.randn(b, c, h, w, generator=torch.Generator().manual_seed(2)).requires_grad_()
    X = A.Unfold.apply(act, k, stride, pad)
    many = torch.randn(4, *X.shape, generator=torch.Generator().manual_seed(3))
    got, = torch.autograd.grad(X, act, many, is_grads_batched=True, retain_graph=True)
    for g, one in zip(got, many):
        assert torch.equal(g, torch.autograd.grad(X, act, one, retain_graph=True)[0])


def test_forward_mode_through_the_gradient(library):
    """A tangent of the matrix's gradient comes out as the tangent of the activation's."""
    import torch.autograd.forward_ad as fa
    g = torch.Generator().manual_seed(4)
    dX, tangent = torch.randn(72, 32 * 9, generator=g), torch.randn(72, 32 * 9, generator=g)
    geometry = ((2, 32, 6, 6), 3, 3, 1, 1, 1)
    with fa.dual_level():
        got = fa.unpack_dual(A._fold(fa.make_dual(dX, tangent), *geometry))
    assert torch.equal(got.primal, _col2im(dX, *geometry)) and torch.equal(got.tangent, _col2im(tangent, *geometry))


def test_a_refused_layer_does_not_decide_for_others(monkeypatch):
    """What hdqt_conv_bwd takes depends on the output channels and the quantization too: a layer that
    it refused leaves the next one of the same input shape alone, and is itself not asked again."""
    asked, unfolded = [], []

    def conv_fwd(act, kh, kw, W, fwd, bww):
        return torch.zeros(act.shape[0] * act.shape[2] * act.shape[3], W.shape[1]), torch.zeros(1)

    def conv_bwd(G, W, saved, shape, kh, kw, bwi, bww):
        asked.append((W.shape[1], bwi.A.b, bwi.s, bwi.acc_bits))
        if W.shape[1] % 32 or bwi.A.b > 4 or bwi.s % 32 or bwi.acc_bits > 8:
            raise B.HdqtError(-13, "hdqt_conv_bwd")
        return torch.zeros(shape), torch.zeros_like(W)

    def layer_bwd(G, W, saved, K, bwi, bww):
        unfolded.append(W.shape[1])
        return torch.zeros(G.shape[0], K), torch.zeros_like(W)

    monkeypatch.setattr(B, "conv_fwd", conv_fwd)
    monkeypatch.setattr(B, "conv_bwd", conv_bwd)
    monkeypatch.setattr(B, "layer_bwd", layer_bwd)
    monkeypatch.setattr(B, "col2im", _col2im)

    def step(cout, **cfg):
        act = torch.randn(2, 32, 8, 8).requires_grad_()
        W = torch.randn(32 * 9, cout).requires_grad_()
        A.HdqtConvMatmul.apply(act, W, A.LayerConfig(**cfg), 0, 3, 3).sum().backward()

    for refused in (dict(cout=16), dict(cout=64, bits=8, acc_bits=16), dict(cout=64, s=48), dict(cout=64, acc_bits=12)):
        asked.clear(), unfolded.clear()
        step(**refused)
        assert len(asked) == 1 and len(unfolded) == 1
        step(cout=64)
        assert len(asked) == 2 and len(unfolded) == 1, refused
        step(**refused)
        assert len(asked) == 2 and len(unfolded) == 2


def test_gradient_that_does_not_start_on_16_bytes(library):
    """The matrix as a part of something larger: its gradient is a view at any float."""
    act = torch.randn(2, 33, 6, 6, generator=torch.Generator().manual_seed(5)).requires_grad_()
    got = []
    for unfold in (A.Unfold.apply, _plain):
        X = unfold(act, 3, 1, 1)
        whole = torch.cat([torch.ones(1, X.shape[1]), X])
        weights = torch.randn(whole.shape, generator=torch.Generator().manual_seed(6))
        assert weights[1:].data_ptr() % 16
        got.append(torch.autograd.grad(whole, act, weights)[0])
    assert torch.equal(*got)
