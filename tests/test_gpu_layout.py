"""GPU parity of the layout kernels against PyTorch's own unfold, fold and transpose, bit for bit (the
terms of a folded element are added in the order of the matrix rows, as its fold does)."""
import pytest
import torch

from paper_2310_03675_amd import autograd as A
from paper_2310_03675_amd import binding as B
from launches import launched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,c,h,w,k,stride,pad", [
    (1, 1, 1, 1, 1, 1, 0), (2, 3, 32, 32, 3, 1, 1), (3, 65, 8, 8, 3, 2, 1), (5, 64, 16, 16, 1, 2, 0), (4, 130, 4, 4, 3, 1, 1),
    (2, 33, 7, 9, 5, 1, 2), (3, 20, 11, 6, 3, 3, 0), (7, 512, 4, 4, 3, 1, 1), (2, 8, 5, 5, 2, 2, 0), (1, 300, 9, 33, 3, 2, 2),
    (3, 33, 7, 9, 3, 8, 1), (2, 33, 7, 9, 3, 2**31 - 1, 1), (2, 5, 4, 6, 1, 2**31 - 1, 0)])
def test_unfold_and_fold(b, c, h, w, k, stride, pad):
    print(f"layout: act [{b},{c},{h},{w}] window {k} stride {stride} pad {pad}", flush=True)
    g = torch.Generator().manual_seed(b * 1000 + c)
    act = torch.randn(b, c, h, w, generator=g).cuda()
    cols = torch.nn.functional.unfold(act, kernel_size=k, padding=pad, stride=stride)
    assert torch.equal(B.im2col(act, k, k, stride, pad, pad), cols.transpose(1, 2).reshape(-1, c * k * k))
    dX = torch.randn(b * cols.shape[2], c * k * k, generator=g).cuda()
    want = torch.nn.functional.fold(dX.reshape(b, -1, c * k * k).transpose(1, 2).contiguous(), output_size=(h, w),
                                    kernel_size=k, padding=pad, stride=stride)
    assert torch.equal(B.col2im(dX, (b, c, h, w), k, k, stride, pad, pad), want)


@pytest.mark.parametrize("b,c,h,w,kh,kw,stride,ph,pw", [
    (2, 17, 9, 65, 3, 3, 1, 1, 1),        # rows of 17 * 9 elements: single ones; two tiles across, the second shorter
    (2, 68, 13, 40, 3, 3, 2, 1, 1),       # a block of 4 channels behind those of 16; rows of windows that end inside a tile
    (3, 20, 33, 7, 2, 2, 3, 0, 0),        # pixels between the windows
    (3, 130, 14, 14, 1, 1, 2, 0, 0), (1, 6, 200, 5, 7, 7, 3, 3, 3), (2, 12, 1, 130, 1, 3, 1, 0, 1),
    (2, 12, 6, 130, 1, 5, 1, 0, 2),       # more taps in a row than a tile's pixel holds
    (1, 2, 120, 110, 100, 100, 40, 5, 0), # windows that do not fit LDS
    (1, 1, 300, 260, 9, 9, 4, 4, 4), (40, 513, 2, 2, 3, 3, 1, 1, 1)])
def test_unfold_and_fold_tiles(b, c, h, w, kh, kw, stride, ph, pw):
    """Edges of the tiles: images, channels and windows that end inside one, do not fill one, or have none."""
    print(f"layout: tiles of act [{b},{c},{h},{w}] window {kh}x{kw} stride {stride} pad {ph},{pw}", flush=True)
    g = torch.Generator().manual_seed(b * 1000 + c)
    act = torch.randn(b, c, h, w, generator=g).cuda()
    cols = torch.nn.functional.unfold(act, kernel_size=(kh, kw), padding=(ph, pw), stride=stride)
    assert torch.equal(B.im2col(act, kh, kw, stride, ph, pw), cols.transpose(1, 2).reshape(-1, c * kh * kw))
    dX = torch.randn(b * cols.shape[2], c * kh * kw, generator=g).cuda()
    want = torch.nn.functional.fold(dX.reshape(b, -1, c * kh * kw).transpose(1, 2).contiguous(), output_size=(h, w),
                                    kernel_size=(kh, kw), padding=(ph, pw), stride=stride)
    assert torch.equal(B.col2im(dX, (b, c, h, w), kh, kw, stride, ph, pw), want)


@pytest.mark.parametrize("b,c,h,w,kh,kw,stride,ph,pw,unfolds,folds", [
    # few windows or pixels per image, little of X per tile, few tiles, padding for the most part: a thread's column
    (400, 64, 1, 1, 1, 1, 1, 0, 0, False, False), (500, 64, 1, 3, 3, 3, 1, 1, 1, False, False), (500, 64, 2, 2, 3, 3, 1, 1, 1, False, True),
    (300, 4, 1, 20, 1, 2, 1, 0, 0, False, True), (40, 516, 4, 4, 3, 3, 1, 1, 1, False, True), (400, 64, 1, 25, 3, 3, 3, 1, 1, False, True),
    # tiles: blocks of 4 channels behind those of 16 and 64, tiles cut off by the last row and the last column, pixels
    # between the windows, rows of a window longer than its stride
    (60, 68, 13, 40, 3, 3, 2, 1, 1, True, True), (50, 516, 4, 4, 3, 3, 1, 1, 1, True, True), (100, 20, 33, 7, 2, 2, 3, 0, 0, True, True),
    (3, 132, 14, 14, 1, 1, 2, 0, 0, True, True), (100, 8, 200, 5, 7, 7, 3, 3, 3, True, True), (300, 12, 1, 130, 1, 3, 1, 0, 1, True, True),
    (120, 12, 6, 130, 1, 5, 1, 0, 2, True, False)])
def test_which_layouts_go_in_tiles(b, c, h, w, kh, kw, stride, ph, pw, unfolds, folds):
    test_unfold_and_fold_tiles(b, c, h, w, kh, kw, stride, ph, pw)
    act = torch.zeros(b, c, h, w, device="cuda")
    X = B.im2col(act, kh, kw, stride, ph, pw)
    assert ("im2col_tile_kernel" in launched(lambda: B.im2col(act, kh, kw, stride, ph, pw))) == unfolds
    assert ("col2im_tile_kernel" in launched(lambda: B.col2im(X, act.shape, kh, kw, stride, ph, pw))) == folds


@pytest.mark.parametrize("b,r,c", [(1, 1, 1), (3, 64, 64), (2, 65, 63), (5, 16, 512), (2, 1, 130), (4, 1024, 64)])
def test_transpose(b, r, c):
    x = torch.randn(b, r, c, generator=torch.Generator().manual_seed(r)).cuda()
    assert torch.equal(B.transpose(x), x.transpose(1, 2).contiguous())


@pytest.mark.parametrize("b,c,h,w,k,stride,pad", [(168, 3, 224, 224, 7, 2, 3),        # 2.1 M rows of 147
                                                  (4112, 3, 30, 34, 7, 1, 3)])        # 4194240, the most there may be
def test_unfold_many_rows(b, c, h, w, k, stride, pad):
    """More runs of rows than the second axis of a grid holds (65535, of 32 rows each)."""
    print(f"layout: act [{b},{c},{h},{w}] window {k} stride {stride} pad {pad}", flush=True)
    act = torch.randn(b, c, h, w, generator=torch.Generator().manual_seed(b)).cuda()
    X = B.im2col(act, k, k, stride, pad, pad)
    per = X.shape[0] // b
    assert X.shape[0] > 65535 * 32
    for first in (0, 65535 * 32 // per - 1, b - 2):
        cols = torch.nn.functional.unfold(act[first:first + 2], kernel_size=k, padding=pad, stride=stride)
        assert torch.equal(X[first * per:(first + 2) * per], cols.transpose(1, 2).reshape(-1, c * k * k))


@pytest.mark.parametrize("b,c,h,w,k,stride,pad", [(335, 32, 112, 112, 3, 2, 1),      # 4.2 M pixels, 1.05 M rows
                                                  (5, 1, 8192, 8192, 16, 16, 0)])    # 2^23 workgroups, and a second turn
def test_fold_many_pixels(b, c, h, w, k, stride, pad):
    """Strided layers: many times the pixels that the matrix has rows."""
    print(f"layout: fold to [{b},{c},{h},{w}] window {k} stride {stride} pad {pad}", flush=True)
    rows = ((h + 2 * pad - k) // stride + 1) * ((w + 2 * pad - k) // stride + 1)
    dX = torch.randn(b * rows, c * k * k, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    got = B.col2im(dX, (b, c, h, w), k, k, stride, pad, pad)
    for first in (0, b // 2, b - 2):
        part = dX[first * rows:(first + 2) * rows].reshape(2, rows, c * k * k).transpose(1, 2).contiguous()
        want = torch.nn.functional.fold(part, output_size=(h, w), kernel_size=k, padding=pad, stride=stride)
        assert torch.equal(got[first:first + 2], want)


@pytest.mark.parametrize("shape,stride", [((3, 40, 8, 6), 1), ((3, 40, 8, 6), 2), ((50, 65, 26, 25), 1),
                                          ((2, 2, 2049, 2048), 2)])
@pytest.mark.parametrize("layout", ["innermost", "misaligned", "transposed", "part"])
def test_unfold_of_any_layout(shape, stride, layout):
    """Activations with their channels innermost (the library's own transposition where it takes the
    sizes: at most 4194240 pixels), off the 16-byte grid, and in orders it does not take."""
    print(f"layout: {layout} act {shape} stride {stride}", flush=True)
    b, c, h, w = shape
    act = torch.randn(shape, generator=torch.Generator().manual_seed(c))
    if layout in ("innermost", "misaligned"):
        room = torch.empty(act.numel() + 1, device="cuda")[layout == "misaligned":][:act.numel()]
        x = room.reshape(b, h, w, c).permute(0, 3, 1, 2)
        assert (x.data_ptr() % 16 != 0) == (layout == "misaligned")
    elif layout == "transposed":
        x = torch.empty(b, c, w, h, device="cuda").transpose(2, 3)
    else:
        x = torch.empty(b, c + 1, h, w, device="cuda")[:, :c]
    x.copy_(act)
    assert not x.is_contiguous()
    x.requires_grad_()
    X = A.Unfold.apply(x, 1 if stride > 1 else 3, stride, 0 if stride > 1 else 1)
    k, pad = (1, 0) if stride > 1 else (3, 1)
    want = torch.nn.functional.unfold(act.cuda(), kernel_size=k, padding=pad, stride=stride)
    assert torch.equal(X, want.transpose(1, 2).reshape(-1, c * k * k))
    X.backward(torch.ones_like(X))
    fold = torch.nn.functional.fold(torch.ones_like(want), output_size=(h, w), kernel_size=k, padding=pad, stride=stride)
    assert torch.equal(x.grad, fold)


@pytest.mark.parametrize("shape,k,stride", [((32, 64, 32, 32), 3, 1), ((33, 64, 32, 32), 3, 2), ((40, 52, 32, 32), 1, 2),
                                            ((8, 64, 32, 32), 3, 1)])       # the last: too small to be turned
def test_gradient_in_the_layout_of_its_activation(shape, k, stride):
    """Channels innermost or planes: the same gradients, each in its activation's layout."""
    print(f"layout: gradient of act {shape} window {k} stride {stride}", flush=True)
    b, c, h, w = shape
    act = torch.randn(shape, generator=torch.Generator().manual_seed(c)).cuda()
    grads = []
    for innermost in (False, True):
        layer = A.HdqtConv2d(c, 32, kernel_size=k, padding=k // 2, stride=stride, cfg=A.LayerConfig(), device="cuda")
        with torch.no_grad():
            layer.weight.copy_(torch.randn(layer.weight.shape, generator=torch.Generator().manual_seed(1)))
        leaf = act.clone().requires_grad_()
        x = leaf * 1.0
        if innermost:
            x = x.permute(0, 2, 3, 1).contiguous().permute(0, 3, 1, 2)
        x.retain_grad()
        seen = []
        x.register_hook(lambda grad: seen.append(grad.stride()))
        z = layer(x)
        z.backward(torch.randn(z.shape, generator=torch.Generator().manual_seed(2)).cuda())
        turned = innermost and act.numel() >= 1 << 21
        assert seen[0] == (x.stride() if turned else act.stride())
        grads.append((leaf.grad, layer.weight.grad))
    for p, q in zip(*grads):
        assert torch.equal(p, q)
