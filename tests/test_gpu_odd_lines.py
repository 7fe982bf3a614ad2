"""Odd contractions inside a layer's calls, whose codes lie in padded lines: bit for bit the three products on their own
(whose codes lie as hdqt_codes_pitch says), from workspaces full of ones."""
import pytest
import torch

from paper_2310_03675_amd import binding as B

pytestmark = pytest.mark.gpu
NE, ST = B.ROUND_NEAREST, B.ROUND_STOCHASTIC


# odd in one dimension and in all, one code and one line, lines that end one code behind a piece of 16 bytes and one before;
# tiles inside a line, of 16 codes, longer than the contraction, and of no whole step
@pytest.mark.parametrize("M,K,N", [(4097, 27, 64), (128, 561, 11), (33, 65, 1), (1, 31, 33), (1023, 64, 129), (20001, 95, 97), (70, 1, 5)])
@pytest.mark.parametrize("b,acc,s", [(4, 8, 32), (4, 8, 64), (3, 16, 16), (4, 8, 1000), (8, 16, 32), (6, 12, 128), (4, 10, 24)])
def test_layer_calls(M, K, N, b, acc, s):
    print(f"M={M} K={K} N={N} b={b} acc={acc} s={s}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(M + K + N)
    X, W, G = (torch.randn(shape, generator=g, device="cuda:0") for shape in ((M, K), (K, N), (M, N)))
    X = torch.relu(X)
    op = lambda rnd, t: B.Operand(b, rnd, 1.0, t)
    prm = [B.Params(had_block=16, acc_bits=acc, s=s, seed=3, A=x, B=y)
           for x, y in ((op(NE, 0), op(NE, 1)), (op(ST, 6), op(NE, 5)), (op(NE, 8), op(ST, 10)))]
    want = [B.gemm(k, P, Q, M, K, N, p)[0] for k, (P, Q), p in zip((B.GEMM_FWD, B.GEMM_BWD_INPUT, B.GEMM_BWD_WEIGHT),
                                                                 ((X, W), (G, W), (X, G)), prm)]
    ones = lambda n: torch.full((max(n, 256),), 255, dtype=torch.uint8, device="cuda:0")
    ws = ones(B.layer_step_workspace_size(M, K, N, *prm))
    for got, w in zip(B.layer_step(X, W, G, *prm, workspace=ws)[:3], want):
        assert torch.equal(got, w)
    Z, saved = B.layer_fwd(X, W, prm[0], prm[2])
    dX, dW = B.layer_bwd(G, W, saved, K, prm[1], prm[2])
    masked, _ = B.layer_bwd(G, W, saved, K, prm[1], prm[2], mask=X)
    assert torch.equal(Z, want[0]) and torch.equal(dX, want[1]) and torch.equal(dW, want[2])
    assert torch.equal(masked, torch.where(X > 0, want[1], torch.zeros_like(want[1])))


# workspaces of the next larger layer of even sizes, which have no room for zeros behind the codes; nothing behind them is written
@pytest.mark.parametrize("M,K,N", [(4097, 27, 64), (128, 561, 11), (1023, 64, 129), (20001, 95, 97), (12001, 3, 64)])
@pytest.mark.parametrize("b,acc,s", [(4, 8, 32), (4, 8, 1000), (8, 16, 32)])
def test_smaller_workspaces(M, K, N, b, acc, s):
    print(f"M={M} K={K} N={N} b={b} acc={acc} s={s}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(M + K + N)
    X, W, G = (torch.randn(shape, generator=g, device="cuda:0") for shape in ((M, K), (K, N), (M, N)))
    op = lambda rnd, t: B.Operand(b, rnd, 1.0, t)
    prm = [B.Params(had_block=16, acc_bits=acc, s=s, seed=3, A=x, B=y)
           for x, y in ((op(NE, 0), op(NE, 1)), (op(ST, 6), op(NE, 5)), (op(NE, 8), op(ST, 10)))]
    lib, even = B.load(), (M + M % 2, K + K % 2, N + N % 2)
    pf, pi, pw = (p.c() for p in prm)
    sizes = lambda dims: (lib.hdqt_layer_step_workspace_size(*dims, pf, pi, pw), lib.hdqt_layer_fwd_workspace_size(*dims, pf, pw),
                          lib.hdqt_layer_bwd_workspace_size(*dims, pi, pw))
    small, full = sizes(even), sizes((M, K, N))
    assert any(a < b for a, b in zip(small, full))
    blocks = [torch.full((n + 4096,), 255, dtype=torch.uint8, device="cuda:0") for n in small]
    room = [t[:n] for t, n in zip(blocks, small)]
    want = B.layer_step(X, W, G, *prm)[:3]
    for got, w in zip(B.layer_step(X, W, G, *prm, workspace=room[0])[:3], want):
        assert torch.equal(got, w)
    Z, saved = B.layer_fwd(X, W, prm[0], prm[2], workspace=room[1])
    dX, dW = B.layer_bwd(G, W, saved, K, prm[1], prm[2], workspace=room[2])
    assert torch.equal(Z, want[0]) and torch.equal(dX, want[1]) and torch.equal(dW, want[2])
    for t, n in zip(blocks, small):
        assert bool((t[n:] == 255).all())


# odd numbers of output channels are not folded inside the product: the gradient of the activation is the layer's, folded
# tap by tap in fp32
@pytest.mark.parametrize("N", [33, 65])
def test_convolutions_with_odd_channels(N):
    from paper_2310_03675_amd import autograd as A
    batch, C, side = 4, 64, 16
    g = torch.Generator(device="cuda:0").manual_seed(N)
    act, G, W = (torch.randn(s, generator=g, device="cuda:0") for s in ((batch, C, side, side), (batch * side * side, N), (9 * C, N)))
    op = lambda rnd, t: B.Operand(4, rnd, 1.0, t)
    fwd, bwi, bww = (B.Params(had_block=16, acc_bits=8, s=32, seed=3, A=a, B=b)
                     for a, b in ((op(NE, 0), op(NE, 1)), (op(ST, 6), op(NE, 5)), (op(NE, 8), op(ST, 10))))
    _, saved = B.conv_fwd(act, 3, 3, W, fwd, bww)
    with pytest.raises(B.HdqtError) as e:
        B.conv_bwd(G, W, saved, act.shape, 3, 3, bwi, bww)
    assert e.value.code == -13
    grads = []
    for folds in (True, False):
        m = A.HdqtConv2d(C, N, cfg=A.LayerConfig(layer_id=3, seed=2, fold_in_matmul=folds), device="cuda:0")
        m.weight.data.copy_(W)
        x = act.clone().requires_grad_(True)
        z = m(x)
        (z * torch.linspace(-1, 1, z.numel(), device="cuda:0").reshape(z.shape)).sum().backward()
        grads.append((z.detach(), x.grad, m.weight.grad))
    assert all(torch.equal(a, b) for a, b in zip(*grads))
