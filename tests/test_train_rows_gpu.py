"""The training kernel's last, partly filled row tile: rows past the end add
nothing to the loss or the gradient, whatever the weights hold. With an
infinite first-layer weight the unit saturates (tanh = +-1) on every row and
loss and gradient stay finite, while a row of zeros in its place would give 0
times infinity.

Tolerance as for the other gradients against FP64 autograd: 1e-5 of the
largest entry."""
import pytest

from paper_2509_19171_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("indexed", [False, True])
@pytest.mark.parametrize("n", [1, 17, 4100])
def test_gradient_with_an_infinite_weight(n, indexed):
    from paper_2509_19171_amd import sel

    g = torch.Generator().manual_seed(n)
    X, y = torch.randn((n, 6), generator=g), torch.rand((n,), generator=g)
    p = torch.from_numpy(I.closure_blob(3, mean=[0.0] * 6, std=[1.0] * 6))
    p[12 + 6 * 5 + 2] = float("inf")
    idx = torch.randperm(n, generator=g).to(torch.int32) if indexed else None
    w = p[12:8845].double().requires_grad_(True)
    W1, b1, W2, b2, W3, b3, w4, b4 = torch.split(w, [384, 64, 4096, 64, 4096, 64, 64, 1])
    h = X.double()
    for W, b, k in ((W1, b1, 6), (W2, b2, 64), (W3, b3, 64)):
        h = torch.tanh(h @ W.view(64, k).T + b)
    loss = ((torch.nn.functional.softplus(h @ w4 + b4) - y.double()) ** 2).mean()
    loss.backward()
    ref, loss = w.grad, loss.item()
    assert torch.isfinite(ref).all()
    got, l = sel.mlp_gradient(p.cuda(), X.cuda(), y.cuda(), idx=None if idx is None else idx.cuda())
    print(f"[gpu] n {n} indexed {indexed}: {(got.cpu().double() - ref).abs().max():.2e}", flush=True)
    assert (got.cpu().double() - ref).abs().max() < 1e-5 * ref.abs().max()
    assert abs(l - loss) < 1e-5 * loss
