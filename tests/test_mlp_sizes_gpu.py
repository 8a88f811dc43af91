"""Closure inference at the row counts where it changes between its two
kernels (16 k, 32 k and 64 k rows and their remainders) and where either has a
partly filled last tile, against FP64 on the same FP32 weights. Tolerance as for
the other sizes: |dz| <= 2e-5 (1 + |z|), and the increment follows z."""
import pytest

from paper_2509_19171_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [16384, 16385, 24577, 32767, 32769, 65533, 65537, 98305, 131073, 700001])
def test_forward_on_both_sides_of_the_choice(n):
    from paper_2509_19171_amd import sel

    X = torch.randn((n, 6), generator=torch.Generator().manual_seed(n))
    p = torch.from_numpy(I.closure_blob(5, mean=[0.1] * 6, std=[1.5] * 6, b4=-0.5))
    W1, b1, W2, b2, W3, b3, w4, b4 = torch.split(p[12:8845].double(), [384, 64, 4096, 64, 4096, 64, 64, 1])
    h = (X.double() - p[:6].double()) / p[6:12].double()
    for W, b, k in ((W1, b1, 6), (W2, b2, 64), (W3, b3, 64)):
        h = torch.tanh(h @ W.view(64, k).T + b)
    ref, tau = h @ w4 + b4, 0.02
    z, d = sel.mlp_forward(p.cuda(), X.cuda(), tau)
    err = ((z.cpu().double() - ref).abs() / (1 + ref.abs())).max().item()
    print(f"[gpu] n {n}: {err:.2e}", flush=True)
    assert err < 2e-5
    assert (d.cpu().double() - tau * torch.nn.functional.softplus(ref)).abs().max() < 4e-5 * tau * (1 + ref.abs().max())
