"""Infinite activations in the one-kernel network passes, widths that do and do
not fill their 16-wide tiles: with positive weights an infinite feature gives
+inf in its row, as the network in 64 bits does, and leaves the other rows
alone; in the gradient the output layer's entries are +inf for the neurons
that exist."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H", [1, 20, 33, 63, 64])
def test_infinite_rows(H):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm as F
    m, rng = F.Mlp(H), np.random.default_rng(H)
    sizes = [(H, F.MLP_INPUTS), (H, H), (H, H), (5, H)]
    Ws = [rng.uniform(0.5, 1.5, s).astype(np.float32) / s[1] for s in sizes]
    w = np.concatenate([np.concatenate([W.ravel(), np.zeros(W.shape[0], np.float32)]) for W in Ws]
                       + [np.ones(5, np.float32), np.zeros(5, np.float32)])
    X = rng.uniform(0.1, 1.0, (37, F.MLP_INPUTS)).astype(np.float32)
    X[5, 3] = np.inf
    X[21, 12] = np.inf
    a = X.astype(np.float64)
    for W in Ws[:-1]:
        z = a @ W.T.astype(np.float64)
        a = z / (1.0 + np.exp(-z))
    ref = a @ Ws[-1].T.astype(np.float64)
    wd, Xd = torch.as_tensor(w).cuda(), torch.as_tensor(X).cuda()
    out = m.forward(wd, Xd).cpu().numpy()
    bad = np.isin(np.arange(37), (5, 21))
    assert np.all(np.isposinf(ref[bad])) and np.all(np.isposinf(out[bad])), out[bad]
    assert np.allclose(out[~bad], ref[~bad], rtol=1e-5, atol=0.0)
    g, loss = m.grad(wd, Xd, torch.zeros(37, 5, device="cuda"))
    n3 = sum(a * (b + 1) for a, b in sizes[:-1])
    assert torch.isposinf(loss).all() and torch.isposinf(g[n3:n3 + 5 * H + 5]).all()
