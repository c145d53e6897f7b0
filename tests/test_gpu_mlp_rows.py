"""Edges of the one-kernel network passes: hidden widths around the 16-wide
tiles and the widest one, batches around the 16-row blocks, one and several
workgroups, against FP64 backpropagation.  Tolerance: sums of up to 64 FP32
products through seven layers (about 64 x 6e-8 x 7 = 3e-5), times a few for
the cancellation in Y - T of a single row."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H", [1, 15, 16, 17, 33, 48, 63, 64, 65])
@pytest.mark.parametrize("B", [1, 15, 16, 17, 47, 4099])
def test_forward_and_gradient_at_tile_edges(H, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm
    rng = np.random.default_rng(100 * H + B)
    w = (omlp.init(H, seed=H) + 0.05 * rng.standard_normal(omlp.n_params(H))).astype(np.float32)
    w[-10:-5] = rng.uniform(0.5, 2.0, 5)
    w[-5:] = rng.uniform(-1, 1, 5)
    X = rng.standard_normal((B, omlp.N_IN)).astype(np.float32)
    T = rng.standard_normal((B, 5)).astype(np.float32)
    loss_ref, g_ref = omlp.loss_and_grad(w.astype(np.float64), X.astype(np.float64), T.astype(np.float64), H)
    y_ref = omlp.predict(w.astype(np.float64), X.astype(np.float64), H)
    net = frdvm.Mlp(H)
    wd, Xd, Td = (torch.as_tensor(a).cuda() for a in (w, X, T))
    y = net.forward(wd, Xd).cpu().numpy()
    assert np.linalg.norm(y - y_ref) <= 1e-4 * np.linalg.norm(y_ref)
    g1, l1 = net.grad(wd, Xd, Td)
    g2, l2 = net.grad(wd, Xd, Td)
    assert torch.equal(g1, g2) and torch.equal(l1, l2)  # fixed order of the sums
    g = g1.cpu().numpy()
    assert abs(l1.item() - loss_ref) < 2e-4 * loss_ref
    o = 0
    for (m, k) in omlp.layer_shapes(H):
        for n_ in (m * k, m):
            seg = slice(o, o + n_)
            assert np.linalg.norm(g[seg] - g_ref[seg]) <= 2e-4 * np.linalg.norm(g_ref[seg]), (m, k, n_)
            o += n_
    assert np.all(g[o:] == 0)
