"""The equilibrium of a moment vector has the same bits whatever batch it is
solved in: the first n of a batch against a batch of those n, on both sides of
every line where the lanes per point change (axis of N nodes: 128 N, 512 N,
2048 N points), cold and learned starts, axes that the eight node classes do
and do not divide, and axes shorter than them."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nv", [(12, 7, 9), (17, 19, 18), (8, 16, 24), (3, 33, 5)])
def test_bits_do_not_depend_on_the_batch(nv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm as F
    h = F.FrDvm(W.box_mesh(1), 1, W.grid_spec(nv, 5.0), {"model": 0, "mu_ref": 1.0, "newton_max_iter": 100})
    H = 24
    h.mlp_set_weights((0.02 * np.random.default_rng(0).uniform(-1, 1, F.Mlp(H).n)).astype(np.float32))
    N = 2048 * max(nv) + 700
    g = torch.Generator().manual_seed(sum(nv))
    rho = torch.exp(torch.randn(N, generator=g, dtype=torch.float64))
    U = torch.empty(N, 3, dtype=torch.float64).uniform_(-1, 1, generator=g)
    th = 0.5 * max(10.0 / (m - 1) for m in nv) ** 2 * (0.8 + torch.rand(N, generator=g, dtype=torch.float64))
    th = th.clamp(max=4.0)
    Q = torch.cat([rho[:, None], rho[:, None] * U, (0.5 * rho * (U * U).sum(1) + 1.5 * rho * th)[:, None]], 1).cuda()
    for guess in (F.GUESS_COLD, F.GUESS_MLP):
        whole = h.equilibrium(Q, guess)
        for n in (1, 128 * max(nv), 128 * max(nv) + 1, 512 * max(nv), 512 * max(nv) + 9, 2048 * max(nv)):
            part = h.equilibrium(Q[:n].contiguous(), guess)
            for a, b in zip(whole, part):
                assert torch.equal(a[:n], b), (guess, n)
        k = N - 5  # and elsewhere in the batch
        assert torch.equal(h.equilibrium(Q[k:].contiguous(), guess)[0], whole[0][k:])
