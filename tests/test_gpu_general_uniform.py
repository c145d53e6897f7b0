"""A state uniform in space on the general-mesh path at p = 1 in FP32 (values
with random mantissas, one per velocity).  Both sides of a face form the same
trace from the same values, so no jump is left, and the residual is the
rounding of one product per direction, D F with |D| = sqrt(3)/2: at most 2^-24
relative, uniformly distributed, 0.577 x 0.866 = 0.50 of 2^-24 |F| in root
mean square.  A trace rounded in another order than the one it is compared
with would add its own rounding times the correction, 1.37 x 1.37."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rk_first", [False, True])
def test_no_jump_in_a_uniform_state(rk_first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm as F
    mesh, _ = W.reorient_elements(W.box_mesh((2, 2, 2)), seed=2)  # sides 1/2: metrics exact in FP32
    grid = W.grid_spec((19, 17, 18), 5.0)
    s = F.FrDvm(mesh, 1, grid, {"model": 2, "mu_ref": 1.0, "precision": F.FP32})
    val = np.random.default_rng(1).uniform(1.0, 2.0, s.nu).astype(np.float32)
    f = torch.as_tensor(val).cuda().repeat(s.ne * s.ns, 1).reshape(s.shape).contiguous()
    if rk_first:
        s.rk_step(f, 0.0)  # (dt = 0: the traces a stage leaves, of the same state)
        assert torch.equal(f, torch.as_tensor(val).cuda().repeat(s.ne * s.ns, 1).reshape(s.shape))
    R = torch.empty_like(f)
    s.residual(f, R)
    ax = [np.linspace(-5.0, 5.0, n) for n in grid["n"]]
    u = np.stack(np.meshgrid(ax[2], ax[1], ax[0], indexing="ij"), -1)[..., ::-1].reshape(-1, 3)
    flux = np.abs(u).sum(1) * 4.0 * val  # |a^d . u| / |J| f, summed over the directions (2 / h = 4)
    rel = R.double().cpu().numpy().reshape(-1, s.nu) / flux * 2.0 ** 24
    rms = np.sqrt(np.mean(rel ** 2))
    print(f"rms {rms:.3f} of 2^-24 |F|, largest {np.abs(rel).max():.2f}", flush=True)
    assert rms <= 0.52
